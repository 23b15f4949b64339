// Host-side launch interface of the score chain that starts from hidden states and projection
// weights (Eq. 1 / Eq. 5 as written), bf16 or fp32 inputs.  Every launcher enqueues on the given stream
// and returns hipGetLastError().
#pragma once
#include "launch.hpp"

namespace vscan {

constexpr int kFusedQtPlanes = 3;  // bf16 planes carrying the hidden-space query (all 24 bits)
struct FusedArgs {
    int is_bf16 = 1;           // element type of hidden, w_q, w_k_t (else fp32)
    const void *hidden;        // [B, S, Dh]; visual tokens are rows vis_start .. vis_start+V
    const void *w_q;           // [Hq*dh, Dh]   rows = output features
    const void *w_k_t;         // [Dh, Hkv*dh]  rows = input features
    float *c_q;                // [ks_q][B*Tq][Hq*dh] partial sums of q
    uint16_t *q_planes;        // bf16 inputs: [3][B*Tq][Hq*dh] bf16; fp32 inputs: [B*Tq][Hq*dh] floats
    uint16_t *qt_planes;       // bf16 inputs: [kFusedQtPlanes][Hkv][B*(Hq/Hkv)*Tq][Dh] bf16; fp32
                               // inputs: [Hkv][B*(Hq/Hkv)*Tq][Dh] floats
    float *c_l;                // [ks_l][B][Hq*Tq][nk] partial sums of the unscaled logits; the
                               // first slot becomes the softmax weights
    float *part;               // [B][V] sums over the query rows
    int B, S, Dh, Hq, Hkv, dh, Tq, vis_start, V, k0, nk;
    int q_row0;                // first of the Tq query rows of a sequence
    int causal;                // query position t sees all but the last Tq-1-t keys of the domain
    // ragged batch (device table, else NULL): a sequence's query rows are its own last Tq rows,
    // its key domain is its visual span, or with `causal` its whole length; S, V, nk are then
    // capacities (tensor strides)
    const SeqMeta *meta = nullptr;
    int ks_q, ks_l;            // shares of the contraction axis (fused_ksplit)
    float scale;
    SelectSeed seed;           // for the selection launch that follows the chain
    int keep_rows = 0;         // the chain ends with the rows' softmax weights in c_l (fused_keep_rows)
};
// Whether q leaves launch_fused_q in its final form (no launch_fused_split_q): few query rows, no more
// than one workgroup of sixteen output features for each CU, and weight rows of which a wave's eighth is
// one batch of loads (17 to 32 query rows, which take twice the registers), two, or (fp32, whose split
// form is the slower one, up to 8 query rows) four.  Stage-2 calls with q in one launch and with the axis
// split over workgroups, us (features out x in, query rows):
//   bf16  4096 x 4096  1: 33.6, 40.5;  8: 42.1, 45.3;  16: 49.0, 51.2;  24: 88.7, 88.6;  32: 112.2, 110.5
//         2048 x 2048  1: 29.1, 32.8;  16: 39.4, 43.7;  17: 51.9, 54.4;  32: 54.7, 56.6
//         2560 x 2560  8: 40.0, 41.3;  16: 48.2, 47.3;  17: 61.1, 58.6;  32: 65.3, 61.2
//         2048 x 5120  1: 34.4, 35.1;  8: 42.1, 40.5;  16: 48.5, 44.0   (rows of 10 KiB)
//         8192 x 2048  1: 35.8, 38.9;  8: 44.3, 43.4;  16: 49.9, 49.3   (two workgroups on a CU)
//         5120 x 5120  1: 50.6, 43.7;  8: 61.2, 49.0;  16: 72.8, 56.5   (both)
//   fp32  1024 x 1024  1: 29.1, 33.3;  16: 38.9, 43.1;  17: 50.4, 53.1;  32: 52.2, 54.7
//         2048 x 2048  1: 31.6, 34.1;  8: 36.2, 41.1;  16: 42.0, 45.4;  17: 60.4, 60.0;  32: 64.1, 62.6
//         4096 x 2560  1: 38.1, 43.7;  8: 45.3, 46.4;  16: 52.5, 50.0
//         4096 x 4096  1: 44.4, 51.9;  8: 50.8, 55.2;  16: 58.5, 59.1;  17: 76.9, 75.7
//         1024 x 4096  1: 39.8, 41.3;  8: 46.7, 49.5;  16: 54.8, 52.0
//         4096 x 5120  1: 53.5, 55.7;  8: 60.9, 59.8;  16: 72.0, 66.7
constexpr int kThinQueries = 32, kThinOutputs = 4096;
inline bool fused_q_whole(const FusedArgs &a) {
    const int64_t rows = (int64_t)a.B * a.Tq, row_bytes = (int64_t)a.Dh * (a.is_bf16 ? 2 : 4);
    const int64_t most = rows <= 8 && !a.is_bf16 ? 16384 : rows <= 16 ? 8192 : 4096;
    return rows <= kThinQueries && a.Hq * a.dh <= kThinOutputs && row_bytes <= most;
}
// Whether the selection adds the R rows of softmax weights up itself, as it does the heads of the
// Q/K forms (no launch_fused_colsum): its key domain is the visual tokens, and the one workgroup that
// selects for a sequence has no more than 64 rows and 128 KiB of them to read.  A launch goes (3 to 5 us);
// the selection takes longer, and beside it in an out-of-place call the copies slow its reads down.
// Stage-2 calls with the rows added by the selection and by a launch of their own, us (bf16):
//   16 rows, hidden 1024  1 x 576 tokens: 26.0, 28.4;  16 x 576: 33.6, 36.2;  32 x 1000: 44.1, 46.7
//   28 rows, hidden 3584  1 x 576: 36.8, 39.4;  16 x 576: 70.7, 73.0;  32 x 1000: 137.2, 137.5
//   32 rows, hidden 4096  1 x 576: 43.7, 44.9;  16 x 576: 65.6, 66.1;  24 x 576: 87.1, 86.5
//   64 rows, hidden 4096  1 x 500: 46.9, 47.2;  8 x 500: 60.1, 60.0
//   128 rows, hidden 4096  1 x 250: 54.8, 54.1;  8 x 250: 72.2, 71.0;  256 rows  4 x 125: 80.4, 76.9
inline bool fused_keep_rows(int R, int nk, int V) {
    return nk == V && R <= 64 && (int64_t)R * nk <= 32768;
}
// shares of the contraction axis for a contraction of Z problems of rows_s x rows_p outputs
int fused_ksplit(int rows_s, int rows_p, int Z, int k_elems, int elem_bytes);
hipError_t launch_fused_q(const FusedArgs &a, hipStream_t s);
hipError_t launch_fused_split_q(const FusedArgs &a, hipStream_t s);
hipError_t launch_fused_qt(const FusedArgs &a, hipStream_t s);
hipError_t launch_fused_logits(const FusedArgs &a, hipStream_t s);
hipError_t launch_fused_softmax(const FusedArgs &a, hipStream_t s);
hipError_t launch_fused_colsum(const FusedArgs &a, hipStream_t s);

// Mean-attention scoring (last sentence of "Global Scan") from hidden states: every token is a
// query, so Q and K are projected outright, in one launch - out[bc][h][t][e] = sum_k hidden[bc][t][k] *
// w[h*dh + e][k], fp32, in the layout the mean-attention kernels read - and those kernels run
// on the result.  `w` has its rows along the output features; W_K arrives the other way round
// and is transposed first.
struct ProjectArgs {
    int is_bf16 = 1;      // element type of hidden and w (else fp32)
    const void *hidden;   // [BC, S, Dh]
    const void *w, *w_k;  // [H*dh, Dh] each
    float *out, *out_k;   // [BC, H, S, dh] each
    int BC, S, Dh, H, dh;
};
hipError_t launch_fused_project(const ProjectArgs &a, hipStream_t s);
// out[c][r] = in[r][c], elements of 2 or 4 bytes
hipError_t launch_transpose(const void *in, void *out, int rows, int cols, int elem_bytes,
                            hipStream_t s);

}  // namespace vscan
