// Host-side launch interface between the C ABI layer and the kernel files.
// Every launcher enqueues on the given stream and returns hipGetLastError().
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace vscan {

// Dynamic LDS above 64 KB has to be allowed per kernel.  The limit is raised to the most one
// workgroup can have, once per kernel instantiation and device: `done` is a static of the
// calling instantiation, one bit per device.  Later launches only read the bit.  A kernel that
// also has static LDS passes a `limit` that leaves room for it.
constexpr int kMaxDynamicLds = 160 * 1024;
template <typename Kernel>
inline hipError_t allow_large_lds(Kernel kernel, std::atomic<uint64_t> &done,
                                  int limit = kMaxDynamicLds) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, limit);
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
    return e;
}


// encoder attention scoring (Eq. 1-2)
struct ScoreArgs {
    const void *q, *k;    // [BC, H, S, dh]
    float *head_scores;   // [BC, H, N] un-averaged per-head scores; mean mode [BC, H, parts, N]
    float *lse;           // [BC, H, N] scratch, mean mode only; parts > 1: [BC, H, parts, N] pairs
    int BC, H, S, dh, N;
    int has_cls, domain_all, is_bf16;
    float scale;
    bool pipelined = false;  // mean_pipelined
    // a second pair for the pipelined form to take along, or NULL: pass 1 always may, pass 2 where
    // head_scores2 is given
    const void *q2 = nullptr, *k2 = nullptr;
    float *lse2 = nullptr;
    int parts = 1;        // mean_parts
    float *head_scores2 = nullptr;
};
// Which of its two forms mean attention takes (per call: both passes the same).  The pipelined form has 256
// resident rows to a workgroup (128 for fp32 rows of more than 80), takes streamed rows in parts and, with Q and K
// given (`pair`: a second pair comes along), both pairs in a launch; fp32 goes as bf16 planes there.  The plain one
// has 128 rows and two workgroups a CU: better where the last 256 rows of a head would be mostly padding.  GPU time
// of a call, us, plain and pipelined (N x heads, one pair unless said):
//   bf16, 64 wide: 64 x 16 19.9, 22.0; 64 x 2048 30, 49; 256 x 64 26.8, 28.3; 256 x 1024 54, 63; 289 x 16 31.0, 31.3;
//   289 x 160 35.6, 45.7; 380 x 64 33.9, 36.3; 380 x 512 59, 70; but 420 x 4 34.4, 30.1; 506 x 64 38.5, 38.0; 506 x 256 54.6,
//   56.9; 650 x 16 46, 42; 650 x 512 132, 131; two pairs 64 x 16 24.9, 22.2; 289 x 16 44, 34; 64 x 256 27.0, 29.5
//   (48 x 180, where the host's launches count, 32.7, 29).
//   fp32, 80 wide: 64 x 16 26, 29; 121 x 2048 139, 179; 132 x 16 37, 35.5; 256 x 1024 231, 169; 289 x 64 60, 47; 289 x 160
//   89, 96; 289 x 256 121, 102; 600 x 160 263, 153; two pairs 64 x 16 38, 31; 121 x 256 59, 65.
//   fp32, 16 wide (padded to 32): 256 x 64 27, 29; 380 x 256 53, 61; 600 x 16 43, 40; 900 x 160 138, 142; 900 x 16 57, 46;
//   40 wide (to 64): 169 x 64 30, 34; 441 x 64 48, 47; 441 x 160 87, 93; 600 x 256 172, 177; 600 x 160 143, 124; 900 x 256 373,
//   325; 96 wide (to 128): 132 x 64 40, 37; 132 x 512 94, 111; 289 x 512 219, 228; 600 x 512 621, 609; 128 wide: 100 x 256
//   43, 38; 100 x 2048 170, 180; 64 x 16 28, 28.3; 132 x 1024 202, 204; 256 x 1024 299, 269.
inline bool mean_pipelined(int is_bf16, int dh, int64_t heads, int N, bool pair) {
    if (is_bf16 && dh > 80) return false;
    if (pair && heads <= (is_bf16 ? 192 : 64)) return true;  // two launches instead of four
    if (is_bf16) return N > 384 || (N > 256 && heads < 64);
    if (dh <= 16) return N >= 600 && heads <= 64;
    if (dh <= 96 && N <= 128) return false;
    if (dh <= 32 || (dh > 40 && dh <= 80)) return N <= 256 || N > 400 || heads <= 128 || heads >= 256;
    if (dh <= 40) return N > 800 || (N > 400 && heads <= 64);
    if (dh <= 96) return N >= 400 || heads <= 64;
    return N >= 200 || heads <= (N >= 100 ? 256 : 0);
}

// Into how many parts the streamed rows of mean attention are cut.  A workgroup owns 256 (128) resident
// rows of a head and takes as long as its stages of streamed rows and about 0.8 more (its own rows, the
// first stage, the sums at the end); the launch takes as long as the CU with most workgroups.  (With 1.5
// instead of 0.8 fewer calls are cut: 2745 tokens 127 us instead of 114.)
// A call in one part and in the number chosen, us (bf16, 16 heads of 80 unless said): 324 tokens 42, 37 (3
// parts); 576 and a second pair 60, 45 (2, joined); 1023: 66, 50 (4); 1296, 8 heads of 64: 71, 49 (4); 2000:
// 98, 77 (2); 7200, 12 heads of 64: 399, 340; 10000: 811, 724.  fp32: 324 tokens 65, 48; 1023: 133, 80;
// 10000: 3064, 2777.  Near the line: 2745 tokens 125, 114 (4), in fp32 314, 308; 2 x 3120, 64 wide 190, 181;
// 3 x 714 and a second pair in fp32, 128 wide 276, 264 (2).
// Left in one part, and what two would take: 3 x 848 in fp32 138, 149; 2 x 850 in fp32, 128 wide 150, 166; 3234 from
// hidden states, 64 wide 318, 336; 3 x 3640, 64 wide 312, 313; 5776 and a second pair 507, 510; 7200 457, 457; 8000
// 515, 509; 4096 179, 171; 3 x 522 and a second pair, 64 wide 66, 58.  Of 105 calls, 256 to 9000 tokens, none took
// more than 1 % longer with the number chosen than in one part.
constexpr int kMeanMaxParts = 4;
constexpr int kMeanStageRows = 128;
constexpr double kMeanStart = 0.8;  // stages
inline int mean_block_rows(int is_bf16, int dh) { return !is_bf16 && dh > 80 ? 128 : 256; }
inline double mean_cost(int64_t heads, int N, int block_rows, int parts) {
    const int64_t items = heads * ((N + block_rows - 1) / block_rows);
    const int stages = (N + kMeanStageRows - 1) / kMeanStageRows;
    return (double)((items * parts + 255) / 256) * ((stages + parts - 1) / parts + kMeanStart);
}
inline int mean_parts(int is_bf16, int dh, int64_t heads, int N) {  // pipelined form
    int best = 1;
    const int stages = (N + kMeanStageRows - 1) / kMeanStageRows, rows = mean_block_rows(is_bf16, dh);
    for (int p = 2; p <= kMeanMaxParts && p <= stages; ++p)
        if (mean_cost(heads, N, rows, p) < 0.95 * mean_cost(heads, N, rows, best)) best = p;
    return best;
}
hipError_t launch_score_cls(const ScoreArgs &a, hipStream_t s);
hipError_t launch_score_mean_lse(const ScoreArgs &a, hipStream_t s);     // pass 1
hipError_t launch_score_mean_colsum(const ScoreArgs &a, hipStream_t s);  // pass 2

// local + global selection (Eq. 2-3, footnote on priority)
struct EncSelectArgs {
    const float *head_global;  // [BC, H, N]
    const float *head_local;   // [BC, H, N] or NULL (= head_global)
    int B, C, H, gh, gw, wr, wc;
    int kw;                    // per window
    int kg;                    // per segment, remainder of the local budget included
    float norm;                // 1/H or 1/(H*N)
    int32_t *kept_idx;         // [B, C*(W*kw+kg)]
    int32_t *drop_idx;         // [B, C*N - K]
    uint64_t *best;            // [B, C*N] packed (similarity key, ~slot)
    float *scores_out;         // optional [B, C*N]
    // scratch for large segments, where the local scan runs as a kernel of its own:
    // global-scan keys [BC, N] and local-scan flags [BC, N]
    uint32_t *pre_key_ws = nullptr;
    uint8_t *pre_flag_ws = nullptr;
    // set by the launcher for the second kernel of that form
    const uint32_t *pre_key = nullptr;
    const uint8_t *pre_flag = nullptr;
};
hipError_t launch_encoder_select(const EncSelectArgs &a, hipStream_t s);
size_t encoder_select_lds_bytes(int N, int has_local);

// cosine assignment (Sec. 4.1 "Token Merging") and Eq. 4
struct MergeArgs {
    const void *x;             // [B, T, D]
    const int32_t *kept_idx;   // [B, K]
    const int32_t *drop_idx;   // [B, U]
    uint64_t *best;            // [B, T]
    void *merged;              // [B, K, D]
    int32_t *assign_out;       // optional [B, T]
    float *inv_norm;           // [B, K] scratch: 1 / ||x_s|| of the kept rows (large form only)
    int B, T, D, K, is_bf16;
};
hipError_t launch_sim_argmax(const MergeArgs &a, hipStream_t s);
hipError_t launch_merge(const MergeArgs &a, hipStream_t s);

// Per-sequence lengths of a ragged stage-2 batch (same layout as vscan_seq_meta).  Where an
// args struct carries a non-NULL `meta` (a DEVICE array of B entries), the kernels take
// seq_len / vis_start / vis_len / keep of sequence b from meta[b]; the struct's own S, V, keep
// then are capacities: tensor strides and LDS sizes.
struct SeqMeta {
    int32_t seq_len, vis_start, vis_len, keep;
};

// Puts a host table of `batch` entries into device memory on the stream, without a copy that
// would make the host wait (ragged_entry.hip).
using TableUpload = hipError_t (*)(SeqMeta *table, const SeqMeta *from_host, int batch, hipStream_t s);

// The kept indices are what the selection launch of an out-of-place call hands over through: the
// scoring kernel before it sets them to kNotYetKept.
constexpr int32_t kNotYetKept = -2;
struct SelectSeed {
    int32_t *kept = nullptr;   // [n_kept]
    int64_t n_kept = 0;
};
// Looks (about a microsecond apart) that a gathering workgroup of that launch takes at an index
// before it makes the selection itself: well above the longest selection.
constexpr int kSelectPolls = 1024;

// stage 2 scoring (Eq. 5)
struct LlmScoreArgs {
    const void *q;             // [B, Hq, Tq, dh]
    const void *k;             // [B, Hkv, S, dh]
    float *part;               // [B, Hkv, V] un-averaged sums over the query rows of a kv head
    int B, Hq, Hkv, Tq, S, dh, vis_start, V;
    int domain_all, is_bf16;
    float scale;
    const SeqMeta *meta = nullptr;
    // scratch of the form that cuts long key domains into chunks (llm_score_split_chunks > 0):
    // logits [B*Hkv, rows, V] and per-chunk (maximum, sum) pairs [B*Hkv, chunks, rows, 2]
    float *split_e = nullptr, *split_stats = nullptr;
    SelectSeed seed;
};
hipError_t launch_llm_score(const LlmScoreArgs &a, hipStream_t s);
int llm_score_split_chunks(int B, int Hkv, int rows, int nk);
// rows = (Hq/Hkv)*Tq query rows per kv head, nk = keys in the softmax domain
bool llm_score_supported(int rows, int nk, int row_bytes);

struct CompactArgs;
struct LlmSelectArgs {
    const float *part;         // [B, Hkv, V]
    int B, Hkv, V, keep;
    float norm;                // 1/(Tq*Hq)
    int32_t *kept_idx;         // [B, keep]; ragged: entries past a sequence's own keep are -1
    float *scores_out;         // optional [B, V]
    const SeqMeta *meta = nullptr;
    int zero_tail = 0;         // ragged: scores past a sequence's own span are set to zero
    // out-of-place compaction (host pointer, NULL in place): done by this launch too
    const CompactArgs *copy = nullptr;
    int polls = kSelectPolls;  // with `copy`; 0: every gathering workgroup selects
};
hipError_t launch_llm_select(const LlmSelectArgs &a, hipStream_t s);
size_t llm_select_lds_bytes(int V);

// order-preserving compaction ("Remarks on KV Cache"); launch_compact is the in-place form
struct CompactArgs {
    void *k, *v, *hidden;              // sources (and destinations when in_place)
    void *k_out, *v_out, *hidden_out;  // NULL when in_place
    const int32_t *kept_idx;           // [B, keep]; at least one readable int when keep == 0
    int B, Hkv, S, dh, Dh, vis_start, V, keep, elem_bytes, in_place;
    // rows between consecutive slabs of the destinations: S - V + keep for the dense
    // out-of-place result, S when compacting in place or into tensors shaped like the inputs
    int out_rows;
    // out of place: rows outside the visual span of the sequence that has most of them (S - V
    // when every sequence is alike); with `zero_tail`, the most rows any sequence has in the
    // destinations besides its kept ones
    int max_static_rows;
    int zero_tail = 0;  // ragged, out of place: rows past a sequence's result are set to zero
    const SeqMeta *meta = nullptr;
};
hipError_t launch_compact(const CompactArgs &a, hipStream_t s);

}  // namespace vscan
