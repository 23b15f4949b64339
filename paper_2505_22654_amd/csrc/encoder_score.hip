// Attention scoring of encoder tokens (Sec. 4.1 "Global Scan", Eq. 1-2).
//
// Both modes write one UN-AVERAGED value per (segment, head, patch token) into
// `head_scores` [BC, H, N]; the selection kernel sums the heads in a fixed order
// and applies the 1/H (or 1/(H*N)) factor of Eq. 2.
//
//   [CLS] mode   head_scores[h][j] = softmax_j(scale * q_CLS^h . k_j^h)
//   mean mode    head_scores[h][j] = sum_i softmax_row_i(scale * q_i^h . k^h)_j
//                (two passes over Q K^T on the matrix cores: row log-sum-exp,
//                then column sums of exp(s - lse_i); the N x N matrix is never
//                stored)
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "launch.hpp"

namespace vscan {

// ---------------------------------------------------------------------------
// [CLS] row.  One workgroup per (segment, head): a batched GEMV over the keys,
// bound by reading K once.  A key row is split into 16-byte pieces over adjacent
// lanes, so a wave reads whole rows contiguously.
// ---------------------------------------------------------------------------
// Three forms (THREADS threads with UNR loads each in flight; launch_score_cls_t): 512 threads have the loads of most
// waves on a CU in flight at the same time and the fewest rounds of softmax; short key blocks, and many of them,
// take 256 threads, with less work for nothing in a workgroup.

// Rows of any number of pieces: as many whole rows as fit a wave per load, a row's pieces added in a tree of lane
// shifts (STEPS: its depth).  With 256 threads, four guarded loads and one shuffle per piece, heads of 80: 576 bf16
// tokens 45.2 us a call, now 37; 8 x 900 64.8, 46; fp32, 1296 tokens 163, 71.
template <typename T, int STEPS, int THREADS, int UNR>
__global__ __launch_bounds__(THREADS) void score_cls_generic_kernel(const T *__restrict__ q,
                                                        const T *__restrict__ k,
                                                        float *__restrict__ head_scores, int H,
                                                        int S, int dh, int first_key, int col0,
                                                        int N, float scale_log2e) {
    constexpr int E = ElemTraits<T>::kPer16B;
    extern __shared__ __align__(16) unsigned char smem[];
    float *red = reinterpret_cast<float *>(smem);  // 16 floats
    float *qf = red + 16;                           // dh floats (dh <= 256)
    float *z = qf + 256;                            // n_keys floats

    const int h = blockIdx.x, bc = blockIdx.y;
    const int64_t head_row0 = ((int64_t)bc * H + h) * S;
    const T *qrow = q + head_row0 * dh;
    const T *kbase = k + (head_row0 + first_key) * dh;
    const int n_keys = S - first_key;
    const int tid = threadIdx.x;

    const int cpr = dh / E;          // 16-byte pieces per key row (<= 64)
    const int rpw = kWave / cpr;     // key rows per wave per load; the lanes past them repeat the last row's
    const int lane = lane_id();
    const int row_in_wave = min(lane / cpr, rpw - 1);
    const int piece = lane < rpw * cpr ? lane - row_in_wave * cpr : cpr - 1;
    constexpr int nw = THREADS / kWave;
    const int64_t row_bytes = (int64_t)dh * sizeof(T);
    auto row_of = [&](int base, int u) { return base + (u * nw + wave_id()) * rpw + row_in_wave; };
    auto fetch = [&](int base, uint4(&raw)[UNR]) {  // clamped: independent loads, in flight together
#pragma unroll
        for (int u = 0; u < UNR; ++u)
            raw[u] = load16_stream(kbase, min(row_of(base, u), n_keys - 1) * row_bytes + piece * 16);
    };
    uint4 raw[UNR];
    fetch(0, raw);
    for (int e = tid; e < dh; e += THREADS) qf[e] = load_elem<T>(qrow + e) * scale_log2e;
    __syncthreads();
    float qreg[E];
#pragma unroll
    for (int e = 0; e < E; ++e) qreg[e] = qf[piece * E + e];

    const int step = nw * rpw * UNR;
    for (int base = 0; base < n_keys; base += step) {
        uint4 nxt[UNR];
        if (base + step < n_keys) fetch(base + step, nxt);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            if (base + (u * nw + wave_id()) * rpw >= n_keys) continue;  // none of this wave's rows
            float kv[E];
            unpack16<T>(raw[u], kv);
            float part = 0.f;
#pragma unroll
            for (int e = 0; e < E; ++e) part = fmaf(kv[e], qreg[e], part);
            // a row's pieces sit in adjacent lanes: lane d adds lane d + n while both belong to the row
#pragma unroll
            for (int n = 1 << (STEPS - 1); n >= 1; n >>= 1) {
                const float up = __shfl_down(part, n, kWave);
                if (piece + n < min(2 * n, cpr)) part += up;
            }
            if (piece == 0 && row_of(base, u) < n_keys) z[row_of(base, u)] = part;
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) raw[u] = nxt[u];
    }
    __syncthreads();

    float m = -INFINITY;
    for (int j = tid; j < n_keys; j += THREADS) m = fmaxf(m, z[j]);
    m = block_max(m, red);
    float sum = 0.f;
    for (int j = tid; j < n_keys; j += THREADS) {
        const float e = __builtin_amdgcn_exp2f(z[j] - m);
        z[j] = e;
        sum += e;
    }
    sum = block_sum(sum, red);
    const float inv = 1.0f / sum;
    float *out = head_scores + ((int64_t)bc * H + h) * N;
    for (int j = tid; j < N; j += THREADS) out[j] = z[col0 + j] * inv;
}

// Same computation for rows whose piece count is a power of two (every common head
// size).  The key block is read as one flat, fully coalesced stream with all of a batch's
// independent 16-byte loads in flight: at these sizes the kernel's time is the number of
// serialised memory round-trips.  With 256 threads and 16 or 20 loads: a call 16 x 576 35.4
// us, now 34.3, 24 x 576 37.7, 35.0, 8 x 5 x 576 61.4, 58.9, one image in fp32 (9232 pieces)
// 32.6, 30.8.
template <typename T, int LOG2_CPR, int THREADS, int UNR>
__global__ __launch_bounds__(THREADS) void score_cls_kernel(const T *__restrict__ q,
                                                        const T *__restrict__ k,
                                                        float *__restrict__ head_scores, int H,
                                                        int S, int dh, int first_key, int col0,
                                                        int N, float scale_log2e) {
    constexpr int E = ElemTraits<T>::kPer16B;
    constexpr int cpr = 1 << LOG2_CPR;  // 16-byte pieces per key row
    constexpr int shift = LOG2_CPR;
    extern __shared__ __align__(16) unsigned char smem[];
    float *red = reinterpret_cast<float *>(smem);  // 16 floats
    float *qf = red + 16;                           // dh floats (dh <= 256)
    float *z = qf + 256;                            // n_keys floats

    const int h = blockIdx.x, bc = blockIdx.y;
    const int64_t head_row0 = ((int64_t)bc * H + h) * S;
    const T *qrow = q + head_row0 * dh;
    const unsigned char *kbase = reinterpret_cast<const unsigned char *>(k + (head_row0 + first_key) * dh);
    const int n_keys = S - first_key;
    const int tid = threadIdx.x;

    const int total = n_keys << shift;  // 16-byte pieces in the key block
    uint4 raw[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
        // clamped, not predicated: the loads of a batch stay independent of each other; what a
        // thread past the end fetched is dropped where the logits are filed
        const int p = min(u * THREADS + tid, total - 1);
        raw[u] = load16_stream(kbase, (int64_t)p * 16);
    }
    for (int e = tid; e < dh; e += THREADS) qf[e] = load_elem<T>(qrow + e) * scale_log2e;
    __syncthreads();
    float qreg[E];
    const int piece = tid & (cpr - 1);
#pragma unroll
    for (int e = 0; e < E; ++e) qreg[e] = qf[piece * E + e];

    for (int base = 0; base < total; base += THREADS * UNR) {
        uint4 nxt[UNR];
        if (base + THREADS * UNR < total) {
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const int p = min(base + THREADS * UNR + u * THREADS + tid, total - 1);
                nxt[u] = load16_stream(kbase, (int64_t)p * 16);
            }
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int p = base + u * THREADS + tid;
            // none of this wave's pieces (ten loads are one batch, mostly full: there the test itself costs 1 %)
            if (UNR < 10 && base + u * THREADS + wave_id() * kWave >= total) continue;
            float kv[E];
            unpack16<T>(raw[u], kv);
            float part = 0.f;
#pragma unroll
            for (int e = 0; e < E; ++e) part = fmaf(kv[e], qreg[e], part);
            part = group_sum<cpr>(part);
            if (piece == 0 && p < total) z[p >> shift] = part;
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) raw[u] = nxt[u];
    }
    __syncthreads();

    // softmax with one exchange between the waves: every wave normalises against its own
    // maximum, posts (maximum, sum) and rescales by what the pairs combine to
    float m = -INFINITY;
    for (int j = tid; j < n_keys; j += THREADS) m = fmaxf(m, z[j]);
    m = wave_max(m);
    float sum = 0.f;
    for (int j = tid; j < n_keys; j += THREADS) {
        const float e = __builtin_amdgcn_exp2f(z[j] - m);
        z[j] = e;  // read again below by this same thread only
        sum += e;
    }
    sum = wave_sum(sum);
    if (lane_id() == 0) {
        red[wave_id()] = m;
        qf[wave_id()] = sum;  // (the query is in registers)
    }
    __syncthreads();
    constexpr int NW = THREADS / kWave;
    float mx = red[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) mx = fmaxf(mx, red[w]);
    float denom = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) denom += qf[w] * __builtin_amdgcn_exp2f(red[w] - mx);
    // a wave without keys posted (-inf, 0): its term is 0 * 0
    const float f = __builtin_amdgcn_exp2f(m - mx) / denom;
    float *out = head_scores + ((int64_t)bc * H + h) * N;
    for (int j = tid; j < n_keys; j += THREADS)
        if (j >= col0 && j - col0 < N) out[j - col0] = z[j] * f;
}

// ---------------------------------------------------------------------------
// Mean attention received, on the matrix cores.
// ---------------------------------------------------------------------------
constexpr int kMeanBlock = 128;  // rows (pass 1) / keys (pass 2) owned by a workgroup
// rows of the streamed operand per LDS stage (smaller for wide rows: static LDS <= 64 KB)
__host__ __device__ constexpr int mean_tile_rows(int nc) { return nc > 8 ? 32 : 64; }

// Stages ROWS rows of NC 32-byte chunks through registers into LDS.
template <int NC, int ROWS>
struct TileStage {
    static constexpr int kPiecesPerRow = NC * 2;
    static constexpr int kPieces = ROWS * kPiecesPerRow;
    static constexpr int kPerThread = (kPieces + 255) / 256;
    static constexpr int kStride = NC * 32 + 16;  // bytes, padded against bank conflicts
    static constexpr int kBytes = ROWS * kStride;
    uint4 regs[kPerThread];

    // rows [row0, row0+ROWS) of a [*, row_bytes] matrix at `base`.  The loads carry no
    // condition: a row >= row_end re-reads row row_end - 1 and a piece past the end of a row
    // re-reads the row's last piece.  What lands in LDS for them is finite data that the
    // consumers neutralise (rows past the end are masked or carry an infinite log-sum-exp; the
    // register-resident operand is zero in the bytes past the row).
    __device__ __forceinline__ void load(const void *base, int row0, int row_end, int row_bytes) {
#pragma unroll
        for (int it = 0; it < kPerThread; ++it) {
            const int p = min((int)threadIdx.x + it * 256, kPieces - 1);
            const int r = p / kPiecesPerRow;
            const int piece = p - r * kPiecesPerRow;
            const int row = min(row0 + r, row_end - 1);
            regs[it] = load16(base, (int64_t)row * row_bytes + min(piece * 16, row_bytes - 16));
        }
    }
    __device__ __forceinline__ void store(unsigned char *lds) const {
#pragma unroll
        for (int it = 0; it < kPerThread; ++it) {
            const int p = threadIdx.x + it * 256;
            const int r = p / kPiecesPerRow;
            const int piece = p - r * kPiecesPerRow;
            if (p < kPieces) *reinterpret_cast<uint4 *>(lds + r * kStride + piece * 16) = regs[it];
        }
    }
};

// work item -> (segment*head, block) with each XCD walking a contiguous range of
// items, so the workgroups resident on one XCD share one head's Q/K in its L2
__device__ __forceinline__ int xcd_contiguous_item(int total) {
    const int id = blockIdx.x;
    const int per = (total + 7) / 8;
    return (id & 7) * per + (id >> 3);
}

// log2 of a sum of exponentials.  The hardware logarithm rounds one way: a whole row's weights would be
// too large by the same 2e-7 to 3e-7 in every row (measured), so its residual, which the hardware
// exponential shows, is added back.
__device__ __forceinline__ float log2_sum(float l) {
    const float y = __builtin_amdgcn_logf(l);
    return y + 1.4426950408889634f * fmaf(l, __builtin_amdgcn_exp2f(-y), -1.0f);
}

// The two half-waves hold disjoint streamed rows of the same resident row: reference and sum over both.
__device__ __forceinline__ void join_half_waves(float m, float l, float &M, float &L) {
    const float m_o = __shfl_xor(m, 32, kWave), l_o = __shfl_xor(l, 32, kWave);
    M = fmaxf(m, m_o);
    L = 0.f;
    if (m > -INFINITY) L += l * __builtin_amdgcn_exp2f(m - M);
    if (m_o > -INFINITY) L += l_o * __builtin_amdgcn_exp2f(m_o - M);
}

// The plain form of both passes (mean_pipelined).
// Pass 1: lse2[i] = log2 sum_j 2^(sl2 * q_i . k_j) over the key domain.
template <typename T, int NC>
__global__ __launch_bounds__(256, 2) void mean_lse_kernel(const T *__restrict__ q,
                                                          const T *__restrict__ k,
                                                          float *__restrict__ lse, int n_heads_total,
                                                          int S, int dh, int row_first, int N,
                                                          int key_first, int n_keys, float sl2) {
    constexpr int kMeanTile = mean_tile_rows(NC);
    using Stage = TileStage<NC, kMeanTile>;
    __shared__ __align__(16) unsigned char lds[2][Stage::kBytes];
    const int nblk = (N + kMeanBlock - 1) / kMeanBlock;
    const int total = n_heads_total * nblk;
    const int item = xcd_contiguous_item(total);
    if (item >= total) return;
    const int bh = item / nblk, rb = item - bh * nblk;
    const int row_bytes = dh * (int)sizeof(T);
    const unsigned char *qbase =
        reinterpret_cast<const unsigned char *>(q) + ((int64_t)bh * S + row_first) * row_bytes;
    const unsigned char *kbase =
        reinterpret_cast<const unsigned char *>(k) + ((int64_t)bh * S + key_first) * row_bytes;

    const int lane = lane_id(), g = lane >> 5, w = wave_id();
    const int qrow = rb * kMeanBlock + w * 32 + (lane & 31);
    uint4 qfrag[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
        qfrag[c] = load16_guard(qbase, (int64_t)qrow * row_bytes + 32 * c + 16 * g,
                                qrow < N && 32 * c + 16 * g < row_bytes);

    float m_run = -INFINITY, l_run = 0.f;
    bool have_ref = false;
    Stage st;
    const int ntiles = (n_keys + kMeanTile - 1) / kMeanTile;
    st.load(kbase, 0, n_keys, row_bytes);
    st.store(lds[0]);
    __syncthreads();
    for (int t = 0; t < ntiles; ++t) {
        const unsigned char *cur = lds[t & 1];
        if (t + 1 < ntiles) st.load(kbase, (t + 1) * kMeanTile, n_keys, row_bytes);
#pragma unroll
        for (int sub = 0; sub < kMeanTile / 32; ++sub) {
            f32x16_t acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
            const unsigned char *arow = cur + (sub * 32 + (lane & 31)) * Stage::kStride + 16 * g;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const uint4 a = *reinterpret_cast<const uint4 *>(arow + 32 * c);
                mma32_chunk<T>(acc, a, qfrag[c]);
            }
            // acc[r] = q_row(lane%32) . k_(key0 + acc_row(r)); mask the ragged tail
            const int key0 = t * kMeanTile + sub * 32;
            if (key0 + 32 > n_keys) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (key0 + acc_row(r) >= n_keys) acc[r] = -INFINITY;
            }
            // Lazy reference: exponentials are taken against a per-lane reference m_run that
            // is an actual logit of the row (so the sum is >= 1 and small terms may underflow
            // harmlessly) and is only raised when the partial sum threatens to overflow.  That
            // removes the per-element running max; the rescue path is rare.  (As a function of its
            // own this part costs calls of 800 to 3300 tokens 1.5 to 3 %.)
            if (!have_ref) {
                float mx = -INFINITY;
#pragma unroll
                for (int r = 0; r < 16; ++r) mx = fmaxf(mx, acc[r]);
                if (mx > -INFINITY) {
                    m_run = mx * sl2;
                    have_ref = true;
                }
            }
            if (have_ref) {
                float add = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    add += __builtin_amdgcn_exp2f(fmaf(acc[r], sl2, -m_run));
                if (add < 0x1p100f) {
                    l_run += add;
                } else {  // a logit far above the reference: re-base on this tile's maximum
                    float mx = -INFINITY;
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, acc[r]);
                    const float m_new = fmaxf(m_run, mx * sl2);
                    add = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        add += __builtin_amdgcn_exp2f(fmaf(acc[r], sl2, -m_new));
                    l_run = l_run * __builtin_amdgcn_exp2f(m_run - m_new) + add;
                    m_run = m_new;
                }
            }
        }
        if (t + 1 < ntiles) st.store(lds[(t + 1) & 1]);
        __syncthreads();
    }
    float M, L;
    join_half_waves(m_run, l_run, M, L);
    if (g == 0 && qrow < N) lse[(int64_t)bh * N + qrow] = M + log2_sum(L);
}

// Pass 2: head_scores[j] = sum_i 2^(sl2 * q_i . k_j - lse2[i]) for patch keys j.
template <typename T, int NC>
__global__ __launch_bounds__(256, 2) void mean_colsum_kernel(const T *__restrict__ q,
                                                             const T *__restrict__ k,
                                                             const float *__restrict__ lse,
                                                             float *__restrict__ head_scores,
                                                             int n_heads_total, int S, int dh,
                                                             int row_first, int N, float sl2) {
    constexpr int kMeanTile = mean_tile_rows(NC);
    using Stage = TileStage<NC, kMeanTile>;
    __shared__ __align__(16) unsigned char lds[2][Stage::kBytes];
    __shared__ __align__(16) float lse_s[2][kMeanTile];
    const int nblk = (N + kMeanBlock - 1) / kMeanBlock;
    const int total = n_heads_total * nblk;
    const int item = xcd_contiguous_item(total);
    if (item >= total) return;
    const int bh = item / nblk, kb = item - bh * nblk;
    const int row_bytes = dh * (int)sizeof(T);
    // queries and keys are both the patch rows here
    const unsigned char *qbase =
        reinterpret_cast<const unsigned char *>(q) + ((int64_t)bh * S + row_first) * row_bytes;
    const unsigned char *kbase =
        reinterpret_cast<const unsigned char *>(k) + ((int64_t)bh * S + row_first) * row_bytes;
    const float *lse_h = lse + (int64_t)bh * N;

    const int lane = lane_id(), g = lane >> 5, w = wave_id();
    const int key = kb * kMeanBlock + w * 32 + (lane & 31);
    uint4 kfrag[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
        kfrag[c] = load16_guard(kbase, (int64_t)key * row_bytes + 32 * c + 16 * g,
                                key < N && 32 * c + 16 * g < row_bytes);

    float colsum = 0.f;
    Stage st;
    const int ntiles = (N + kMeanTile - 1) / kMeanTile;
    const int tid = threadIdx.x;
    float lse_reg = 0.f;
    st.load(qbase, 0, N, row_bytes);
    if (tid < kMeanTile) lse_reg = tid < N ? lse_h[tid] : INFINITY;
    st.store(lds[0]);
    if (tid < kMeanTile) lse_s[0][tid] = lse_reg;
    __syncthreads();
    for (int t = 0; t < ntiles; ++t) {
        const unsigned char *cur = lds[t & 1];
        const float *lcur = lse_s[t & 1];
        if (t + 1 < ntiles) {
            st.load(qbase, (t + 1) * kMeanTile, N, row_bytes);
            const int r = (t + 1) * kMeanTile + tid;
            if (tid < kMeanTile) lse_reg = r < N ? lse_h[r] : INFINITY;
        }
#pragma unroll
        for (int sub = 0; sub < kMeanTile / 32; ++sub) {
            f32x16_t acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
            const unsigned char *arow = cur + (sub * 32 + (lane & 31)) * Stage::kStride + 16 * g;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const uint4 a = *reinterpret_cast<const uint4 *>(arow + 32 * c);
                mma32_chunk<T>(acc, a, kfrag[c]);
            }
            // acc[r] = q_(row0 + acc_row(r)) . k_key ; rows past N carry lse = +inf -> 0.  (A lane per query
            // row, as in the form below, saves no matrix instruction here and adds sums over the lanes at the
            // end: 3306 tokens, 4 heads of 96, 119 -> 121 us a call, 884 of 16 49.4 -> 50.2.)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const float4 l4 = *reinterpret_cast<const float4 *>(lcur + sub * 32 + 8 * rg + 4 * g);
                colsum += __builtin_amdgcn_exp2f(fmaf(acc[4 * rg + 0], sl2, -l4.x));
                colsum += __builtin_amdgcn_exp2f(fmaf(acc[4 * rg + 1], sl2, -l4.y));
                colsum += __builtin_amdgcn_exp2f(fmaf(acc[4 * rg + 2], sl2, -l4.z));
                colsum += __builtin_amdgcn_exp2f(fmaf(acc[4 * rg + 3], sl2, -l4.w));
            }
        }
        if (t + 1 < ntiles) {
            st.store(lds[(t + 1) & 1]);
            if (tid < kMeanTile) lse_s[(t + 1) & 1][tid] = lse_reg;
        }
        __syncthreads();
    }
    colsum += __shfl_xor(colsum, 32, kWave);
    if (g == 0 && key < N) head_scores[(int64_t)bh * N + key] = colsum;
}

// ---------------------------------------------------------------------------
// Both passes for bf16 rows of up to 160 bytes and for fp32, software-pipelined inside each wave.
//
// Measured on this GPU (issue rates in core cycles per wave instruction): v_fma / v_mul / v_add
// 4, v_exp_f32 8, a 32x32x16 matrix instruction occupies the matrix pipe for 32 and takes about
// 10 from the vector issue port.  A 32 x 32 tile of logits therefore costs 16 x (4 + 8 + 4) = 256
// cycles of vector work per lane against 160 cycles of matrix work (80-element rows): the
// vector ALU is the bound, and the matrix instructions have to be hidden under it.  A wave that
// multiplies, waits and then exponentiates leaves both pipes idle in turn, so here every wave
// keeps two accumulator sets: the matrix instructions of tile t+1 are issued while the
// exponentials of tile t run, and the LDS reads of tile t+2's operands are already under way.
//
// A workgroup (4 waves) owns 4 x 32 x HALVES resident rows, held in registers as matrix
// operands (pass 1: query rows, pass 2: key rows).  The other operand streams through LDS in
// stages of 128 rows (4 tiles), two stages in LDS, the next one in flight in registers: one
// workgroup barrier per 128 streamed rows.
//   PASS 1: lse2[i] = log2 sum_j 2^(sl2 * q_i . k_j)      (resident i, streamed j)
//   PASS 2: head_scores[j] = sum_i 2^(sl2 * q_i . k_j - lse2[i])   (resident j, streamed i)
// In both passes a lane's sixteen logits of a tile belong to one query row, whose reference is one
// register: in pass 1 the resident rows are the columns of the accumulator (a lane owns resident row
// lane % 32 and sixteen streamed rows), in pass 2 its rows (a lane owns streamed row lane % 32 and sums
// for its sixteen resident rows; the lanes are added once, at the end).  Subtracting the reference is
// the multiply-add that scales the logit.  (Pass 2 had the log-sum-exp as one more 32-byte chunk of the
// contraction before, a sixth more matrix instructions: 16384 tokens, 16 heads of 80, 850 -> 800 us.)  Rows past
// the end carry -inf and contribute 2^-inf = 0.
//
// With `parts` > 1 the streamed rows are cut into runs of whole stages with a workgroup each
// (mean_parts): pass 1 leaves a reference m and l = sum_j 2^(sl2 * q_i . k_j - m) per row and part, which
// pass 2 adds up where it fetches them, and pass 2 a row of sums per part, which the selection adds like
// further heads.
// ---------------------------------------------------------------------------

// 16-byte loads from global memory straight into LDS (no pass through vector registers, no LDS
// write instruction): lane l's data lands 16*l bytes behind the wave-uniform LDS address.  Issued
// from inline assembly so that the compiler's wait-count bookkeeping does not see them - it would
// otherwise make every LDS read wait for them, whichever buffer they fill; the kernel waits for
// them itself (wait_direct_loads) before the barrier that publishes the stage.
__device__ __forceinline__ unsigned lds_byte_address(const void *p) {
    return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}
__device__ __forceinline__ void direct_load16(const void *src, unsigned lds_address) {
    // (M0 carries the LDS address.  It is a reserved register that compiler-generated code
    // loads right before each instruction that reads it, never keeps live across statements,
    // and that the kernels of this file use for nothing else.)
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off"
                 :
                 : "s"(lds_address), "v"(src)
                 : "memory");
}
// every outstanding vector-memory load of this wave has arrived (vmcnt 0, the other counters
// left alone)
__device__ __forceinline__ void wait_direct_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

struct MeanPair {
    const unsigned char *resident, *streamed;
    float *lse;          // [n_heads, rows], or [n_heads, parts, rows] pairs (m, l)
    float *head_scores;  // [n_heads, parts, rows], pass 2
};

// lse2 of a row from its parts' pairs, two of them in either lane of a pair of lanes
__device__ __forceinline__ float merged_lse(const float2 (&p)[kMeanMaxParts / 2], int first, int parts) {
    static_assert(kMeanMaxParts == 4, "two parts a lane");
    const auto larger = [](float a, float b) { return fmaxf(a, b); };
    // (past the last part its pair is repeated: no weight, and the maximum stays)
    const float m = group_reduce<2>(fmaxf(p[0].x, p[1].x), larger);
    float l = first < parts ? p[0].y * __builtin_amdgcn_exp2f(p[0].x - m) : 0.f;
    l += first + 1 < parts ? p[1].y * __builtin_amdgcn_exp2f(p[1].x - m) : 0.f;
    return m + log2_sum(group_sum<2>(l));
}

// fp32 on the bf16 matrix instructions (the method of Henry, Tang and Heinecke, "Leveraging the bfloat16 artificial
// intelligence datatype for higher-precision computations", 2019): an fp32 value is the sum of three bf16 values
// (each the rounding of what the previous ones left over: 24 significant bits, the same exponents), a product of
// two fp32 values the sum of nine products of bf16 values, which are exact.  Six are formed.  The three left out
// (mid x lo, lo x mid, lo x lo) come to at most 2^-24 of the product (mid up to 2^-8 of the value, lo up to 2^-17;
// below 2^-26 for 97 % of mantissas), which is what rounding an fp32 product may cost.  The small products are added
// first, so that only the last, hi x hi, are rounded at the size of the result: 5 roundings for rows of 80 instead of
// the 40 of fp32 instructions.  Error of the scores against 64 bits (2-norm; 324 to 1023 tokens, three seeds of four
// shapes): given rows 2.8e-7 on average and 5.6e-7 at worst with fp32 instructions, 0.9e-7 and 1.6e-7 so;
// projected rows 7.0e-7 and 12.8e-7, 2.6e-7 and 4.8e-7; rows of values that leave out the most 1.9 to 4.2e-7, 0.7
// to 3.3e-7.  Below 2^-110 (7.7e-34) the low planes run out of exponents; what a value loses there, less than
// 2^-126, is seen in a logit only against values of 2^100 and more.
// Six bf16 instructions take the matrix pipe 192 cycles, the eight fp32 instructions for the same chunk 512.
// That is still four times what the vector work of a tile takes, so the matrix pipe is the bound: one
// workgroup a CU (up to 512 registers a lane), whose waves never wait for anything but the pipe: the planes of
// the resident rows and of a whole tile of streamed rows are in registers, and the streamed rows are split
// once per workgroup on their way into LDS, a few at a time between the matrix instructions.
// 2688 tokens, 16 heads of 80: 277 + 276 -> 145 + 134 us for the two passes; 16384 tokens, a call: 13.2 -> 7.2 ms,
// 1.2 PFLOP/s in the passes, which is what an 8192^3 product of the bf16 library reaches on this card.
template <typename T>
struct MeanForm;
template <>
struct MeanForm<bf16_t> {
    static constexpr int kPlanes = 1, kProducts = 1;
    static constexpr int kWorkgroupsPerCu = 2;
    static __device__ constexpr int streamed_plane(int) { return 0; }
    static __device__ constexpr int resident_plane(int) { return 0; }
};
template <>
struct MeanForm<float> {
    static constexpr int kPlanes = 3, kProducts = 6;  // planes hi, mid, lo
    static constexpr int kWorkgroupsPerCu = 1;
    static __device__ constexpr int streamed_plane(int p) { return p == 0 ? 2 : p < 3 ? 1 : 0; }
    static __device__ constexpr int resident_plane(int p) { return p == 1 || p == 4 ? 1 : p == 3 ? 2 : 0; }
};

// eight consecutive elements -> their planes.  From 3.396e38 on, rounding would make hi infinite and the other
// planes NaN: hi stops at the largest finite bf16 value and the others take the rest, exactly.  (The clamp costs a
// call 0 to 0.5 % up to heads of 80 and 2 % at 128: 1600 tokens, 8 heads, 132 -> 134.6 us.)
__device__ __forceinline__ void split_planes(const uint4 &a, const uint4 &b, uint4 *out) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    constexpr float kLargestBf16 = 0x1.fep127f;
    float v[8];
    unpack16<float>(a, v);
    unpack16<float>(b, v + 4);
#pragma unroll
    for (int p = 0; p < MeanForm<float>::kPlanes; ++p) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f32x2_t two = {v[2 * i], v[2 * i + 1]};
            if (p == 0) {
                two.x = __builtin_amdgcn_fmed3f(two.x, -kLargestBf16, kLargestBf16);
                two.y = __builtin_amdgcn_fmed3f(two.y, -kLargestBf16, kLargestBf16);
            }
            w[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2_t));
            v[2 * i] -= bf16_lo(w[i]);  // exact
            v[2 * i + 1] -= bf16_hi(w[i]);
        }
        out[p] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// Sum over the 32 streamed rows that the lanes of a half-wave hold, for each of the sixteen resident rows
// of a 32x32 accumulator: lane l < 16 of half g gets the sum of resident row acc_row(l).  Every step
// adds pairs of lanes and leaves each lane with half of the rows (31 exchanges instead of 80).
template <int ROWS>  // lanes n < ROWS apart have yet to be added, ROWS rows are left to this one
__device__ __forceinline__ float resident_row_sum(float (&v)[16]) {
    if constexpr (ROWS == 16) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] += __shfl_xor(v[r], 16, kWave);
    }
    if constexpr (ROWS > 1) {
        constexpr int n = ROWS / 2;
        const bool upper = (lane_id() & n) != 0;
#pragma unroll
        for (int r = 0; r < n; ++r) {
            const float mine = upper ? v[r + n] : v[r], other = upper ? v[r] : v[r + n];
            v[r] = mine + __shfl_xor(other, n, kWave);
        }
        return resident_row_sum<n>(v);
    } else {
        return v[0];
    }
}

// f(0), ..., f(N - 1) with constants
template <int... I, typename F>
__device__ __forceinline__ void for_constants(std::integer_sequence<int, I...>, F f) {
    (f(std::integral_constant<int, I>{}), ...);
}

// LDS of the kernel below: two stages of kRows streamed rows, in dynamic LDS where they pass 64 KB.
template <typename T, int NC>
struct MeanLds {
    static constexpr int kPlanes = MeanForm<T>::kPlanes;
    static constexpr int kRows = kPlanes * NC * 32 * 2 * 128 > 144 * 1024 ? 64 : 128;
    static constexpr int kStride = kPlanes * NC * 32 + (kPlanes == 1 && (NC & 1) ? 0 : 16);
    static constexpr int kBytes = 2 * kRows * kStride;
    static constexpr bool kDynamic = kBytes > 62 * 1024;
};

// PARTED, pass 2: the statistics come in parts.  A branch on `parts` where they are fetched would wait,
// where its sides join, for every load in flight.
template <typename T, int NC, int HALVES, int PASS, bool PARTED>
__global__ __launch_bounds__(256, MeanForm<T>::kWorkgroupsPerCu) void mean_pipe_kernel(
    MeanPair first, MeanPair second, int pairs, int n_heads, int S, int dh, int res_first, int n_res,
    int str_first, int n_streamed, int parts, float sl2) {
    using Form = MeanForm<T>;
    constexpr int PL = Form::kPlanes;
    constexpr bool SPLIT = PL > 1;
    // With an odd number of 32-byte chunks per row the unpadded row pitch serves the 16-byte
    // operand reads at 92 % of the LDS rate (measured; 25 % for an even number), and a stage
    // is then one contiguous block in memory and in LDS alike: it is fetched with direct loads.
    // Otherwise: padded rows (an odd number of 16-byte pieces, conflict-free) staged through registers.
    constexpr bool DIRECT = !SPLIT && (NC & 1) != 0;
    using Lds = MeanLds<T, NC>;
    constexpr int ROWS = Lds::kRows, TILES = ROWS / 32, STRIDE = Lds::kStride;
    constexpr int PPR = NC * 2;                        // 16-byte pieces per plane of a streamed row
    constexpr int PER = (ROWS * PPR + 255) / 256;      // pieces per thread and stage
    constexpr int RB = 4 * 32 * HALVES;                // resident rows per workgroup
    constexpr int NM = Form::kProducts * NC * HALVES;  // matrix instructions per tile
    constexpr int NL = 16 * HALVES;                    // logits per lane and tile
    static_assert(ROWS * PPR == 256 * PER, "PER pieces per thread and stage");
    static_assert((TILES & (TILES - 1)) == 0 && kMeanStageRows % ROWS == 0, "whole stages per part");
    extern __shared__ __align__(16) unsigned char dynamic_lds[];
    __shared__ __align__(16) unsigned char static_lds[Lds::kDynamic ? 16 : 2 * ROWS * STRIDE];
    unsigned char *const lds_base = Lds::kDynamic ? dynamic_lds : static_lds;
    auto lds = [&](int buffer) { return lds_base + buffer * (ROWS * STRIDE); };
    __shared__ __align__(16) float neg_lse[2][PASS == 2 ? ROWS : 1];

    const int nblk = (n_res + RB - 1) / RB;
    const int total = pairs * n_heads * parts * nblk;
    const int item = xcd_contiguous_item(total);
    if (item >= total) return;
    const int run = item / nblk;  // (pair, head, part)
    const int blk = item - run * nblk;
    int bh = run / parts;
    const int part = run - bh * parts;
    const bool is_second = bh >= n_heads;
    if (is_second) bh -= n_heads;
    const int row_bytes = dh * (int)sizeof(T);
    // this part's stages of the streamed rows
    const int all_stages = (n_streamed + kMeanStageRows - 1) / kMeanStageRows;
    const int row0 = part * all_stages / parts * kMeanStageRows;
    const int n_str = min((part + 1) * all_stages / parts * kMeanStageRows, n_streamed) - row0;
    const unsigned char *__restrict__ rbase = (is_second ? second.resident : first.resident) +
                                              ((int64_t)bh * S + res_first) * row_bytes;
    const unsigned char *__restrict__ sbase = (is_second ? second.streamed : first.streamed) +
                                              ((int64_t)bh * S + str_first + row0) * row_bytes;
    float *__restrict__ lse = is_second ? second.lse : first.lse;
    float2 *__restrict__ pair = reinterpret_cast<float2 *>(lse);  // parts > 1
    const int64_t at = PASS == 1 ? ((int64_t)bh * parts + part) * n_res : (int64_t)bh * parts * n_streamed + row0;

    const int tid = threadIdx.x, lane = lane_id(), g = lane >> 5, w = wave_id();
    uint4 kf[HALVES][NC][PL];
#pragma unroll
    for (int h = 0; h < HALVES; ++h) {
        const int row = blk * RB + (w * HALVES + h) * 32 + (lane & 31);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int64_t off = (int64_t)row * row_bytes + (16 * c + 8 * g) * (int)sizeof(T);
            const bool valid = row < n_res && 16 * c + 8 * g < dh;  // dh is a multiple of eight
            const uint4 a = load16_guard(rbase, off, valid);
            if constexpr (SPLIT)
                split_planes(a, load16_guard(rbase, off + 16, valid), kf[h][c]);
            else
                kf[h][c][0] = a;
        }
    }
    const int ntiles = (n_str + 31) >> 5;
    const int nstages = (n_str + ROWS - 1) / ROWS;

    // ---- staging of the streamed operand: thread t carries pieces t, t + 256, ... of a stage
    // (fp32: of eight elements, which become a piece of every plane)
    uint4 sreg[DIRECT ? 1 : PER][SPLIT ? 2 : 1];
    // pass 2: threads 2r and 2r + 1 carry the statistics of a stage's row r, two parts each
    float2 stat_reg[PARTED ? kMeanMaxParts / 2 : 1];
    const int first_part = (tid & 1) * (kMeanMaxParts / 2);
    auto stage_load = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < PER; ++it) {
            const int p = tid + it * 256;
            const int r = p / PPR, piece = p - r * PPR;
            // clamped, not predicated: rows past the end re-read the last row (finite data that
            // the consumers neutralise), pieces past the end of a row its last piece (the
            // resident operand is zero there)
            const int row = min(s * ROWS + r, n_str - 1);
            const int64_t off = (int64_t)row * row_bytes + min(piece * 8, dh - 8) * (int)sizeof(T);
            if constexpr (DIRECT) {
                // piece p of the stage goes to byte 16 p of the stage's buffer: the wave's 64
                // pieces of this round form one contiguous kilobyte
                direct_load16(sbase + off, __builtin_amdgcn_readfirstlane(lds_byte_address(
                                               lds(s & 1) + 16 * (it * 256 + w * kWave))));
            } else {
                sreg[it][0] = load16(sbase, off);
                if constexpr (SPLIT) sreg[it][1] = load16(sbase, off + 16);
            }
        }
        if constexpr (PASS == 2) {
            const int64_t row = at + min(s * ROWS + min(tid >> 1, ROWS - 1), n_str - 1);
            if constexpr (!PARTED) {
                stat_reg[0].x = lse[row];
            } else {
#pragma unroll
                for (int u = 0; u < kMeanMaxParts / 2; ++u)
                    stat_reg[u] = pair[row + (int64_t)min(first_part + u, parts - 1) * n_streamed];
            }
        }
    };
    auto piece_store = [&](int s, int it) __attribute__((always_inline)) {
        const int p = tid + it * 256;
        const int r = p / PPR, piece = p - r * PPR;
        unsigned char *dst = lds(s & 1) + r * STRIDE + piece * 16;
        uint4 out[PL];
        if constexpr (SPLIT)
            split_planes(sreg[it][0], sreg[it][1], out);
        else
            out[0] = sreg[it][0];
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) *reinterpret_cast<uint4 *>(dst + pl * NC * 32) = out[pl];
    };
    // `spread`: the pieces are in LDS already
    auto stage_store = [&](int s, bool spread) __attribute__((always_inline)) {
        if constexpr (DIRECT) {
            wait_direct_loads();  // this wave's share of the stage is in LDS
        } else if (!spread) {
#pragma unroll
            for (int it = 0; it < PER; ++it) piece_store(s, it);
        }
        if constexpr (PASS == 2) {
            float x;
            if constexpr (PARTED)
                x = merged_lse(stat_reg, first_part, parts);
            else
                x = stat_reg[0].x;
            if ((tid & 1) == 0 && tid < 2 * ROWS)
                neg_lse[s & 1][tid >> 1] = s * ROWS + (tid >> 1) < n_str ? -x : -INFINITY;
        }
    };

    u32x4_t fr[PL][NC];      // streamed operand of one tile in matrix-operand layout, refilled in place
    f32x16_t acc[2][HALVES];
    auto frag_ptr = [&](int t) {
        return lds((t / TILES) & 1) + ((t & (TILES - 1)) * 32 + (lane & 31)) * STRIDE + 16 * g;
    };
    // chunk c of a tile in matrix-operand layout (`base` = frag_ptr(t))
    auto read_frag = [&](const unsigned char *base, int pl, int c) {
        return *reinterpret_cast<const u32x4_t *>(base + 32 * (pl * NC + c));
    };
    // product p of chunk c
    auto multiply = [&](const f32x16_t &sum, int h, int p, int c) {
        union {
            uint4 u;
            bf16x8_t v;
        } x;
        x.u = kf[h][c][Form::resident_plane(p)];
        const bf16x8_t y = __builtin_bit_cast(bf16x8_t, fr[Form::streamed_plane(p)][c]);
        return PASS == 1 ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(y, x.v, sum, 0, 0, 0)
                         : __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.v, y, sum, 0, 0, 0);
    };
    // pass 2: -lse2 of this lane's streamed row, of the present and of the next tile
    float row_lse[2];
    auto read_lse = [&](int t) { return neg_lse[(t / TILES) & 1][(t & (TILES - 1)) * 32 + (lane & 31)]; };

    float m_run[HALVES], l_run[HALVES], colsum[HALVES][PASS == 2 ? 16 : 1];
    bool have_ref[HALVES];
#pragma unroll
    for (int h = 0; h < HALVES; ++h) {
        m_run[h] = -INFINITY;
        l_run[h] = 0.f;
        have_ref[h] = false;
        if constexpr (PASS == 2) {
#pragma unroll
            for (int r = 0; r < 16; ++r) colsum[h][r] = 0.f;
        }
    }

    // One pipeline step: the vector work of tile t (accumulators `cur`), with the matrix instructions of
    // tile t + 1 (operands in `fr`, accumulators `nxt`) issued in between; every operand chunk is refilled
    // with tile t + 2's right after its last use, and `between(m)` runs behind matrix instruction m.
    // (Past the last tile the refills read what lies there and nobody uses it.)  LAST: tile t is the last
    // one, nothing is multiplied.
    auto step = [&](int t, f32x16_t(&cur)[HALVES], f32x16_t(&nxt)[HALVES], auto last_tag,
                    auto between) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(last_tag)::value;
        float ref[HALVES], part[HALVES];
        const float now = PASS == 2 ? row_lse[t & 1] : 0.f;
        if constexpr (PASS == 1) {
            if (LAST && (n_str & 31) != 0) {
#pragma unroll
                for (int h = 0; h < HALVES; ++h)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (t * 32 + acc_row(r) >= n_str) cur[h][r] = -INFINITY;
            }
            // Lazy reference: exponentials are taken against a per-lane reference that is an
            // actual logit of the row (so the sum is >= 1 and small terms may underflow
            // harmlessly) and is only raised when the partial sum threatens to overflow.
#pragma unroll
            for (int h = 0; h < HALVES; ++h) {
                if (!have_ref[h]) {
                    float mx = -INFINITY;
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, cur[h][r]);
                    if (mx > -INFINITY) {
                        m_run[h] = mx * sl2;
                        have_ref[h] = true;
                    }
                }
                ref[h] = have_ref[h] ? m_run[h] : 0.f;  // without a reference every logit is -inf
            }
        }
#pragma unroll
        for (int h = 0; h < HALVES; ++h) part[h] = 0.f;
        const unsigned char *next_frags = frag_ptr(t + 2);
        // Slot by slot: one matrix instruction, the LDS read that refills an operand chunk
        // after its last use, and a slice of tile t's logits (one plane: about three, forty cycles of
        // vector work, which is what one matrix instruction keeps its pipe busy for).  (Pinning
        // this order with scheduling groups, or tying the step's inputs to this point with
        // empty asm statements, measured the same as leaving the order to the compiler.)
        for_constants(std::make_integer_sequence<int, NM>{}, [&](auto slot) __attribute__((always_inline)) {
            constexpr int m = decltype(slot)::value;
            if constexpr (!LAST) {
                constexpr int p = m / (NC * HALVES), c = m / HALVES % NC, h = m % HALVES;
                // (the first chunk starts from a constant zero: no registers to clear)
                const f32x16_t zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                                       0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                nxt[h] = multiply(m < HALVES ? zero : nxt[h], h, p, c);
                constexpr int sp = Form::streamed_plane(p);
                constexpr bool used = p + 1 == Form::kProducts || Form::streamed_plane(p + 1) != sp;
                if constexpr (h == HALVES - 1 && used) fr[sp][c] = read_frag(next_frags, sp, c);
            }
#pragma unroll
            for (int i = m * NL / NM; i < (m + 1) * NL / NM; ++i) {
                const int h = i / 16, r = i % 16;
                if constexpr (PASS == 1)
                    part[h] += __builtin_amdgcn_exp2f(fmaf(cur[h][r], sl2, -ref[h]));
                else
                    colsum[h][r] += __builtin_amdgcn_exp2f(fmaf(cur[h][r], sl2, now));
            }
            between(slot);
        });
        if constexpr (PASS == 2 && !LAST) row_lse[t & 1] = read_lse(t + 2);
        if constexpr (PASS == 1) {
#pragma unroll
            for (int h = 0; h < HALVES; ++h) {
                if (part[h] < 0x1p100f) {
                    l_run[h] += part[h];
                } else {  // a logit far above the reference: re-base on this tile's maximum
                    float mx = -INFINITY;
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, cur[h][r]);
                    const float m_new = fmaxf(m_run[h], mx * sl2);
                    float add = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        add += __builtin_amdgcn_exp2f(fmaf(cur[h][r], sl2, -m_new));
                    l_run[h] = l_run[h] * __builtin_amdgcn_exp2f(m_run[h] - m_new) + add;
                    m_run[h] = m_new;
                }
            }
        }
        // keep the steps apart: left alone, the compiler gathers the matrix instructions of
        // several steps into one burst right behind the LDS reads they wait for
        __builtin_amdgcn_sched_barrier(0);
    };
    using yes = std::integral_constant<bool, true>;
    using no = std::integral_constant<bool, false>;

    // ---- prologue: stage 0 in LDS, stage 1 in flight, tile 0 multiplied, tile 1's operands read
    stage_load(0);
    stage_store(0, false);
    __syncthreads();
    if (nstages > 1) stage_load(1);
    {
        const unsigned char *f0 = frag_ptr(0);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int pl = 0; pl < PL; ++pl) fr[pl][c] = read_frag(f0, pl, c);
        if constexpr (PASS == 2) row_lse[0] = read_lse(0);
#pragma unroll
        for (int h = 0; h < HALVES; ++h) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[0][h][r] = 0.f;
#pragma unroll
            for (int m = 0; m < Form::kProducts * NC; ++m) acc[0][h] = multiply(acc[0][h], h, m / NC, m % NC);
        }
        if (ntiles > 1) {
            const unsigned char *f1 = frag_ptr(1);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int pl = 0; pl < PL; ++pl) fr[pl][c] = read_frag(f1, pl, c);
            if constexpr (PASS == 2) row_lse[1] = read_lse(1);
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    const auto nothing = [](auto) {};
    int t0 = 0;
    // Steady state, one stage per trip: straight-line code.  The next stage goes to LDS (its loads were
    // issued a stage ago) before the last two tiles, the first to fetch operands from it, and the one
    // after it takes over the staging registers.  Where it is split on the way, the pieces go one by one
    // between the matrix instructions of the tiles before: their place in LDS has been free since the
    // last barrier.
    constexpr bool SPREAD = SPLIT && TILES == 4;
    for (; t0 + TILES + 2 <= ntiles; t0 += TILES) {
        const int s = t0 / TILES;
        for_constants(std::make_integer_sequence<int, TILES>{}, [&](auto tile) __attribute__((always_inline)) {
            constexpr int j = decltype(tile)::value;
            if constexpr (j == TILES - 2) {
                stage_store(s + 1, SPREAD);
                __syncthreads();
                if (s + 2 < nstages) stage_load(s + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            step(t0 + j, acc[j & 1], acc[(j + 1) & 1], no{}, [&](auto slot) __attribute__((always_inline)) {
                constexpr int m = decltype(slot)::value;
                constexpr int EACH = (PER + 1) / 2, GAP = NM / EACH;  // pieces per tile of the first two
                constexpr int piece = j * EACH + m / GAP;
                if constexpr (SPREAD && j < 2 && m % GAP == GAP / 2 && m / GAP < EACH && piece < PER)
                    piece_store(s + 1, piece);
            });
        });
    }
    // The last tiles.
    for (; t0 + 1 < ntiles; t0 += TILES) {
        const int s = t0 / TILES;
        for_constants(std::make_integer_sequence<int, TILES>{}, [&](auto tile) __attribute__((always_inline)) {
            constexpr int j = decltype(tile)::value;
            if (t0 + j + 1 < ntiles) {
                if (j == TILES - 2 && s + 1 < nstages) {
                    stage_store(s + 1, false);
                    __syncthreads();
                    if (s + 2 < nstages) stage_load(s + 2);
                }
                step(t0 + j, acc[j & 1], acc[(j + 1) & 1], no{}, nothing);
            }
        });
    }
    if (ntiles & 1)
        step(ntiles - 1, acc[0], acc[1], yes{}, nothing);
    else
        step(ntiles - 1, acc[1], acc[0], yes{}, nothing);

#pragma unroll
    for (int h = 0; h < HALVES; ++h) {
        const int first_row = blk * RB + (w * HALVES + h) * 32, l = lane & 31;
        if constexpr (PASS == 1) {
            const int row = first_row + l;
            float M, L;
            join_half_waves(m_run[h], l_run[h], M, L);
            if (g == 0 && row < n_res) {
                if (parts == 1)
                    lse[at + row] = M + log2_sum(L);
                else
                    pair[at + row] = make_float2(M, L);
            }
        } else {
            const float sum = resident_row_sum<16>(colsum[h]);
            const int row = first_row + 8 * (l >> 2) + 4 * g + (l & 3);
            if (l < 16 && row < n_res)
                (is_second ? second.head_scores : first.head_scores)[((int64_t)bh * parts + part) * n_res + row] = sum;
        }
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <typename T, int THREADS, int UNR>
static hipError_t launch_score_cls_form(const ScoreArgs &a, hipStream_t s) {
    const int first_key = a.domain_all ? 0 : 1;
    const int n_keys = a.S - first_key;
    const size_t smem = (16 + 256 + (size_t)n_keys) * sizeof(float);
    const int cpr = a.dh / ElemTraits<T>::kPer16B;
    auto launch = [&](auto kernel, std::atomic<uint64_t> &lds_allowed) {
        if (smem > 64 * 1024) {
            hipError_t e = allow_large_lds(kernel, lds_allowed);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3(a.H, a.BC), dim3(THREADS), smem, s, (const T *)a.q, (const T *)a.k,
                           a.head_scores, a.H, a.S, a.dh, first_key, 1 - first_key, a.N,
                           a.scale * 1.4426950408889634f);
        return hipGetLastError();
    };
    static std::atomic<uint64_t> lds_allowed[12];  // one per kernel
    if ((cpr & (cpr - 1)) == 0) {
        switch (__builtin_ctz(cpr)) {
            case 0: return launch(score_cls_kernel<T, 0, THREADS, UNR>, lds_allowed[0]);
            case 1: return launch(score_cls_kernel<T, 1, THREADS, UNR>, lds_allowed[1]);
            case 2: return launch(score_cls_kernel<T, 2, THREADS, UNR>, lds_allowed[2]);
            case 3: return launch(score_cls_kernel<T, 3, THREADS, UNR>, lds_allowed[3]);
            case 4: return launch(score_cls_kernel<T, 4, THREADS, UNR>, lds_allowed[4]);
            case 5: return launch(score_cls_kernel<T, 5, THREADS, UNR>, lds_allowed[5]);
            case 6: return launch(score_cls_kernel<T, 6, THREADS, UNR>, lds_allowed[6]);
        }
    }
    if (cpr < 4) return launch(score_cls_generic_kernel<T, 2, THREADS, UNR>, lds_allowed[7]);
    if (cpr < 8) return launch(score_cls_generic_kernel<T, 3, THREADS, UNR>, lds_allowed[8]);
    if (cpr < 16) return launch(score_cls_generic_kernel<T, 4, THREADS, UNR>, lds_allowed[9]);
    if (cpr < 32) return launch(score_cls_generic_kernel<T, 5, THREADS, UNR>, lds_allowed[10]);
    return launch(score_cls_generic_kernel<T, 6, THREADS, UNR>, lds_allowed[11]);
}

// 256 threads with four loads up to one batch of them, and up to three where a CU has more than three workgroups;
// 512 threads with ten where that is one batch and five would be two, for workgroups with a CU to themselves (a
// call 16 x 576, on keys that are in no cache, 36.6 us, with five 36.9; warm, 4608 x 256 30.4, 30.3); 512 threads with
// five otherwise.  GPU time of a call, us, with 512 x 5 and with 256 threads (16-byte pieces of a key block x
// workgroups; rows of 8 pieces, then of 10):  448 x 16 16.3, 16.1;  448 x 4800 31.4, 25.1;  880 x 256 21.6, 21.6;
// 2048 x 16 18.8, 19.2;  2048 x 640 22.1, 21.9;  2048 x 1600 27.5, 26.9;  2888 x 1600 39.0, 37.8;  2888 x 4800 72.2, 73.3;
// 3872 x 4800 88.6, 90.0;  6960 x 256 37.8, 39.6;  10:  490 x 4800 41.9, 29.4;  900 x 256 21.9, 21.8;  1440 x 256 21.6,
// 22.3;  2100 x 640 24.5, 25.5;  2100 x 1024 26.9, 25.2;  2890 x 4800 78, 74.5;  4000 x 4800 91.8, 93.3.  With 512 x 10 for
// all of these 448 x 4800 takes 41.9, 2888 x 640 29.4 (five: 28.8), 10: 2100 x 1600 53.  Past one workgroup a CU, on
// keys that are in no cache, with five and with ten: 4608 x 320 25.4, 26.1;  x 640 30.2, 30.8 (in a call 8 x 5 x 576
// of wide features 58.9, 58.5);  x 1600 51.8, 53.4;  10: 4800 x 320 27.0, 32.0.
template <typename T>
static hipError_t launch_score_cls_t(const ScoreArgs &a, hipStream_t s) {
    const int64_t pieces = (int64_t)(a.S - (a.domain_all ? 0 : 1)) * (a.dh / ElemTraits<T>::kPer16B);
    const int64_t workgroups = (int64_t)a.H * a.BC;
    if (pieces <= 1024 || (pieces <= 3072 && workgroups > 3 * kCus)) return launch_score_cls_form<T, 256, 4>(a, s);
    if (pieces > 2560 && pieces <= 5120 && workgroups <= kCus) return launch_score_cls_form<T, 512, 10>(a, s);
    return launch_score_cls_form<T, 512, 5>(a, s);
}

hipError_t launch_score_cls(const ScoreArgs &a, hipStream_t s) {
    return a.is_bf16 ? launch_score_cls_t<bf16_t>(a, s) : launch_score_cls_t<float>(a, s);
}

template <typename T, int NC>
static hipError_t launch_score_mean_nc(const ScoreArgs &a, hipStream_t s, int pass) {
    const int row_first = a.has_cls;
    const int key_first = a.domain_all ? 0 : a.has_cls;
    const int n_keys = a.S - key_first;
    const int nblk = (a.N + kMeanBlock - 1) / kMeanBlock;
    const int total = a.BC * a.H * nblk;
    const int grid = ((total + 7) / 8) * 8;
    const float sl2 = a.scale * 1.4426950408889634f;
    if (pass == 1)
        hipLaunchKernelGGL((mean_lse_kernel<T, NC>), dim3(grid), dim3(256), 0, s, (const T *)a.q,
                           (const T *)a.k, a.lse, a.BC * a.H, a.S, a.dh, row_first, a.N, key_first,
                           n_keys, sl2);
    else
        hipLaunchKernelGGL((mean_colsum_kernel<T, NC>), dim3(grid), dim3(256), 0, s,
                           (const T *)a.q, (const T *)a.k, a.lse, a.head_scores, a.BC * a.H, a.S,
                           a.dh, row_first, a.N, sl2);
    return hipGetLastError();
}

// The pipelined form, which takes pairs and parts.
template <typename T, int NC, int HALVES>
static hipError_t launch_mean_pipe(const ScoreArgs &a, hipStream_t s, int pass) {
    const int row_first = a.has_cls;
    const int key_first = a.domain_all ? 0 : a.has_cls;
    const int n_keys = a.S - key_first;
    constexpr int RB = 4 * 32 * HALVES;
    const int pairs = (pass == 1 ? a.q2 != nullptr : a.head_scores2 != nullptr) ? 2 : 1;
    const int total = pairs * a.BC * a.H * a.parts * ((a.N + RB - 1) / RB);
    const int grid = ((total + 7) / 8) * 8;
    const float sl2 = a.scale * 1.4426950408889634f;
    using Bytes = const unsigned char *;
    constexpr auto pass1 = mean_pipe_kernel<T, NC, HALVES, 1, false>, pass2 = mean_pipe_kernel<T, NC, HALVES, 2, false>,
                   pass2_parted = mean_pipe_kernel<T, NC, HALVES, 2, true>;
    using Lds = MeanLds<T, NC>;
    constexpr int lds = Lds::kDynamic ? Lds::kBytes : 0;
    if constexpr (Lds::kDynamic) {
        static std::atomic<uint64_t> allowed[3];
        hipError_t e = pass == 1 ? allow_large_lds(pass1, allowed[0], lds)
                       : a.parts > 1 ? allow_large_lds(pass2_parted, allowed[1], lds)
                                     : allow_large_lds(pass2, allowed[2], lds);
        if (e != hipSuccess) return e;
    }
    if (pass == 1)  // resident query rows (patch rows), streamed keys of the softmax domain
        hipLaunchKernelGGL(pass1, dim3(grid), dim3(256), lds, s,
                           (MeanPair{(Bytes)a.q, (Bytes)a.k, a.lse, nullptr}),
                           (MeanPair{(Bytes)a.q2, (Bytes)a.k2, a.lse2, nullptr}), pairs,
                           a.BC * a.H, a.S, a.dh, row_first, a.N, key_first, n_keys, a.parts, sl2);
    else            // resident patch keys, streamed query rows (patch rows) with their log-sum-exps
        hipLaunchKernelGGL((a.parts > 1 ? pass2_parted : pass2), dim3(grid), dim3(256), lds, s,
                           (MeanPair{(Bytes)a.k, (Bytes)a.q, a.lse, a.head_scores}),
                           (MeanPair{(Bytes)a.k2, (Bytes)a.q2, a.lse2, a.head_scores2}), pairs,
                           a.BC * a.H, a.S, a.dh, row_first, a.N, row_first, a.N, a.parts, sl2);
    return hipGetLastError();
}

// The plain kernels, by the 32-byte chunks of a row.
template <typename T>
static hipError_t launch_score_mean_plain(const ScoreArgs &a, hipStream_t s, int pass) {
    const int nc = (a.dh * (int)sizeof(T) + 31) / 32;
    if (nc <= 2) return launch_score_mean_nc<T, 2>(a, s, pass);
    if (nc <= 4) return launch_score_mean_nc<T, 4>(a, s, pass);
    if (nc <= 5) return launch_score_mean_nc<T, 5>(a, s, pass);
    if (nc <= 8) return launch_score_mean_nc<T, 8>(a, s, pass);
    if (nc <= 12) return launch_score_mean_nc<T, 12>(a, s, pass);
    if (nc <= 16) return launch_score_mean_nc<T, 16>(a, s, pass);
    return hipErrorInvalidValue;  // rows wider than 512 bytes are rejected by the ABI layer
}

static hipError_t launch_score_mean(const ScoreArgs &a, hipStream_t s, int pass) {
    if (!a.pipelined)
        return a.is_bf16 ? launch_score_mean_plain<bf16_t>(a, s, pass) : launch_score_mean_plain<float>(a, s, pass);
    const int nc = (a.dh + 15) / 16;  // chunks of sixteen elements
    if (!a.is_bf16) {
        if (nc <= 2) return launch_mean_pipe<float, 2, 2>(a, s, pass);
        if (nc <= 4) return launch_mean_pipe<float, 4, 2>(a, s, pass);
        if (nc <= 5) return launch_mean_pipe<float, 5, 2>(a, s, pass);
        return launch_mean_pipe<float, 8, 1>(a, s, pass);
    }
    if (nc <= 2) return launch_mean_pipe<bf16_t, 2, 2>(a, s, pass);
    if (nc <= 4) return launch_mean_pipe<bf16_t, 4, 2>(a, s, pass);
    return launch_mean_pipe<bf16_t, 5, 2>(a, s, pass);
}

hipError_t launch_score_mean_lse(const ScoreArgs &a, hipStream_t s) { return launch_score_mean(a, s, 1); }
hipError_t launch_score_mean_colsum(const ScoreArgs &a, hipStream_t s) { return launch_score_mean(a, s, 2); }

}  // namespace vscan
