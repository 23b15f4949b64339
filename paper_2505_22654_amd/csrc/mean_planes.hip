// Mean attention received (last sentence of "Global Scan") for fp32 queries and keys.
//
// The fp32 matrix instructions run at a sixteenth of the fp16 rate, so every fp32 value is carried
// as a pair of fp16 values, x = 2^-e (hi + lo) with e common to a block of 128 rows (the largest
// magnitude of the block lands in [2^14, 2^15)), and a logit is
//     q . k = 2^-(eq + ek) (lo_q . hi_k + hi_q . lo_k + hi_q . hi_k) ,
// three fp16 contractions with fp32 accumulation.  hi + lo holds 22 to 23 bits of every value down
// to 2^-18 of the block's maximum (below that, 2^-40 of the maximum), the dropped lo_q . lo_k is
// below 2^-22 of a product.  Relative error of the scores against 64 bits, this form and the fp32
// instructions (2688 tokens, 16 heads of 80): mean 3.1e-7 and -6.6e-7, deviation 1.5e-7 and 2.4e-7,
// largest 0.9e-6 and 1.3e-6.  (In the 2-norm, which the few large scores decide and where the lean of
// the fp32 form on the small ones does not count: 6e-7 and 1.2e-7 to 1.9e-7.)
//
// Measured, lse + column sums, fp32 instructions -> this form: 2688 tokens, 16 heads of 80:
// 266 + 266 us -> 76 + 71 us and 10 us for the planes; 6400 tokens: 1236 + 1237 -> 336 + 316 us
// (630 TFLOP/s of fp16 products); 1600 tokens, 16 heads of 64: 64 + 62 -> 27 + 26 us.
#include <type_traits>

#include "mean.hpp"

namespace vscan {
namespace {

typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));

// Rows in the order the kernels walk them: the N patch rows first, a [CLS] row (row 0 of the
// matrix) after them.  Blocks of kPlaneBlock rows are counted in this order.
__device__ __forceinline__ int matrix_row(int r, int N, int row_first) {
    return r < N ? row_first + r : 0;
}

// A workgroup turns one block of one head's q or k into planes: a row of dh floats becomes dh
// halves of hi and dh halves of lo in the same number of bytes, possibly in place (all of the
// block is in registers before anything is written, and no other workgroup touches its rows).
// Bound by memory: read and written once.
template <int NI>
__global__ __launch_bounds__(256) void planes_kernel(const float *q, const float *k,
                                                     unsigned char *q_planes, unsigned char *k_planes,
                                                     int32_t *__restrict__ exps, int n_heads_total,
                                                     int nblk, int S, int dh, int row_first, int N,
                                                     int n_rows) {
    __shared__ uint32_t red[4];
    const int bh = blockIdx.x / nblk, blk = blockIdx.x - bh * nblk;
    const bool is_k = blockIdx.y != 0;
    const float *src = (is_k ? k : q) + (int64_t)bh * S * dh;
    unsigned char *dst = (is_k ? k_planes : q_planes) + (int64_t)bh * S * dh * 4;
    const int ppr = dh >> 2, r0 = blk * kPlaneBlock;
    const int total = min(kPlaneBlock, n_rows - r0) * ppr;  // 16-byte pieces of the block
    uint4 raw[NI];
    int at[NI];  // where the piece's hi halves go, from the head's first byte
    uint32_t amax = 0;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int p = min((int)threadIdx.x + i * 256, total - 1);  // clamped: all loads in flight
        const int r = p / ppr, piece = p - r * ppr;
        const int row = matrix_row(r0 + r, N, row_first);
        at[i] = row * dh * 4 + piece * 8;
        raw[i] = load16(src, (int64_t)row * dh * 4 + piece * 16);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
        amax = max(max(amax, max(raw[i].x & 0x7fffffffu, raw[i].y & 0x7fffffffu)),
                   max(raw[i].z & 0x7fffffffu, raw[i].w & 0x7fffffffu));
    amax = wave_umax_dpp(amax);
    if (lane_id() == 0) red[wave_id()] = amax;
    __syncthreads();
    amax = max(max(red[0], red[1]), max(red[2], red[3]));
    // block maximum 1.m x 2^x -> 2^14; zero, infinite and NaN blocks stay as they are.  The bounds
    // keep 2^e and the values in range (subnormal blocks are scaled by 2^110 only).
    const int ex = (int)(amax >> 23);
    const int e = amax == 0 || ex == 255 ? 0 : min(14 - (ex - 127), 110);
    const float f = ldexpf(1.f, e);
    if (threadIdx.x == 0) exps[((int64_t)(is_k ? n_heads_total : 0) + bh) * nblk + blk] = e;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        if ((int)threadIdx.x + i * 256 >= total) break;
        float v[4];
        unpack16<float>(raw[i], v);
        f16x4_t hi, lo;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float x = v[j] * f;
            hi[j] = (_Float16)x;
            lo[j] = (_Float16)(x - (float)hi[j]);
        }
        *reinterpret_cast<f16x4_t *>(dst + at[i]) = hi;
        *reinterpret_cast<f16x4_t *>(dst + at[i] + dh * 2) = lo;
    }
}

// ---------------------------------------------------------------------------
// Both passes, pipelined like mean_pipe_kernel (encoder_score.hip): a workgroup of four waves owns
// 4 x 32 x HALVES resident rows in registers as matrix operands, the other operand streams through
// LDS in stages of 32 ST rows (two stages, fetched straight into LDS), every wave keeps two
// accumulator sets, and the matrix instructions of tile t + 1 are issued between the exponentials
// of tile t.
//   PASS 1: lse2[i] = log2 sum_j 2^(sl2 * q_i . k_j)               (resident i, streamed j)
//   PASS 2: head_scores[j] = sum_i 2^(sl2 * q_i . k_j - lse2[i])   (resident j, streamed i)
// Bound by the matrix cores: a tile takes 3 NC HALVES instructions of 32 cycles against 256 HALVES
// cycles of vector work.  Stages of 64 rows leave room for two workgroups on a CU.
// A plane's rows lie in LDS without padding (direct loads allow none).  An odd number of 32-byte
// chunks per row spreads the 16-byte operand reads over the banks by itself; otherwise the row's
// 16-byte columns are permuted by the row's low bits.
// ---------------------------------------------------------------------------
template <int NC, int ST>
constexpr int planes_lds_bytes() {
    return 2 * ST * 32 * NC * 64 + 3 * ST * 32 * 4;
}

template <int NC, int HALVES, int PASS, int ST>
__global__ __launch_bounds__(256, 2) void mean_planes_kernel(
    const unsigned char *__restrict__ resident, const unsigned char *__restrict__ streamed,
    const int32_t *__restrict__ res_exp, const int32_t *__restrict__ str_exp,
    const float *__restrict__ lse_in, float *__restrict__ out, int n_heads_total, int nblk_exp, int S,
    int dh, int row_first, int N, int n_str, float sl2) {
    constexpr int PPR = NC * 2;                  // 16-byte pieces per row of a plane
    constexpr int ROWS = 32 * ST;                // rows per stage
    constexpr int PLANE = ROWS * NC * 32;        // bytes of a stage's plane
    constexpr int NI = 2 * ROWS * PPR / 256;     // direct loads per thread and stage
    constexpr int RB = 4 * 32 * HALVES;
    constexpr int NM = 3 * NC * HALVES, NL = 16 * HALVES;
    static_assert(2 * ROWS * PPR % 256 == 0 && ROWS * PPR % kWave == 0,
                  "whole rounds of loads, each wave's inside one plane");
    static_assert(kPlaneBlock % ROWS == 0, "a stage has one exponent");
    extern __shared__ __align__(16) unsigned char smem[];
    auto stage_buf = [&](int s) { return smem + (s & 1) * 2 * PLANE; };
    // three deep: a wave that stores for stage s + 2 may meet one that still reads stage s
    float *neg_lse = reinterpret_cast<float *>(smem + 4 * PLANE);

    const int nblk = (N + RB - 1) / RB;
    const int total = n_heads_total * nblk;
    const int item = xcd_contiguous_item(total);
    if (item >= total) return;
    const int bh = item / nblk, blk = item - bh * nblk;
    const int row_bytes = dh * 4, plane_bytes = dh * 2;
    const unsigned char *rbase = resident + (int64_t)bh * S * row_bytes;
    const unsigned char *sbase = streamed + (int64_t)bh * S * row_bytes;
    const float *lse_h = PASS == 2 ? lse_in + (int64_t)bh * N : nullptr;
    const int32_t *sexp = str_exp + (int64_t)bh * nblk_exp;

    const int tid = threadIdx.x, lane = lane_id(), g = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(wave_id());
    f16x8_t kf[HALVES][2][NC];
    int rexp[HALVES];
#pragma unroll
    for (int h = 0; h < HALVES; ++h) {
        const int row = blk * RB + (w * HALVES + h) * 32 + (lane & 31);
        rexp[h] = res_exp[(int64_t)bh * nblk_exp +
                          min((blk * RB + (w * HALVES + h) * 32) / kPlaneBlock, nblk_exp - 1)];
#pragma unroll
        for (int pl = 0; pl < 2; ++pl)
#pragma unroll
            for (int c = 0; c < NC; ++c)
                kf[h][pl][c] = __builtin_bit_cast(
                    f16x8_t, load16_guard(rbase, (int64_t)(row_first + row) * row_bytes +
                                                     pl * plane_bytes + 32 * c + 16 * g,
                                          row < N && 32 * c + 16 * g < plane_bytes));
    }

    const int ntiles = (n_str + 31) >> 5;
    const int nstages = (n_str + ROWS - 1) / ROWS;

    // 16-byte column of a row where its piece lies (an involution)
    auto swizzle = [](int r, int piece) {
        if constexpr (NC & 1) return piece;
        if constexpr (PPR == 4) return piece ^ ((r >> 1) & 3);
        return piece ^ (r & (PPR - 1));
    };
    float lse_reg = 0.f;
    auto stage_load = [&](int s) {
        const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_byte_address(stage_buf(s)));
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int both = tid + it * 256, lo = both >= ROWS * PPR;
            const int p = both - (lo ? ROWS * PPR : 0);  // piece of the plane
            const int r = p / PPR, piece = swizzle(r, p - r * PPR);
            // clamped, not predicated: rows past the end re-read the last row and pieces past the
            // end of a row its last piece (finite data; masked, or against zeros of the resident
            // operand)
            const int row = matrix_row(min(s * ROWS + r, n_str - 1), N, row_first);
            const int64_t off = (int64_t)row * row_bytes + (lo ? plane_bytes : 0) +
                                min(piece * 16, plane_bytes - 16);
            direct_load16(sbase + off, __builtin_amdgcn_readfirstlane(
                                           lds0 + 16 * (it * 256 + w * kWave)));
        }
        if (PASS == 2 && tid < ROWS) lse_reg = lse_h[min(s * ROWS + tid, n_str - 1)];
    };
    auto stage_store = [&](int s) {
        wait_direct_loads();  // this wave's share of the stage is in LDS
        if (PASS == 2 && tid < ROWS)
            neg_lse[s % 3 * ROWS + tid] = s * ROWS + tid < n_str ? -lse_reg : -INFINITY;
    };

    f16x8_t fr[2][NC];  // streamed operand of one tile, refilled in place
    f32x16_t acc[2][HALVES];
    auto read_frag = [&](int t, int pl, int c) {
        const int r = t % ST * 32 + (lane & 31);
        return *reinterpret_cast<const f16x8_t *>(stage_buf(t / ST) + pl * PLANE + r * (NC * 32) +
                                                  swizzle(r, 2 * c + g) * 16);
    };
    const f32x16_t zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                           0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // The small products of all chunks go first, while the accumulator is small.
    // Product i of chunk c: lo_k hi_q, hi_k lo_q, hi_k hi_q.  Both passes add in this order, whichever
    // side streams: a logit has the same bits in both, so its rounding leaves the large weights
    // (2^(s - lse) with lse close to s) alone.
    constexpr int kLo = PASS == 1 ? 0 : 1;  // the product that takes the streamed lo plane
    auto multiply = [&](f32x16_t(&to)[HALVES], int c, int i, int h) {
        to[h] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fr[i == kLo ? 1 : 0][c],
                                                       kf[h][i == 1 - kLo ? 1 : 0][c],
                                                       c == 0 && i == 0 ? zero : to[h], 0, 0, 0);
    };

    float m_run[HALVES], l_run[HALVES], colsum[HALVES];
    float sc[HALVES];  // logit in units of log2 per unit of the accumulator, this stage
    bool have_ref[HALVES];
#pragma unroll
    for (int h = 0; h < HALVES; ++h) {
        m_run[h] = -INFINITY;
        l_run[h] = 0.f;
        colsum[h] = 0.f;
        have_ref[h] = false;
    }
    int next_exp = sexp[0];
    auto enter_stage = [&](int s) {
#pragma unroll
        for (int h = 0; h < HALVES; ++h) sc[h] = ldexpf(sl2, -(rexp[h] + next_exp));
        next_exp = sexp[min(s + 1, nstages - 1) * ROWS / kPlaneBlock];
    };

    // One pipeline step: the vector work of tile t (accumulators `cur`), between it the matrix
    // instructions of tile t + 1 (MULT) and the operand reads of tile t + 2 (REFILL).  MASK: tile t
    // is the ragged last tile of pass 1.
    auto step = [&](int t, f32x16_t(&cur)[HALVES], f32x16_t(&nxt)[HALVES], auto mult_tag,
                    auto refill_tag, auto mask_tag) {
        constexpr bool MULT = decltype(mult_tag)::value, REFILL = decltype(refill_tag)::value,
                       MASK = decltype(mask_tag)::value;
        float ref[HALVES], part[HALVES], nl[16];
        if constexpr (PASS == 1) {
            if constexpr (MASK) {
#pragma unroll
                for (int h = 0; h < HALVES; ++h)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (t * 32 + acc_row(r) >= n_str) cur[h][r] = -INFINITY;
            }
            // Lazy reference: exponentials are taken against an actual logit of the row (so the
            // sum is >= 1), raised only when the partial sum threatens to overflow.
#pragma unroll
            for (int h = 0; h < HALVES; ++h) {
                if (!have_ref[h]) {
                    float mx = -INFINITY;
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, cur[h][r]);
                    if (mx > -INFINITY) {
                        m_run[h] = mx * sc[h];
                        have_ref[h] = true;
                    }
                }
                ref[h] = have_ref[h] ? m_run[h] : 0.f;
            }
        } else {
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const float4 l4 = *reinterpret_cast<const float4 *>(
                    neg_lse + t / ST % 3 * ROWS + t % ST * 32 + 8 * rg + 4 * g);
                nl[4 * rg] = l4.x;
                nl[4 * rg + 1] = l4.y;
                nl[4 * rg + 2] = l4.z;
                nl[4 * rg + 3] = l4.w;
            }
        }
#pragma unroll
        for (int h = 0; h < HALVES; ++h) part[h] = 0.f;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            if constexpr (MULT) {
                const int n = m / HALVES, h = m % HALVES;
                const int i = n < 2 * NC ? n & 1 : 2, c = n < 2 * NC ? n >> 1 : n - 2 * NC;
                multiply(nxt, c, i, h);
                if constexpr (REFILL) {
                    if (h == HALVES - 1 && i == kLo) fr[1][c] = read_frag(t + 2, 1, c);
                    if (h == HALVES - 1 && i == 2) fr[0][c] = read_frag(t + 2, 0, c);
                }
            }
#pragma unroll
            for (int i = m * NL / NM; i < (m + 1) * NL / NM; ++i) {
                const int h = i / 16, r = i % 16;
                part[h] += __builtin_amdgcn_exp2f(
                    fmaf(cur[h][r], sc[h], PASS == 1 ? -ref[h] : nl[r]));
            }
        }
#pragma unroll
        for (int h = 0; h < HALVES; ++h) {
            if constexpr (PASS == 2) {
                colsum[h] += part[h];
            } else {
                if (part[h] < 0x1p100f) {
                    l_run[h] += part[h];
                } else {  // a logit far above the reference: re-base on this tile's maximum
                    float mx = -INFINITY;
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, cur[h][r]);
                    const float m_new = fmaxf(m_run[h], mx * sc[h]);
                    float add = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        add += __builtin_amdgcn_exp2f(fmaf(cur[h][r], sc[h], -m_new));
                    l_run[h] = l_run[h] * __builtin_amdgcn_exp2f(m_run[h] - m_new) + add;
                    m_run[h] = m_new;
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);  // keep the steps apart
    };
    using yes = std::integral_constant<bool, true>;
    using no = std::integral_constant<bool, false>;

    // ---- prologue: stage 0 in LDS, stage 1 in flight, tile 0 multiplied, tile 1's operands read
    stage_load(0);
    stage_store(0);
    __syncthreads();
    if (nstages > 1) stage_load(1);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        fr[0][c] = read_frag(0, 0, c);
        fr[1][c] = read_frag(0, 1, c);
    }
#pragma unroll
    for (int n = 0; n < 3 * NC; ++n)
#pragma unroll
        for (int h = 0; h < HALVES; ++h)
            multiply(acc[0], n < 2 * NC ? n >> 1 : n - 2 * NC, n < 2 * NC ? n & 1 : 2, h);
    if (ntiles > 1) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            fr[0][c] = read_frag(1, 0, c);
            fr[1][c] = read_frag(1, 1, c);
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    const bool ragged = PASS == 1 && (n_str & 31) != 0;
    int t0 = 0;
    // steady state, one stage per trip: every step has a tile t + 2 to fetch operands for
    for (; t0 + ST + 2 <= ntiles; t0 += ST) {
        enter_stage(t0 / ST);
#pragma unroll
        for (int j = 0; j < ST; ++j) {
            if (j == ST - 2) {  // tile t + 2 is the next stage's first
                const int s = t0 / ST;
                stage_store(s + 1);
                __syncthreads();
                if (s + 2 < nstages) stage_load(s + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            step(t0 + j, acc[j & 1], acc[(j + 1) & 1], yes{}, yes{}, no{});
        }
    }
    for (; t0 < ntiles; t0 += ST) {
        enter_stage(t0 / ST);
#pragma unroll
        for (int j = 0; j < ST; ++j) {
            const int t = t0 + j;
            if (t < ntiles) {
                if (j == ST - 2) {
                    const int s = t0 / ST;
                    if (s + 1 < nstages) {
                        stage_store(s + 1);
                        __syncthreads();
                        if (s + 2 < nstages) stage_load(s + 2);
                    }
                }
                if (t + 2 < ntiles) {
                    step(t, acc[j & 1], acc[(j + 1) & 1], yes{}, yes{}, no{});
                } else if (t + 1 < ntiles) {
                    step(t, acc[j & 1], acc[(j + 1) & 1], yes{}, no{}, no{});
                } else if (ragged) {
                    step(t, acc[j & 1], acc[(j + 1) & 1], no{}, no{}, yes{});
                } else {
                    step(t, acc[j & 1], acc[(j + 1) & 1], no{}, no{}, no{});
                }
            }
        }
    }

    // the two half-waves hold disjoint streamed rows of the same resident row
#pragma unroll
    for (int h = 0; h < HALVES; ++h) {
        const int row = blk * RB + (w * HALVES + h) * 32 + (lane & 31);
        if constexpr (PASS == 1) {
            const float m_o = __shfl_xor(m_run[h], 32, kWave), l_o = __shfl_xor(l_run[h], 32, kWave);
            const float M = fmaxf(m_run[h], m_o);
            float L = 0.f;
            if (m_run[h] > -INFINITY) L += l_run[h] * __builtin_amdgcn_exp2f(m_run[h] - M);
            if (m_o > -INFINITY) L += l_o * __builtin_amdgcn_exp2f(m_o - M);
            if (g == 0 && row < N) out[(int64_t)bh * N + row] = M + log2f(L);
        } else {
            const float c = colsum[h] + __shfl_xor(colsum[h], 32, kWave);
            if (g == 0 && row < N) out[(int64_t)bh * N + row] = c;
        }
    }
}

template <int NC, int HALVES, int PASS>
hipError_t launch_pass(const ScoreArgs &a, hipStream_t s) {
    constexpr int ST = 2, RB = 4 * 32 * HALVES;
    constexpr int lds = planes_lds_bytes<NC, ST>();
    if constexpr (lds > 64 * 1024) {
        static std::atomic<uint64_t> lds_allowed{0};
        hipError_t e = allow_large_lds(mean_planes_kernel<NC, HALVES, PASS, ST>, lds_allowed);
        if (e != hipSuccess) return e;
    }
    const int BH = a.BC * a.H, nblk_exp = (a.N + a.has_cls + kPlaneBlock - 1) / kPlaneBlock;
    const int total = BH * ((a.N + RB - 1) / RB);
    const unsigned char *q = reinterpret_cast<const unsigned char *>(a.q_planes);
    const unsigned char *k = reinterpret_cast<const unsigned char *>(a.k_planes);
    const int32_t *qe = a.plane_exps, *ke = a.plane_exps + (int64_t)BH * nblk_exp;
    const float sl2 = a.scale * 1.4426950408889634f;
    // pass 1: resident queries, streamed keys of the softmax domain (patch keys, then [CLS]);
    // pass 2: resident patch keys, streamed queries with their lse
    const int n_str = PASS == 1 && a.domain_all ? a.N + a.has_cls : a.N;
    hipLaunchKernelGGL((mean_planes_kernel<NC, HALVES, PASS, ST>), dim3((total + 7) / 8 * 8), dim3(256),
                       lds, s, PASS == 1 ? q : k, PASS == 1 ? k : q, PASS == 1 ? qe : ke,
                       PASS == 1 ? ke : qe, PASS == 1 ? nullptr : a.lse,
                       PASS == 1 ? a.lse : a.head_scores, BH, nblk_exp, a.S, a.dh, a.has_cls, a.N,
                       n_str, sl2);
    return hipGetLastError();
}

template <int NC>
hipError_t launch_pass_nc(const ScoreArgs &a, hipStream_t s, int pass) {
    // 64 resident rows per wave serve twice the matrix instructions per operand read, 32 make
    // twice the workgroups.  Where every CU has several of the larger ones the reads decide (6400
    // tokens, 16 heads of 80: 336 + 316 us against 359 + 346); where there is at most one, the
    // second workgroup on some CUs pays for itself (2688 tokens: 83 + 70 us against 76 + 71).
    // (Rows of 256 bytes a plane leave registers for 32 only.)
    if constexpr (NC <= 5) {
        const int64_t heads = (int64_t)a.BC * a.H;
        const int64_t two = (heads * ((a.N + 255) / 256) + kCus - 1) / kCus;
        const int64_t one = (heads * ((a.N + 127) / 128) + kCus - 1) / kCus;
        if (2 * two <= one && two > 1)
            return pass == 1 ? launch_pass<NC, 2, 1>(a, s) : launch_pass<NC, 2, 2>(a, s);
    }
    return pass == 1 ? launch_pass<NC, 1, 1>(a, s) : launch_pass<NC, 1, 2>(a, s);
}

template <int NI>
hipError_t launch_planes(const ScoreArgs &a, hipStream_t s) {
    const int n_rows = a.N + a.has_cls, nblk = (n_rows + kPlaneBlock - 1) / kPlaneBlock;
    hipLaunchKernelGGL(planes_kernel<NI>, dim3(a.BC * a.H * nblk, 2), dim3(256), 0, s,
                       (const float *)a.q, (const float *)a.k, (unsigned char *)a.q_planes,
                       (unsigned char *)a.k_planes, a.plane_exps, a.BC * a.H, nblk, a.S, a.dh,
                       a.has_cls, a.N, n_rows);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_mean_planes(const ScoreArgs &a, hipStream_t s, int pass) {
    if (pass == 1) {
        const hipError_t e = a.dh <= 32   ? launch_planes<4>(a, s)
                             : a.dh <= 64 ? launch_planes<8>(a, s)
                             : a.dh <= 80 ? launch_planes<10>(a, s)
                                          : launch_planes<16>(a, s);
        if (e != hipSuccess) return e;
    }
    if (a.dh <= 32) return launch_pass_nc<2>(a, s, pass);
    if (a.dh <= 64) return launch_pass_nc<4>(a, s, pass);
    if (a.dh <= 80) return launch_pass_nc<5>(a, s, pass);
    if (a.dh <= 128) return launch_pass_nc<8>(a, s, pass);
    return hipErrorInvalidValue;  // 512-byte rows are the limit of fp32 mean mode
}

}  // namespace vscan
