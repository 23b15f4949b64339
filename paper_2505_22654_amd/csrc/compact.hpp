// Compaction ("Remarks on KV Cache"): where rows come from and go to, and the device code of the
// out-of-place form, which runs inside the stage-2 selection launch.
#pragma once
#include "common.hpp"
#include "launch.hpp"

namespace vscan {

// ---------------------------------------------------------------------------
// Compaction.  New row p of a sequence comes from old row
//   p                          p <  vis_start
//   vis_start + kept[p - vs]   p <  vis_start + keep
//   p + (V - keep)             otherwise
// so sources never lie below destinations.  A "strip" is up to 256 bytes of one
// row of one slab (K or V: one (sequence, kv head); hidden: one sequence).
// ---------------------------------------------------------------------------
struct Strip {
    unsigned char *src, *dst;  // first byte of row 0 of the strip
    int64_t src_stride, dst_stride;
    int width;                 // bytes, multiple of 16, <= 256
    int b;
};

// slab bases only: valid before the per-sequence lengths of a ragged batch are known
__device__ __forceinline__ Strip decode_strip(const CompactArgs &a, int id) {
    const int kv_w = a.dh * a.elem_bytes, hid_w = a.Dh * a.elem_bytes;
    const int kv_strips = (kv_w + 255) / 256, hid_strips = (hid_w + 255) / 256;
    const int n_kv = a.B * a.Hkv * kv_strips;
    Strip s;
    if (id < 2 * n_kv) {
        const bool is_v = id >= n_kv;
        const int r = is_v ? id - n_kv : id;
        const int slab = r / kv_strips, strip = r - slab * kv_strips;
        unsigned char *in = reinterpret_cast<unsigned char *>(is_v ? a.v : a.k);
        unsigned char *out = reinterpret_cast<unsigned char *>(is_v ? a.v_out : a.k_out);
        s.b = slab / a.Hkv;
        s.src_stride = kv_w;
        s.dst_stride = kv_w;
        s.src = in + (int64_t)slab * a.S * kv_w + strip * 256;
        s.dst = a.in_place ? s.src : out + (int64_t)slab * a.out_rows * kv_w + strip * 256;
        s.width = min(256, kv_w - strip * 256);
    } else {
        const int r = id - 2 * n_kv;
        const int b = r / hid_strips, strip = r - b * hid_strips;
        unsigned char *in = reinterpret_cast<unsigned char *>(a.hidden);
        unsigned char *out = reinterpret_cast<unsigned char *>(a.hidden_out);
        s.b = b;
        s.src_stride = hid_w;
        s.dst_stride = hid_w;
        s.src = in + (int64_t)b * a.S * hid_w + strip * 256;
        s.dst = a.in_place ? s.src : out + (int64_t)b * a.out_rows * hid_w + strip * 256;
        s.width = min(256, hid_w - strip * 256);
    }
    return s;
}

inline int compact_strips(const CompactArgs &a) {
    const int kv_strips = (a.dh * a.elem_bytes + 255) / 256;
    const int hid_strips = (a.Dh * a.elem_bytes + 255) / 256;
    return 2 * a.B * a.Hkv * kv_strips + a.B * hid_strips;
}
constexpr int kCompactTile = 128;  // rows of a strip that are moved together

// Visual and kept tokens of a sequence of a ragged batch.  The table is device memory, and what the
// host validated is its copy: the counts stay inside the capacities, and no more is kept than there
// is, so that the selection writes every index that a copy waits for.
struct SpanCounts {
    int V, keep;
};
__device__ __forceinline__ SpanCounts span_counts(const SeqMeta &m, int V_cap, int keep_cap) {
    SpanCounts c;
    c.V = min(max(m.vis_len, 1), V_cap);
    c.keep = min(max(m.keep, 0), min(c.V, keep_cap));
    return c;
}

// Ragged batch: replace the lengths in the (by-value) argument block by those of sequence b.
// Returns the kept-index row of the sequence.
__device__ __forceinline__ const int32_t *sequence_view(CompactArgs &a, int b) {
    const int32_t *kept_b = a.kept_idx + (int64_t)b * a.keep;  // a.keep is still the stride here
    if (a.meta) {
        const SeqMeta m = a.meta[b];
        const SpanCounts c = span_counts(m, a.V, a.keep);  // (both are still the capacities)
        a.S = m.seq_len;
        a.vis_start = m.vis_start;
        a.V = c.V;
        a.keep = c.keep;
    }
    return kept_b;
}

// ---------------------------------------------------------------------------
// Out of place, one launch does the selection and the copies.  The selection is bound by latency
// (a workgroup per sequence, the rest of the chip idle for 5-20 us), the copies by memory, and
// every boundary between launches drains the chip (3 us).  Workgroups in launch order:
//   selection   one per sequence
//   static rows the rows before the visual span and after it go to places known beforehand:
//               byte o of "all rows of a slab but the visual ones" comes from o, or o + V rows
//               once it lies past the prefix, and goes to o, or o + keep rows.  (A slab is one
//               (sequence, kv head) of K or V, or one sequence of the hidden states; where a
//               ragged result is to end in zero rows, they simply continue that range.)
//   kept rows   a gather of kCompactTile rows of one strip, for which the kept indices have to
//               be there: a thread re-reads its entries until none is kNotYetKept
// Kept indices are written and polled with device-scope accesses, which pass the L2s of the eight
// XCDs; an index is its own flag, so no ordering between memory operations is relied upon.
// A gathering workgroup waits a bounded time; then it makes its sequence's selection itself.  A
// selection waits for nobody, writes all of its sequence's indices whatever the scores are, and
// writes the same ones whoever makes it, so every workgroup ends, in whatever order they start and
// whatever else writes to the kept indices meanwhile.
// Measured (kernel durations): 16 sequences of 192 visual tokens, hidden 4096: 5.7 + 28.8 us for
// selection and compaction as two launches, 27.2 us as one (154 MB: 5.7 TB/s); 12 ragged
// sequences of up to 1500 tokens: 10.6 + 25.6 us and 30 us of fills -> 39 us with the zero rows.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int32_t device_load(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void device_store(int32_t *p, int32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// part of the kernel before the selection launch: workgroup `wg` of `nwg`
__device__ __forceinline__ void seed_selection(const SelectSeed &s, int wg, int nwg) {
    const int64_t first = (int64_t)wg * blockDim.x + threadIdx.x, step = (int64_t)nwg * blockDim.x;
    for (int64_t i = first; i < s.n_kept; i += step) s.kept[i] = kNotYetKept;
}
constexpr int kCopyPieces = 4;  // 16-byte pieces per thread of a static unit

struct CopyUnits {
    int per_kv, per_hidden;  // static units per slab of K or V, and of the hidden states
    int n_static, n_kept;    // units in all: static rows, kept rows
    int strips;
};
inline CopyUnits copy_units(const CompactArgs &a, int threads) {
    const int64_t unit = (int64_t)threads * 16 * kCopyPieces;
    const int64_t kv = (int64_t)a.max_static_rows * a.dh * a.elem_bytes;
    const int64_t hid = (int64_t)a.max_static_rows * a.Dh * a.elem_bytes;
    CopyUnits u;
    u.per_kv = (int)((kv + unit - 1) / unit);
    u.per_hidden = (int)((hid + unit - 1) / unit);
    u.n_static = 2 * a.B * a.Hkv * u.per_kv + a.B * u.per_hidden;
    u.strips = compact_strips(a);
    u.n_kept = u.strips * ((a.keep + kCompactTile - 1) / kCompactTile);
    return u;
}

__device__ __forceinline__ void copy_static_rows(CompactArgs a, const CopyUnits &u, int id) {
    const int n_kv = a.B * a.Hkv * u.per_kv;
    const unsigned char *src;
    unsigned char *dst;
    int64_t row_bytes;
    int unit, b;
    if (id < 2 * n_kv) {
        const bool is_v = id >= n_kv;
        const int r = is_v ? id - n_kv : id, slab = r / u.per_kv;
        unit = r - slab * u.per_kv;
        b = slab / a.Hkv;
        row_bytes = (int64_t)a.dh * a.elem_bytes;
        src = reinterpret_cast<const unsigned char *>(is_v ? a.v : a.k) + (int64_t)slab * a.S * row_bytes;
        dst = reinterpret_cast<unsigned char *>(is_v ? a.v_out : a.k_out) +
              (int64_t)slab * a.out_rows * row_bytes;
    } else {
        const int r = id - 2 * n_kv;
        b = r / u.per_hidden;
        unit = r - b * u.per_hidden;
        row_bytes = (int64_t)a.Dh * a.elem_bytes;
        src = reinterpret_cast<const unsigned char *>(a.hidden) + (int64_t)b * a.S * row_bytes;
        dst = reinterpret_cast<unsigned char *>(a.hidden_out) + (int64_t)b * a.out_rows * row_bytes;
    }
    sequence_view(a, b);
    const int64_t prefix = a.vis_start * row_bytes, rows = (a.S - a.V) * row_bytes;  // rows > 0
    const int64_t end = a.zero_tail ? (a.out_rows - a.keep) * row_bytes : rows;
    const int64_t skip = a.V * row_bytes, shift = a.keep * row_bytes;
    const int64_t o0 = ((int64_t)unit * kCopyPieces * blockDim.x + threadIdx.x) * 16;
    const int64_t step = (int64_t)blockDim.x * 16;
    if (o0 >= end) return;
    uint4 v[kCopyPieces];
    if (o0 < rows) {
#pragma unroll
        for (int i = 0; i < kCopyPieces; ++i) {  // clamped, not predicated: all in flight together
            const int64_t o = min(o0 + i * step, rows - 16);
            v[i] = load16(src, o < prefix ? o : o + skip);
        }
    }
#pragma unroll
    for (int i = 0; i < kCopyPieces; ++i) {
        const int64_t o = o0 + i * step;
        if (o < end)
            store16_stream(dst + (o < prefix ? o : o + shift), o < rows ? v[i] : zero16());
    }
}

// A kept unit: positions first .. last of the kept rows of one strip.
struct KeptUnit {
    Strip s;
    const int32_t *kept_b;
    int first, last, vis_start, V;
};
// false: the sequence keeps no row of that tile
__device__ __forceinline__ bool kept_unit(CompactArgs a, const CopyUnits &u, int id, KeptUnit *k) {
    k->s = decode_strip(a, id % u.strips);
    k->kept_b = sequence_view(a, k->s.b);
    k->first = id / u.strips * kCompactTile;
    k->last = min(k->first + kCompactTile, a.keep) - 1;
    k->vis_start = a.vis_start;
    k->V = a.V;
    return k->first < a.keep;
}

// sixteen threads span a strip; a thread's rows of the unit
template <int NT>
struct KeptRows {
    static constexpr int RPT = kCompactTile * 16 / NT;
    static_assert(RPT >= 1 && NT * RPT == kCompactTile * 16, "sixteen threads span a strip");
    int kv[RPT];
    // true: all of them are there
    __device__ __forceinline__ bool load(const KeptUnit &u) {
#pragma unroll
        for (int i = 0; i < RPT; ++i)  // clamped positions: the loads are in flight together
            kv[i] = device_load(u.kept_b + min(u.first + (int)(threadIdx.x >> 4) + i * (NT / 16), u.last));
        bool there = true;
#pragma unroll
        for (int i = 0; i < RPT; ++i) there &= kv[i] != kNotYetKept;
        return there;
    }
};

// Waits for the unit's indices, `polls` looks at the last one at most: whether they are there (for
// every thread of the workgroup alike).  `lds`: two free words, free again after a barrier.
template <int NT>
__device__ __forceinline__ bool wait_kept_rows(const KeptUnit &u, KeptRows<NT> &rows, int polls, int *lds) {
    // one thread waits for the tile's last index first: a thousand workgroups that poll with
    // every thread are traffic the selection has to get through
    if (threadIdx.x == 0) {
        int left = polls;
        while (left > 0 && device_load(u.kept_b + u.last) == kNotYetKept) {
            __builtin_amdgcn_s_sleep(16);
            --left;
        }
        lds[0] = left;
        lds[1] = 0;
    }
    __syncthreads();
    const int left = lds[0];
    if (left <= 0) return false;
    bool there = rows.load(u);
    for (int i = 0; i < left && !there; ++i) {  // the tile's other indices may be under way still
        __builtin_amdgcn_s_sleep(8);
        there = rows.load(u);
    }
    if (!there) lds[1] = 1;
    __syncthreads();
    return lds[1] == 0;
}

template <int NT>
__device__ __forceinline__ void copy_kept_rows(const KeptUnit &u, const KeptRows<NT> &rows) {
    constexpr int RPT = KeptRows<NT>::RPT;
    const int piece = threadIdx.x & 15, row0 = u.first + (threadIdx.x >> 4);
    if (piece * 16 >= u.s.width) return;
    uint4 v[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        // clamped: the index comes from device memory
        const int src = u.vis_start + min(max(rows.kv[i], 0), u.V - 1);
        v[i] = load16(u.s.src, (int64_t)src * u.s.src_stride + piece * 16);
    }
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int r = row0 + i * (NT / 16);
        if (r <= u.last)
            store16_stream(u.s.dst + (int64_t)(u.vis_start + r) * u.s.dst_stride + piece * 16, v[i]);
    }
}

}  // namespace vscan
