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

// Ragged batch: replace the lengths in the (by-value) argument block by those of sequence b.
// Returns the kept-index row of the sequence.
__device__ __forceinline__ const int32_t *sequence_view(CompactArgs &a, int b) {
    const int32_t *kept_b = a.kept_idx + (int64_t)b * a.keep;  // a.keep is still the stride here
    if (a.meta) {
        const SeqMeta m = a.meta[b];
        a.S = m.seq_len;
        a.vis_start = m.vis_start;
        a.V = m.vis_len;
        a.keep = m.keep;
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
// No workgroup waits for one that has not started: the workgroup that selects for a sequence
// is whoever claims it first (`claim`, one atomic exchange), normally the one launched for it; a
// gathering workgroup that finds its sequence unclaimed makes the selection itself.  A selection
// waits for nobody and writes all of its sequence's indices, whatever the scores are.
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
    for (int64_t i = first; i < s.n_claim; i += step) s.claim[i] = 0u;
}
// whether this workgroup selects for sequence b; one that is here to gather (`patient`) leaves the
// workgroup launched for it a few microseconds to start
__device__ __forceinline__ bool claim_selection(uint32_t *claim, int b, bool patient, int *lds) {
    if (threadIdx.x == 0) {
        auto taken = [&]() {
            return __hip_atomic_load(claim + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
        };
        bool gone = false;
        for (int i = 0; patient && i < 8 && !gone; ++i) {
            gone = taken();
            if (!gone) __builtin_amdgcn_s_sleep(8);
        }
        *lds = !gone &&
               __hip_atomic_exchange(claim + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u;
    }
    __syncthreads();
    return *lds != 0;
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

// sequence of a kept unit
__device__ __forceinline__ int kept_unit_sequence(const CompactArgs &a, const CopyUnits &u, int id) {
    return decode_strip(a, id % u.strips).b;
}

template <int NT>
__device__ __forceinline__ void copy_kept_rows(CompactArgs a, const CopyUnits &u, int id) {
    constexpr int RPT = kCompactTile * 16 / NT;  // rows per thread
    static_assert(RPT >= 1 && NT * RPT == kCompactTile * 16, "sixteen threads span a strip");
    const Strip s = decode_strip(a, id % u.strips);
    const int tile = id / u.strips;
    const int32_t *kept_b = sequence_view(a, s.b);
    const int piece = threadIdx.x & 15, row0 = tile * kCompactTile + (threadIdx.x >> 4);
    if (tile * kCompactTile >= a.keep) return;
    // one thread waits for the tile's last index first: a thousand workgroups that poll with
    // every thread are traffic the selection has to get through
    if (threadIdx.x == 0) {
        const int32_t *last = kept_b + min((tile + 1) * kCompactTile, a.keep) - 1;
        while (device_load(last) == kNotYetKept) __builtin_amdgcn_s_sleep(16);
    }
    __syncthreads();
    if (piece * 16 >= s.width) return;
    int kv[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i)  // clamped positions: the loads are in flight together
        kv[i] = device_load(kept_b + min(row0 + i * (NT / 16), a.keep - 1));
    for (;;) {
        bool wait = false;
#pragma unroll
        for (int i = 0; i < RPT; ++i) wait |= kv[i] == kNotYetKept;
        if (!wait) break;
        __builtin_amdgcn_s_sleep(8);
#pragma unroll
        for (int i = 0; i < RPT; ++i)
            kv[i] = device_load(kept_b + min(row0 + i * (NT / 16), a.keep - 1));
    }
    uint4 v[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        // clamped: the index comes from device memory
        const int src = a.vis_start + min(max(kv[i], 0), a.V - 1);
        v[i] = load16(s.src, (int64_t)src * s.src_stride + piece * 16);
    }
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int r = row0 + i * (NT / 16);
        if (r < a.keep)
            store16_stream(s.dst + (int64_t)(a.vis_start + r) * s.dst_stride + piece * 16, v[i]);
    }
}

}  // namespace vscan
