// Calls the stage-2 selection launcher of the built library directly, for
// tests/test_gpu_select_wait.py: the public entry points do not let a caller choose how long a
// gathering workgroup waits.  Host code only.
#include "../paper_2505_22654_amd/csrc/launch.hpp"

extern "C" int vscan_test_select_compact(const int *dims, int polls, const float *part, const int *meta,
                                         int *kept, float *scores, void *const *src, void *const *dst,
                                         void *stream) {
    using namespace vscan;
    // dims: B, Hkv, S, dh, Dh, vis_start, V, keep, elem_bytes
    CompactArgs ca{};
    ca.k = src[0], ca.v = src[1], ca.hidden = src[2];
    ca.k_out = dst[0], ca.v_out = dst[1], ca.hidden_out = dst[2];
    ca.kept_idx = kept;
    ca.B = dims[0], ca.Hkv = dims[1], ca.S = dims[2], ca.dh = dims[3], ca.Dh = dims[4];
    ca.vis_start = dims[5], ca.V = dims[6], ca.keep = dims[7], ca.elem_bytes = dims[8];
    ca.max_static_rows = ca.S - ca.V;
    ca.out_rows = ca.S - ca.V + ca.keep;
    ca.meta = reinterpret_cast<const SeqMeta *>(meta);
    LlmSelectArgs a{};
    a.part = part;
    a.B = ca.B, a.Hkv = ca.Hkv, a.V = ca.V, a.keep = ca.keep;
    a.norm = 1.0f;
    a.kept_idx = kept;
    a.scores_out = scores;
    a.meta = ca.meta;
    a.copy = &ca;
    if (polls >= 0) a.polls = polls;
    return (int)launch_llm_select(a, static_cast<hipStream_t>(stream));
}
