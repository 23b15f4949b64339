// Stand-ins for the kernel launchers, for a CPU-only build of the host layer (api.cpp,
// budget.cpp) under AddressSanitizer and UndefinedBehaviorSanitizer.  Nothing here launches or
// dereferences anything.  Each stand-in checks what the host layer hands to a launcher: every
// scratch region (start and extent, worked out from the dimensions in the argument struct) must
// lie inside the workspace window the test announced, 16-byte aligned, and the regions of one
// call must not overlap.  The test reads the tally through vscan_test_report.
#include <stdint.h>
#include <stdio.h>

#include <algorithm>
#include <utility>
#include <vector>

#include "../include/vscan.h"
#include "../paper_2505_22654_amd/csrc/fused.hpp"
#include "../paper_2505_22654_amd/csrc/launch.hpp"

namespace {
uintptr_t g_lo = 0, g_hi = 0;
int g_calls = 0, g_regions = 0, g_violations = 0;
vscan::SelectSeed g_seed;  // what the last scoring launch was asked to prepare
std::vector<std::pair<const void *, size_t>> g_lse;  // statistics left by the first pass of mean attention
int g_parted = 0, g_joined = 0, g_chunked = 0;       // second passes in parts, for both pairs; ragged chunks

void region(const char *who, const char *what, const void *p, size_t bytes) {
    ++g_regions;
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    if (!p || (a & 15u) || a < g_lo || a + bytes > g_hi || a + bytes < a) {
        ++g_violations;
        fprintf(stderr, "host_stubs: %s: %s [%p, +%zu) outside the window or unaligned\n", who, what,
                p, bytes);
    }
}
// regions that must be distinct from one another within a call
void distinct(const char *who, std::vector<std::pair<const void *, size_t>> rs) {
    std::vector<std::pair<uintptr_t, uintptr_t>> v;
    for (auto &r : rs)
        if (r.first && r.second) v.push_back({(uintptr_t)r.first, (uintptr_t)r.first + r.second});
    std::sort(v.begin(), v.end());
    for (size_t i = 1; i < v.size(); ++i)
        if (v[i].first < v[i - 1].second) {
            ++g_violations;
            fprintf(stderr, "host_stubs: %s: scratch regions overlap\n", who);
        }
}
void expect(const char *who, const char *what, bool ok) {
    if (ok) return;
    ++g_violations;
    fprintf(stderr, "host_stubs: %s: %s\n", who, what);
}
}  // namespace

extern "C" void vscan_test_window(const void *lo, size_t bytes) {
    g_seed = {};
    g_lse.clear();
    g_lo = reinterpret_cast<uintptr_t>(lo);
    g_hi = g_lo + bytes;
}
extern "C" void vscan_test_report(int *calls, int *regions, int *violations) {
    *calls = g_calls;
    *regions = g_regions;
    *violations = g_violations;
}
extern "C" void vscan_test_forms(int *parted, int *joined, int *chunked) {
    *parted = g_parted;
    *joined = g_joined;
    *chunked = g_chunked;
}

namespace vscan {

hipError_t launch_score_cls(const ScoreArgs &a, hipStream_t) {
    ++g_calls;
    expect("score_cls", "parts of a form without them", a.parts == 1);
    region("score_cls", "head_scores", a.head_scores, (size_t)a.BC * a.H * a.N * sizeof(float));
    return hipSuccess;
}

// Mean attention: scores of all parts of the streamed rows, and a row's statistics, of one pair or of both.
static size_t mean_scores_bytes(const ScoreArgs &a) { return (size_t)a.BC * a.H * a.parts * a.N * sizeof(float); }
static size_t mean_lse_bytes(const ScoreArgs &a) { return mean_scores_bytes(a) * (a.parts > 1 ? 2 : 1); }
static void check_mean(const char *who, const ScoreArgs &a, bool both) {
    ++g_calls;
    const int stages = (a.N + kMeanStageRows - 1) / kMeanStageRows;
    expect(who, "more parts than stages or than the kernels add",
           a.parts >= 1 && a.parts <= kMeanMaxParts && a.parts <= stages);
    expect(who, "parts or two pairs in a form of one",
           a.pipelined || (a.parts == 1 && !both));
    if (both) expect(who, "second pair without rows", a.q2 && a.k2);
}
hipError_t launch_score_mean_lse(const ScoreArgs &a, hipStream_t) {
    const char *who = "score_mean_lse";
    check_mean(who, a, a.q2 != nullptr);
    expect(who, "statistics of the launch before not read", g_lse.empty());
    g_lse = {{a.lse, mean_lse_bytes(a)}};
    if (a.q2) g_lse.push_back({a.lse2, mean_lse_bytes(a)});
    for (const auto &r : g_lse) region(who, "lse", r.first, r.second);
    distinct(who, g_lse);
    return hipSuccess;
}
hipError_t launch_score_mean_colsum(const ScoreArgs &a, hipStream_t) {
    const char *who = "score_mean_colsum";
    const bool both = a.head_scores2 != nullptr;
    check_mean(who, a, both);
    std::vector<std::pair<const void *, size_t>> all = g_lse;  // read here or by the next launch
    auto one = [&](float *scores, float *lse) {
        region(who, "head_scores", scores, mean_scores_bytes(a));
        all.push_back({scores, mean_scores_bytes(a)});
        const auto mine = std::find(g_lse.begin(), g_lse.end(), std::pair<const void *, size_t>(lse, mean_lse_bytes(a)));
        expect(who, "statistics that the launch before did not leave", mine != g_lse.end());
        if (mine != g_lse.end()) g_lse.erase(mine);
    };
    one(a.head_scores, a.lse);
    if (both) one(a.head_scores2, a.lse2);
    distinct(who, all);
    g_joined += both;
    g_parted += a.parts > 1;
    return hipSuccess;
}

hipError_t launch_encoder_select(const EncSelectArgs &a, hipStream_t) {
    ++g_calls;
    const size_t N = (size_t)a.gh * a.gw, BC = (size_t)a.B * a.C;
    const size_t K = (size_t)a.C * ((size_t)a.wr * a.wc * a.kw + a.kg);
    const size_t head = BC * a.H * N * sizeof(float);
    region("encoder_select", "head_global", a.head_global, head);
    if (a.head_local) region("encoder_select", "head_local", a.head_local, head);
    region("encoder_select", "drop_idx", a.drop_idx, (size_t)a.B * (a.C * N - K) * 4);
    region("encoder_select", "best", a.best, BC * N * 8);
    region("encoder_select", "pre_key", a.pre_key_ws, BC * N * 4);
    region("encoder_select", "pre_flag", a.pre_flag_ws, BC * N);
    distinct("encoder_select", {{a.head_global, head},
                                {a.head_local, head},
                                {a.drop_idx, (size_t)a.B * (a.C * N - K) * 4},
                                {a.best, BC * N * 8},
                                {a.pre_key_ws, BC * N * 4},
                                {a.pre_flag_ws, BC * N}});
    return hipSuccess;
}
size_t encoder_select_lds_bytes(int N, int has_local) {
    return 1024 + (size_t)N * 4 * (has_local ? 2 : 1) + (size_t)N;
}

static void check_merge(const char *who, const MergeArgs &a) {
    ++g_calls;
    const size_t U = (size_t)a.T - a.K;
    region(who, "drop_idx", a.drop_idx, (size_t)a.B * U * 4);
    region(who, "best", a.best, (size_t)a.B * a.T * 8);
    region(who, "inv_norm", a.inv_norm, (size_t)a.B * a.K * 4);
    distinct(who, {{a.drop_idx, (size_t)a.B * U * 4},
                   {a.best, (size_t)a.B * a.T * 8},
                   {a.inv_norm, (size_t)a.B * a.K * 4}});
}
hipError_t launch_sim_argmax(const MergeArgs &a, hipStream_t) {
    check_merge("sim_argmax", a);
    return hipSuccess;
}
hipError_t launch_merge(const MergeArgs &a, hipStream_t) {
    check_merge("merge", a);
    return hipSuccess;
}

int llm_score_split_chunks(int B, int Hkv, int rows, int nk) {
    if (rows > 16 || nk < 1024 || (int64_t)B * Hkv > 64) return 0;
    return (nk + 63) / 64;
}
bool llm_score_supported(int rows, int, int row_bytes) { return rows <= 64 && row_bytes <= 512; }
hipError_t launch_llm_score(const LlmScoreArgs &a, hipStream_t) {
    ++g_calls;
    const size_t items = (size_t)a.B * a.Hkv, rows = (size_t)(a.Hq / a.Hkv) * a.Tq;
    const size_t part = items * a.V * 4;
    region("llm_score", "part", a.part, part);
    const int nk = a.domain_all ? a.S : a.V;
    const int chunks = llm_score_split_chunks(a.B, a.Hkv, (int)rows, nk);
    if (chunks > 0) {
        const size_t e = items * rows * a.V * 4, st = items * chunks * rows * 2 * 4;
        region("llm_score", "split_e", a.split_e, e);
        region("llm_score", "split_stats", a.split_stats, st);
        distinct("llm_score", {{a.part, part}, {a.split_e, e}, {a.split_stats, st}});
        g_chunked += a.meta != nullptr;
    }
    g_seed = a.seed;
    return hipSuccess;
}
hipError_t launch_llm_select(const LlmSelectArgs &a, hipStream_t) {
    ++g_calls;
    region("llm_select", "part", a.part, (size_t)a.B * a.Hkv * a.V * 4);
    // out of place the indices are handed over inside the launch, and the scoring launch before it
    // must have been asked to prepare every one of them; in place none
    if (a.copy) {
        expect("llm_select", "indices not prepared",
               g_seed.kept == a.kept_idx && g_seed.n_kept == (int64_t)a.B * a.keep);
        expect("llm_select", "copies other indices",
               (a.keep == 0 || a.copy->kept_idx == a.kept_idx) && !a.copy->in_place);
        expect("llm_select", "copies another table", a.copy->meta == a.meta && a.copy->B == a.B);
        expect("llm_select", "does not wait", a.polls > 0);
    } else {
        expect("llm_select", "indices prepared in place", g_seed.n_kept == 0);
    }
    g_seed = {};
    return hipSuccess;
}
size_t llm_select_lds_bytes(int V) { return 1024 + (size_t)V * 5; }
hipError_t launch_compact(const CompactArgs &, hipStream_t) {
    ++g_calls;
    return hipSuccess;
}

int fused_ksplit(int, int, int, int k_elems, int) { return k_elems >= 512 ? 2 : 1; }
static hipError_t check_fused(const char *who, const FusedArgs &a) {
    ++g_calls;
    const size_t M = (size_t)a.B * a.Tq, N = (size_t)a.Hq * a.dh, R = (size_t)a.Hq * a.Tq;
    const size_t cq = (size_t)a.ks_q * M * N * 4, qp = a.is_bf16 ? 3 * M * N * 2 : M * N * 4;
    const size_t qt = (a.is_bf16 ? (size_t)kFusedQtPlanes * 2 : 4) * a.B * R * a.Dh;
    const size_t cl = (size_t)a.ks_l * a.B * R * a.nk * 4;
    region(who, "c_q", a.c_q, cq);
    region(who, "q_planes", a.q_planes, qp);
    region(who, "qt_planes", a.qt_planes, qt);
    region(who, "c_l", a.c_l, cl);
    region(who, "part", a.part, (size_t)a.B * a.V * 4);
    distinct(who, {{a.c_q, cq}, {a.q_planes, qp}, {a.qt_planes, qt}, {a.c_l, cl},
                   {a.part, (size_t)a.B * a.V * 4}});
    if (a.keep_rows)
        expect(who, "softmax rows of another length than the span", a.nk == a.V && !a.causal);
    return hipSuccess;
}
hipError_t launch_fused_project(const ProjectArgs &a, hipStream_t) {
    ++g_calls;
    const size_t out = (size_t)a.BC * a.H * a.S * a.dh * 4;
    const size_t w = (size_t)a.H * a.dh * a.Dh * (a.is_bf16 ? 2 : 4);
    region("fused_project", "out", a.out, out);
    region("fused_project", "out_k", a.out_k, out);
    region("fused_project", "w_k", a.w_k, w);  // transposed into the workspace by the launch before
    distinct("fused_project", {{a.out, out}, {a.out_k, out}, {a.w_k, w}});
    return hipSuccess;
}
hipError_t launch_transpose(const void *, void *out, int rows, int cols, int es, hipStream_t) {
    ++g_calls;
    region("fused_transpose", "out", out, (size_t)rows * cols * es);
    return hipSuccess;
}
hipError_t launch_fused_q(const FusedArgs &a, hipStream_t) { return check_fused("fused_q", a); }
hipError_t launch_fused_split_q(const FusedArgs &a, hipStream_t) { return check_fused("fused_split_q", a); }
hipError_t launch_fused_qt(const FusedArgs &a, hipStream_t) { return check_fused("fused_qt", a); }
hipError_t launch_fused_logits(const FusedArgs &a, hipStream_t) { return check_fused("fused_logits", a); }
hipError_t launch_fused_softmax(const FusedArgs &a, hipStream_t) {
    if (a.keep_rows) g_seed = a.seed;  // the last launch before the selection
    return check_fused("fused_softmax", a);
}
hipError_t launch_fused_colsum(const FusedArgs &a, hipStream_t) {
    expect("fused_colsum", "launched although the selection adds the rows", !a.keep_rows);
    g_seed = a.seed;
    return check_fused("fused_colsum", a);
}

// The padded ragged calls (api.cpp), with an upload that checks where the table goes: at the start
// of the window, and everything else behind it.
size_t ragged_table_bytes(int batch);
int llm_prune_ragged_padded(const vscan_llm_desc *d, const vscan_seq_meta *meta_host,
                            TableUpload upload, const void *q, void *k, void *v, void *hidden,
                            int32_t *kept_idx, void *k_out, void *v_out, void *hidden_out,
                            float *scores_out, void *workspace, size_t workspace_bytes, void *stream);
int llm_prune_fused_ragged_padded(const vscan_llm_desc *d, const vscan_seq_meta *meta_host,
                                  TableUpload upload, void *hidden, const void *w_q,
                                  const void *w_k_t, int32_t *kept_idx, void *hidden_out,
                                  float *scores_out, void *workspace, size_t workspace_bytes,
                                  void *stream);

}  // namespace vscan

static hipError_t checking_upload(vscan::SeqMeta *table, const vscan::SeqMeta *from_host, int batch,
                                  hipStream_t) {
    ++g_calls;
    region("table_upload", "table", table, (size_t)batch * sizeof(vscan::SeqMeta));
    expect("table_upload", "not at the start of the workspace", reinterpret_cast<uintptr_t>(table) == g_lo);
    expect("table_upload", "no host table", from_host != nullptr);
    g_lo += (size_t)batch * sizeof(vscan::SeqMeta);
    return hipSuccess;
}
extern "C" size_t vscan_test_table_bytes(int batch) { return vscan::ragged_table_bytes(batch); }
extern "C" int vscan_test_ragged_padded(const vscan_llm_desc *d, const vscan_seq_meta *meta, void *t,
                                        void *out, int from_hidden, void *ws, size_t bytes) {
    // `t` stands for every input tensor, `out` for every out-of-place result (NULL in place)
    int32_t *kept = static_cast<int32_t *>(t);
    float *scores = static_cast<float *>(t);
    return from_hidden ? vscan::llm_prune_fused_ragged_padded(d, meta, checking_upload, t, t, t, kept, out,
                                                              scores, ws, bytes, nullptr)
                       : vscan::llm_prune_ragged_padded(d, meta, checking_upload, t, t, t, t, kept, out,
                                                        out, out, scores, ws, bytes, nullptr);
}
