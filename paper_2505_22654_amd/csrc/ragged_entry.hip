// Ragged stage-2 calls for a caller whose table of lengths is on the host only: the call puts the
// table into the workspace itself, and defines what the other ragged entry points leave alone
// (destination rows and scores past a sequence's results are zero).
//
// A copy of the table from pageable host memory makes the host wait for the stream - 30 us of a
// call whose kernels take 50 - so it travels in the arguments of a one-workgroup kernel instead.
// The zero rows are written by the launch that copies the rows around the visual span.
#include <hip/hip_runtime.h>
#include <string.h>

#include <algorithm>

#include "../../include/vscan.h"
#include "launch.hpp"
#include "log.hpp"

namespace vscan {
// api.cpp
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

namespace {

using namespace vscan;

constexpr int kTableChunk = 128;  // entries per launch: 2 KiB of kernel arguments
struct TableChunk {
    SeqMeta m[kTableChunk];
};
__global__ __launch_bounds__(kTableChunk) void table_upload_kernel(TableChunk chunk, SeqMeta *table,
                                                                   int count) {
    if ((int)threadIdx.x < count) table[threadIdx.x] = chunk.m[threadIdx.x];
}

hipError_t upload(SeqMeta *table, const SeqMeta *from_host, int batch, hipStream_t s) {
    for (int b = 0; b < batch; b += kTableChunk) {
        const int count = std::min(kTableChunk, batch - b);
        TableChunk chunk;
        memset(&chunk, 0, sizeof(chunk));
        memcpy(chunk.m, from_host + b, count * sizeof(SeqMeta));
        hipLaunchKernelGGL(table_upload_kernel, dim3(1), dim3(kTableChunk), 0, s, chunk, table + b, count);
    }
    return hipGetLastError();
}

int finish(const char *entry, int rc) {
    if (rc != VSCAN_OK) logf("%s -> %d (%s)", entry, rc, vscan_status_string(rc));
    return rc;
}

}  // namespace

extern "C" {

int vscan_llm_ragged_workspace_size(const vscan_llm_desc *desc, int from_hidden, size_t *bytes) {
    if (!desc || !bytes) return VSCAN_ERR_NULL;
    if (desc->struct_size != sizeof(*desc)) return VSCAN_ERR_VERSION;
    vscan_llm_desc caps = *desc;
    caps.vis_start = 0;
    const int rc = from_hidden ? vscan_llm_fused_workspace_size(&caps, bytes)
                               : vscan_llm_workspace_size(&caps, bytes);
    if (rc == VSCAN_OK) *bytes += ragged_table_bytes(desc->batch);
    return rc;
}

int vscan_llm_prune_ragged_padded(const vscan_llm_desc *desc, const vscan_seq_meta *meta_host,
                                  const void *q, void *k, void *v, void *hidden, int32_t *kept_idx,
                                  void *k_out, void *v_out, void *hidden_out, float *scores_out,
                                  void *workspace, size_t workspace_bytes, void *stream) {
    return finish("vscan_llm_prune_ragged_padded",
                  llm_prune_ragged_padded(desc, meta_host, upload, q, k, v, hidden, kept_idx, k_out,
                                          v_out, hidden_out, scores_out, workspace,
                                          workspace_bytes, stream));
}

int vscan_llm_prune_fused_ragged_padded(const vscan_llm_desc *desc, const vscan_seq_meta *meta_host,
                                        void *hidden, const void *w_q, const void *w_k_t,
                                        int32_t *kept_idx, void *hidden_out, float *scores_out,
                                        void *workspace, size_t workspace_bytes, void *stream) {
    return finish("vscan_llm_prune_fused_ragged_padded",
                  llm_prune_fused_ragged_padded(desc, meta_host, upload, hidden, w_q, w_k_t, kept_idx,
                                                hidden_out, scores_out, workspace, workspace_bytes,
                                                stream));
}

}  // extern "C"
