// Shared by the mean-attention kernels (encoder_score.hip).
#pragma once
#include "common.hpp"
#include "launch.hpp"

namespace vscan {

// work item -> (segment*head, block) with each XCD walking a contiguous range of
// items, so the workgroups resident on one XCD share one head's Q/K in its L2
__device__ __forceinline__ int xcd_contiguous_item(int total) {
    const int id = blockIdx.x;
    const int per = (total + 7) / 8;
    return (id & 7) * per + (id >> 3);
}

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
    // and that these kernels use for nothing else.)
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off"
                 :
                 : "s"(lds_address), "v"(src)
                 : "memory");
}
// every outstanding vector-memory load of this wave has arrived (vmcnt 0, the other counters
// left alone)
__device__ __forceinline__ void wait_direct_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

}  // namespace vscan
