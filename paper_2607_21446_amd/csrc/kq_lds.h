// Loads straight into LDS and bare barriers, for kernels that pipeline stages of
// operands through LDS with explicit waits (kq_gemm.hip, kq_calib.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kq {

// Lane l's 16 bytes at base + voff land at the wave-uniform LDS address lds + 16 l.  As asm:
// the compiler puts a vmcnt(0) before LDS reads that may alias a load into LDS it knows of,
// which would drain the stages in flight.  The caller waits (s_waitcnt vmcnt), and the load
// has no register result.
__device__ __forceinline__ void lds_dma16(uint32_t lds, uint32_t voff, const uint8_t* base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base)
                 : "memory", "m0");
}

// A barrier that waits for no load in flight.
__device__ __forceinline__ void stage_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace kq
