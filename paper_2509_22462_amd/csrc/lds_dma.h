// Waits of the kernels that fill LDS by DMA (gemm_dma.hip, gemm_pk.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace nnc {

typedef __attribute__((address_space(3))) void* lds_ptr;

// s_waitcnt immediate: at most `vm` vector-memory and `lgkm` LDS operations of
// this wave outstanding (expcnt at its maximum).
constexpr int waitcnt_imm(int vm, int lgkm) { return (vm & 15) | 0x70 | (lgkm << 8) | ((vm >> 4) << 14); }

// Until at most N of this wave's vector-memory operations are outstanding.
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(N, 15));
}

// Between two steps of a pipeline of LDS stages: all but this wave's N newest
// loads have landed and every one of its LDS reads has returned, then the
// workgroup's barrier.  After it the stage of the step before may be filled
// again: another wave's DMA must not find a read of it on the way, whatever
// order the compiler gave the multiplications that use what was read.  (No
// memory fence, which would wait for the N newest loads too.)
template <int N>
__device__ __forceinline__ void wait_stage() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(N, 0));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

}  // namespace nnc
