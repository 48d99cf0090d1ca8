// Direct global->LDS copies and their waits, shared by the kernels that stage
// keys through LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace kara {
namespace {

// Direct global->LDS copy of 16 bytes per lane; lane i's bytes land at
// lds_wave_base + 16*i (global_load_lds_dwordx4 with the LDS base in M0).
// Issued through inline assembly: the compiler then inserts no wait of its
// own before LDS reads (it cannot tell the ring stages apart and would drain
// every copy); the kernel waits explicitly.  The wait state between the
// scalar write of M0 and the load that reads it is written here, as the
// compiler adds none inside an asm block.  M0 is restored.
__device__ inline void copy16(const void* g, char* lds_wave_base) {
  const uint32_t lds = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds_wave_base);
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "v"(g), "s"(lds)
      : "memory");
}

// Workgroup barrier for LDS traffic only.  __syncthreads() would also drain
// every outstanding global->LDS copy (its release fence waits on vmcnt),
// defeating a prefetch ring; the copies this barrier must cover are waited
// for explicitly first.
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int N>
__device__ inline void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

}  // namespace
}  // namespace kara
