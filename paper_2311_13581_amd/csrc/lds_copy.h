// Copies from memory straight into LDS, past the register file, and the waits that go with them.  A compute unit draws 59 B
// per clock out of its die's L2 this way, through registers 36 (measured with all units on a 1 MB buffer).
#ifndef PASS_LDS_COPY_H
#define PASS_LDS_COPY_H
#include <hip/hip_runtime.h>

#include <cstdint>

namespace pass {

// 64 x 16 bytes from memory (one address per lane) to 1 KB of LDS (wavefront-uniform); NT: data that is read once.  In
// assembly because the compiler, which cannot tell the stages of a ring of buffers apart, would wait for every copy in
// flight before each LDS read; it has no register result.  The copies of a wavefront complete in order.
template <bool NT = false>
__device__ __forceinline__ void copy_to_lds(const void *src, void *dst) {
  const uint32_t off = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)dst;
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(src), "s"(off) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(off) : "memory", "m0");
}
// 64 x 4 bytes to 256 bytes of LDS
__device__ __forceinline__ void copy1_to_lds(const void *src, void *dst) {
  const uint32_t off = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)dst;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "s"(off) : "memory", "m0");
}
// until no more than the wavefront's youngest N copies are in flight
template <int N>
__device__ __forceinline__ void wait_copies() {
  static_assert(N >= 0 && N < 64, "six bits");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
}
// until what the wavefront has read out of LDS has arrived: only then may a copy overwrite it
__device__ __forceinline__ void wait_lds_reads() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0xC07F);
}
// the workgroup meets; neither the compiler nor the instruction scheduler moves memory accesses across
__device__ __forceinline__ void meet() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}

}  // namespace pass
#endif
