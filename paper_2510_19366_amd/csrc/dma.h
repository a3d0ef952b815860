// Wave-wide copies global -> LDS and the waits that go with them, shared by the kernels whose
// operands do not pass through registers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace mp {

__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// One wave-wide copy: lane i's 16 bytes at base + voff land at LDS address lds + 16 i.  m0 carries
// the LDS address; the compiler reserves m0 and does not accept it in a clobber list, so the value
// it may be keeping there is saved and put back.
__device__ __forceinline__ void copy_to_lds16(const void* base, uint32_t voff, uint32_t lds) {
  uint32_t keep;
  asm volatile(
      "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\t"
      "global_load_lds_dwordx4 %1, %2\n\ts_mov_b32 m0, %0"
      : "=&s"(keep)
      : "v"(voff), "s"(base), "s"(lds)
      : "memory");
}

// the same with a 64-bit address per lane
__device__ __forceinline__ void copy_to_lds16_addr(uint64_t addr, uint32_t lds) {
  uint32_t keep;
  asm volatile(
      "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
      : "=&s"(keep)
      : "v"(addr), "s"(lds)
      : "memory");
}

// until at most N of this wave's vector memory operations are pending (they retire in issue order)
template <int N>
__device__ __forceinline__ void wait_vmem() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// A 16-byte LDS read into the register it is given (tied), not tracked by the compiler, and the
// wait for all but the youngest N of this wave's LDS reads, behind which the given values may be used.
// (Kernels at the register limit: the compiler rotates reads through twice the registers.)
template <int OFF, class V>
__device__ __forceinline__ void read_lds16(V& v, uint32_t addr) {
  static_assert(sizeof(V) == 16);
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "+v"(v) : "v"(addr), "n"(OFF));
}
template <int N, class V>
__device__ __forceinline__ void wait_lds(V& a, V& b) {
  asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N));
}
template <int N, class V>
__device__ __forceinline__ void wait_lds(V& a, V& b, V& c) {
  asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(a), "+v"(b), "+v"(c) : "n"(N));
}
template <int N, class V>
__device__ __forceinline__ void wait_lds(V& a, V& b, V& c, V& d) {
  asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "n"(N));
}

// s_barrier without the wait for outstanding copies that __syncthreads() would add; LDS accesses
// stay on their side of it
__device__ __forceinline__ void raw_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// f(integral_constant<I>) for I = BEGIN .. END - 1: a loop whose index can be a template argument
template <int BEGIN, int END, class F>
__device__ __forceinline__ void static_loop(F&& f) {
  if constexpr (BEGIN < END) {
    f(std::integral_constant<int, BEGIN>{});
    static_loop<BEGIN + 1, END>(f);
  }
}

}  // namespace mp
