// Direct global -> LDS loads (gfx950): 16 bytes per lane, no registers, no vector instruction.  The 64
// lanes of an instruction fill 1 KiB of LDS, lane L at base + 16 L, from whatever address each lane names.
//
// The load is emitted as inline assembly (M0 = LDS base of the instruction, then the load).  The
// compiler's own builtin works, but it cannot tell which LDS stage such a load writes and so
// waits for ALL outstanding loads before every later LDS read, which serialises the look-ahead.
// Ordering is done by hand instead: a vmcnt wait plus a barrier before a stage is read.  So are the wait states, which the
// compiler does not look for inside a string: one between the write of M0 and the load (the s_nop), and five between a
// vector instruction that writes the scalar base (uniform_pointer) and the load, which the address arithmetic in between
// provides (the CPU tests follow both through the compiled code).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ifkv {

__device__ __forceinline__ uint32_t lds_address(const void *p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void *)p));
}
// per-lane 64-bit global address; lds_dst: wavefront-uniform LDS byte address of the instruction
__device__ __forceinline__ void dma16(const void *global_src, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(global_src), "s"(lds_dst) : "memory");
}
// the same with 4 bytes per lane: lane L's land at lds_dst + 4 L
__device__ __forceinline__ void dma4_base(const void *uniform_base, uint32_t lane_offset, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
               :
               : "v"(lane_offset), "s"(uniform_base), "s"(lds_dst)
               : "memory");
}
// wavefront-uniform 64-bit base + per-lane 32-bit byte offset
__device__ __forceinline__ void dma16_base(const void *uniform_base, uint32_t lane_offset, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(lane_offset), "s"(uniform_base), "s"(lds_dst)
               : "memory");
}
// a pointer that is the same in every lane, as a scalar
__device__ __forceinline__ const char *uniform_pointer(const char *p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
  return reinterpret_cast<const char *>((static_cast<uint64_t>(hi) << 32) | lo);
}
// waits until at most N (0 .. 63) of the wavefront's vector memory operations are outstanding
template <int N>
__device__ __forceinline__ void wait_vmem() {
  static_assert(N >= 0 && N <= 63, "six bits, the upper two apart from the lower four");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | (N >> 4) << 14);
  asm volatile("" : : : "memory");  // no LDS read moves up
}
// waits until the wavefront's LDS reads have returned (before a direct load overwrites what they read)
__device__ __forceinline__ void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }

}  // namespace ifkv
