// Loads from memory straight to LDS, and waiting for them: shared by the kernels whose weights lie in memory as they lie in LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ppc {

// a wave-uniform address, in scalar registers
__device__ __forceinline__ const void* uniform_address(const void* p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (const void*)(((uint64_t)hi << 32) | lo);
}
// 64 lanes x 16 bytes from base + off to the 1 KB of LDS at lds_dst (wave-uniform)
__device__ __forceinline__ void load_lds16(uint32_t off, const void* base, uint32_t lds_dst) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds_dst) : "memory", "m0");
}
// ... 4 bytes, to 256 bytes
__device__ __forceinline__ void load_lds4(uint32_t off, const void* base, uint32_t lds_dst) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(base), "s"(lds_dst) : "memory", "m0");
}
// s_waitcnt's operand for vmcnt(n) alone
constexpr int wait_vmcnt(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

}  // namespace ppc
