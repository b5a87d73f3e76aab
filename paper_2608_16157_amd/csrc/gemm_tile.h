// LDS-DMA and pipeline helpers shared by the MFMA expert kernels (gemm.hip, skinny_tile.h); internal.
#pragma once

#include <type_traits>

#include "ftmoe_device.h"

namespace ftmoe {

enum { GEMM_GATEUP = 0, GEMM_DOWN = 1 };

template <int V> using ic = std::integral_constant<int, V>;

// Calls f(ic<S>) for S = B .. E-1.
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (B < E) {
        f(ic<B>{});
        static_for<B + 1, E>(f);
    }
}

// Block index b of n working blocks -> logical tile index such that logical tiles [x*q + min(x,r),
// ...) run on XCD x (blocks are dealt to the 8 XCDs round-robin).  n counts only blocks that have a
// tile: with idle blocks among the n, the tiles would crowd onto the first XCDs.
__device__ __forceinline__ int xcd_remap(int b, int n) {
    const int q = n / 8, r = n % 8, x = b % 8, i = b / 8;
    return x * q + min(x, r) + i;
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}
__device__ __forceinline__ void wait_lgkmcnt0() {
    __builtin_amdgcn_s_waitcnt(0xF | (0x7 << 4) | (0x0 << 8) | (0x3 << 14));
}

// Workgroup barrier between pipeline stages.  The empty asm statements are compiler-level memory
// fences: they keep LDS reads of a stage from being moved across the barrier, without the
// wait-for-everything a __syncthreads fence adds.
__device__ __forceinline__ void stage_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Position of 16-byte chunk c in LDS row r.  A 16-byte-per-lane LDS read serves 16 lanes (256
// bytes, all 64 banks) per pass; the operand reads give those lanes 16 consecutive rows and one
// chunk index, so the XOR spreads the same chunk of 16 consecutive rows over all 16 chunk
// positions of a 256-byte window: a 256-byte row holds 16 chunks (XOR r mod 16), a 128-byte row 8
// (XOR (r / 2) mod 8), a 64-byte row 4 (XOR (r / 4) mod 4), a 32-byte row 2 (XOR (r / 8) mod 2).
template <int ROW_BYTES>
__device__ __forceinline__ int swz(int r, int c) {
    static_assert(ROW_BYTES == 32 || ROW_BYTES == 64 || ROW_BYTES == 128 || ROW_BYTES == 256, "row size");
    if constexpr (ROW_BYTES == 256) return c ^ (r & 15);
    else if constexpr (ROW_BYTES == 128) return c ^ ((r >> 1) & 7);
    else if constexpr (ROW_BYTES == 64) return c ^ ((r >> 2) & 3);
    else return c ^ ((r >> 3) & 1);
}

// LDS DMA: lane i of the instruction writes LDS bytes [16 i, 16 i + 16) (dma4: [4 i, 4 i + 4)) of
// the block at LDS byte address `lds`, from its own global address.  Written as assembly because
// the compiler makes every later LDS read wait for all outstanding DMAs into the same LDS object,
// and the rings here are one object whose slots are chosen at run time.  The instructions have no
// register outputs; the waits are the explicit ones of the main loops (loads return in order, so
// waits that the compiler adds for its own loads are at worst longer than needed).  Each sets M0, the
// LDS address, for itself (nothing else in these kernels uses it; the compiler reserves it and takes
// no clobber of it); the ISA asks for one wait state between that write and the DMA, which neither
// the hardware checks nor the compiler inserts inside an assembly string.
__device__ __forceinline__ void dma16(const uint8_t *g, uint32_t lds) {
    lds = __builtin_amdgcn_readfirstlane(lds);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(g), "s"(lds) : "memory");
}
// the same with a wave-uniform base and a 32-bit offset per lane
__device__ __forceinline__ const uint8_t *uniform_ptr(const uint8_t *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
    return reinterpret_cast<const uint8_t *>(static_cast<uint64_t>(hi) << 32 | lo);
}
__device__ __forceinline__ void dma16(const uint8_t *base, uint32_t off, uint32_t lds) {
    base = uniform_ptr(base);
    lds = __builtin_amdgcn_readfirstlane(lds);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds) : "memory");
}
__device__ __forceinline__ void dma4(const uint8_t *base, uint32_t off, uint32_t lds) {
    base = uniform_ptr(base);
    lds = __builtin_amdgcn_readfirstlane(lds);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" : : "v"(off), "s"(base), "s"(lds) : "memory");
}

// A load through the scalar cache from a wave-uniform address of memory that this kernel does not
// write.  It is counted apart from the vector loads, so waiting for it waits for no DMA.
__device__ __forceinline__ int scalar_load(const int32_t *p) {
    return __builtin_amdgcn_readfirstlane(*(const __attribute__((address_space(4))) int32_t *)p);
}

__device__ __forceinline__ void dma4(const uint8_t *g, uint32_t lds) {
    lds = __builtin_amdgcn_readfirstlane(lds);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" : : "v"(g), "s"(lds) : "memory");
}

// LDS byte address of a shared object, for the DMAs
__device__ __forceinline__ uint32_t lds_address(uint8_t *p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t *)p));
}

}  // namespace ftmoe
