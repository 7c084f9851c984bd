// Direct-to-LDS loads and the explicit waits that go with them, for kernels
// that keep a ring of stages in flight.
//
// The loads are issued from inline asm so that the compiler's wait
// insertion, which cannot tell ring stages apart and would drain every load
// before each LDS read, stays out of the way; such a load writes no
// register.  The kernel waits for each stage itself (s_waitcnt vmcnt counts
// the loads in issue order, then s_barrier where other wavefronts read them).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qlk {

__device__ inline constexpr int dma_vmcnt(int v)
{
    // gfx9 s_waitcnt encoding: vmcnt[3:0] + vmcnt[5:4] at bits 15:14;
    // expcnt (bits 6:4) and lgkmcnt (bits 11:8) left at "no wait"
    return (v & 15) | (((v >> 4) & 3) << 14) | (7 << 4) | (15 << 8);
}

// wave-uniform 64-bit base in an SGPR pair (readfirstlane returns int: widen
// through uint32_t)
__device__ inline uint64_t dma_base(const void *p)
{
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

// LDS byte address of a pointer into LDS (the low half of the generic one)
__device__ inline uint32_t dma_lds(const void *p) { return (uint32_t)(uintptr_t)p; }

// 16 (4) bytes per lane from wave-uniform base + per-lane offset to LDS:
// lane t's data lands at lds + t * 16 (t * 4)
__device__ inline void dma_load16(const void *base, uint32_t off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(off), "s"(dma_base(base)), "s"(__builtin_amdgcn_readfirstlane(lds))
                 : "memory");
}
__device__ inline void dma_load4(const void *base, uint32_t off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                 :
                 : "v"(off), "s"(dma_base(base)), "s"(__builtin_amdgcn_readfirstlane(lds))
                 : "memory");
}

// Wait until at most y * LOADS (+ nothing else) of the wavefront's loads
// are still in flight, y <= Y known at run time.
template <int LOADS, int Y>
__device__ inline void dma_wait(int y)
{
    if constexpr (Y > 0) {
        if (y >= Y)
            __builtin_amdgcn_s_waitcnt(dma_vmcnt(Y * LOADS));
        else
            dma_wait<LOADS, Y - 1>(y);
    } else {
        __builtin_amdgcn_s_waitcnt(dma_vmcnt(0));
    }
}

// An empty statement the compiler keeps in order with the scheduling
// barriers: a value passed through it is computed where it is written.
template <typename T>
__device__ inline void dma_pin(T &v)
{
    asm volatile("" : "+v"(v));
}

}  // namespace qlk
