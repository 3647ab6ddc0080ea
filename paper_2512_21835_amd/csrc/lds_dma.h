// Copies from global memory straight into LDS, and the waits and the barrier of kernels that order them
// themselves.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace stg {

// Copies 16 bytes per lane from global memory straight into LDS (global_load_lds_dwordx4): lane l
// of the wavefront reads base + off and writes LDS bytes [lds_addr + 16 l, lds_addr + 16 l + 16).
// Issued as inline assembly so that the compiler does not wait for every such load before each LDS
// read (it cannot tell which LDS bytes a DMA load writes); the kernel waits for them itself
// (wait_vm).  m0 holds the wavefront-uniform LDS address; nothing else in the kernel uses m0.  An
// LDS DMA must not directly follow a scalar write of m0 (gfx9 asks for one wait state there; the
// compiler inserts it in code it generates, not inside inline assembly), hence the s_nop.
// NT: non-temporal, for bytes that no other workgroup reads.
template <bool NT = false>
__device__ __forceinline__ void dma16(uint32_t off, const void *base, uint32_t lds_addr) {
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(off), "s"(base), "s"(lds_addr)
                     : "memory");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds_addr)
                     : "memory");
}

// s_waitcnt vmcnt(N), other counters untouched.
template <int N>
__device__ __forceinline__ void wait_vm() {
    __builtin_amdgcn_s_waitcnt(0x3F70 | (N & 0xF) | ((N >> 4) << 14));
}

// s_waitcnt lgkmcnt(N), other counters untouched.
template <int N>
__device__ __forceinline__ void wait_lgkm() {
    static_assert(N >= 0 && N < 16, "lgkmcnt is four bits");
    __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
}

// Workgroup barrier for kernels that order their LDS traffic themselves (wait_vm and wait_lgkm before
// it); no LDS access moves across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace stg
