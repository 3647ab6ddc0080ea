// The exact-sum bf16 pair of an fp32 value (hi = bf16(x), lo = bf16(x - hi), both rounded to nearest
// even) in the interleaved layout the prefill GEMMs read (pair_at, stage_kernels.h).  Shared by the
// kernels that produce GEMM operands: RMSNorm, SwiGLU, and the prefill attention output.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace stg {

// The pairs of a (low half) and b (high half): two v_cvt_pk_bf16_f32 (nearest even, NaN kept quiet).
__device__ __forceinline__ void split_pair2(float a, float b, uint32_t &hi, uint32_t &lo) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    hi = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
    lo = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)(a - __uint_as_float(hi << 16)),
                                             (__bf16)(b - __uint_as_float(hi & 0xFFFF0000u))});
}

__device__ __forceinline__ void split_pair(float v, uint16_t &hi, uint16_t &lo) {
    uint32_t h, l;
    split_pair2(v, 0.f, h, l);
    hi = (uint16_t)h;
    lo = (uint16_t)l;
}

// The hi and lo of four consecutive elements of a 32-wide block (p: the first one's hi, 8-byte
// aligned): two 8-byte stores, the lo 32 elements further.
__device__ __forceinline__ void store_pair4(uint16_t *p, float4 v) {
    uint2 h, l;
    split_pair2(v.x, v.y, h.x, l.x);
    split_pair2(v.z, v.w, h.y, l.y);
    *reinterpret_cast<uint2 *>(p) = h;
    *reinterpret_cast<uint2 *>(p + 32) = l;
}

}  // namespace stg
