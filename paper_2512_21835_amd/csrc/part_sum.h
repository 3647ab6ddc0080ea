// Sum of the partial products of a GEMM whose k ranges ran in different workgroups: SP of them, `stride`
// floats apart, four columns at p.  Groups of up to four neighbours ascending, then the groups (a
// workgroup that runs such a group itself adds it the same way, so the grouping does not change the
// result).  Every load is issued before the first sum.
#pragma once

#include <hip/hip_runtime.h>

namespace stg {

__device__ __forceinline__ float4 add4(float4 a, float4 b) {
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

template <int SP>   // 1 to 4, or 8
__device__ __forceinline__ float4 part_sum(const float *p, size_t stride) {
    float4 v[SP];
#pragma unroll
    for (int i = 0; i < SP; ++i) v[i] = *reinterpret_cast<const float4 *>(p + i * stride);
#pragma unroll
    for (int i = 0; i < SP; ++i)
        if (i % 4) v[i / 4 * 4] = add4(v[i / 4 * 4], v[i]);
    if constexpr (SP == 8) return add4(v[0], v[4]);
    return v[0];
}

}  // namespace stg
