// RoPE and KV-cache store, block-table updates and dense <-> paged KV copies.
#include "part_sum.h"
#include "stage_kernels.h"

namespace stg {
namespace {

// fp32 -> bf16 bits, round to nearest even (NaN kept quiet).
__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Four consecutive values at element e of the cache.
__device__ __forceinline__ void store_kv4(void *pool, size_t e, float4 v, int kv_fp32) {
    if (kv_fp32) {
        *reinterpret_cast<float4 *>(static_cast<float *>(pool) + e) = v;
    } else {
        *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(pool) + e) =
            make_uint2(to_bf16(v.x) | ((uint32_t)to_bf16(v.y) << 16), to_bf16(v.z) | ((uint32_t)to_bf16(v.w) << 16));
    }
}

// Rotates q and k (pairs (i, i + d/2) by p * theta^(-2i/d), from the per-position cos/sin tables),
// writes rotated q, and stores rotated k and v into the row's position of the paged cache in the KV
// element type.  A thread takes four neighbouring pairs of a q or k head, or four values of a v head
// (d % 8 == 0), of row blockIdx.x; SP > 1: it adds the projection's partial products first.  Bound by
// its bytes at many rows (1200 rows of the 13B-shaped stage, fp32 cache: 41 -> 28 us with 16-byte
// accesses), by two dependent loads (metadata, then the cache position) at few: a row over several
// workgroups instead of one takes 8.4 -> 4.0 us at 37 rows of the 8B-shaped stage.
template <int SP>
__global__ __launch_bounds__(256) void rope_kv_kernel(RopeKvArgs a) {
    const int row = blockIdx.x;
    const int d = a.kv.head_dim, half = d / 2, per = half / 4;   // threads per q or k head
    const int hq = a.n_q_heads, hkv = a.kv.n_kv_heads;
    const int t = blockIdx.y * 256 + threadIdx.x, rot = (hq + hkv) * per;
    if (t >= rot + hkv * 2 * per) return;
    const size_t ld = (size_t)(hq + 2 * hkv) * d, stride = (size_t)a.rows * ld;
    const float *src = a.qkv + row * ld;
    const int sidx = row / a.meta.rows_per_seq;
    const int pos = a.meta.pos0(sidx) + row % a.meta.rows_per_seq;
    const int slot = a.meta.seq_slot(sidx);
    const size_t head_stride = (size_t)kBlockTokens * d;
    auto cache = [&]() {   // the row's position of head 0 of K
        const int block = a.kv.block_table[(size_t)slot * a.kv.max_blocks + pos / kBlockTokens];
        return (size_t)block * 2 * hkv * head_stride + (size_t)(pos % kBlockTokens) * d;
    };
    if (t >= rot) {
        const int i = 4 * (t - rot), g = i / d, c = i % d;
        const float4 v = part_sum<SP>(src + (size_t)(hq + hkv) * d + i, stride);
        store_kv4(a.kv.pool, cache() + (size_t)(hkv + g) * head_stride + c, v, a.kv_fp32);
        return;
    }
    const int h = t / per, j = 4 * (t % per);
    const float4 x1 = part_sum<SP>(src + h * d + j, stride), x2 = part_sum<SP>(src + h * d + j + half, stride);
    const float4 c = *reinterpret_cast<const float4 *>(a.cos_t + (size_t)pos * half + j);
    const float4 s = *reinterpret_cast<const float4 *>(a.sin_t + (size_t)pos * half + j);
    const float4 r1 = make_float4(x1.x * c.x - x2.x * s.x, x1.y * c.y - x2.y * s.y, x1.z * c.z - x2.z * s.z,
                                  x1.w * c.w - x2.w * s.w);
    const float4 r2 = make_float4(x1.x * s.x + x2.x * c.x, x1.y * s.y + x2.y * c.y, x1.z * s.z + x2.z * c.z,
                                  x1.w * s.w + x2.w * c.w);
    if (h < hq) {
        float *q = a.q_out + row * (size_t)hq * d + h * d + j;
        *reinterpret_cast<float4 *>(q) = r1;
        *reinterpret_cast<float4 *>(q + half) = r2;
    } else {
        const size_t e = cache() + (size_t)(h - hq) * head_stride + j;
        store_kv4(a.kv.pool, e, r1, a.kv_fp32);
        store_kv4(a.kv.pool, e + half, r2, a.kv_fp32);
    }
}

__global__ void meta_write_kernel(CallMeta m, CallMeta *dst) {
    const int *src = reinterpret_cast<const int *>(&m);
    int *d = reinterpret_cast<int *>(dst);
    for (int i = threadIdx.x; i < (int)(sizeof(CallMeta) / sizeof(int)); i += blockDim.x) d[i] = src[i];
}

constexpr int kTableChunk = 240;
struct TableChunk {
    int *table;
    int n;
    int idx[kTableChunk];
    int val[kTableChunk];
};

__global__ void table_write_kernel(TableChunk c) {
    const int i = threadIdx.x;
    if (i < c.n) c.table[c.idx[i]] = c.val[i];
}

// The general form, one element at a time: dense buffers off 16-byte boundaries.
template <typename T>
__global__ __launch_bounds__(256) void kv_copy_kernel(KvCopyArgs a) {
    const int t = blockIdx.x, layer = blockIdx.y;
    const int pos = a.pos0 + t;
    const int d = a.head_dim, hkv = a.n_kv_heads;
    const int block = a.block_table[(size_t)a.slot * a.max_blocks + pos / kBlockTokens];
    T *pool = reinterpret_cast<T *>(static_cast<char *>(a.pool_base) + (size_t)layer * a.layer_stride);
    const size_t pbase = (size_t)block * 2 * hkv * kBlockTokens * d + (size_t)(pos % kBlockTokens) * d;
    const size_t dbase = ((size_t)layer * a.n + t) * hkv * d;
    T *dk = static_cast<T *>(a.k);
    T *dv = static_cast<T *>(a.v);
    for (int i = threadIdx.x; i < hkv * d; i += blockDim.x) {
        const int g = i / d, c = i % d;
        const size_t pk = pbase + (size_t)g * kBlockTokens * d + c;
        const size_t pv = pbase + (size_t)(hkv + g) * kBlockTokens * d + c;
        if (a.to_pool) {
            pool[pk] = dk[dbase + i];
            pool[pv] = dv[dbase + i];
        } else {
            dk[dbase + i] = pool[pk];
            dv[dbase + i] = pool[pv];
        }
    }
}

// 16-byte chunks, kCopyDeep of K and of V in flight per thread; a head vector is 2^row_bits chunks,
// contiguous on both sides.  Bound by its bytes once enough of them are in flight: 500 tokens of 16
// 70B-shaped layers (32.8 MB read, 32.8 MB written per direction) 19.4 us with an element per access ->
// 10.8 us (6.1 TB/s).
constexpr int kCopyDeep = 4;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // (arrays of the uint4 struct would not stay in registers)
template <bool TO_POOL>
__global__ __launch_bounds__(256) void kv_copy_wide_kernel(KvCopyArgs a, int row_bits, uint32_t chunks) {
    const int layer = blockIdx.y, hkv = a.n_kv_heads;
    u32x4 *const pool = reinterpret_cast<u32x4 *>(static_cast<char *>(a.pool_base) + (size_t)layer * a.layer_stride);
    const size_t head = (size_t)kBlockTokens << row_bits, dense0 = (size_t)layer * chunks;   // (chunks: of K, per layer)
    u32x4 *const dk = static_cast<u32x4 *>(a.k) + dense0, *const dv = static_cast<u32x4 *>(a.v) + dense0;
    const int *const table = a.block_table + (size_t)a.slot * a.max_blocks;
    const uint32_t c0 = blockIdx.x * (256u * kCopyDeep) + threadIdx.x;
    size_t at[kCopyDeep];   // the chunk's place in the pool (K; V is hkv heads further)
#pragma unroll
    for (int u = 0; u < kCopyDeep; ++u) {   // chunks past the last: the last one (in bounds, not stored)
        const uint32_t c = min(c0 + 256u * u, chunks - 1), row = c >> row_bits;
        const int pos = a.pos0 + (int)(row / hkv), g = (int)(row % hkv);
        at[u] = ((size_t)table[pos / kBlockTokens] * 2 * hkv + g) * head + ((size_t)(pos % kBlockTokens) << row_bits) +
                (c & ((1u << row_bits) - 1));
    }
    u32x4 k[kCopyDeep], v[kCopyDeep];
#pragma unroll
    for (int u = 0; u < kCopyDeep; ++u) {
        const uint32_t c = min(c0 + 256u * u, chunks - 1);
        const u32x4 *const pk = TO_POOL ? dk + c : pool + at[u], *const pv = TO_POOL ? dv + c : pool + at[u] + hkv * head;
        k[u] = *pk;
        v[u] = *pv;
    }
#pragma unroll
    for (int u = 0; u < kCopyDeep; ++u) {
        const uint32_t c = c0 + 256u * u;
        if (c < chunks) {
            *(TO_POOL ? pool + at[u] : dk + c) = k[u];
            *(TO_POOL ? pool + at[u] + hkv * head : dv + c) = v[u];
        }
    }
}

// 16-byte chunks, four in flight per lane, on kParkWorkgroups workgroups: the traffic crosses
// the host link at a few tens of GB/s, and a full-grid copy would hold every compute unit's
// memory pipeline behind slow host accesses while decode kernels wait for HBM.
__global__ __launch_bounds__(256) void kv_park_kernel(KvParkArgs a) {
    const int row_chunks = a.head_dim * a.elem_bytes / 16;  // one (token, head) vector
    const size_t per_layer = (size_t)a.n * a.n_kv_heads * row_chunks;
    const size_t total = 2 * (size_t)a.n_layers * per_layer;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const size_t head_bytes = (size_t)kBlockTokens * a.head_dim * a.elem_bytes;
    char *pool = static_cast<char *>(a.pool_base);
    uint4 *host = static_cast<uint4 *>(a.host);
    auto pool_chunk = [&](size_t c) -> uint4 * {
        const int j = (int)(c % row_chunks);
        size_t r = c / row_chunks;
        const int g = (int)(r % a.n_kv_heads);
        r /= a.n_kv_heads;
        const int t = (int)(r % a.n);
        r /= a.n;
        const int layer = (int)(r % a.n_layers);
        const int kv = (int)(r / a.n_layers);
        const int pos = a.pos0 + t;
        const int block = a.block_table[(size_t)a.slot * a.max_blocks + pos / kBlockTokens];
        const size_t off = (size_t)layer * a.layer_stride + (((size_t)block * 2 + kv) * a.n_kv_heads + g) * head_bytes +
                           (size_t)(pos % kBlockTokens) * a.head_dim * a.elem_bytes + (size_t)j * 16;
        return reinterpret_cast<uint4 *>(pool + off);
    };
    for (size_t c0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c0 < total; c0 += 4 * stride) {
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t c = c0 + u * stride;
            if (c < total) v[u] = a.to_pool ? host[c] : *pool_chunk(c);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t c = c0 + u * stride;
            if (c < total) {
                if (a.to_pool) *pool_chunk(c) = v[u];
                else host[c] = v[u];
            }
        }
    }
}

}  // namespace

hipError_t launch_kv_park(const KvParkArgs &a, hipStream_t st) {
    if (a.n <= 0) return hipSuccess;
    STG_LAUNCH(kv_park_kernel, dim3(kParkWorkgroups), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_rope_kv_store(const RopeKvArgs &a, hipStream_t st) {
    if (a.rows <= 0) return hipSuccess;
    const int d = a.kv.head_dim, threads = (a.n_q_heads + a.kv.n_kv_heads) * (d / 8) + a.kv.n_kv_heads * (d / 4);
    if (d % 8 != 0) return hipErrorInvalidValue;
    const dim3 grid(a.rows, (threads + 255) / 256);
    switch (a.n_part) {
        case 1: STG_LAUNCH(rope_kv_kernel<1>, grid, dim3(256), 0, st, a); break;
        case 2: STG_LAUNCH(rope_kv_kernel<2>, grid, dim3(256), 0, st, a); break;
        case 3: STG_LAUNCH(rope_kv_kernel<3>, grid, dim3(256), 0, st, a); break;
        case 4: STG_LAUNCH(rope_kv_kernel<4>, grid, dim3(256), 0, st, a); break;
        case 8: STG_LAUNCH(rope_kv_kernel<8>, grid, dim3(256), 0, st, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_meta_write(const CallMeta &m, CallMeta *dst, hipStream_t st) {
    STG_LAUNCH(meta_write_kernel, dim3(1), dim3(256), 0, st, m, dst);
    return hipGetLastError();
}

hipError_t launch_table_write(int *table, const int *idx, const int *val, int n, hipStream_t st) {
    for (int b = 0; b < n; b += kTableChunk) {
        TableChunk c;
        c.table = table;
        c.n = n - b < kTableChunk ? n - b : kTableChunk;
        for (int i = 0; i < c.n; ++i) {
            c.idx[i] = idx[b + i];
            c.val[i] = val[b + i];
        }
        STG_LAUNCH(table_write_kernel, dim3(1), dim3(256), 0, st, c);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_kv_copy(const KvCopyArgs &a, hipStream_t st) {
    if (a.n <= 0) return hipSuccess;
    // whole 16-byte chunks where both dense buffers start on such a boundary (a device buffer of the
    // caller's may not; the pool's head vectors always do) and a layer's chunks count in 31 bits
    const int row_bytes = a.head_dim * (a.kv_fp32 ? 4 : 2);
    const size_t chunks = (size_t)a.n * a.n_kv_heads * row_bytes / 16;
    const bool pow2 = row_bytes >= 16 && (row_bytes & (row_bytes - 1)) == 0;
    if (pow2 && chunks < (size_t(1) << 31) && ((uintptr_t)a.k | (uintptr_t)a.v) % 16 == 0) {
        int row_bits = 0;
        while (16 << row_bits < row_bytes) ++row_bits;
        const dim3 grid((unsigned)((chunks + 256 * kCopyDeep - 1) / (256 * kCopyDeep)), a.n_layers);
        if (a.to_pool) STG_LAUNCH(kv_copy_wide_kernel<true>, grid, dim3(256), 0, st, a, row_bits, (uint32_t)chunks);
        else STG_LAUNCH(kv_copy_wide_kernel<false>, grid, dim3(256), 0, st, a, row_bits, (uint32_t)chunks);
        return hipGetLastError();
    }
    dim3 grid(a.n, a.n_layers);
    if (a.kv_fp32)
        STG_LAUNCH(kv_copy_kernel<float>, grid, dim3(256), 0, st, a);
    else
        STG_LAUNCH(kv_copy_kernel<uint16_t>, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace stg
