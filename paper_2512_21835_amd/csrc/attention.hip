// Causal grouped-query attention over the paged KV cache, fp32 arithmetic.
//
// Prefill (split_keys == 0): flash-attention tiling on the matrix cores, the G = Hq/Hkv query heads
// that share a KV head in one workgroup; attn_prefill_mfma with a bf16 cache (operands as bf16 hi/lo
// pairs), attn_prefill_f32 with an fp32 one.  Decode (split_keys > 0): the context is
// cut into splits of split_keys keys so that one token's attention still fills the GPU, and a
// second launch (attn_merge) merges each row's splits.  With a bf16 cache and 128-wide heads the
// splits run on the matrix cores (attn_decode_mfma: the G query heads of a KV head are the N
// dimension of S^T = K Q^T, then O = P V; with G = 8 the vector form spends 16 multiply-adds per
// cached element and is bound by them); otherwise attn_decode_kernel.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lanes.h"
#include "lds_dma.h"
#include "pair.h"
#include "stage_kernels.h"

namespace stg {
namespace {

// 16 bytes in registers (arrays of HIP's uint4 and float4 structs may go to scratch memory)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kChunk = 64;
constexpr int kMaxDecodeSplits = 256;  // splits one row may have (max_context / split_keys)

__device__ __forceinline__ float bf16lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }

template <bool F32KV>
__device__ __forceinline__ void load8(const void *pool, size_t elem, float f[8]) {
    if (F32KV) {
        const float4 *p = reinterpret_cast<const float4 *>(static_cast<const float *>(pool) + elem);
        const float4 a = p[0], b = p[1];
        f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
        f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
    } else {
        const uint4 v = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(pool) + elem);
        f[0] = bf16lo(v.x); f[1] = bf16hi(v.x);
        f[2] = bf16lo(v.y); f[3] = bf16hi(v.y);
        f[4] = bf16lo(v.z); f[5] = bf16hi(v.z);
        f[6] = bf16lo(v.w); f[7] = bf16hi(v.w);
    }
}

template <int G, int D>
struct DecodeSmem {
    float wm[4][G], wl[4][G];
    float o[4][G][D];
};

// Decode: one workgroup per (key split, KV head, row); a split holds at most kChunk keys.  K and V
// of the lane's keys are fetched together up front, scores are reduced across the D/8 lanes of a
// key, the split's maximum and sum across the workgroup through LDS once, and the partial output
// (unnormalised, with its max and sum) goes to global memory for attn_merge.  FINAL (every
// row of the call within one split): the output o / l directly, the value the merge would compute
// from the single split (weight exp(m - m) = 1), so no merge launch follows.
template <int G, int D, bool F32KV, bool FINAL>
__device__ __forceinline__ void attn_decode_task(const AttnArgs &a, int split, int g, int row,
                                                 DecodeSmem<G, D> &sm) {
    constexpr int LPK = D / 8;
    constexpr int KPW = 64 / LPK;
    constexpr int KPS = 4 * KPW;
    constexpr int STEPS = kChunk / KPS;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kl = lane / LPK, sub = lane % LPK, c0 = sub * 8;
    const int hq_total = a.n_q_heads;
    const size_t q_ld = (size_t)hq_total * D;
    // the queries first: they depend on the row only
    const float scale = 1.f / sqrtf((float)D);
    float q[G][8];
#pragma unroll
    for (int h = 0; h < G; ++h) {
        const float *qp = a.q + row * q_ld + (size_t)(g * G + h) * D + c0;
#pragma unroll
        for (int j = 0; j < 8; ++j) q[h][j] = qp[j] * scale;
    }
    const int sidx = row / a.rows_per_seq;
    const int pos = a.meta.pos0(sidx) + row % a.rows_per_seq;
    const int slot = a.meta.seq_slot(sidx);
    const int ctx = pos + 1;
    const int kbeg = split * a.split_keys;
    if (kbeg >= ctx || slot < 0) return;  // (slot tested so that both metadata loads go out together)
    const int n = min(a.split_keys, ctx - kbeg);

    const int hkv = a.kv.n_kv_heads;
    const int *table = a.kv.block_table + (size_t)slot * a.kv.max_blocks;
    const size_t blk_stride = (size_t)2 * hkv * kBlockTokens * D;

    // keys of this lane: kk = st * KPS + wave * KPW + kl.  Slots past the split's last key load that
    // key again (in bounds; their scores are masked below), so that the loads carry no branches and
    // all block-table loads, then all K/V loads, are in flight together: two round trips in all.
    int blk[STEPS];
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const int key = kbeg + min(st * KPS + wave * KPW + kl, n - 1);
        blk[st] = table[key / kBlockTokens];
    }
    float kf[STEPS][8], vf[STEPS][8];
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const int key = kbeg + min(st * KPS + wave * KPW + kl, n - 1);
        const size_t e = (size_t)blk[st] * blk_stride + ((size_t)g * kBlockTokens + key % kBlockTokens) * D + c0;
        load8<F32KV>(a.kv.pool, e, kf[st]);
        load8<F32KV>(a.kv.pool, e + (size_t)hkv * kBlockTokens * D, vf[st]);
    }
    __builtin_amdgcn_sched_barrier(0);  // every K and V load in flight before any is used

    float sc[STEPS][G];
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const bool valid = st * KPS + wave * KPW + kl < n;
#pragma unroll
        for (int h = 0; h < G; ++h) {
            float p = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) p = fmaf(q[h][j], kf[st][j], p);
#pragma unroll
            for (int o2 = LPK / 2; o2 >= 1; o2 >>= 1) p += lane_xor(p, o2);
            sc[st][h] = valid ? p : -INFINITY;
        }
    }
    // split maximum per head
#pragma unroll
    for (int h = 0; h < G; ++h) {
        float m = sc[0][h];
#pragma unroll
        for (int st = 1; st < STEPS; ++st) m = fmaxf(m, sc[st][h]);
#pragma unroll
        for (int o2 = 32; o2 >= LPK; o2 >>= 1) m = fmaxf(m, lane_xor(m, o2));
        if (lane == 0) sm.wm[wave][h] = m;
    }
    __syncthreads();
    float mh[G];
#pragma unroll
    for (int h = 0; h < G; ++h) mh[h] = fmaxf(fmaxf(sm.wm[0][h], sm.wm[1][h]), fmaxf(sm.wm[2][h], sm.wm[3][h]));

    float l[G], o[G][8];
#pragma unroll
    for (int h = 0; h < G; ++h) {
        l[h] = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) o[h][j] = 0.f;
    }
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
#pragma unroll
        for (int h = 0; h < G; ++h) {
            const float p = sc[st][h] == -INFINITY ? 0.f : expf(sc[st][h] - mh[h]);
            l[h] += p;
#pragma unroll
            for (int j = 0; j < 8; ++j) o[h][j] = fmaf(p, vf[st][j], o[h][j]);
        }
    }
#pragma unroll
    for (int h = 0; h < G; ++h) {
#pragma unroll
        for (int o2 = 32; o2 >= LPK; o2 >>= 1) l[h] += lane_xor(l[h], o2);
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int o2 = 32; o2 >= LPK; o2 >>= 1)   // G >= 8: the VALU is the bound, the LDS crossbar is idle
                o[h][j] += G >= 8 ? __shfl_xor(o[h][j], o2, 64) : lane_xor(o[h][j], o2);
    }
    if (kl == 0) {
#pragma unroll
        for (int h = 0; h < G; ++h)
#pragma unroll
            for (int j = 0; j < 8; ++j) sm.o[wave][h][c0 + j] = o[h][j];
    }
    if (lane == 0) {
#pragma unroll
        for (int h = 0; h < G; ++h) sm.wl[wave][h] = l[h];
    }
    __syncthreads();
    for (int i = tid; i < G * D; i += 256) {
        const int h = i / D, c = i % D;
        if (FINAL) {
            const float o_sum = ((sm.o[0][h][c] + sm.o[1][h][c]) + sm.o[2][h][c]) + sm.o[3][h][c];
            const float l_sum = ((sm.wl[0][h] + sm.wl[1][h]) + sm.wl[2][h]) + sm.wl[3][h];
            const int col = (g * G + h) * D + c;
            if (row < a.pair_rows) {
                uint16_t *p = a.out_pair + row * a.out_pair_ld + pair_at(col);
                split_pair(o_sum / l_sum, p[0], p[32]);
            } else {
                a.out[row * q_ld + col] = o_sum / l_sum;
            }
            continue;
        }
        const size_t pi = ((size_t)row * hq_total + g * G + h) * a.max_splits + split;
        a.part_o[pi * D + c] = ((sm.o[0][h][c] + sm.o[1][h][c]) + sm.o[2][h][c]) + sm.o[3][h][c];
        if (c == 0) {
            a.part_ml[pi * 2 + 0] = fmaxf(fmaxf(sm.wm[0][h], sm.wm[1][h]), fmaxf(sm.wm[2][h], sm.wm[3][h]));
            a.part_ml[pi * 2 + 1] = ((sm.wl[0][h] + sm.wl[1][h]) + sm.wl[2][h]) + sm.wl[3][h];
        }
    }
}


template <int G, int D, bool F32KV, bool FINAL>
__global__ __launch_bounds__(256) void attn_decode_kernel(AttnArgs a) {
    __shared__ DecodeSmem<G, D> sm;
    attn_decode_task<G, D, F32KV, FINAL>(a, blockIdx.y, blockIdx.x, blockIdx.z, sm);
}

// The split states (maximum m, sum l and unnormalised output o of each 64-key split) are merged in a
// fixed order: groups of kMergeGroup consecutive splits first, then the groups of a lane, then the lanes
// (attn_merge).  Where a call has splits enough to fill the GPU with a workgroup per group, the splits'
// kernel writes the groups' states instead of the splits': a quarter of the partial outputs.
constexpr int kMergeGroup = 4;
// A group's maximum and its splits' weights exp(m - maximum) (0 for a split without a score above
// -inf; n splits).
__device__ __forceinline__ float group_weights(const float m[kMergeGroup], int n, float w[kMergeGroup]) {
    float mg = -INFINITY;
#pragma unroll
    for (int u = 0; u < kMergeGroup; ++u)
        if (u < n) mg = fmaxf(mg, m[u]);
    const float ref = mg == -INFINITY ? 0.f : mg;
#pragma unroll
    for (int u = 0; u < kMergeGroup; ++u) w[u] = expf(m[u] - ref);
    return mg;
}
__device__ __forceinline__ float group_sum(const float v[kMergeGroup], const float w[kMergeGroup], int n) {
    float s = w[0] * v[0];
#pragma unroll
    for (int u = 1; u < kMergeGroup; ++u)
        if (u < n) s = fmaf(w[u], v[u], s);
    return s;
}

// Merge of the decode splits: one workgroup per (row, query head).  Thread t owns the 4 output
// columns 4 (t % (D/4)) .. + 3 and the groups with index % SL == t / (D/4) (SL = 1024 / D split
// lanes: 8 for 128-wide heads, 16 for 64-wide).  Per round it issues the loads of kMergePer states per
// lane (splits, or with GROUPED whole groups) at once, addresses clamped to the call's longest row
// (a.grid_splits), before the row's own split count arrives from the metadata: one round trip for
// contexts up to kMergePer * SL states.  A lane merges its groups in ascending order (online: rescaled
// to the running maximum); the SL lane states then meet in LDS and are added in lane order.  The order
// depends on the row's split count only, never on the other rows of the call nor on who combined the
// groups; for a single split the result is exactly o / l (weights exp(0) = 1, empty lanes add 0).
constexpr int kMergePer = 8;
template <int D, bool GROUPED>
__global__ __launch_bounds__(256) void attn_merge(AttnArgs a) {
    constexpr int CG = D / 4, SL = 256 / CG;
    constexpr int GS = GROUPED ? 1 : kMergeGroup, GPL = kMergePer / GS;   // states per group, groups per lane and round
    __shared__ float s_m[SL][CG], s_l[SL][CG];
    __shared__ float4 s_o[SL][CG];
    const int cg = threadIdx.x % CG, sl = threadIdx.x / CG;
    const int hq = blockIdx.x, row = blockIdx.y, hq_total = a.n_q_heads;
    const size_t pi0 = ((size_t)row * hq_total + hq) * a.max_splits;
    const float2 *ml = reinterpret_cast<const float2 *>(a.part_ml) + pi0;
    const float4 *po = reinterpret_cast<const float4 *>(a.part_o + pi0 * D) + cg;
    const int per = GROUPED ? kMergeGroup * a.split_keys : a.split_keys;   // keys per state
    const int lim = GROUPED ? (a.grid_splits + kMergeGroup - 1) / kMergeGroup : a.grid_splits;
    float mx = -INFINITY, den = 0.f;
    float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
    int nst = -1;   // the row's states
    for (int s0 = 0; s0 < lim; s0 += kMergePer * SL) {
        const int ngr = min(GPL, ((lim - s0 + GS - 1) / GS + SL - 1) / SL);  // same for every thread
        float2 v[kMergePer];
        float4 o[kMergePer];
#pragma unroll
        for (int j = 0; j < kMergePer; ++j)
            if (j / GS < ngr) {
                const int s = min(s0 + (j / GS * SL + sl) * GS + j % GS, lim - 1);
                v[j] = ml[s];
                o[j] = po[(size_t)s * (D / 4)];
            }
        if (nst < 0) {
            const int sidx = row / a.rows_per_seq;
            const int ctx = a.meta.pos0(sidx) + row % a.rows_per_seq + 1;
            nst = min((ctx + per - 1) / per, lim);
        }
        if (s0 >= nst) break;
#pragma unroll
        for (int gi = 0; gi < GPL; ++gi) {
            const int first = s0 + (gi * SL + sl) * GS, n = min(GS, nst - first);
            if (gi >= ngr || n <= 0) continue;
            float mg, lg;
            float4 og;
            if constexpr (GROUPED) {
                mg = v[gi].x;
                lg = v[gi].y;
                og = o[gi];
            } else {
                float m[GS], w[GS], t[GS];
                auto sum = [&](auto get) {
#pragma unroll
                    for (int u = 0; u < GS; ++u) t[u] = get(GS * gi + u);
                    return group_sum(t, w, n);
                };
#pragma unroll
                for (int u = 0; u < GS; ++u) m[u] = v[GS * gi + u].x;
                mg = group_weights(m, n, w);
                lg = sum([&](int j) { return v[j].y; });
                og = make_float4(sum([&](int j) { return o[j].x; }), sum([&](int j) { return o[j].y; }),
                                 sum([&](int j) { return o[j].z; }), sum([&](int j) { return o[j].w; }));
            }
            if (gi == 0 && s0 == 0) {   // the lane's first: weight 1, nothing before it
                mx = mg;
                den = lg;
                num = og;
                continue;
            }
            const float m = fmaxf(mx, mg), ref = m == -INFINITY ? 0.f : m;
            const float r = expf(mx - ref), w = expf(mg - ref);
            den = fmaf(w, lg, den * r);
            num.x = fmaf(w, og.x, num.x * r);
            num.y = fmaf(w, og.y, num.y * r);
            num.z = fmaf(w, og.z, num.z * r);
            num.w = fmaf(w, og.w, num.w * r);
            mx = m;
        }
    }
    s_m[sl][cg] = mx;
    s_l[sl][cg] = den;
    s_o[sl][cg] = num;
    __syncthreads();
    if (sl != 0) return;
    float L = 0.f;
    float4 O = make_float4(0.f, 0.f, 0.f, 0.f);
    auto add_lanes = [&](auto count) {
        constexpr int N = decltype(count)::value;
        float M = -INFINITY;
#pragma unroll
        for (int i = 0; i < N; ++i) M = fmaxf(M, s_m[i][cg]);
        const float ref = M == -INFINITY ? 0.f : M;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float w = expf(s_m[i][cg] - ref);   // (a lane without a group: 0, and its sums are 0)
            const float4 oi = s_o[i][cg];
            L = fmaf(w, s_l[i][cg], L);
            O.x = fmaf(w, oi.x, O.x);
            O.y = fmaf(w, oi.y, O.y);
            O.z = fmaf(w, oi.z, O.z);
            O.w = fmaf(w, oi.w, O.w);
        }
    };
    // rows of up to 4 lanes' groups (1024 keys) leave the empty lanes out, most of the 16 at 64-wide heads
    if (nst <= 4 * GS) add_lanes(std::integral_constant<int, 4>{});
    else add_lanes(std::integral_constant<int, SL>{});
    const float4 v = make_float4(O.x / L, O.y / L, O.z / L, O.w / L);
    const int col = hq * D + 4 * cg;
    if (row < a.pair_rows) store_pair4(a.out_pair + row * a.out_pair_ld + pair_at(col), v);
    else *reinterpret_cast<float4 *>(a.out + (size_t)row * hq_total * D + col) = v;
}

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

__device__ __forceinline__ bf16x8_t as_bf(uint4 v) {
    bf16x8_t r;
    __builtin_memcpy(&r, &v, 16);
    return r;
}
// x as an exact-sum pair of bf16 vectors: hi = bf16(x), lo = bf16(x - hi), both nearest even.
__device__ __forceinline__ void split8(const float *x, bf16x8_t &hi, bf16x8_t &lo) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        hi[j] = (__bf16)x[j];                   // v_cvt_pk_bf16_f32: nearest even
        lo[j] = (__bf16)(x[j] - (float)hi[j]);
    }
}

// 16 bytes of the cache, which one workgroup reads once per call.  STREAM: non-temporal (see AttnArgs).
template <bool STREAM>
__device__ __forceinline__ u32x4 load_cache16(const uint16_t *p) {
    if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return *reinterpret_cast<const u32x4 *>(p);
}

// Decode attention of (up to UNITS consecutive 64-key splits, KV head g, row) on the matrix cores (bf16
// KV, D = 128, G <= 16): S^T = K Q^T with the K rows of the split's cache blocks as the A operand (one
// 16-key block per wavefront) and Q as a bf16 hi/lo pair; softmax statistics per head from the MFMA
// layout; O = P V with P (hi/lo) from LDS and V read transposed from an LDS tile.  UNITS == 1: partial
// outputs as attn_decode_task writes them, or with FINAL the output o / l.  UNITS == kMergeGroup: the
// state of the whole group of splits, combined as attn_merge combines the splits' own (the same bits),
// with the K (V) rows of the next split loaded while this one is multiplied.
template <int G, int D, bool FINAL, int UNITS, bool STREAM>
__global__ __launch_bounds__(256, UNITS == 1 ? 5 : 4) void attn_decode_mfma(AttnArgs a) {
    static_assert(D == 128 && G <= 16, "one 128-wide head, up to 16 query heads per KV head");
    static_assert(UNITS == 1 || (UNITS == kMergeGroup && !FINAL), "one split, or a merge group");
    constexpr int VROW = D + 8;                     // V tile row stride in bf16 (272 bytes)
    // UNITS == 1: one LDS area for the K tile (until the first barrier: each wavefront reads only its
    // own 16 keys) and then the V tile
    __shared__ uint4 v_tile[kChunk * VROW * 2 / 16];
    __shared__ uint4 k_tile[UNITS > 1 ? kChunk * D * 2 / 16 : 1];
    uint4 (*const ks)[D / 8] = reinterpret_cast<uint4 (*)[D / 8]>(UNITS > 1 ? k_tile : v_tile);   // [key][chunk ^ key % 16]
    uint16_t (*const vs)[VROW] = reinterpret_cast<uint16_t (*)[VROW]>(v_tile);
    __shared__ uint4 pf[2][2][64];                  // P A-fragments [key step][hi, lo][lane]
    __shared__ float wm[UNITS][4][16], wl[UNITS][4][16];
    const int split0 = blockIdx.y * UNITS, g = blockIdx.x, row = blockIdx.z;
    const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int hq_total = a.n_q_heads, hkv = a.kv.n_kv_heads;
    // Q^T fragments first (they depend on the row only): head l16 (heads past G load head G - 1 and
    // are zeroed below), d 32 s + 8 lq
    const float *qp = a.q + (size_t)row * hq_total * D + (size_t)(g * G + min(l16, G - 1)) * D + 8 * lq;
    float4 qv[4][2];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        qv[s][0] = *reinterpret_cast<const float4 *>(qp + 32 * s);
        qv[s][1] = *reinterpret_cast<const float4 *>(qp + 32 * s + 4);
    }
    const int sidx = row / a.rows_per_seq;
    const int pos = a.meta.pos0(sidx) + row % a.rows_per_seq;
    const int slot = a.meta.seq_slot(sidx);
    const int ctx = pos + 1, kbeg0 = split0 * a.split_keys;
    if (kbeg0 >= ctx || slot < 0) return;  // (slot tested so that both metadata loads go out together)
    const int units = UNITS > 1 ? min(UNITS, (ctx - kbeg0 + a.split_keys - 1) / a.split_keys) : 1;
    const size_t blk_stride = (size_t)2 * hkv * kBlockTokens * D;
    const uint16_t *pool = static_cast<const uint16_t *>(a.kv.pool);
    // every key of wavefront w (16 w .. 16 w + 15 of a split, clamped into it) lies in one cache
    // block (splits start on a block boundary): one block-table entry per wavefront and split
    const int *table = a.kv.block_table + (size_t)slot * a.kv.max_blocks;
    int blk[UNITS];
#pragma unroll
    for (int u = 0; u < UNITS; ++u)
        blk[u] = table[min(kbeg0 + u * a.split_keys + 16 * wave, ctx - 1) / kBlockTokens];
    // K and V rows, 4 keys x 256 contiguous bytes per load instruction (16 keys x 64 bytes, the
    // MFMA fragment layout read straight from memory, streams poorly): instruction i, lane l: key
    // 16 wave + 4 i + lq of the split (clamped into it); K: 16-byte d chunk l16 ^ (4 i + lq),
    // stored in the K tile at [key][l16]; V: chunk l16
    u32x4 kr[4], vr[4];
    auto load_k = [&](int u) {
        const uint16_t *kb = pool + (size_t)blk[u] * blk_stride + (size_t)g * kBlockTokens * D;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int key = min(kbeg0 + u * a.split_keys + 16 * wave + 4 * i + lq, ctx - 1);
            kr[i] = load_cache16<STREAM>(kb + (size_t)(key % kBlockTokens) * D + 8 * (l16 ^ (4 * i + lq)));
        }
    };
    auto load_v = [&](int u) {
        const uint16_t *vb = pool + (size_t)blk[u] * blk_stride + (size_t)(hkv + g) * kBlockTokens * D;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int key = min(kbeg0 + u * a.split_keys + 16 * wave + 4 * i + lq, ctx - 1);
            vr[i] = load_cache16<STREAM>(vb + (size_t)(key % kBlockTokens) * D + 8 * l16);
        }
    };
    load_k(0);
    load_v(0);
    // every K and V load in flight before any is used (left alone, the scheduler issues half of
    // them after the first products, a second round trip to memory)
    __builtin_amdgcn_sched_barrier(0);
    // Q^T as a bf16 hi/lo pair, scaled by 1/sqrt(d)
    const float scale = 1.f / sqrtf((float)D);
    bf16x8_t qh[4], ql[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const float q8[8] = {qv[s][0].x, qv[s][0].y, qv[s][0].z, qv[s][0].w,
                             qv[s][1].x, qv[s][1].y, qv[s][1].z, qv[s][1].w};
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = l16 < G ? q8[j] * scale : 0.f;
        split8(x, qh[s], ql[s]);
    }
    // o[u][nb][i]: split u, head 4 lq + i, d 32 wave + 16 nb + l16
    f32x4_t o[UNITS][2];
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        if (u > 0 && u >= units) break;
        const int n = min(a.split_keys, ctx - kbeg0 - u * a.split_keys);
        const bool more = u + 1 < UNITS && u + 1 < units;
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4 *>(&ks[16 * wave + 4 * i + lq][l16]) = kr[i];
        if (more) load_k(u + 1);
        __builtin_amdgcn_sched_barrier(0);
        // K fragments: key 16 wave + l16, d 32 s + 8 lq, i.e. chunk 4 s + lq (the tile holds chunk c of
        // key k at c ^ k % 16: every 16 lanes of a read meet distinct banks)
        f32x4_t sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const bf16x8_t kf = as_bf(ks[16 * wave + l16][(4 * s + lq) ^ l16]);
            sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qh[s], sc, 0, 0, 0);
            sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, ql[s], sc, 0, 0, 0);
        }
        // sc[i]: score of key 16 wave + 4 lq + i for head l16
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (16 * wave + 4 * lq + i >= n) sc[i] = -INFINITY;
            mx = fmaxf(mx, sc[i]);
        }
        mx = fmaxf(mx, lane_xor(mx, 16));
        mx = fmaxf(mx, lane_xor(mx, 32));
        if (lane < 16) wm[u][wave][lane] = mx;
        // every wavefront's K reads (UNITS == 1) and its reads of the last split's V and P are done
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4 *>(&vs[16 * wave + 4 * i + lq][8 * l16]) = vr[i];
        if (more) load_v(u + 1);
        __builtin_amdgcn_sched_barrier(0);
        const float mh = fmaxf(fmaxf(wm[u][0][l16], wm[u][1][l16]), fmaxf(wm[u][2][l16], wm[u][3][l16]));
        float p[4], ls = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = sc[i] == -INFINITY ? 0.f : expf(sc[i] - mh);
            ls += p[i];
        }
        ls += lane_xor(ls, 16);
        ls += lane_xor(ls, 32);
        if (lane < 16) wl[u][wave][lane] = ls;
        // P fragment slot of key 16 wave + 4 lq + i: key step wave / 2, lane l16 + 16 (2 (wave % 2) + lq / 2),
        // elements 4 (lq % 2) + i
        {
            uint16_t hb[4], lb[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const __bf16 h = (__bf16)p[i];
                const __bf16 l = (__bf16)(p[i] - (float)h);
                hb[i] = __builtin_bit_cast(uint16_t, h);
                lb[i] = __builtin_bit_cast(uint16_t, l);
            }
            const int L = l16 + 16 * (2 * (wave & 1) + (lq >> 1));
            uint2 h2 = make_uint2(hb[0] | ((uint32_t)hb[1] << 16), hb[2] | ((uint32_t)hb[3] << 16));
            uint2 l2 = make_uint2(lb[0] | ((uint32_t)lb[1] << 16), lb[2] | ((uint32_t)lb[3] << 16));
            reinterpret_cast<uint2 *>(&pf[wave >> 1][0][L])[lq & 1] = h2;
            reinterpret_cast<uint2 *>(&pf[wave >> 1][1][L])[lq & 1] = l2;
        }
        __syncthreads();
        // O block (heads 0..15) x (d 32 wave + 16 nb .. + 15), K = the split's 64 keys in two steps
        o[u][0] = o[u][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const bf16x8_t ph = as_bf(pf[t][0][lane]), pl = as_bf(pf[t][1][lane]);
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                const int d = 32 * wave + 16 * nb + l16;
                bf16x8_t vb;
#pragma unroll
                for (int j = 0; j < 8; ++j) vb[j] = __builtin_bit_cast(__bf16, vs[32 * t + 8 * lq + j][d]);
                o[u][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph, vb, o[u][nb], 0, 0, 0);
                o[u][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl, vb, o[u][nb], 0, 0, 0);
            }
        }
    }
    auto unit_max = [&](int u, int h) {
        return fmaxf(fmaxf(wm[u][0][h], wm[u][1][h]), fmaxf(wm[u][2][h], wm[u][3][h]));
    };
    auto unit_sum = [&](int u, int h) { return ((wl[u][0][h] + wl[u][1][h]) + wl[u][2][h]) + wl[u][3][h]; };
    if (FINAL) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int h = 4 * lq + i;
            if (h >= G) continue;
            const float l_sum = unit_sum(0, h);
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                const int col = (g * G + h) * D + 32 * wave + 16 * nb + l16;
                if (row < a.pair_rows) {
                    uint16_t *p = a.out_pair + row * a.out_pair_ld + pair_at(col);
                    split_pair(o[0][nb][i] / l_sum, p[0], p[32]);
                } else {
                    a.out[(size_t)row * hq_total * D + col] = o[0][nb][i] / l_sum;
                }
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int h = 4 * lq + i;
        if (h >= G) continue;
        const size_t pi = ((size_t)row * hq_total + g * G + h) * a.max_splits + blockIdx.y;
        if constexpr (UNITS == 1) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) a.part_o[pi * D + 32 * wave + 16 * nb + l16] = o[0][nb][i];
            if (wave == 0 && l16 == 0) {
                a.part_ml[pi * 2 + 0] = unit_max(0, h);
                a.part_ml[pi * 2 + 1] = unit_sum(0, h);
            }
        } else {
            float m[UNITS], l[UNITS], w[UNITS];
#pragma unroll
            for (int u = 0; u < UNITS; ++u) m[u] = u < units ? unit_max(u, h) : -INFINITY;
            const float mg = group_weights(m, units, w);
#pragma unroll
            for (int u = 0; u < UNITS; ++u) l[u] = u < units ? unit_sum(u, h) : 0.f;
            const float lg = group_sum(l, w, units);
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                float v[UNITS];
#pragma unroll
                for (int u = 0; u < UNITS; ++u) v[u] = u < units ? o[u][nb][i] : 0.f;
                a.part_o[pi * D + 32 * wave + 16 * nb + l16] = group_sum(v, w, units);
            }
            if (wave == 0 && l16 == 0) {
                a.part_ml[pi * 2 + 0] = mg;
                a.part_ml[pi * 2 + 1] = lg;
            }
        }
    }
}

constexpr int KT = 32;                 // keys per tile of the prefill kernel
typedef short s16x4_t __attribute__((ext_vector_type(4)));

// One workgroup: 128 query rows = G heads x (128 / G) consecutive positions of one sequence, one
// KV head.  Wave w owns rows 32 w .. 32 w + 31 (row r: head r / BQ, position offset r % BQ).
// Per 32-key tile: S^T = K Q^T (lane = one query column, 16 keys), online softmax in-lane,
// O^T += V^T P^T.  q and p enter the MFMAs as bf16 hi + lo pairs.
//
// K and V tiles are copied as they lie in the cache (rows of D elements) into a ring of S stages of LDS by
// global_load_lds, two tiles ahead of their use, one barrier per tile; no registers stage them.  The
// 16-byte chunks of a row are permuted by the copies' lane addresses so that the K fragments' reads (16
// rows, one chunk) and the transposing reads of V (4 rows x 64 bytes) meet distinct banks.  A wavefront
// multiplies tile t + 1's K by Q while it takes the softmax of tile t: the two are independent, and with
// one wavefront per SIMD (a prompt's chunk of 500 tokens is 256 workgroups) nothing else fills the
// matrix pipe during the softmax.  Before, tiles went through registers into padded LDS rows, V element by
// element into its transpose, between two barriers per tile.  4 x 2048 tokens of the 70B-shaped stage 940
// -> 590 us, 500 tokens of the 32B-shaped one after 0 to 3000 others 130 -> 92 us on average, 1024 of the
// 8B-shaped one 70 -> 54 us; bit-identical.
template <int G, int D>
__global__ __launch_bounds__(256, 2) void attn_prefill_mfma(AttnArgs a) {
    constexpr int BQ = 128 / G;
    constexpr int KK = D / 16;          // k16 steps over d
    constexpr int NB = D / 32;          // 32-row blocks of d in O^T
    constexpr int S = 4;                // stages
    constexpr int ROW = 2 * D, CH = D / 8;                // bytes and 16-byte chunks of a key's row
    constexpr int TILE = KT * ROW, STAGE = 2 * TILE;      // K tile, then V tile
    constexpr int KPC = 1024 / ROW, CP = KT / KPC / 4;    // keys per copy; copies of K (and of V) per wavefront
    __shared__ __align__(256) char lds[S * STAGE];   // (whole rows: addresses are permuted by XOR)
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const int qb = gridDim.z - 1 - blockIdx.z, g = blockIdx.x, sidx = blockIdx.y;  // the longest blocks of all first
    const int T = a.rows_per_seq;
    const int pos0 = a.meta.pos0(sidx), slot = a.meta.seq_slot(sidx);
    const int hkv = a.kv.n_kv_heads, hq_total = a.n_q_heads;
    const size_t q_ld = (size_t)hq_total * D;
    const int *table = a.kv.block_table + (size_t)slot * a.kv.max_blocks;
    const size_t blk_bytes = (size_t)2 * hkv * kBlockTokens * ROW, v_off = (size_t)hkv * kBlockTokens * ROW;
    const char *pool = static_cast<const char *>(a.kv.pool) + (size_t)g * kBlockTokens * ROW;

    // keys of the block's last query, and tiles; of the wavefront's own rows: the tiles that they see, and
    // their first position (a tile that ends before it hides nothing)
    const int n_keys = pos0 + min(T, (qb + 1) * BQ), n_tiles = (n_keys + KT - 1) / KT;
    const int first = BQ > 32 ? 32 * wave % BQ : 0;
    const int wave_min = pos0 + min(qb * BQ + first, T - 1);
    const int wave_tiles = qb * BQ + first >= T ? 0 : (pos0 + min(T, qb * BQ + (BQ > 32 ? first + 32 : BQ)) + KT - 1) / KT;

    // The copies of one tile by this wavefront: 8 consecutive keys of K and of V (one cache block).  Keys past
    // the last one: that one (in bounds; their scores are masked).
    const int lr = lane / CH, lc = lane % CH;
    auto wave_key = [&](int tile) { return min(tile * KT + 8 * wave, n_keys - 1); };
    auto copy = [&](int tile, int blk) {
        const int k0 = wave_key(tile) & ~7, last = n_keys - 1 - k0;   // (8 keys start at a multiple of 8)
        const char *const kp = pool + (size_t)blk * blk_bytes + (size_t)(k0 % kBlockTokens) * ROW;
        const uint32_t st = lds_base + tile % S * STAGE + 8 * wave * ROW;
#pragma unroll
        for (int i = 0; i < CP; ++i) {
            const int r = KPC * i + lr, row = 8 * wave + r;   // key of the copy's eight, and row of the tile
            const int kx = D == 128 ? row & 15 : (row >> 1) & 7, vx = D == 128 ? (row & 3) << 2 : (row & 2) << 1;
            const uint32_t src = (uint32_t)min(r, last) * ROW;
            dma16(src + 16 * (lc ^ kx), kp, st + 1024 * i);
            dma16(src + 16 * (lc ^ vx), kp + v_off, st + TILE + 1024 * i);
        }
    };
    // (a scalar load: the memory clobbers of the copies would have the compiler take a vector load, whose
    // wait would take in the copies ahead of it)
    typedef const __attribute__((address_space(4))) int *const_ints;
    auto block_of = [&](int tile) { return ((const_ints)(uintptr_t)table)[wave_key(tile) / kBlockTokens]; };
    int blk[S];
#pragma unroll
    for (int t = 0; t < S; ++t) blk[t] = block_of(t);
#pragma unroll
    for (int t = 0; t < S - 1; ++t) copy(t, blk[t]);   // (tiles past the last: its keys again, never read)
    int next_blk = blk[S - 1];

    // this lane's query (column) and its position
    const int r = wave * 32 + col, hh = r / BQ, t_q = qb * BQ + r % BQ;
    const bool qvalid = t_q < T;
    const int qpos = pos0 + (qvalid ? t_q : T - 1);
    const size_t qrow = (size_t)(sidx * T + (qvalid ? t_q : T - 1));
    // Q^T fragments: B[k = d 16 kk + 8 half + j][query col]
    bf16x8_t qh[KK], ql[KK];
    {
        const float scale = 1.4426950408889634f / sqrtf((float)D);   // log2(e) / sqrt(d): scores in base 2
        const float *qp = a.q + qrow * q_ld + (size_t)(g * G + hh) * D + 8 * half;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            float x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = qp[16 * kk + j] * scale;
            split8(x, qh[kk], ql[kk]);
        }
    }
    f32x16_t o[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[b][i] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    // S^T[key][query] = sum_d K[key][d] Q[query][d]: A = K (lane: key col, d 16 kk + 8 half)
    typedef const __attribute__((address_space(3))) u32x4 *lds16;
    typedef __attribute__((address_space(3))) s16x4_t *lds8;
    const uint32_t k_at = lds_base + col * ROW + 16 * (half ^ (D == 128 ? col & 15 : (col >> 1) & 7));
    auto scores = [&](int tile) {
        const uint32_t L = k_at + tile % S * STAGE;
        f32x16_t s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const bf16x8_t kf = __builtin_bit_cast(bf16x8_t, *(lds16)(L ^ (32 * kk)));   // chunk 2 kk + half, permuted
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qh[kk], s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, ql[kk], s, 0, 0, 0);
        }
        return s;
    };
    // lane holds keys k0 + 8 (i / 4) + 4 half + i % 4 for query column col
    auto mask = [&](f32x16_t &s, int k0) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (k0 + 8 * (i / 4) + 4 * half + (i % 4) > qpos) s[i] = -INFINITY;
    };
    // The softmax of a tile's scores s in pieces: scores -> p (as a pair) and the factor of what came before.
    constexpr int PIECES = 11;
    bf16x8_t ph[2], pl[2];
    float ref, alpha, p[16], ps;
    auto pair_of = [&](int i) {   // p[2 i] and p[2 i + 1]
#pragma unroll
        for (int j = 2 * i; j < 2 * i + 2; ++j) {
            ph[j / 8][j % 8] = (__bf16)p[j];
            pl[j / 8][j % 8] = (__bf16)(p[j] - (float)ph[j / 8][j % 8]);
        }
    };
    auto piece = [&](const f32x16_t &s, int x) {
        if (x == 0) {
            ref = s[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) ref = fmaxf(ref, s[i]);
        } else if (x == 1) {
            const float m_new = fmaxf(m_run, fmaxf(ref, lane_xor(ref, 32)));
            ref = m_new == -INFINITY ? 0.f : m_new;
            alpha = __builtin_amdgcn_exp2f(m_run - ref);   // (0 on the first tile)
            m_run = m_new;
            ps = 0.f;
        } else if (x < PIECES - 1) {
            const int i = x - 2;
#pragma unroll
            for (int j = 2 * i; j < 2 * i + 2; ++j) {
                p[j] = __builtin_amdgcn_exp2f(s[j] - ref);
                ps += p[j];
            }
            if (i > 0) pair_of(i - 1);
        } else {
            pair_of(7);
            ps += lane_xor(ps, 32);
            l_run = l_run * alpha + ps;
        }
    };
    // The scores of `tile`, with the pieces of s's softmax behind the MFMAs (schedule fences keep them there).
    auto scores_and_softmax = [&](int tile, f32x16_t &s) {
        const uint32_t L = k_at + tile % S * STAGE;
        auto key_frag = [&](int kk) { return __builtin_bit_cast(bf16x8_t, *(lds16)(L ^ (32 * kk))); };
        f32x16_t n;
#pragma unroll
        for (int i = 0; i < 16; ++i) n[i] = 0.f;
        bf16x8_t kf[2] = {key_frag(0), key_frag(1)};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 2 * KK; ++q) {
            const int kk = q / 2;
            n = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk & 1], q & 1 ? ql[kk] : qh[kk], n, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if ((q & 1) && kk + 2 < KK) kf[kk & 1] = key_frag(kk + 2);
#pragma unroll
            for (int x = 0; x < PIECES; ++x)
                if (x * 2 * KK / PIECES == q) piece(s, x);
            __builtin_amdgcn_sched_barrier(0);
        }
        s = n;
    };
    // O^T[d][query] += sum_key V[key][d] P[query][key]; k index (8 half + j) of MFMA m is the lane's key
    // 16 m + 8 (j / 4) + 4 half + j % 4 = its p[8 m + j].  A transposing read gives 16 lanes the 4 keys x
    // 16 d that they point at (lane i: key i / 4, d 4 (i % 4) .. + 3) column-wise: lane i all keys of d i.
    const int vk = 4 * half + (lane & 15) / 4;   // key of this lane's piece, within 8
    const uint32_t v_at = lds_base + TILE + vk * ROW + 8 * (lane & 1) +
                          16 * ((((lane >> 4) & 1) * 2 + (lane & 3) / 2) ^ (D == 128 ? (vk & 3) << 2 : (vk & 2) << 1));
    auto values = [&](int tile) {
        if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {   // some lane's maximum moved
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[b][i] *= alpha;
        }
        const uint32_t L = v_at + tile % S * STAGE;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const uint32_t p = (L ^ (64 * b)) + 16 * m * ROW;
                const s16x4_t v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds8)p);
                const s16x4_t v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds8)(p + 8 * ROW));
                const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
                o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, ph[m], o[b], 0, 0, 0);
                o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pl[m], o[b], 0, 0, 0);
            }
    };

    wait_vm<(S - 2) * 2 * CP>();   // tile 0 has landed (this wavefront's share)
    lds_barrier();
    f32x16_t s = scores(0);
    for (int t = 0; t < n_tiles; ++t) {
        // tile t + 1 has landed everywhere; tile t - 1 has been read by all: its stage takes tile t + S - 1
        if (t + S - 2 < n_tiles) wait_vm<(S - 3) * 2 * CP>();
        else wait_vm<0>();   // (no copies behind it)
        wait_lgkm<0>();
        lds_barrier();
        if (t + S - 1 < n_tiles) {
            copy(t + S - 1, next_blk);
            next_blk = block_of(t + S);
        }
        if (t >= wave_tiles) continue;   // wave-uniform, as the following: past them every key is masked
        if (t * KT + KT - 1 > wave_min) mask(s, t * KT);
        scores_and_softmax(t + 1, s);   // (past the wavefront's last tile: scores of no meaning, not used)
        values(t);
    }
    if (!qvalid) return;
    // O^T[d = 32 b + 8 (i / 4) + 4 half + i % 4][query col]
    const float inv = 1.f / l_run;
    uint16_t *prow = a.out_pair + qrow * a.out_pair_ld;   // four consecutive d of one 32-wide block per store
    const int k0 = (g * G + hh) * D;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            store_pair4(prow + pair_at(k0 + 32 * b + 8 * j + 4 * half),
                        make_float4(o[b][4 * j] * inv, o[b][4 * j + 1] * inv, o[b][4 * j + 2] * inv,
                                    o[b][4 * j + 3] * inv));
}

// Prefill attention over an fp32 cache, in fp32 throughout, on v_mfma_f32_32x32x2_f32 (fp32 operands,
// products and sums; twice the vector ALUs' rate and none of their operand traffic).  One workgroup: 64
// query rows = G heads x 64 / G consecutive positions of one sequence, one KV head.  Wavefront w: rows
// 32 (w % 2) .. + 31 (row r: head r / BQ, position offset r % BQ) over the keys of half w / 2 of each
// 64-key tile; the two halves' states are merged through LDS at the end.  Where the call's blocks are few
// (prefill_key_ranges), the keys are cut into ranges of kRangeKeys, each a workgroup of its own, and attn_merge
// adds a row's states.  A row's result depends on its position and on which of the two its call is.  S^T = K Q^T, softmax in-lane, O^T += V^T P^T, where the lane layout of S^T is
// already the one of P^T's operand.  The k index of an MFMA is 8 u + j for lanes 0..31 and 8 u + 4 + j
// for the rest, so that operands load 16 bytes at a time.
// Bound by its MFMAs; 68 KB of LDS leave two workgroups per compute unit, one of which multiplies
// while the other loads.  2 x 600 tokens of the 13B-shaped stage (40 heads): a workgroup per row and
// KV head on the vector ALUs 700 us -> 186 us, without the pass that made the O projection's operand pair (9 us).
constexpr int kRangeKeys = 128;   // (whole tiles)
template <int G, int D>
__global__ __launch_bounds__(256, 2) void attn_prefill_f32(AttnArgs a) {
    constexpr int KEYS = 64, BQ = 64 / G;
    constexpr int KROW = D + 4, VROW32 = D + 8;   // row strides (padding: lanes on distinct banks)
    constexpr int QU = D / 8, NB = D / 32;
    __shared__ __align__(16) float sk[KEYS * KROW];
    __shared__ __align__(16) float sv[KEYS * VROW32];
    static_assert(KEYS * KROW >= 64 * (16 * NB + 2), "a wavefront's state fits where K (V) was");
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wq = wave & 1, kh = wave >> 1;
    const int ranges = a.grid_splits, range = blockIdx.z % ranges;
    const int qb = (gridDim.z - 1 - blockIdx.z) / ranges, g = blockIdx.x, sidx = blockIdx.y;  // the longest blocks of all first
    const int T = a.rows_per_seq;
    const int pos0 = a.meta.pos0(sidx), slot = a.meta.seq_slot(sidx);
    const int hkv = a.kv.n_kv_heads, hq_total = a.n_q_heads;
    const size_t q_ld = (size_t)hq_total * D;
    const int *table = a.kv.block_table + (size_t)slot * a.kv.max_blocks;
    const float *pool = static_cast<const float *>(a.kv.pool);
    const size_t blk_stride = (size_t)2 * hkv * kBlockTokens * D;

    // this lane's query (column) and its position
    const int r = 32 * wq + col, hh = r / BQ, t = qb * BQ + r % BQ;
    const bool qvalid = t < T;
    const int qpos = pos0 + (qvalid ? t : T - 1);
    const size_t qrow = (size_t)sidx * T + (qvalid ? t : T - 1);
    float q[QU][4];   // d 8 u + 4 half + j, scaled by 1 / sqrt(d)
    {
        const float scale = 1.f / sqrtf((float)D);
        const float *qp = a.q + qrow * q_ld + (size_t)(g * G + hh) * D + 4 * half;
#pragma unroll
        for (int u = 0; u < QU; ++u) {
            const float4 v = *reinterpret_cast<const float4 *>(qp + 8 * u);
            q[u][0] = v.x * scale;
            q[u][1] = v.y * scale;
            q[u][2] = v.z * scale;
            q[u][3] = v.w * scale;
        }
    }
    f32x16_t o[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[b][i] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    // the last and the first position of the block, the last of this wavefront (keys past it are
    // masked in every one of its rows)
    const int block_min = pos0 + qb * BQ;
    // the keys that this workgroup takes: first_key .. n_keys - 1
    const int first_key = range * kRangeKeys, all_keys = pos0 + min(T, (qb + 1) * BQ);
    const int n_keys = ranges > 1 ? min(all_keys, first_key + kRangeKeys) : all_keys;
    const int wave_max = pos0 + min(T, BQ > 32 ? qb * BQ + 32 * wq + 32 : (qb + 1) * BQ) - 1;

    for (int base = first_key; base < n_keys; base += KEYS) {
        __syncthreads();            // the previous tile's LDS reads are done
        // 64 keys x D of K and of V, 16 bytes per access; keys past the block's last: that one (their
        // scores are masked).  A row whose mask hides a key must not meet its V, which may hold an
        // infinity or NaN (0 x inf): a tile that hides keys notes whether any V of it does.
        constexpr int CH = D / 4, PER = 4;
        bool odd = false;
#pragma unroll 1
        for (int c0 = tid; c0 < KEYS * CH; c0 += 256 * PER) {
            f32x4_t kr[PER], vr[PER];
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int c = c0 + 256 * i, kp = min(base + c / CH, n_keys - 1);
                const float *p = pool + (size_t)table[kp / kBlockTokens] * blk_stride +
                                 ((size_t)g * kBlockTokens + kp % kBlockTokens) * D + c % CH * 4;
                kr[i] = *reinterpret_cast<const f32x4_t *>(p);
                vr[i] = *reinterpret_cast<const f32x4_t *>(p + (size_t)hkv * kBlockTokens * D);
            }
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int c = c0 + 256 * i;
                *reinterpret_cast<f32x4_t *>(sk + c / CH * KROW + c % CH * 4) = kr[i];
                *reinterpret_cast<f32x4_t *>(sv + c / CH * VROW32 + c % CH * 4) = vr[i];
                const float big = fmaxf(fmaxf(fabsf(vr[i].x), fabsf(vr[i].y)), fmaxf(fabsf(vr[i].z), fabsf(vr[i].w)));
                const float sum = (vr[i].x + vr[i].y) + (vr[i].z + vr[i].w);   // (NaN if any is)
                odd = odd || !(big < INFINITY) || sum != sum;
            }
        }
        const bool hides = base + KEYS - 1 > block_min;
        const bool careful = __syncthreads_or(hides && odd);
        const int k0 = base + 32 * kh;
        if (k0 > wave_max) continue;           // wave-uniform: every key of this half is masked
        f32x16_t s, s1;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = s1[i] = 0.f;
        const float *kp = sk + (32 * kh + col) * KROW + 4 * half;
#pragma unroll
        for (int u = 0; u < QU; u += 2) {
            const float4 x = *reinterpret_cast<const float4 *>(kp + 8 * u), y = *reinterpret_cast<const float4 *>(kp + 8 * u + 8);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, q[u][0], s, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(y.x, q[u + 1][0], s1, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, q[u][1], s, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(y.y, q[u + 1][1], s1, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, q[u][2], s, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(y.z, q[u + 1][2], s1, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, q[u][3], s, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(y.w, q[u + 1][3], s1, 0, 0, 0);
            if (u % 8 == 6) __builtin_amdgcn_sched_barrier(0);   // (all K reads at once would not fit the registers)
        }
        // register i: key k0 + 8 (i / 4) + 4 half + i % 4 of query column col
        float mt = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            s[i] = k0 + 8 * (i / 4) + 4 * half + i % 4 > qpos ? -INFINITY : s[i] + s1[i];
            mt = fmaxf(mt, s[i]);
        }
        mt = fmaxf(mt, lane_xor(mt, 32));
        const float m_new = fmaxf(m_run, mt);
        const float alpha = m_run == -INFINITY ? 0.f : expf(m_run - m_new);
        float ps = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            s[i] = s[i] == -INFINITY ? 0.f : expf(s[i] - m_new);
            ps += s[i];
        }
        ps += lane_xor(ps, 32);
        l_run = l_run * alpha + ps;
        m_run = m_new;
        if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {   // some lane's maximum moved
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[b][i] *= alpha;
        }
        if (careful) {   // key by key, hidden keys left out; in the order of the MFMAs' sums: the same bits
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float other = lane_xor(s[i], 32);
#pragma unroll 1
                for (int e = 0; e < 2; ++e) {
                    const int key = 8 * (i / 4) + 4 * e + i % 4;
                    if (k0 + key > qpos) continue;
                    const float p = e == half ? s[i] : other;
                    const float *vr = sv + (32 * kh + key) * VROW32 + 4 * half;
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
#pragma unroll
                        for (int j = 0; j < 16; ++j) o[b][j] = fmaf(p, vr[32 * b + 8 * (j / 4) + j % 4], o[b][j]);
                        __builtin_amdgcn_sched_barrier(0);   // (registers)
                    }
                }
            }
            continue;
        }
        const float *vp = sv + (32 * kh + 4 * half) * VROW32 + col;
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int b = 0; b < NB; ++b)
                o[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(vp[(8 * (i / 4) + i % 4) * VROW32 + 32 * b], s[i], o[b], 0, 0, 0);
    }

    // the second key half's state joins the first's (which holds the first key: empty for no row that sees it)
    __syncthreads();
    float *const st = (wq ? sv : sk) + lane;
    if (kh == 1) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) st[64 * (16 * b + i)] = o[b][i];
        st[64 * 16 * NB] = m_run;
        st[64 * (16 * NB + 1)] = l_run;
    }
    __syncthreads();
    if (kh == 1 || !qvalid || first_key > qpos) return;
    const float m1 = st[64 * 16 * NB], l1 = st[64 * (16 * NB + 1)];
    const float m = fmaxf(m_run, m1);
    const bool both = m1 > -INFINITY || l1 != 0.f;   // (l1 is NaN, too, if every score of the half is)
    const float w0 = expf(m_run - m), w1 = both ? expf(m1 - m) : 0.f;
    const float l = both ? fmaf(l1, w1, l_run * w0) : l_run * w0;
    const int k0 = (g * G + hh) * D;
    const size_t state = (qrow * hq_total + g * G + hh) * a.max_splits + range;   // ranges > 1
    if (ranges > 1 && half == 0) {
        a.part_ml[2 * state + 0] = m;
        a.part_ml[2 * state + 1] = l;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j) {   // O^T[d = 32 b + 8 j + 4 half + x][query col]
            float v[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int i = 4 * j + x;
                v[x] = o[b][i] * w0;
                if (both) v[x] = fmaf(st[64 * (16 * b + i)], w1, v[x]);
                if (ranges == 1) v[x] /= l;
            }
            const int c = 32 * b + 8 * j + 4 * half;
            const float4 v4 = make_float4(v[0], v[1], v[2], v[3]);
            if (ranges > 1) *reinterpret_cast<float4 *>(a.part_o + state * D + c) = v4;
            else store_pair4(a.out_pair + qrow * a.out_pair_ld + pair_at(k0 + c), v4);
        }
}

template <int G, int D>
hipError_t launch_gd(const AttnArgs &a, hipStream_t st) {
    const int hkv = a.kv.n_kv_heads;
    if (a.split_keys == 0) {
        if (a.n_seqs * a.rows_per_seq != a.rows || a.pair_rows != a.rows) return hipErrorInvalidValue;
        if (a.kv_fp32) {
            constexpr int BQ = 64 / G;
            if (a.grid_splits < 1) return hipErrorInvalidValue;
            dim3 grid(hkv, a.n_seqs, (a.rows_per_seq + BQ - 1) / BQ * a.grid_splits);
            STG_LAUNCH((attn_prefill_f32<G, D>), grid, dim3(256), 0, st, a);
            if (a.grid_splits > 1) {
                AttnArgs m = a;
                m.split_keys = kRangeKeys;
                STG_LAUNCH((attn_merge<D, false>), dim3((unsigned)a.n_q_heads, (unsigned)a.rows), dim3(256), 0, st, m);
            }
        } else {
            constexpr int BQ = 128 / G;
            dim3 grid(hkv, a.n_seqs, (a.rows_per_seq + BQ - 1) / BQ);
            STG_LAUNCH((attn_prefill_mfma<G, D>), grid, dim3(256), 0, st, a);
        }
        return hipGetLastError();
    }
    if (a.split_keys != kChunk || a.max_splits > kMaxDecodeSplits || a.rows_per_seq <= 0)
        return hipErrorInvalidValue;
    // KV heads fastest: workgroups that start together read the heads of the same cache blocks, which lie
    // side by side (64 KB of a 70B-shaped block, 4 KB per head and workgroup).  With the splits fastest they read the
    // same 4 KB of every 64: 16 rows at 7900 tokens of the 70B-shaped stage 116 -> 99 us, 8 rows at 7000 of
    // the 8B-shaped one 44 -> 40.
    dim3 grid(hkv, a.grid_splits, a.rows);
    auto merge = [&](auto grouped) {
        STG_LAUNCH((attn_merge<D, decltype(grouped)::value>), dim3((unsigned)a.n_q_heads, (unsigned)a.rows), dim3(256), 0, st, a);
        return hipGetLastError();
    };
    [[maybe_unused]] auto mfma = [&](auto units) {
        constexpr int U = decltype(units)::value;
        if constexpr (D == 128) {
            if (a.stream_kv) STG_LAUNCH((attn_decode_mfma<G, D, false, U, true>), grid, dim3(256), 0, st, a);
            else STG_LAUNCH((attn_decode_mfma<G, D, false, U, false>), grid, dim3(256), 0, st, a);
        }
    };
    if (a.grid_splits == 1) {   // every row within one split: its output directly, no merge
        if (a.kv_fp32)
            STG_LAUNCH((attn_decode_kernel<G, D, true, true>), grid, dim3(256), 0, st, a);
        else if constexpr (D == 128)
            STG_LAUNCH((attn_decode_mfma<G, D, true, 1, false>), grid, dim3(256), 0, st, a);
        else
            STG_LAUNCH((attn_decode_kernel<G, D, false, true>), grid, dim3(256), 0, st, a);
        return hipGetLastError();
    }
    if constexpr (D == 128) {
        // A workgroup per group of splits where there are at least 48 group outputs per compute unit (groups of
        // the longest row x query heads x rows): the partial outputs, 512 bytes per split and query head written
        // and read again, then cost more than what the larger workgroups lose (with four wavefronts per SIMD
        // instead of five, and a coarser last round).  Splits and merge, a workgroup per split -> per group:
        // 70B-shaped 16 rows at 7900 tokens (31744 outputs) 113 -> 104 us, 32 at 2000 (16384) 61.9 -> 57.5,
        // 8 at 7900 (15872) 60.2 -> 57.8, 8B-shaped 64 at 2000 (16384) 101 -> 96; below, 64 at 1100 (10240) 59.9
        // against 61.9, 16 at 4000 (8192) 52.0 against 54.6, 13B-shaped 16 at 2000 (5120) 105.8 against 111.
        const int groups = (a.grid_splits + kMergeGroup - 1) / kMergeGroup;
        if (!a.kv_fp32 && (long)groups * a.n_q_heads * a.rows >= 48L * device_compute_units()) {
            grid.y = groups;
            mfma(std::integral_constant<int, kMergeGroup>{});
            const hipError_t e = hipGetLastError();
            return e != hipSuccess ? e : merge(std::true_type{});
        }
    }
    if (a.kv_fp32)
        STG_LAUNCH((attn_decode_kernel<G, D, true, false>), grid, dim3(256), 0, st, a);
    else if constexpr (D == 128)
        mfma(std::integral_constant<int, 1>{});
    else
        STG_LAUNCH((attn_decode_kernel<G, D, false, false>), grid, dim3(256), 0, st, a);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : merge(std::false_type{});
}

}  // namespace

hipError_t launch_attention(const AttnArgs &a, hipStream_t st) {
    if (a.rows <= 0) return hipSuccess;
    const int G = a.n_q_heads / a.kv.n_kv_heads;
    const int D = a.kv.head_dim;
#define STG_ATTN_CASE(GG, DD) \
    if (G == GG && D == DD) return launch_gd<GG, DD>(a, st);
    STG_ATTN_CASE(1, 64) STG_ATTN_CASE(2, 64) STG_ATTN_CASE(4, 64) STG_ATTN_CASE(8, 64)
    STG_ATTN_CASE(1, 128) STG_ATTN_CASE(2, 128) STG_ATTN_CASE(4, 128) STG_ATTN_CASE(8, 128)
#undef STG_ATTN_CASE
    return hipErrorInvalidValue;
}

// A block alone takes 3.6 us (d = 64) to 6.5 us (d = 128) per 64 keys, one tile after the other; with few blocks
// nothing else runs meanwhile, and a workgroup per row, as it was before the tiles, was faster over long contexts.
// Calls of an fp32 cache, one layer, us, a workgroup per row / blocks with all keys / key ranges: tiny stage, 2
// tokens after 4000 others 158 / 284 / 65; hkv 2, G 4, d 128, 300 tokens after 4000 490 / 577 / 196; 8B-shaped, 16
// after 4000 795 / 533 / 141; 13B-shaped, 8 after 8000 1136 / 1094 / 321.  Up to 64 blocks: from 88 on (700 tokens,
// hkv 2, G 4) all keys in a block beat the workgroup per row at every context (436 against 529 at 4000), and the
// states of 64 blocks' rows stay below 70 MB per 4000 tokens of context.  Ranges of 256 keys: 5-10 us slower below
// 500 tokens, 3-5% faster at 3000.
int prefill_key_ranges(int n_seqs, int T, int longest, int n_q_heads, int n_kv_heads, bool kv_fp32) {
    const int per = 64 / (n_q_heads / n_kv_heads);   // positions of a query block
    if (!kv_fp32 || (long)n_kv_heads * n_seqs * ((T + per - 1) / per) > 64) return 1;
    return (longest + kRangeKeys - 1) / kRangeKeys;
}

bool attention_supported(int group, int head_dim) {
    return (group == 1 || group == 2 || group == 4 || group == 8) && (head_dim == 64 || head_dim == 128);
}

}  // namespace stg
