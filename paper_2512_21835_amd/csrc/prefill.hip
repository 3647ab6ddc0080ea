// Projections of prefill, and of decode calls of more than 16 rows, on the matrix cores: C[M, N] =
// A[M, K] . W[N, K]^T with bf16 weights W and
// an fp32 activation A taken as the exact-sum pair A = hi + lo of two bf16 matrices (hi = bf16(A),
// lo = bf16(A - hi); the pair keeps ~16 bits of A's mantissa, a single bf16 only 8).  Each 16-wide
// k step issues v_mfma_f32_32x32x16_bf16 twice per output block, hi then lo, accumulating in fp32.
// The pair is stored interleaved by 32-wide k blocks (hi block, then lo block, per row), so the
// operand bytes of one k tile of a row are 128 contiguous bytes.
//
// Tiling: gemm_tile_kernel (K a multiple of 32), a workgroup of 4 wavefronts per tile of C, copies its
// operands global -> LDS directly into a ring of three stages.  Up to 32 and 64 rows 32 x 128 and 64 x 128
// (or 112 columns), beyond that 256 x 256, 128 x 256 or 128 x 128 by the least estimated time; up to
// kFewRows rows K may be cut into ranges besides (gemm_plan).  gemm_kernel (any K) stages 128 x 128 tiles
// through registers into two LDS stages, one tile ahead.  Every fragment read is one
// conflict-free ds_read_b128 per lane.  Workgroups that share a weight tile are adjacent in launch
// order (x over M tiles), so each weight tile is read from HBM once and re-served from L2.
//
// The producers of A write the hi/lo pair directly: RMSNorm (before QKV and gate/up), the
// attention output (before O) and the SwiGLU of the gate/up output (before down).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "lanes.h"
#include "lds_dma.h"
#include "pair.h"
#include "part_sum.h"
#include "stage_kernels.h"

namespace stg {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int BM = 128, BN = 128, BK = 32;
constexpr int kFrag = (BM / 32) * (BK / 16) * 64;  // 16-byte fragment slots per operand tile (512)

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4 &v) {
    bf16x8 r;
    __builtin_memcpy(&r, &v, 16);
    return r;
}

// LDS slot of 16-byte chunk `ch` (k offset 8 ch) of tile row `row`.
__device__ __forceinline__ int frag_slot(int row, int ch) {
    return ((row >> 5) * (BK / 16) + (ch >> 1)) * 64 + (row & 31) + 32 * (ch & 1);
}

// Stores one 32 x 32 accumulator block (rows mb .. mb + 31, this lane's column c): register r of
// lane l is row mb + 8 (r / 4) + 4 (l / 32) + r % 4.  RESIDUAL: for a block inside M all 16
// residual values are loaded before any sum is stored, in straight-line code, so their loads are in
// flight together and the stores wait for nothing (out may alias res: each element is read and
// written by this lane only, read first).  A block crossing M stores element by element.
template <int MODE>
__device__ __forceinline__ void store_block(const GemmArgs &a, const f32x16 &acc, int mb, int M, int c, int lane) {
    const size_t o0 = (size_t)(mb + 4 * (lane >> 5)) * a.ldo + c;
    auto off = [&](int r) { return o0 + (size_t)(8 * (r >> 2) + (r & 3)) * a.ldo; };
    if (mb + 32 <= M) {   // the same for the whole wavefront
        float rv[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) rv[r] = MODE == GEMM_RESIDUAL ? a.res[off(r)] : 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) a.out[off(r)] = MODE == GEMM_RESIDUAL ? rv[r] + acc[r] : acc[r];
        return;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int m = mb + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (m < M) a.out[off(r)] = MODE == GEMM_RESIDUAL ? a.res[off(r)] + acc[r] : acc[r];
    }
}

template <int MODE>
__global__ __launch_bounds__(256) void gemm_kernel(GemmArgs a) {
    __shared__ uint4 lds[2][3][kFrag];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
    const uint16_t *W = a.w[blockIdx.z];
    const int M = a.M, N = a.N, K = a.K;

    // global -> register tile load: chunk q = tid + 256 i, row q / 4, 16-byte chunk q % 4
    uint4 rh[2], rl[2], rw[2];
    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = tid + 256 * i, row = q >> 2, ch = q & 3, k = k0 + ch * 8;
            const bool kin = k < K;
            const int m = m0 + row, n = n0 + row;
            rh[i] = rl[i] = rw[i] = make_uint4(0, 0, 0, 0);
            if (kin && m < M) {
                const uint16_t *p = a.a + (size_t)m * a.lda + pair_at(k);
                rh[i] = *reinterpret_cast<const uint4 *>(p);
                rl[i] = *reinterpret_cast<const uint4 *>(p + 32);
            }
            if (kin && n < N) rw[i] = *reinterpret_cast<const uint4 *>(W + (size_t)n * K + k);
        }
    };
    auto store = [&](int st) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = tid + 256 * i;
            const int s = frag_slot(q >> 2, q & 3);
            lds[st][0][s] = rh[i];
            lds[st][1][s] = rl[i];
            lds[st][2][s] = rw[i];
        }
    };

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    load(0);
    store(0);
    int st = 0;
    for (int k0 = 0; k0 < K; k0 += BK) {
        __syncthreads();
        const bool more = k0 + BK < K;
        if (more) load(k0 + BK);
#pragma unroll
        for (int step = 0; step < BK / 16; ++step) {
            bf16x8 ah[2], al[2], bw[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int sa = ((wm * 2 + b) * (BK / 16) + step) * 64 + lane;
                const int sb = ((wn * 2 + b) * (BK / 16) + step) * 64 + lane;
                ah[b] = as_bf16x8(lds[st][0][sa]);
                al[b] = as_bf16x8(lds[st][1][sa]);
                bw[b] = as_bf16x8(lds[st][2][sb]);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bw[j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], bw[j], acc[i][j], 0, 0, 0);
                }
        }
        if (more) store(st ^ 1);
        st ^= 1;
    }

    // result register r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32 of the block
    const int col_off = a.out_col[blockIdx.z];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = n0 + wn * 64 + j * 32 + (lane & 31);
            if (n >= N) continue;
            store_block<MODE>(a, acc[i][j], m0 + wm * 64 + i * 32, M, col_off + n, lane);
        }
}

constexpr int kTurn = 896;   // a whole number of the gate/up rows of any tile: 56, 64 or 128

// Workgroup tile of gemm_tile_kernel: 4 wavefronts as WM x WN, each MB x NB blocks of 32 x 32; K
// advances BK (32 or 64) at a time through S stages of LDS.  ONE: calls of at most TM rows, whose
// weights no other workgroup reads.
template <int WM_, int WN_, int MB_, int NB_, int BK_, int S_, bool ONE_ = false>
struct Tile {
    static constexpr bool ONE = ONE_;
    static constexpr int WM = WM_, WN = WN_, MB = MB_, NB = NB_, TK = BK_, S = S_;
    static constexpr int TM = 32 * WM * MB, TN = 32 * WN * NB;   // rows of the activation and weight tiles
    static constexpr int STEPS = TK / 16;                        // MFMA k steps per k tile
    static constexpr int A_BYTES = TM * TK * 4, W_BYTES = TN * TK * 2, STAGE = A_BYTES + W_BYTES;
    static constexpr int AI = A_BYTES / 4096, WI = W_BYTES / 4096, D = AI + WI;   // copies per wavefront per k tile
    static constexpr int LDS = S * STAGE;
    static_assert(WM * WN == 4 && (TK == 32 || TK == 64) && S >= 2, "four wavefronts");
    static_assert(LDS <= 160 * 1024, "LDS of a compute unit");
};

// The same product as gemm_kernel (same MFMAs in the same order for every tile shape: bit-identical
// results) for K a multiple of TK, with the operand tiles copied into a ring of S LDS stages by
// global_load_lds, so that no registers stage them.
//
// LDS layout.  Both tiles hold 128-byte rows of eight 16-byte segments (weights: 64 k; activation:
// the hi and lo of 32 k, one sub-tile per 32 k), segment g of row r at slot 8 r + (g ^ ((r >> 1) &
// 7)): one copy instruction moves 8 rows x 128 contiguous bytes (full cache lines), and the 32 x 32
// fragment reads (lane l: row l % 32, 8 k at l / 32) touch every LDS bank once per 16 lanes.  With
// TK = 32 a weight row is 64 bytes, four segments, segment s of row r at slot 4 r + (s ^ ((r >> 2)
// & 3)): 16 rows x 64 bytes per copy.
//
// Pipeline.  One wavefront per SIMD with the large tiles: nothing else hides a wavefront's stalls, so
// the instruction order is fixed by hand.  While the MFMAs of one 16-deep k step run, the fragments
// of the next are read into a second register set and a share of the copies of a later tile is
// issued, each behind an MFMA of its own (schedule fences keep them there): copies issued three in
// a row, and a step's fragment reads in one burst ahead of its MFMAs, had left the matrix pipe idle
// while all four wavefronts queued at the LDS and texture units (8192 rows of the 70B-shaped layer,
// before -> now: gate/up 12.06 -> 11.1 ms, down 5.87 -> 5.24, QKV 2.12 -> 1.91; pipe busy 66 ->
// 82-91% of the cycles, the clock falling from 1.82 to 1.6 GHz: the power limit is the bound now.
// 1024 rows of the 8B-shaped layer, 128 x 128 tiles: down 277 -> 211 us, O 84 -> 66).
// The barrier of tile t stands before its last step, by when every wavefront has read its last
// fragment of the tile: the stage then takes tile t + S, whose copies are issued over that last
// step and the first steps of tile t + 1; what the barrier waits for is tile t + 1, issued S - 1
// tiles before.
//
// K ranges (calls of up to kFewRows rows).  blockIdx.z runs GR neighbouring ranges of a.kr tiles, each
// summed from zero, and adds them as part_sum does; GEMM_PARTIAL writes that sum to a.part.
template <int MODE, class C, int GR>
__global__ __launch_bounds__(256, 1) void gemm_tile_kernel(GemmArgs a) {
    constexpr int MB = C::MB, NB = C::NB, S = C::S, TK = C::TK, STEPS = C::STEPS;
    constexpr int AI = C::AI, WI = C::WI, D = C::D;
    __shared__ __align__(16) char lds[C::LDS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int cols = C::ONE ? a.cols : C::TN;   // of the tile's TN columns, those that are this workgroup's
    const int m0 = blockIdx.x * C::TM, n0 = blockIdx.y * cols;
    const int M = a.M, K = a.K;
    // this workgroup's k tiles: t0 .. t0 + nk - 1
    const int kr = a.kr * (64 / TK);
    const int t0 = MODE == GEMM_PARTIAL ? blockIdx.z * GR * kr : 0;
    const int nk = MODE == GEMM_PARTIAL ? min(GR * kr, K / TK - t0) : K / TK;

    // Copies of this wavefront: uniform bases that advance with the tile, and a 32-bit byte offset
    // per lane.  Activation copy q = wave * AI + i: 8 rows of sub-tile q / (TM / 8); weight copy q =
    // wave * WI + i.  Rows past M or N are clamped (in bounds), their results are never stored.
    // SWIGLU: the weight tile's rows alternate between Wg and Wu rows n0 / 2 .., 32 of each at a
    // time (16 with one 32-wide block per wavefront, so that each block holds its own pairs).
    constexpr int HALF = NB % 2 == 0 ? 32 : 16;
    const char *const base_a = reinterpret_cast<const char *>(a.a + (size_t)m0 * a.lda + (size_t)t0 * (2 * TK));
    const int nrow0 = MODE == GEMM_SWIGLU ? n0 / 2 : n0;
    const int N = min(a.N, nrow0 + (MODE == GEMM_SWIGLU ? cols / 2 : cols));   // end of this workgroup's columns
    // SWIGLU of few rows: the groups of kTurn rows of Wg and Wu start their k loops at different tiles.
    // In step, every workgroup would read the same 128-byte columns of rows a power of two apart, which
    // crowds some memory channels (64 rows of the 8B-shaped layer, with non-temporal weight copies and
    // 112 columns per workgroup: 59 -> 49 us; a bare copy loop 48.6 -> 42.2 us from this alone).
    const int turn = MODE == GEMM_SWIGLU && M <= kFewRows && K % 64 == 0
                         ? (int)((long)(nrow0 / kTurn) * (K / 64) / ((a.N + kTurn - 1) / kTurn)) * (64 / TK) : 0;
    const char *const base_w = reinterpret_cast<const char *>(a.w[0] + (size_t)nrow0 * K + (size_t)t0 * TK);
    const long up = MODE == GEMM_SWIGLU ? reinterpret_cast<const char *>(a.w[1]) - reinterpret_cast<const char *>(a.w[0]) : 0;
    uint32_t off_a[AI], off_w[WI];
#pragma unroll
    for (int i = 0; i < AI; ++i) {
        const int q = wave * AI + i, sub = q / (C::TM / 8), r = 8 * (q % (C::TM / 8)) + (lane >> 3);
        const int g = (lane & 7) ^ ((r >> 1) & 7);
        off_a[i] = (uint32_t)min(r, M - 1 - m0) * (uint32_t)a.lda * 2 + 128 * sub + 16 * g;
    }
    long mat[WI];   // where the matrix of copy i's rows begins (wavefront-uniform)
#pragma unroll
    for (int i = 0; i < WI; ++i) {
        const int q = wave * WI + i;
        const int r = TK == 64 ? 8 * q + (lane >> 3) : 16 * q + (lane >> 2);
        const int seg = TK == 64 ? (lane & 7) ^ ((r >> 1) & 7) : (lane & 3) ^ ((r >> 2) & 3);
        const int n = MODE == GEMM_SWIGLU ? r / (2 * HALF) * HALF + r % HALF : r;
        mat[i] = MODE == GEMM_SWIGLU ? ((TK == 64 ? 8 : 16) * q / HALF & 1) * up : 0;
        off_w[i] = (uint32_t)min(n, N - 1 - nrow0) * (uint32_t)K * 2 + 16 * seg;
    }
    // copy d of tile t into stage st
    auto copy = [&](int t, int st, int d) {
        if constexpr (MODE == GEMM_SWIGLU) t = t + turn >= nk ? t + turn - nk : t + turn;
        if (d < AI)
            dma16(off_a[d], base_a + (size_t)t * (TK * 4), lds_base + st * C::STAGE + (wave * AI + d) * 1024);
        else
            dma16<C::ONE>(off_w[d - AI], base_w + mat[d - AI] + (size_t)t * (TK * 2),
                  lds_base + st * C::STAGE + C::A_BYTES + (wave * WI + d - AI) * 1024);
    };
    // the copies of one tile are issued in STEPS shares
    constexpr auto share = [](int s) { return s * D / STEPS; };

    struct Acc {
        f32x16 v[MB][NB];
    };
    Acc sum, tot;   // the running range; GR > 1: the sum of those before it
    auto &acc = sum.v;
    auto clear = [](Acc &x) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) x.v[i][j][r] = 0.f;
    };
    auto add = [](Acc &x, const Acc &y) {   // x += y
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) x.v[i][j][r] += y.v[i][j][r];
    };
    clear(sum);
    if (GR > 1) clear(tot);

    // byte offsets of this lane's fragments in a stage, without the block and the sub-tile
    const int fr = lane & 31, fk = lane >> 5;   // fragment row and k half of this lane
    int ao[2][2], wo[STEPS];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int hl = 0; hl < 2; ++hl)
            ao[p][hl] = 128 * (32 * wm * MB + fr) + 16 * ((2 * p + fk + 4 * hl) ^ ((fr >> 1) & 7));
#pragma unroll
    for (int p = 0; p < STEPS; ++p)
        wo[p] = TK == 64 ? 128 * (32 * wn * NB + fr) + 16 * ((2 * p + fk) ^ ((fr >> 1) & 7))
                         : 64 * (32 * wn * NB + fr) + 16 * ((2 * p + fk) ^ ((fr >> 2) & 3));
    struct Frags {
        bf16x8 ah[MB], al[MB], bw[NB];
    };
    // fragment r of k step p, in the order the step's MFMAs need them: the first row's hi and lo
    // with the weight blocks, then the other rows
    constexpr int RD = 2 * MB + NB;
    auto read = [&](const char *L, int p, int r, Frags &f) {
        auto ld = [&](int o) { return as_bf16x8(*reinterpret_cast<const uint4 *>(L + o)); };
        const int sub = C::TM * 128 * (p >> 1);
        if (r == 0) f.ah[0] = ld(ao[p & 1][0] + sub);
        else if (r <= NB) f.bw[r - 1] = ld(C::A_BYTES + wo[p] + 32 * (TK * 2) * (r - 1));
        else if (r == NB + 1) f.al[0] = ld(ao[p & 1][1] + sub);
        else if ((r - NB) % 2 == 0) f.ah[(r - NB) / 2] = ld(ao[p & 1][0] + sub + 4096 * ((r - NB) / 2));
        else f.al[(r - NB) / 2] = ld(ao[p & 1][1] + sub + 4096 * ((r - NB) / 2));
    };
    // MFMA q of a step: rows of blocks in turn, hi then lo into each block
    constexpr int MM = 2 * MB * NB;
    auto mma = [&](int q, const Frags &f) {
        const int i = q / (2 * NB), j = q / 2 % NB;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q & 1 ? f.al[i] : f.ah[i], f.bw[j], acc[i][j], 0, 0, 0);
    };

    Frags fa, fb;
    int st = 0;   // stage of the tile being multiplied
    // one step: the MFMAs of `cur`; the fragments of the next step (of stage Ln) into `nxt`; the
    // copies d0 .. d1 - 1 of tile tc into stage sc
    auto step = [&](const Frags &cur, Frags &nxt, const char *Ln, int pn, auto reads, int tc, int sc, auto d0, auto d1) {
        constexpr int R = decltype(reads)::value ? RD : 0, ND = decltype(d1)::value - decltype(d0)::value;
        constexpr int RW = MM >= 8 ? MM - MM / 4 : MM;   // the reads go out behind the first three quarters
#pragma unroll
        for (int q = 0; q < MM; ++q) {
            mma(q, cur);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (r * RW / (R ? R : 1) == q) read(Ln, pn, r, nxt);
#pragma unroll
            for (int d = 0; d < ND; ++d)
                if ((2 * d + 1) * MM / (2 * (ND ? ND : 1)) == q) copy(tc, sc, decltype(d0)::value + d);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using std::integral_constant;
    constexpr integral_constant<int, 0> zero{};
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    // Tile t (stage st).  FIRST: the rest of tile t + S - 1's copies go out over the first steps;
    // LAST: tile t + S's first share over the last step; AHEAD: tiles issued past t + 1 when the
    // barrier waits for t + 1, or -1: t is the last tile (no barrier, no reads past it).
    auto tile = [&](int t, auto first, auto last, auto ahead) {
        constexpr bool FIRST = decltype(first)::value, LAST = decltype(last)::value;
        constexpr int AHEAD = decltype(ahead)::value;
        const char *L = lds + st * C::STAGE;
        const int stn = st + 1 == S ? 0 : st + 1, stp = st == 0 ? S - 1 : st - 1;
        const char *Ln = lds + stn * C::STAGE;
#define STG_STEP(P, CUR, NXT)                                                                                     \
    step(CUR, NXT, L, (P) + 1, yes, t + S - 1, stp, integral_constant<int, FIRST ? share((P) + 1) : 0>{},         \
         integral_constant<int, FIRST ? share((P) + 2) : 0>{})
        STG_STEP(0, fa, fb);
        if constexpr (STEPS == 4) {
            STG_STEP(1, fb, fa);
            STG_STEP(2, fa, fb);
        }
#undef STG_STEP
        if constexpr (AHEAD >= 0) {
            wait_vm<(AHEAD >= 0 ? AHEAD : 0) * D>();   // this wavefront's copies of tile t + 1 have landed
            wait_lgkm<0>();                            // and its reads of tile t are done
            lds_barrier();
            step(fb, fa, Ln, 0, yes, t + S, st, zero, integral_constant<int, LAST ? share(1) : 0>{});
        } else {
            step(fb, fa, Ln, 0, no, 0, 0, zero, zero);
        }
        st = stn;
    };
    auto first_frags = [&]() {
#pragma unroll
        for (int r = 0; r < RD; ++r) read(lds, 0, r, fa);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto tail = [&](auto self, int t, auto j) -> void {   // tiles nk - S + j .. nk - 1
        constexpr int J = decltype(j)::value;
        tile(t, integral_constant<bool, J == 0>{}, no, integral_constant<int, S - 2 - J>{});
        if constexpr (J + 1 < S) self(self, t + 1, integral_constant<int, J + 1>{});
    };
    if (nk >= S) {
#pragma unroll
        for (int u = 0; u < S; ++u)
#pragma unroll
            for (int d = 0; d < (u < S - 1 ? D : share(1)); ++d) copy(u, u, d);
        wait_vm<(S - 2) * D + share(1)>();
        lds_barrier();
        first_frags();
        int t = 0;
        // (a loop, not unrolled: with a copy of the body per range the compiler spills the sums)
#pragma unroll 1
        for (int end = kr; GR > 1 && end < GR * kr; end += kr) {
            for (; t < end; ++t) tile(t, yes, yes, integral_constant<int, S - 2>{});
            add(tot, sum);
            clear(sum);
        }
        for (; t < nk - S; ++t) tile(t, yes, yes, integral_constant<int, S - 2>{});   // (the last range has at least S tiles)
        tail(tail, t, zero);
        if (GR > 1) add(sum, tot);
    } else {   // fewer tiles than stages: all copied at once
        for (int u = 0; u < nk; ++u)
#pragma unroll
            for (int d = 0; d < D; ++d) copy(u, u, d);
        wait_vm<0>();
        lds_barrier();
        first_frags();
        for (int t = 0; t + 1 < nk; ++t) tile(t, no, no, zero);
        tile(nk - 1, no, no, integral_constant<int, -1>{});
    }

    if constexpr (MODE == GEMM_SWIGLU) {
        // h of rows m and m + 1, column n (gates g, ups u), as pairs.  Neighbouring lanes hold neighbouring
        // columns: an even lane takes row m of both columns, an odd one row m + 1, so that a store is 4 bytes.
        // Nothing overlaps a large tile's epilogue, some 7000 instructions per lane at 256 x 256 with pairs
        // rounded by integer arithmetic and stored 2 bytes at a time; with the conversion instructions (pair.h)
        // and 4-byte stores 1024 rows of the 8B-shaped stage, two layers, take 1711 -> 1667 us, 37 rows 272 -> 262.
        auto put2 = [&](int m, int n, float g0, float u0, float g1, float u1, bool mine) {
            auto sw = [](float gt, float up) { return gt / (1.f + expf(-gt)) * up; };
            uint32_t hi, lo;
            split_pair2(sw(g0, u0), sw(g1, u1), hi, lo);
            const uint32_t e0 = (hi & 0xFFFFu) | (lo << 16), e1 = (hi >> 16) | (lo & 0xFFFF0000u);
            const bool odd = lane & 1;
            const uint32_t keep = odd ? e1 : e0, recv = lane_xor_bits(odd ? e0 : e1, 1);
            const uint32_t c0 = odd ? recv : keep, c1 = odd ? keep : recv;   // columns n & ~1 and the next (N is even)
            m += odd;
            n &= ~1;
            if (!mine || m >= M || n >= N) return;
            uint16_t *const o = a.out_pair + (size_t)m * a.ldo + pair_at(n);
            *reinterpret_cast<uint32_t *>(o) = (c0 & 0xFFFFu) | (c1 << 16);
            *reinterpret_cast<uint32_t *>(o + 32) = (c0 >> 16) | (c1 & 0xFFFF0000u);
        };
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int mb = m0 + 32 * (wm * MB + i) + 4 * (lane >> 5);
            if constexpr (NB % 2 == 0) {   // blocks j (gate) and j + 1 (up) hold the same rows of h
#pragma unroll
                for (int j = 0; j < NB; j += 2)
#pragma unroll
                    for (int r = 0; r < 16; r += 2)
                        put2(mb + 8 * (r >> 2) + (r & 3), n0 / 2 + 16 * (wn * NB + j) + (lane & 31), acc[i][j][r],
                             acc[i][j + 1][r], acc[i][j][r + 1], acc[i][j + 1][r + 1], true);
            } else {                       // columns c (gate) and c + 16 (up) of every block
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int r = 0; r < 16; r += 2)
                        put2(mb + 8 * (r >> 2) + (r & 3), n0 / 2 + 16 * (wn * NB + j) + (lane & 15), acc[i][j][r],
                             lane_xor(acc[i][j][r], 16), acc[i][j][r + 1], lane_xor(acc[i][j][r + 1], 16), (lane & 16) == 0);
            }
        }
        return;
    }
    if (MODE == GEMM_PARTIAL) {
        a.out = a.part + (size_t)blockIdx.z * M * a.N;
        a.ldo = a.N;
    }
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int n = n0 + 32 * (wn * NB + j) + (lane & 31);
            if (n >= N) continue;
            store_block<MODE>(a, acc[i][j], m0 + 32 * (wm * MB + i), M, n, lane);
        }
}

// out = res + the sum of SP partial products, [SP][rows][n] with n % 4 == 0, four columns per thread.
template <int SP>
__global__ __launch_bounds__(256) void part_residual_kernel(GemmArgs a) {
    const size_t quads = (size_t)a.M * a.N / 4;
    for (size_t q = blockIdx.x * 256ull + threadIdx.x; q < quads; q += (size_t)gridDim.x * 256) {
        const size_t o = 4 * q / a.N * a.ldo + 4 * q % a.N;
        const float4 r = *reinterpret_cast<const float4 *>(a.res + o);
        *reinterpret_cast<float4 *>(a.out + o) = add4(r, part_sum<SP>(a.part + 4 * q, (size_t)a.M * a.N));
    }
}

// y = x / sqrt(mean(x^2) + eps) * g, written as a pair (row stride ld).  One workgroup per row.
__global__ __launch_bounds__(256) void rmsnorm_split_kernel(const float *x, const uint16_t *g, float eps, int H,
                                                             uint16_t *pair, long ld) {
    const int row = blockIdx.x;
    const float *xr = x + (size_t)row * H;
    // sum of squares: four elements per thread and step (H % 4 == 0), the loads of four steps
    // issued before their products
    float ss = 0.f;
#pragma unroll 4
    for (int i = 4 * threadIdx.x; i < H; i += 1024) {
        const float4 v = *reinterpret_cast<const float4 *>(xr + i);
        ss = fmaf(v.x, v.x, ss);
        ss = fmaf(v.y, v.y, ss);
        ss = fmaf(v.z, v.z, ss);
        ss = fmaf(v.w, v.w, ss);
    }
    __shared__ float red[4];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) ss += lane_xor(ss, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    const float tot = ((red[0] + red[1]) + red[2]) + red[3];
    const float scale = 1.f / sqrtf(tot / (float)H + eps);
    // four elements per thread (H % 4 == 0): one 16-byte load, 8-byte stores of their hi and lo
    for (int i = 4 * threadIdx.x; i < H; i += 1024) {
        const float4 v = *reinterpret_cast<const float4 *>(xr + i);
        const uint2 gg = *reinterpret_cast<const uint2 *>(g + i);
        store_pair4(pair + (size_t)row * ld + pair_at(i),
                    make_float4(v.x * scale * __uint_as_float(gg.x << 16), v.y * scale * __uint_as_float(gg.x & 0xFFFF0000u),
                                v.z * scale * __uint_as_float(gg.y << 16), v.w * scale * __uint_as_float(gg.y & 0xFFFF0000u)));
    }
}

// The same for H = 1024 NV (NV <= 8): a thread's NV float4 of the row stay in registers between
// the sum of squares and the output, so the row is read once (same arithmetic in the same order:
// identical results).
template <int NV>
__global__ __launch_bounds__(256) void rmsnorm_split_rows_kernel(const float *x, const uint16_t *g, float eps,
                                                                 uint16_t *pair, long ld) {
    constexpr int H = 1024 * NV;
    const int row = blockIdx.x;
    const float *xr = x + (size_t)row * H + 4 * threadIdx.x;
    float4 v[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = *reinterpret_cast<const float4 *>(xr + 1024 * j);
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        ss = fmaf(v[j].x, v[j].x, ss);
        ss = fmaf(v[j].y, v[j].y, ss);
        ss = fmaf(v[j].z, v[j].z, ss);
        ss = fmaf(v[j].w, v[j].w, ss);
    }
    __shared__ float red[4];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) ss += lane_xor(ss, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    const float tot = ((red[0] + red[1]) + red[2]) + red[3];
    const float scale = 1.f / sqrtf(tot / (float)H + eps);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int i = 4 * threadIdx.x + 1024 * j;
        const uint2 gg = *reinterpret_cast<const uint2 *>(g + i);
        store_pair4(pair + (size_t)row * ld + pair_at(i),
                    make_float4(v[j].x * scale * __uint_as_float(gg.x << 16), v[j].y * scale * __uint_as_float(gg.x & 0xFFFF0000u),
                                v[j].z * scale * __uint_as_float(gg.y << 16), v[j].w * scale * __uint_as_float(gg.y & 0xFFFF0000u)));
    }
}

// h = silu(gate) * up from gu [rows, 2F] (gate columns first), written as a pair [rows, F] (row
// stride ld; F % 4 == 0), four elements per thread.
__global__ __launch_bounds__(256) void swiglu_split_kernel(const float *gu, int F, int rows, uint16_t *pair,
                                                            long ld) {
    const size_t quads = (size_t)rows * F / 4;
    for (size_t q = blockIdx.x * 256ull + threadIdx.x; q < quads; q += (size_t)gridDim.x * 256) {
        const size_t r = 4 * q / F;
        const int f = (int)(4 * q % F);
        const float4 g4 = *reinterpret_cast<const float4 *>(gu + r * 2 * F + f);
        const float4 u4 = *reinterpret_cast<const float4 *>(gu + r * 2 * F + F + f);
        auto sw = [](float gt, float up) { return gt / (1.f + expf(-gt)) * up; };
        store_pair4(pair + r * ld + pair_at(f), make_float4(sw(g4.x, u4.x), sw(g4.y, u4.y), sw(g4.z, u4.z), sw(g4.w, u4.w)));
    }
}

int grid_for(size_t count) {
    const size_t g = (count + 255) / 256;
    return (int)(g < 8192 ? g : 8192);
}

using Tile256 = Tile<2, 2, 4, 4, 32, 3>;      // 256 x 256
using TileWide = Tile<2, 2, 2, 4, 32, 3>;     // 128 x 256
using Tile128 = Tile<2, 2, 2, 2, 64, 3>;      // 128 x 128
using Tile128K32 = Tile<2, 2, 2, 2, 32, 3>;   // 128 x 128, K an odd multiple of 32
using Tile64 = Tile<2, 2, 1, 2, 64, 3, true>;   // 64 x 128
using Tile32 = Tile<1, 4, 1, 1, 64, 3, true>;   // 32 x 128

// How a GEMM runs: K cut into `ranges` ranges of kr tiles of 64, `group` of them at a time in a
// workgroup; wm x wn tiles.
struct GemmPlan {
    int ranges = 1, group = 1, kr = 0, wm = 0, wn = 0;
    int parts() const { return ranges / group; }
};

// Cut of K, calls of up to kFewRows rows.  Few rows are bound by the weights, and a [N, K] matrix has
// only N / 128 workgroups to read them, so K is cut into as many ranges as leave about one workgroup
// per compute unit, at least 512 deep; fixed by the matrix (see kFewRows).
// 37 rows of the 8B-shaped layer, whole K -> cut, with the pass that adds the parts: down (32
// workgroups -> 256) 204 -> 25 us, O 63 -> 11, QKV 62 -> 18.
//
// Tiles and grouping, more than 64 rows: the least estimated time, from the rounds of workgroups over
// the compute units, the time of a workgroup's 64 k at each tile shape with the chip full (us,
// measured: 256 x 256 2.86, 128 x 256 1.6, 128 x 128 0.88), and the bytes of the partial products
// (written and read back at about 5 TB/s, and a launch to add them).  Before, 256 x 256 wherever that
// gave a workgroup per compute unit, else 128 x 128, with whole K: 1200 rows of the 13B-shaped layer
// gate/up 769 -> 634 us (540 workgroups, 2.1 rounds -> 2160, 8.4), QKV 473 -> 337; 500 rows of the
// 32B-shaped one down 329 -> 271 us (160 workgroups -> 640 of a quarter of K), QKV 136 -> 113 with
// what follows it.
// None of it changes a bit: every tile shape runs the same MFMAs in the same order, and the ranges are
// added in one order however they are grouped.
GemmPlan gemm_plan(int M, int N, int K, bool swiglu, bool cut, size_t cap64) {
    GemmPlan p;
    const int cus = device_compute_units(), nv = swiglu ? 2 * N : N, tiles = K / 64;
    if (cut && !swiglu && M <= kFewRows && K % 64 == 0 && N % 4 == 0)
        for (int r : {8, 4, 3, 2}) {
            const int kr = (tiles + r - 1) / r, last = tiles - (r - 1) * kr;
            if ((long)((N + 127) / 128) * r > cus + cus / 16 || kr < 8 || last < 4 || (size_t)r * 64 * N > cap64) continue;
            p.ranges = r;
            p.kr = kr;
            break;
        }
    if (M <= 64 && K % 64 == 0) {
        p.wm = M <= 32 ? 32 : 64;
        // 112 of a tile's 128 columns where that evens out the last round of workgroups
        auto rounds = [&](int tn) { return ((nv + tn - 1) / tn * p.ranges + cus - 1) / cus * tn; };
        p.wn = rounds(112) < rounds(128) ? 112 : 128;
        return p;
    }
    static const struct { int wm, wn; double us; } shapes[] = {{256, 256, 2.86}, {128, 256, 1.6}, {128, 128, 0.88}};
    double best = 0;
    for (const auto &t : shapes)
        for (int g : {4, 3, 2, 1}) {
            if ((g > 1 && g != std::min(p.ranges, 4)) || (t.wm == 256 && p.ranges > 1)) continue;
            if (K % 64 != 0 && t.wm != t.wn) continue;
            const int parts = p.ranges / g;
            const long wgs = (long)((M + t.wm - 1) / t.wm) * ((nv + t.wn - 1) / t.wn) * parts;
            double us = (double)((wgs + cus - 1) / cus) * tiles / parts * t.us;
            if (parts > 1) us += 3 + 8e-6 * parts * M * N / 5;
            if (best > 0 && us >= best) continue;
            best = us;
            p.group = g;
            p.wm = t.wm;
            p.wn = t.wn;
        }
    return p;
}

template <int MODE, class C, int GR>
void launch_shape(GemmArgs a, const GemmPlan &p, hipStream_t st) {
    const int nv = MODE == GEMM_SWIGLU ? 2 * a.N : a.N;   // SWIGLU tiles span the rows of both matrices
    a.kr = p.kr;
    a.cols = p.wn;
    const dim3 grid((a.M + C::TM - 1) / C::TM, (nv + a.cols - 1) / a.cols, p.parts());
    STG_LAUNCH((gemm_tile_kernel<MODE, C, GR>), grid, dim3(256), 0, st, a);
}

template <int MODE, int GR>
void launch_tile(const GemmArgs &a, const GemmPlan &p, hipStream_t st) {
    if constexpr (GR == 1) {
        if (p.wm == 32) return launch_shape<MODE, Tile32, 1>(a, p, st);
        if (p.wm == 64) return launch_shape<MODE, Tile64, 1>(a, p, st);
        if constexpr (MODE != GEMM_PARTIAL) {
            if (p.wm == 256) return launch_shape<MODE, Tile256, 1>(a, p, st);
            if (a.K % 64 != 0) return launch_shape<MODE, Tile128K32, 1>(a, p, st);
        }
    }
    if constexpr (MODE != GEMM_SWIGLU || GR == 1) {
        if (p.wn == 256) launch_shape<MODE, TileWide, GR>(a, p, st);
        else launch_shape<MODE, Tile128, GR>(a, p, st);
    }
}

// One part: MODE's own epilogue; several: GEMM_PARTIAL.
template <int MODE>
void launch_plan(const GemmArgs &a, const GemmPlan &p, hipStream_t st) {
    auto go = [&](auto mode) {
        constexpr int X = decltype(mode)::value;
        switch (p.group) {
            case 2: launch_tile<X, 2>(a, p, st); break;
            case 3: launch_tile<X, 3>(a, p, st); break;
            case 4: launch_tile<X, 4>(a, p, st); break;
            default: launch_tile<X, 1>(a, p, st);
        }
    };
    if (p.parts() > 1) go(std::integral_constant<int, GEMM_PARTIAL>{});
    else go(std::integral_constant<int, MODE>{});
}

template <int MODE>
void launch_any_k(const GemmArgs &a, int n_mats, hipStream_t st) {
    const dim3 grid((a.M + BM - 1) / BM, (a.N + BN - 1) / BN, n_mats);
    STG_LAUNCH(gemm_kernel<MODE>, grid, dim3(256), 0, st, a);
}

template <int SP>
void launch_part_residual(const GemmArgs &a, hipStream_t st) {
    STG_LAUNCH(part_residual_kernel<SP>, dim3(grid_for((size_t)a.M * a.N / 4)), dim3(256), 0, st, a);
}

}  // namespace

size_t gemm_part_floats(int rows, int N, int K, size_t cap64, size_t most) {
    for (int m = min(rows, kFewRows); m >= 1; --m) {
        const GemmPlan p = gemm_plan(m, N, K, false, true, cap64);
        if (p.ranges == 1 || (size_t)p.ranges * m * N <= most) break;   // (the cut is the same for every m)
        if (p.parts() > 1) most = max(most, (size_t)p.parts() * m * N);
    }
    return most;
}

hipError_t launch_gemm(int mode, const GemmArgs &a, int n_mats, hipStream_t st) {
    if (a.M <= 0) return hipSuccess;
    // variants without a K cut run the same MFMAs in the same order: which of them runs never changes a bit
    if (a.lda < pair_ld(a.K)) return hipErrorInvalidValue;
    if (mode == GEMM_SWIGLU) {
        if (a.K % BK != 0 || n_mats != 1 || !a.out_pair || a.ldo < pair_ld(a.N)) return hipErrorInvalidValue;
        launch_plan<GEMM_SWIGLU>(a, gemm_plan(a.M, a.N, a.K, true, false, 0), st);
    } else if (a.K % BK != 0) {
        if (mode == GEMM_RESIDUAL) launch_any_k<GEMM_RESIDUAL>(a, n_mats, st);
        else launch_any_k<GEMM_STORE>(a, n_mats, st);
    } else if (n_mats != 1 || a.out_col[0] != 0 || mode != GEMM_RESIDUAL) {   // (the QKV product: launch_qkv)
        return hipErrorInvalidValue;
    } else {
        const GemmPlan p = gemm_plan(a.M, a.N, a.K, false, a.part != nullptr, a.part_cap64);
        launch_plan<GEMM_RESIDUAL>(a, p, st);
        switch (p.parts()) {
            case 2: launch_part_residual<2>(a, st); break;
            case 3: launch_part_residual<3>(a, st); break;
            case 4: launch_part_residual<4>(a, st); break;
            case 8: launch_part_residual<8>(a, st); break;
        }
    }
    return hipGetLastError();
}

hipError_t launch_qkv(const GemmArgs &g, RopeKvArgs r, hipStream_t st) {
    if (g.M <= 0) return hipSuccess;
    r.n_part = 1;
    r.qkv = g.out;
    if (g.K % BK != 0) {
        const hipError_t e = launch_gemm(GEMM_STORE, g, 1, st);
        if (e != hipSuccess) return e;
    } else {
        if (g.lda < pair_ld(g.K)) return hipErrorInvalidValue;
        const GemmPlan p = gemm_plan(g.M, g.N, g.K, false, g.part != nullptr, g.part_cap64);
        r.n_part = p.parts();
        if (r.n_part > 1) r.qkv = g.part;
        launch_plan<GEMM_STORE>(g, p, st);
    }
    return launch_rope_kv_store(r, st);
}

hipError_t launch_rmsnorm_split(const float *x, const uint16_t *g, float eps, int rows, int H, uint16_t *pair,
                                long ld, hipStream_t st) {
    if (rows <= 0) return hipSuccess;
    if (ld < pair_ld(H) || H % 4 != 0) return hipErrorInvalidValue;
    // rows of up to 8 whole 1024s in registers (500 rows of 5120: 8.6 us with two reads of the row -> 6.5;
    // 1200 rows 14.4 -> 11.6); others, and longer ones, are read twice
    switch (H % 1024 == 0 ? H / 1024 : 0) {
#define STG_NORM_CASE(NV) \
    case NV: STG_LAUNCH(rmsnorm_split_rows_kernel<NV>, dim3(rows), dim3(256), 0, st, x, g, eps, pair, ld); break;
        STG_NORM_CASE(1) STG_NORM_CASE(2) STG_NORM_CASE(3) STG_NORM_CASE(4)
        STG_NORM_CASE(5) STG_NORM_CASE(6) STG_NORM_CASE(7) STG_NORM_CASE(8)
#undef STG_NORM_CASE
        default: STG_LAUNCH(rmsnorm_split_kernel, dim3(rows), dim3(256), 0, st, x, g, eps, H, pair, ld);
    }
    return hipGetLastError();
}

hipError_t launch_swiglu_split(const float *gu, int F, int rows, uint16_t *pair, long ld, hipStream_t st) {
    if (rows <= 0) return hipSuccess;
    if (ld < pair_ld(F)) return hipErrorInvalidValue;
    if (F % 4 != 0) return hipErrorInvalidValue;
    STG_LAUNCH(swiglu_split_kernel, dim3(grid_for((size_t)rows * F / 4)), dim3(256), 0, st, gu, F, rows, pair, ld);
    return hipGetLastError();
}

}  // namespace stg
