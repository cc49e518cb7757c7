// proj_gemm_f32.hip -- the projection products for fp32 storage, gfx950.
//
// The same three products as proj_gemm.hip (Y = X W, dX = dY W^T,
// dW = X^T dY; section 4.1's matrix-product gradients, no operand transposed
// in memory) for tensors stored in fp32, with fp32 accumulation on
// v_mfma_f32_32x32x2_f32 (eight per 16-deep chunk, cdna4.hpp's fragment
// convention).  Any extents, any leading dimensions, 4-byte alignment.
//
// The fp32 MFMA rate bounds it (157 TFLOP/s; a large library product reaches
// 138): one 32x32x2 product takes 64 cycles, so LDS has time for column reads
// by single floats and any wavefront tile, and what counts is that every CU has
// work and that loads are hidden.  Operands go through registers (16-byte
// loads, 4-byte alignment) into LDS in their stored orientation, the next step's
// loads under the current step's products; small outputs take small tiles whose
// wavefronts split the contraction.  512 tokens x 768 x 3072: Y 112 -> 26, dX
// 336 -> 30, dW 91 -> 28 us (82 .. 94 TFLOP/s) against 64 x 64 tiles staged by
// single floats; 4096 x 2048 x 2048 252 .. 293 us (117 .. 136 TFLOP/s).
#include <algorithm>
#include <array>
#include <utility>

#include "cdna4.hpp"
#include "kernels.hpp"
#include "stage.hpp"

namespace fbl {

namespace {

// A workgroup's output tile (bm x bn), the contraction depth of a step (bk)
// and its wavefronts: a wm x wn grid of wavefront tiles, each computed by wk
// wavefronts that split every step's contraction.
struct F32Tile {
    int bm, bn, bk, wm, wn, wk;
};
constexpr F32Tile kF32Tiles[] = {
    {128, 128, 16, 2, 2, 1},  // 0: wavefronts of 64 x 64
    {128, 64, 32, 2, 2, 1},   // 1: 64 x 32
    {64, 64, 32, 2, 2, 1},    // 2: 32 x 32
    {64, 32, 64, 2, 1, 2},    // 3: 32 x 32 on half of every step
    {32, 32, 64, 1, 1, 4},    // 4: 32 x 32 on a quarter
    {32, 32, 128, 1, 1, 8},   // 5: 32 x 32 on an eighth
};
constexpr int kF32TileCount = (int)(sizeof(kF32Tiles) / sizeof(kF32Tiles[0]));

// LDS tile of ROWS stored rows of COLS floats, filled through registers by NT
// threads in 16-byte chunks.  Rows are padded by 4 floats: 16-byte aligned,
// 16 consecutive rows on 16 different 16-byte bank groups (row reads), and
// rows 8 apart on the other half of the banks (column reads).
template <int ROWS, int COLS, int NT>
struct FTile {
    static constexpr int PITCH = COLS + 4;
    static constexpr int FLOATS = ROWS * PITCH;
    static constexpr int CPR = COLS / 4;
    static constexpr int PER = ROWS * CPR / NT;  // chunks per thread
    static_assert(ROWS * CPR % NT == 0, "whole chunks per thread");
    f32x4 x[PER];
    uint32_t voff[PER];
    FBL_DEV void init(uint32_t row_bytes) {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int q = (int)threadIdx.x + j * NT;
            voff[j] = (uint32_t)(q / CPR) * row_bytes + (uint32_t)(q % CPR) * 16u;
        }
    }
    FBL_DEV void load(__amdgpu_buffer_rsrc_t rs, uint32_t origin) {
#pragma unroll
        for (int j = 0; j < PER; ++j)
            x[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff[j], origin, 0));
    }
    // Zero the contraction positions from krem on: whole rows when the
    // contraction runs down the stored rows (KROWS), else columns.
    template <bool KROWS>
    FBL_DEV void zero_tail(int krem) {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int q = (int)threadIdx.x + j * NT;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((KROWS ? q / CPR : 4 * (q % CPR) + e) >= krem) x[j][e] = 0.f;
        }
    }
    FBL_DEV void store(float* tile) const {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int q = (int)threadIdx.x + j * NT;
            *(FBL_LDS f32x4*)(tile + (q / CPR) * PITCH + 4 * (q % CPR)) = x[j];
        }
    }
    // Fragment of a 16-deep chunk at contraction position k, row/column r0 +
    // lane % 32: lane group g holds elements 8g .. 8g+7.
    template <bool KROWS>
    static FBL_DEV void frag(Frag<float>& f, const float* tile, int r0, int k, int lane) {
        const int r = r0 + (lane & 31), kk = k + 8 * (lane >> 5);
        if constexpr (KROWS) {
#pragma unroll
            for (int e = 0; e < 8; ++e) f.v[e] = *(const FBL_LDS float*)(tile + (kk + e) * PITCH + r);
        } else {
            const f32x4 a = *(const FBL_LDS f32x4*)(tile + r * PITCH + kk);
            const f32x4 b = *(const FBL_LDS f32x4*)(tile + r * PITCH + kk + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) { f.v[e] = a[e]; f.v[4 + e] = b[e]; }
        }
    }
};

// Workgroups of a product: whole groups of 8, one per XCD (xcd_logical_id).
int64_t f32_workgroups(const F32Tile& t, const GemmArgs& p) {
    return ((((int64_t)p.M + t.bm - 1) / t.bm) * (((int64_t)p.N + t.bn - 1) / t.bn) + 7) / 8 * 8;
}

// AT: A stored k-major ([K, M] rows); BT: B stored n-major ([N, K] rows).
template <int I, bool AT, bool BT>
struct F32Cfg {
    static constexpr F32Tile t = kF32Tiles[I];
    static constexpr int NW = t.wm * t.wn * t.wk, NT = 64 * NW;
    using TA = FTile<AT ? t.bk : t.bm, AT ? t.bm : t.bk, NT>;
    using TB = FTile<BT ? t.bn : t.bk, BT ? t.bk : t.bn, NT>;
    static constexpr int TM = t.bm / (32 * t.wm), TN = t.bn / (32 * t.wn);  // 32 x 32 tiles per wavefront
    static constexpr int KCW = t.bk / 16 / t.wk;                            // 16-deep chunks per wavefront and step
    static constexpr int STAGE = TA::FLOATS + TB::FLOATS;
    static constexpr int PART = (t.wk - 1) * t.bm * t.bn;
    static constexpr int BYTES = 4 * (2 * STAGE > PART ? 2 * STAGE : PART);
    static_assert(t.bk % (16 * t.wk) == 0 && BYTES <= 80 * 1024, "whole chunks per wavefront; two workgroups per CU");
};

template <int I, bool AT, bool BT>
__global__ __launch_bounds__((F32Cfg<I, AT, BT>::NT), 2) void proj_gemm_f32(GemmArgs p) {
    using C = F32Cfg<I, AT, BT>;
    using TA = typename C::TA;
    using TB = typename C::TB;
    constexpr F32Tile t = C::t;
    constexpr int TM = C::TM, TN = C::TN;
    extern __shared__ __attribute__((aligned(16))) float f32_smem[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 5;
    const int wm = wave % t.wm, wn = (wave / t.wm) % t.wn, wk = wave / (t.wm * t.wn);
    const int mt = (p.M + t.bm - 1) / t.bm, nt = (p.N + t.bn - 1) / t.bn;
    // consecutive ids share a column block of B and land on one XCD
    const int logical = xcd_logical_id(blockIdx.x, mt * nt, gridDim.x);
    if (logical < 0) return;
    const int m0 = (logical % mt) * t.bm, n0 = (logical / mt) * t.bn;
    const int nk = (p.K + t.bk - 1) / t.bk;

    // Loads past an operand's span return zeros.  Rows and columns past its
    // extents may read other elements of the span: they meet unstored outputs
    // only, except along the contraction, where zero_tail clears them.
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.a), 0, (int)p.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.b), 0, (int)p.b_bytes, 0x00020000);
    TA ta;
    TB tb;
    ta.init((uint32_t)(p.lda * 4));
    tb.init((uint32_t)(p.ldb * 4));
    auto load = [&](int s) __attribute__((always_inline)) {
        const int k0 = s * t.bk;
        ta.load(ra, (uint32_t)((AT ? (int64_t)k0 * p.lda + m0 : (int64_t)m0 * p.lda + k0) * 4));
        tb.load(rb, (uint32_t)((BT ? (int64_t)n0 * p.ldb + k0 : (int64_t)k0 * p.ldb + n0) * 4));
    };
    auto store = [&](int s) __attribute__((always_inline)) {
        float* stage = f32_smem + (s & 1) * C::STAGE;
        if (p.K - s * t.bk < t.bk) {
            ta.template zero_tail<AT>(p.K - s * t.bk);
            tb.template zero_tail<!BT>(p.K - s * t.bk);
        }
        ta.store(stage);
        tb.store(stage + TA::FLOATS);
    };

    f32x16 acc[TM][TN];  // rows = m (acc_row), columns = n (lane)
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) acc[tm][tn] = f32x16{};

    // Two LDS stages: step s is contracted while step s+1 is on its way from
    // memory into registers; it goes to the other stage once step s is done.
    load(0);
    store(0);
    __syncthreads();
    for (int s = 0; s < nk; ++s) {
        if (s + 1 < nk) load(s + 1);
        const float* sa = f32_smem + (s & 1) * C::STAGE;
        const float* sb = sa + TA::FLOATS;
#pragma unroll
        for (int j = 0; j < C::KCW; ++j) {
            const int k = 16 * (wk * C::KCW + j);
            Frag<float> fa[TM], fb[TN];
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) TA::template frag<AT>(fa[tm], sa, (wm * TM + tm) * 32, k, lane);
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) TB::template frag<!BT>(fb[tn], sb, (wn * TN + tn) * 32, k, lane);
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn)
                        acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[tm].v[e], fb[tn].v[e], acc[tm][tn], 0, 0, 0);
        }
        if (s + 1 < nk) store(s + 1);
        __syncthreads();
    }

    if constexpr (t.wk > 1) {
        // Partial sums through LDS (the stages are free), added in the order wk = 1, 2, ...
        float* part = f32_smem + (wn * t.wm + wm) * (TM * TN * 1024) + lane * 4;
        constexpr int kSlot = t.bm * t.bn;
        if (wk > 0) {
#pragma unroll
            for (int i = 0; i < TM * TN * 4; ++i) {
                const f32x16& a = acc[i / (4 * TN)][i / 4 % TN];
                *(FBL_LDS f32x4*)(part + (wk - 1) * kSlot + i * 256) =
                    f32x4{a[4 * (i % 4)], a[4 * (i % 4) + 1], a[4 * (i % 4) + 2], a[4 * (i % 4) + 3]};
            }
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int w = 0; w < t.wk - 1; ++w)
#pragma unroll
            for (int i = 0; i < TM * TN * 4; ++i) {
                const f32x4 v = *(const FBL_LDS f32x4*)(part + w * kSlot + i * 256);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i / (4 * TN)][i / 4 % TN][4 * (i % 4) + e] += v[e];
            }
    }

    // 32 consecutive columns per store and row; stores outside the output go
    // to an offset past the buffer's range, which the hardware drops
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(p.c, 0, (int)p.c_bytes, 0x00020000);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const int n = n0 + (wn * TN + tn) * 32 + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + (wm * TM + tm) * 32 + acc_row(r, g);
                const uint32_t off = m < p.M && n < p.N ? (uint32_t)(((int64_t)m * p.ldc + n) * 4) : 0x80000000u;
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(acc[tm][tn][r]), rc, off, 0, 0);
            }
        }
}

template <int I, bool AT, bool BT>
hipError_t launch_id(const GemmArgs& p, hipStream_t stream) {
    using C = F32Cfg<I, AT, BT>;
    constexpr auto kernel = &proj_gemm_f32<I, AT, BT>;
    const hipError_t once = ensure_dynamic_lds<kernel>(C::BYTES);
    if (once != hipSuccess) return once;
    hipLaunchKernelGGL(kernel, dim3((unsigned)f32_workgroups(C::t, p)), dim3(C::NT), C::BYTES, stream, p);
    return hipGetLastError();
}

using Launcher = hipError_t (*)(const GemmArgs&, hipStream_t);

template <bool AT, bool BT, int... I>
constexpr std::array<Launcher, sizeof...(I)> launchers(std::integer_sequence<int, I...>) {
    return {&launch_id<I, AT, BT>...};
}

template <bool AT, bool BT>
hipError_t launch_tile(int tile, const GemmArgs& p, hipStream_t stream) {
    static constexpr auto table = launchers<AT, BT>(std::make_integer_sequence<int, kF32TileCount>{});
    return table[tile](p, stream);
}

// The tile of a product: least rounds x area x cost, where rounds is the number
// of workgroups the busiest of the 256 CUs gets and cost the measured time per
// output element and contraction element of a CU -- lower for tiles that read
// less LDS and L2 per product, higher when a CU has a single workgroup (nothing
// covers its barriers and loads).  Measured over 18 products of 64 .. 4096 rows
// and columns and their gradients (relative units; us per tile there, e.g.
// 512 x 3072 from 768: 59 / 33 / 32 / 26 / 29 and 2048^3: 152 / 146 / 144 / 167
// / 179 for tiles 0 .. 4; the picks are within 10% of the best of each).  Few
// small tiles with a deep contraction split it over 8 wavefronts: 33 x 2048
// from 2048 17.6 -> 16.0 us, 128 x 768 from 3072 25.2 -> 22.2 us.
// A launch holds less than 2^32 threads: a 2 GB column of outputs (2^29 rows of
// one) has too many 32-row tiles for it.
int f32_tile(const GemmArgs& p) {
    constexpr double kCost[5][2] = {{3.5, 3.0}, {4.0, 3.2}, {4.7, 3.6}, {4.8, 4.1}, {5.2, 4.4}};  // one round, more
    int best = 0;
    double best_cost = 0;
    for (int i = 0; i < 5; ++i) {
        const F32Tile& t = kF32Tiles[i];
        const int64_t tiles = f32_workgroups(t, p);
        if (i > 0 && tiles * 256 > UINT32_MAX) break;
        const int64_t rounds = (tiles + 255) / 256;
        const double cost = (double)rounds * (t.bm * t.bn) * kCost[i][rounds > 1];
        if (i == 0 || cost < best_cost) best = i, best_cost = cost;
    }
    return best == 4 && f32_workgroups(kF32Tiles[4], p) <= 256 && p.K >= 768 ? 5 : best;
}

hipError_t launch_f32(int a_kmajor, int b_nmajor, int tile, const GemmArgs& p, hipStream_t stream) {
    if (a_kmajor && b_nmajor) return hipErrorInvalidValue;  // no product reads both that way
    if (a_kmajor) return launch_tile<true, false>(tile, p, stream);
    return b_nmajor ? launch_tile<false, true>(tile, p, stream) : launch_tile<false, false>(tile, p, stream);
}

}  // namespace

hipError_t launch_proj_gemm_f32(int a_kmajor, int b_nmajor, const GemmArgs& p, hipStream_t stream) {
    return launch_f32(a_kmajor, b_nmajor, f32_tile(p), p, stream);
}

void proj_gemm_f32_info(const GemmArgs& p, int32_t* info) {
    const F32Tile& t = kF32Tiles[f32_tile(p)];
    const int32_t v[6] = {t.bm, t.bn, t.bk, t.wm * t.wn * t.wk, t.wk,
                          (int32_t)std::min<int64_t>(f32_workgroups(t, p), INT32_MAX)};
    for (int i = 0; i < 6; ++i) info[i] = v[i];
}

}  // namespace fbl
