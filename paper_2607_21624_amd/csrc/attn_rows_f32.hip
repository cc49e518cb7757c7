// attn_rows_f32.hip -- fp32 attention passes in 128-row workgroups on token-major
// tensors, gfx950: the forward at d = 64 and 128, and the backward's kv and dQ passes at
// d = 128, where the keys (forward, dQ) or queries (kv) to walk are few.
//
// attn_streams.hip deals a walk to four wavefronts and adds their partial results
// through LDS at its end: with one to three steps in the walk the end costs as
// much as a step, and at d = 128 nothing covers it (one workgroup per CU).  Here a
// wavefront owns 32 of a workgroup's 128 rows and walks all of it, so there is no
// end; the tiles are shared by the four wavefronts (one barrier per tile).  What it
// takes is enough rows: a grid of whole rounds of 256 workgroups (f32_rows_* choose).
//
// 128 rows -> 32 rows (us): forward d = 64, 4096 queries on 33 keys, B4 H16 S1024,
// 22.4 -> 35.4; B64 H8 S128 32.5 -> 41.2; B64 H8 S256 94 -> 104; but 288 workgroups of
// 128 rows (B36 H8 S128) 28.2 -> 23.5.  Backward d = 128 (statistics, kv and dQ) B16
// H16 S128 105 -> 146, S64 57.7 -> 65.7, B8 H16 S256 174 -> 194, but B4 H16 S128
// 92 -> 36 and B8 H16 S512 620 -> 627.
#include <algorithm>
#include <type_traits>

#include "cdna4.hpp"
#include "kernels.hpp"
#include "stage.hpp"
#include "tokmap.hpp"

namespace fbl {

namespace {

constexpr int kWaves = 4;
constexpr int kRows = 32 * kWaves;     // queries (forward, dQ) or keys (kv) per workgroup
constexpr int kTile = 64;              // keys per staged tile (forward, dQ)
constexpr int kQTile = 32;             // queries per staged tile (kv; register budget at d = 128)
constexpr float kRescaleSlack = 8.0f;  // log2 of the largest unnormalised probability

int padded8(int n) { return (n + 7) / 8 * 8; }

// Row `p` (8 elements per lane group and 16-deep chunk) of an operand; zeros where !ok.
template <int D>
FBL_DEV void row_frags(Frag<float>* f, const float* p, int g, bool ok, bool neg = false) {
#pragma unroll
    for (int c = 0; c < D / 16; ++c) {
        f32x4 x = f32x4{}, y = f32x4{};
        if (ok) {
            x = __builtin_bit_cast(f32x4, load16(p + 16 * c + 8 * g));
            y = __builtin_bit_cast(f32x4, load16(p + 16 * c + 8 * g + 4));
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            f[c].v[e] = neg ? -x[e] : x[e];
            f[c].v[4 + e] = neg ? -y[e] : y[e];
        }
    }
}

template <int D>
FBL_DEV Rsrc rows_rsrc(const float* head, const TokMap& m, int rows) {
    return make_rsrc(head, (uint32_t)(((int64_t)(rows - 1) * m.ss + D) * 4));
}

// ---------------------------------------------------------------- forward
template <int D>
__global__ __launch_bounds__(256, 1) void attn_fwd_rows_f32(FwdArgs a) {
    constexpr int NC = D / 16, ND = D / 32;
    constexpr int TILE = kTile * D;
    constexpr uint32_t TB = TILE * 4;
    extern __shared__ __attribute__((aligned(1024))) unsigned char rows_fwd_smem[];
    float* smem = reinterpret_cast<float*>(rows_fwd_smem);  // K0 K1 V0 V1
    const uint32_t lds = lds_addr(rows_fwd_smem);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 5, c32 = lane & 31;
    const int S = a.S, Skv = a.Skv;
    const int nqb = (S + kRows - 1) / kRows;
    int rank, bh;
    if (!rank_major_item(blockIdx.x, nqb, a.Hq * a.B, rank, bh)) return;
    const int h = bh % a.Hq, b = bh / a.Hq;
    const int qb = a.mask.causal ? (nqb - 1 - rank) : rank;
    const int hk = h / (a.Hq / a.Hkv);
    int kv_end = Skv;
    if (a.mask.kv_len) kv_end = min(max(a.mask.kv_len[b], 0), Skv);
    const int q0 = qb * kRows;
    const int qi = q0 + wave * 32 + c32;  // this lane's query (column of S^T)
    int k_hi = kv_end;
    if (a.mask.causal) k_hi = min(k_hi, q0 + kRows);
    const int nkb = (k_hi + kTile - 1) / kTile;

    // the softmax FMA below needs a non-negative scale: fold the sign into Q
    const bool neg = a.scale_log2 < 0.f;
    const float c = neg ? -a.scale_log2 : a.scale_log2;
    Frag<float> qf[NC];
    row_frags<D>(qf, static_cast<const float*>(a.q) + a.mq.head_base(b, h) + (int64_t)qi * a.mq.ss, g, qi < S, neg);

    f32x16 oacc[ND];
#pragma unroll
    for (int t = 0; t < ND; ++t) oacc[t] = f32x16{};
    float m = -INFINITY;  // running maximum (log2 units), equal in both lane halves
    float l = 0.f;        // this lane half's share of the running sum

    const Rsrc rk = rows_rsrc<D>(static_cast<const float*>(a.k) + a.mk.head_base(b, hk), a.mk, Skv);
    const Rsrc rv = rows_rsrc<D>(static_cast<const float*>(a.v) + a.mv.head_base(b, hk), a.mv, Skv);
    const uint32_t kbytes = (uint32_t)(a.mk.ss * 4), vbytes = (uint32_t)(a.mv.ss * 4);
    DmaPlan<float, D, kTile, kWaves> dk, dv;
    dk.init(kbytes, wave, lane);
    dv.init(vbytes, wave, lane);

    // Iteration j: wait for K_{j+1}, V_j; barrier; DMA K_{j+2} -> Kbuf[j%2], V_{j+1} ->
    // Vbuf[(j+1)%2]; S_{j+1} = Q K_{j+1}^T; P_j = softmax(S_j); O += P_j V_j.  In pairs, so
    // that buffer and score-array parities are compile-time.
    f32x16 sc[2][2];  // scores of two tiles: [parity][32-key half]
    auto qk = [&](auto par_c, int kbuf) {
        constexpr int P = decltype(par_c)::value;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            sc[P][kt] = f32x16{};
#pragma unroll
            for (int cc = 0; cc < NC; ++cc) {
                Frag<float> kf;
                tile_row_frag<D>(kf, smem + kbuf * TILE, kt * 32 + c32, 16 * cc + 8 * g);
                mma(sc[P][kt], kf, qf[cc]);
            }
        }
    };
    auto softmax_pv = [&](auto par_c, auto mask_c, int k0) {
        constexpr int P = decltype(par_c)::value;
        constexpr bool MASK = decltype(mask_c)::value;
        f32x16* s = sc[P];
        if constexpr (MASK) {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = k0 + kt * 32 + acc_row(r, g);
                    if (key >= kv_end || (a.mask.causal && key > qi)) s[kt][r] = -INFINITY;
                }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kt][r]);
        mx = fmaxf(mx, other_half(mx)) * c;
        if (__any(mx > m + kRescaleSlack)) {
            const float m_new = fmaxf(m, mx);
            const float alpha = (m_new == -INFINITY) ? 1.f : fast_exp2(m - m_new);  // 0 when m was -inf
            l *= alpha;
#pragma unroll
            for (int t = 0; t < ND; ++t) oacc[t] *= alpha;
            m = m_new;
        }
        const float nm = (m == -INFINITY) ? 0.f : -m;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float p = fast_exp2(__builtin_fmaf(s[kt][r], c, nm));
                if constexpr (MASK) {
                    if (s[kt][r] == -INFINITY) p = 0.f;
                }
                s[kt][r] = p;
                l += p;
            }
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int cc = 0; cc < 2; ++cc) {
                Frag<float> pf;
                float pv[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) pv[e] = s[kt][8 * cc + e];
                pack_frag(pf, pv);
#pragma unroll
                for (int t = 0; t < ND; ++t) {
                    Frag<float> vf;
                    const int row0 = kt * 32 + 16 * cc + 4 * g;
                    tile_tr_frag<D>(vf, smem + (2 + P) * TILE, row0, row0 + 8, 32 * t, lane);
                    mma(oacc[t], vf, pf);
                }
            }
    };
    auto step = [&](auto par_c, auto mask_c, int j) {
        constexpr int P = decltype(par_c)::value;
        constexpr int NP = 1 - P;
        wait_vmcnt<0>();
        __syncthreads();  // K_{j+1} and V_j landed; iteration j-1 is done everywhere
        if (j + 2 < nkb) dk.issue(lds + P * TB, rk, (uint32_t)((j + 2) * kTile) * kbytes, wave);
        if (j + 1 < nkb) {
            dv.issue(lds + (2 + NP) * TB, rv, (uint32_t)((j + 1) * kTile) * vbytes, wave);
            qk(std::integral_constant<int, NP>{}, NP);
        }
        softmax_pv(par_c, mask_c, j * kTile);
    };

    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    if (nkb > 0) {
        dk.issue(lds, rk, 0u, wave);
        dv.issue(lds + 2 * TB, rv, 0u, wave);
        if (nkb > 1) dk.issue(lds + TB, rk, (uint32_t)kTile * kbytes, wave);
        wait_vmcnt<0>();
        __syncthreads();
        qk(P0{}, 0);
    }
    // Tiles inside kv_end and (causal) at or below the block's first query need no
    // mask; an even count, so that the masked loop also starts on parity 0.
    const int n_full = min(nkb, min(kv_end, a.mask.causal ? q0 + 1 : Skv) / kTile) & ~1;
    for (int j = 0; j < n_full; j += 2) {
        step(P0{}, std::false_type{}, j);
        step(P1{}, std::false_type{}, j + 1);
    }
    for (int j = n_full; j < nkb; j += 2) {
        step(P0{}, std::true_type{}, j);
        if (j + 1 < nkb) step(P1{}, std::true_type{}, j + 1);
    }

    l += other_half(l);
    if (qi < S) {
        const float inv = (l > 0.f) ? 1.f / l : 0.f;
        float* orow = static_cast<float*>(a.o) + a.mo.head_base(b, h) + (int64_t)qi * a.mo.ss;
#pragma unroll
        for (int t = 0; t < ND; ++t)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
                store4(orow + 32 * t + 8 * rr + 4 * g, oacc[t][4 * rr] * inv, oacc[t][4 * rr + 1] * inv,
                       oacc[t][4 * rr + 2] * inv, oacc[t][4 * rr + 3] * inv);
        if (g == 0) a.lse[((int64_t)b * a.Hq + h) * S + qi] = (l > 0.f) ? (m + __log2f(l)) * kLn2 : -INFINITY;
    }
}

// ------------------------------------------------------- backward: dK, dV
template <int D>
struct KvRows {
    static constexpr int TILE = kQTile * D;  // elements of one Q or dO tile
    static constexpr int TB = TILE * 4;
    // LDS: Q0 Q1 dO0 dO1, then lse2 0/1 and D 0/1 (256 bytes each: one 64-lane dword DMA)
    static constexpr int OFF_STATS = 4 * TB;
    static constexpr int BYTES = OFF_STATS + 4 * 256;
};

template <int D>
__global__ __launch_bounds__(256, 1) void attn_bwd_kv_rows_f32(BwdArgs a) {
    using C = KvRows<D>;
    constexpr int NC = D / 16, ND = D / 32;
    extern __shared__ __attribute__((aligned(1024))) unsigned char rows_kv_smem[];
    const uint32_t lds = lds_addr(rows_kv_smem);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 5, c32 = lane & 31;
    const int S = a.S, Skv = a.Skv;
    const int nkb = (Skv + kRows - 1) / kRows;
    const int logical = xcd_logical_id(blockIdx.x, nkb * a.Hkv * a.B, gridDim.x);
    if (logical < 0) return;
    const int kblk = logical % nkb, hk = (logical / nkb) % a.Hkv, b = logical / (nkb * a.Hkv);
    const int G_ = a.Hq / a.Hkv;
    int kv_end = Skv;
    if (a.mask.kv_len) kv_end = min(max(a.mask.kv_len[b], 0), Skv);
    const int k0 = kblk * kRows;
    const int kw0 = k0 + wave * 32;  // first key of this wave
    const int key = kw0 + c32;       // this lane's key (column of S)

    // K and V rows of this wave's keys: lane <-> key, in-lane d
    Frag<float> kf[NC], vf[NC];
    row_frags<D>(kf, static_cast<const float*>(a.k) + a.mk.head_base(b, hk) + (int64_t)key * a.mk.ss, g, key < Skv);
    row_frags<D>(vf, static_cast<const float*>(a.v) + a.mv.head_base(b, hk) + (int64_t)key * a.mv.ss, g, key < Skv);

    // dK^T and dV^T: accumulator rows = d, columns = keys
    f32x16 dk[ND], dv[ND];
#pragma unroll
    for (int t = 0; t < ND; ++t) dk[t] = dv[t] = f32x16{};

    const int qb_start = a.mask.causal ? k0 / kQTile : 0;
    const int per_head = (S + kQTile - 1) / kQTile - qb_start;
    const int n_iter = k0 < kv_end ? G_ * per_head : 0;
    // blocks of each head that need a mask: all of them when the workgroup's keys run
    // past kv_end; else (causal) those holding a query before one of its keys
    int n_mask = 0;
    if (k0 + kRows > kv_end) n_mask = per_head;
    else if (a.mask.causal) n_mask = min(per_head, (k0 + kRows - 2) / kQTile - qb_start + 1);

    const uint32_t qbytes = (uint32_t)(a.mq.ss * 4), obytes = (uint32_t)(a.mdo.ss * 4);
    DmaPlan<float, D, kQTile, kWaves> pq, po;
    pq.init(qbytes, wave, lane);
    po.init(obytes, wave, lane);
    auto issue = [&](int it) {
        const int buf = it & 1;
        const int h = hk * G_ + it / per_head, q0 = (qb_start + it % per_head) * kQTile;
        pq.issue(lds + buf * C::TB, rows_rsrc<D>(static_cast<const float*>(a.q) + a.mq.head_base(b, h), a.mq, S),
                 (uint32_t)q0 * qbytes, wave);
        po.issue(lds + (2 + buf) * C::TB,
                 rows_rsrc<D>(static_cast<const float*>(a.dout) + a.mdo.head_base(b, h), a.mdo, S),
                 (uint32_t)q0 * obytes, wave);
        if (wave < 2) {  // wave 0: lse2 of the block's queries, wave 1: D
            const float* row = a.stats + (2 * ((int64_t)b * a.Hq + h) + wave) * S;
            dma4(make_rsrc(row, (uint32_t)(S * 4)), lds + C::OFF_STATS + (2 * wave + buf) * 256, (uint32_t)lane * 4u,
                 (uint32_t)q0 * 4u);
        }
    };

    auto compute = [&](auto mask_c, int buf, int q0) {
        constexpr bool MASK = decltype(mask_c)::value;
        const float* sQ = reinterpret_cast<const float*>(rows_kv_smem) + buf * C::TILE;
        const float* sdO = sQ + 2 * C::TILE;
        const uint32_t st = lds + C::OFF_STATS + 256u * buf + 16u * g;
        // S = Q K_w^T and dP = dO V_w^T: lane <-> key, in-lane query acc_row
        f32x16 s = f32x16{}, dp = f32x16{};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            Frag<float> fq, fo;
            tile_row_frag<D>(fq, sQ, c32, 16 * c + 8 * g);
            tile_row_frag<D>(fo, sdO, c32, 16 * c + 8 * g);
            mma(s, fq, kf[c]);
            mma(dp, fo, vf[c]);
        }
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const f32x4 l4 = *(const FBL_LDS f32x4*)(uintptr_t)(st + 32 * rr);
            const f32x4 d4 = *(const FBL_LDS f32x4*)(uintptr_t)(st + 512 + 32 * rr);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 4 * rr + j;
                float p = fast_exp2(__builtin_fmaf(s[r], a.scale_log2, -l4[j]));
                float ds = p * (dp[r] - d4[j]);
                if constexpr (MASK) {  // a masked score or dP may be inf or nan
                    if (key >= kv_end || (a.mask.causal && key > q0 + acc_row(r, g))) p = ds = 0.f;
                }
                s[r] = p;
                dp[r] = ds;
            }
        }
        // dV^T += dO^T P and dK^T += Q^T dS, contracting over the block's queries
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
            Frag<float> pb, dsb;
            float pv[8], dsv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) pv[e] = s[8 * cc + e], dsv[e] = dp[8 * cc + e];
            pack_frag(pb, pv);
            pack_frag(dsb, dsv);
#pragma unroll
            for (int t = 0; t < ND; ++t) {
                Frag<float> fo, fq;
                const int row0 = 16 * cc + 4 * g;
                tile_tr_frag<D>(fo, sdO, row0, row0 + 8, 32 * t, lane);
                tile_tr_frag<D>(fq, sQ, row0, row0 + 8, 32 * t, lane);
                mma(dv[t], fo, pb);
                mma(dk[t], fq, dsb);
            }
        }
    };
    auto step = [&](auto mask_c, int it) {
        wait_vmcnt<0>();
        __syncthreads();  // block `it` landed; block it-1's buffers are free
        if (it + 1 < n_iter) issue(it + 1);
        const int q0 = (qb_start + it % per_head) * kQTile;
        // a wave whose keys all follow every query of the block has nothing to add
        if (!(a.mask.causal && q0 + kQTile - 1 < kw0) && kw0 < kv_end) compute(mask_c, it & 1, q0);
    };
    if (n_iter > 0) issue(0);
    int it = 0;
    for (int hh = 0; hh < G_ && n_iter > 0; ++hh) {
        for (int j = 0; j < n_mask; ++j, ++it) step(std::true_type{}, it);
        for (int j = n_mask; j < per_head; ++j, ++it) step(std::false_type{}, it);
    }

    if (key < Skv) {
        const bool live = key < kv_end;  // else no part in the sums, whatever dO and Q hold
        float* dkrow = static_cast<float*>(a.dk) + a.mdk.head_base(b, hk) + (int64_t)key * a.mdk.ss;
        float* dvrow = static_cast<float*>(a.dv) + a.mdv.head_base(b, hk) + (int64_t)key * a.mdv.ss;
#pragma unroll
        for (int t = 0; t < ND; ++t)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                float x[4], y[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] = live ? dk[t][4 * rr + e] * a.scale : 0.f;
                    y[e] = live ? dv[t][4 * rr + e] : 0.f;
                }
                store4(dkrow + 32 * t + 8 * rr + 4 * g, x[0], x[1], x[2], x[3]);
                store4(dvrow + 32 * t + 8 * rr + 4 * g, y[0], y[1], y[2], y[3]);
            }
    }
}

// ----------------------------------------------------------- backward: dQ
template <int D>
__global__ __launch_bounds__(256, 1) void attn_bwd_q_rows_f32(BwdArgs a) {
    constexpr int NC = D / 16, ND = D / 32;
    constexpr int TILE = kTile / 2 * D;  // 32 keys: two tensors, two buffers
    constexpr int TB = TILE * 4;
    constexpr int KT = kTile / 2;
    extern __shared__ __attribute__((aligned(1024))) unsigned char rows_q_smem[];
    float* smem = reinterpret_cast<float*>(rows_q_smem);  // K0 K1 V0 V1
    const uint32_t lds = lds_addr(rows_q_smem);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 5, c32 = lane & 31;
    const int S = a.S, Skv = a.Skv;
    const int nqb = (S + kRows - 1) / kRows;
    const int logical = xcd_logical_id(blockIdx.x, nqb * a.Hq * a.B, gridDim.x);
    if (logical < 0) return;
    const int rank = logical % nqb, h = (logical / nqb) % a.Hq, b = logical / (nqb * a.Hq);
    const int qb = a.mask.causal ? (nqb - 1 - rank) : rank;
    const int hk = h / (a.Hq / a.Hkv);
    int kv_end = Skv;
    if (a.mask.kv_len) kv_end = min(max(a.mask.kv_len[b], 0), Skv);
    const int q0 = qb * kRows;
    const int qi = q0 + wave * 32 + c32;  // this lane's query (column of S^T)
    int k_hi = kv_end;
    if (a.mask.causal) k_hi = min(k_hi, q0 + kRows);
    const int nkb = (k_hi + KT - 1) / KT;

    Frag<float> qf[NC], of[NC];
    row_frags<D>(qf, static_cast<const float*>(a.q) + a.mq.head_base(b, h) + (int64_t)qi * a.mq.ss, g, qi < S);
    row_frags<D>(of, static_cast<const float*>(a.dout) + a.mdo.head_base(b, h) + (int64_t)qi * a.mdo.ss, g, qi < S);
    float lse2 = INFINITY, drow = 0.f;  // this lane's query row statistics
    if (qi < S) {
        const float* row = a.stats + 2 * ((int64_t)b * a.Hq + h) * S;
        lse2 = row[qi];
        drow = row[S + qi];
    }
    f32x16 dq[ND];  // dQ^T: rows = d, columns = queries
#pragma unroll
    for (int t = 0; t < ND; ++t) dq[t] = f32x16{};

    const Rsrc rk = rows_rsrc<D>(static_cast<const float*>(a.k) + a.mk.head_base(b, hk), a.mk, Skv);
    const Rsrc rv = rows_rsrc<D>(static_cast<const float*>(a.v) + a.mv.head_base(b, hk), a.mv, Skv);
    const uint32_t kbytes = (uint32_t)(a.mk.ss * 4), vbytes = (uint32_t)(a.mv.ss * 4);
    DmaPlan<float, D, KT, kWaves> pk, pv;
    pk.init(kbytes, wave, lane);
    pv.init(vbytes, wave, lane);
    auto issue = [&](int kb) {
        pk.issue(lds + (kb & 1) * TB, rk, (uint32_t)(kb * KT) * kbytes, wave);
        pv.issue(lds + (2 + (kb & 1)) * TB, rv, (uint32_t)(kb * KT) * vbytes, wave);
    };
    const int q_end = a.mask.causal ? min(kv_end, qi + 1) : kv_end;  // the first key the query does not see
    if (nkb > 0) issue(0);
    for (int kb = 0; kb < nkb; ++kb) {
        wait_vmcnt<0>();
        __syncthreads();  // tile kb landed; tile kb-1's buffers are free
        if (kb + 1 < nkb) issue(kb + 1);
        const float* sk = smem + (kb & 1) * TILE;
        const float* sv = sk + 2 * TILE;
        // S^T = K Q^T and dP^T = V dO^T: lane <-> query, in-lane key acc_row
        f32x16 s = f32x16{}, dp = f32x16{};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            Frag<float> fk, fv;
            tile_row_frag<D>(fk, sk, c32, 16 * c + 8 * g);
            tile_row_frag<D>(fv, sv, c32, 16 * c + 8 * g);
            mma(s, fk, qf[c]);
            mma(dp, fv, of[c]);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float p = fast_exp2(__builtin_fmaf(s[r], a.scale_log2, -lse2));
            const float ds = p * (dp[r] - drow);
            dp[r] = kb * KT + acc_row(r, g) >= q_end ? 0.f : ds;  // a masked score or dP may be inf or nan
        }
        // dQ^T += K^T dS^T over the tile's keys
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
            Frag<float> dsb;
            float dsv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) dsv[e] = dp[8 * cc + e];
            pack_frag(dsb, dsv);
#pragma unroll
            for (int t = 0; t < ND; ++t) {
                Frag<float> fk;
                const int row0 = 16 * cc + 4 * g;
                tile_tr_frag<D>(fk, sk, row0, row0 + 8, 32 * t, lane);
                mma(dq[t], fk, dsb);
            }
        }
    }
    if (qi < S) {
        float* dqrow = static_cast<float*>(a.dq) + a.mdq.head_base(b, h) + (int64_t)qi * a.mdq.ss;
#pragma unroll
        for (int t = 0; t < ND; ++t)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
                store4(dqrow + 32 * t + 8 * rr + 4 * g, dq[t][4 * rr] * a.scale, dq[t][4 * rr + 1] * a.scale,
                       dq[t][4 * rr + 2] * a.scale, dq[t][4 * rr + 3] * a.scale);
    }
}

// ---------------------------------------------------------------- the choice
// Times (us) of both forms: workgroups of 128 rows run in whole rounds of 256 (one per
// CU), those of 32 rows in rounds whose last is half paid for, each a fixed part and a
// part per tile or step.  Over 211 shapes (33 .. 2048 keys, 160 .. 1024 workgroups of 128
// rows) the choice is never more than 2% behind 32 rows nor 8% behind 128 (the 8%
// margin).  Forward walks past 320 keys stay with 32 rows, whose four partial sums
// round better; without a mask on full grids they take 5 .. 9% longer there.  A causal walk of
// more than one block is unequal, which 32 rows take better (S200 and up 0.8 .. 1.03).
int64_t blocks(int64_t n, int64_t of) { return (n + of - 1) / of; }
double rounds128(int64_t pairs, int64_t n) { return (double)blocks(pairs * blocks(n, kRows), 256); }
double rounds32(int64_t pairs, int64_t n, int64_t slots) {
    const int64_t wgs = pairs * blocks(n, 32);
    return std::max(1.0, 0.5 * ((double)wgs / (double)slots + (double)blocks(wgs, slots)));
}
bool unequal(const MaskArgs& m, int S) { return m.causal && S > kRows; }

}  // namespace

bool f32_rows_fwd(const FwdArgs& a, int D) {
    if (unequal(a.mask, a.S) || a.Skv > (D == 128 ? kTile : 320)) return false;
    const int64_t pairs = (int64_t)a.B * a.Hq;
    if (D == 128)  // a single tile (two take 72 us a round: the state of d = 128 does not fit)
        return rounds128(pairs, a.S) * 25.5 < 0.92 * rounds32(pairs, a.S, 256) * 9.5;
    const double rows = rounds128(pairs, a.S) * (6.7 + 4.2 * (double)blocks(a.Skv, kTile));
    const double step = (double)blocks(blocks(a.Skv, 32), 4);
    return rows < 0.92 * rounds32(pairs, a.S, 512) * std::max(10.2, 5.0 + 4.33 * step);
}

bool f32_rows_kv(const BwdArgs& a) {
    if (unequal(a.mask, a.S)) return false;
    const int64_t pairs = (int64_t)a.B * a.Hkv, walk = (int64_t)(a.Hq / a.Hkv) * blocks(a.S, 32);
    const double rows = rounds128(pairs, a.Skv) * (11.0 + 10.4 * (double)walk);
    return rows < 0.92 * rounds32(pairs, a.Skv, 256) * (11.0 + 8.4 * (double)blocks(walk, 4));
}

bool f32_rows_q(const BwdArgs& a) {
    if (unequal(a.mask, a.S)) return false;
    const int64_t pairs = (int64_t)a.B * a.Hq, walk = blocks(a.Skv, 32);
    const double rows = rounds128(pairs, a.S) * (11.0 + 7.8 * (double)walk);
    return rows < 0.92 * rounds32(pairs, a.S, 256) * (9.0 + 6.2 * (double)blocks(walk, 4));
}

template <int D>
hipError_t launch_attn_fwd_rows_f32(const FwdArgs& a, hipStream_t stream) {
    constexpr int lds = 4 * kTile * D * 4;
    const hipError_t e = ensure_dynamic_lds<&attn_fwd_rows_f32<D>>(lds);
    if (e != hipSuccess) return e;
    const int n = rank_major_grid((a.S + kRows - 1) / kRows, a.Hq * a.B);
    hipLaunchKernelGGL((attn_fwd_rows_f32<D>), dim3(n), dim3(256), lds, stream, a);
    return hipGetLastError();
}
template hipError_t launch_attn_fwd_rows_f32<64>(const FwdArgs&, hipStream_t);
template hipError_t launch_attn_fwd_rows_f32<128>(const FwdArgs&, hipStream_t);

hipError_t launch_attn_bwd_kv_rows_f32(const BwdArgs& a, hipStream_t stream) {
    constexpr int lds = KvRows<128>::BYTES;
    const hipError_t e = ensure_dynamic_lds<&attn_bwd_kv_rows_f32<128>>(lds);
    if (e != hipSuccess) return e;
    const int n = (a.Skv + kRows - 1) / kRows * a.Hkv * a.B;
    hipLaunchKernelGGL((attn_bwd_kv_rows_f32<128>), dim3(padded8(n)), dim3(256), lds, stream, a);
    return hipGetLastError();
}

hipError_t launch_attn_bwd_q_rows_f32(const BwdArgs& a, hipStream_t stream) {
    constexpr int lds = 4 * (kTile / 2) * 128 * 4;
    const hipError_t e = ensure_dynamic_lds<&attn_bwd_q_rows_f32<128>>(lds);
    if (e != hipSuccess) return e;
    const int n = (a.S + kRows - 1) / kRows * a.Hq * a.B;
    hipLaunchKernelGGL((attn_bwd_q_rows_f32<128>), dim3(padded8(n)), dim3(256), lds, stream, a);
    return hipGetLastError();
}

}  // namespace fbl
