// attn_f32.hip -- attention forward and backward for fp32 storage on
// token-major tensors, gfx950.  (bf16 storage: attn_fwd_bf16.hip,
// attn_bwd_kv.hip, attn_bwd_dq.hip, attn_bwd_q.hip.)
//
// Three kernels of one shape: attn_fwd_f32 (O, LSE), attn_bwd_kv_f32 (dK, dV)
// and attn_bwd_q_f32 (dQ, recomputing S and dP).  A workgroup of 4 wavefronts
// owns 32 rows of one (batch, head) -- queries in the forward and dQ passes,
// keys in the kv pass -- and walks the other side in tiles of 32 rows (the
// R-Tile, paper section 4.2) that stream from the token-major tensors into LDS
// by DMA: row r of a tile is token t0 + r of its head, at
// base + b*sb + (t0 + r)*ss + h*sh, so the head split and transpose of the
// multi-head attention chain (section 4.3.1) are a change of base address,
// never a copy.  No operand needs a physical transpose: one staged tile serves
// row reads, where a product contracts along d, and column reads, where it
// contracts along tokens.
//
// Why this split.  fp32 MFMAs (v_mfma_f32_32x32x2_f32) take 64 cycles each, so
// a 32 x 32 block of one product at d = 64 occupies its SIMD for 2048 cycles,
// and a wavefront that walks a whole row of blocks is a serial chain: with 128
// rows per workgroup, 32 per wavefront, the longest chain alone took 27 us
// (forward) or 55 us (kv) at 500 tokens while 160 of 256 CUs had no work.  Here
// the tiles of a workgroup's walk are dealt to four "streams", one wavefront
// each with its own LDS tiles (so the loop has no barrier), whose partial
// results are combined through LDS at the end in a fixed order.  A tile is
// refilled as soon as its last product is issued and arrives under the next
// one; a second buffer instead (one workgroup per CU at d = 64) measured the
// same at 500 tokens, 8 streams of 32 rows 0 .. 20% slower.
// B2 S500 H12 d64 causal: forward 43 -> 19.4, kv 77 -> 32.5, dQ 63 -> 25.6 us
// (the longest workgroup's chain); B4 S1024 H16 without a mask: 106 / 126 / 126
// TFLOP/s executed at d = 64 against 138 for a large library product.
#include <type_traits>

#include "cdna4.hpp"
#include "kernels.hpp"
#include "stage.hpp"
#include "tokmap.hpp"

namespace fbl {

namespace {

constexpr float kRescaleSlack = 8.0f;  // log2 of the largest unnormalised probability

template <int D>
struct F32Attn {
    static constexpr int NC = D / 16;              // 16-deep chunks over the head dim
    static constexpr int ND = D / 32;              // 32-wide column blocks
    static constexpr int NS = 4;                   // streams: one wavefront each
    static constexpr int TB = 32 * D * 4;          // bytes of one tile
    static constexpr int SB = 2 * TB;              // bytes of a stream: a tile of each of two tensors
    static constexpr int BYTES = NS * SB;
    static constexpr int STATS = BYTES;            // kv pass: [stream][lse2, D][64 floats]
    static constexpr int OWN = STATS + NS * 512;   // kv pass: the workgroup's V rows
    static constexpr int KV_BYTES = OWN + TB;
    static constexpr int QUADS = 4 * ND;           // f32x4 per lane of a 32 x D result
    static constexpr int OCC = D == 128 ? 1 : 2;   // workgroups per CU (registers, LDS)
    using Dma = DmaPlan<float, D, 32, 1>;
    static constexpr int LOADS = Dma::PER_WAVE;    // DMA loads of one tile
    static_assert(KV_BYTES * OCC <= 160 * 1024, "LDS of the workgroups of a CU");
};

// The workgroups of one launch as a grid of two dimensions: one alone holds at
// most 2^32 threads.
constexpr unsigned kGridX = 1u << 22;
FBL_DEV int workgroup_id() { return (int)(blockIdx.y * gridDim.x + blockIdx.x); }
dim3 grid_of(int n) { return dim3((unsigned)n < kGridX ? n : kGridX, ((unsigned)n + kGridX - 1) / kGridX); }

// Wait until at most N of this wave's DMA loads are in flight (what landed may
// be read), or for its LDS reads (what they read may be overwritten).  A
// stream's tiles are its wavefront's own, so no barrier follows that would
// order the compiler's LDS reads: the memory clobber does.
template <int N>
FBL_DEV void wait_tile() {
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
FBL_DEV void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }

template <int D>
FBL_DEV Rsrc head_rsrc(const void* base, const TokMap& m, int b, int h, int rows) {
    return make_rsrc(static_cast<const float*>(base) + m.head_base(b, h),
                     (uint32_t)(((int64_t)(rows - 1) * m.ss + D) * 4));
}

// Row `row` of a head as MFMA operands: lane <-> row, in-lane d = 16c + 8g + e.
template <int D>
FBL_DEV void row_operands(Frag<float>* f, const void* base, const TokMap& m, int b, int h, int row, int rows, int g,
                          bool neg) {
    const float* p = static_cast<const float*>(base) + m.head_base(b, h) + (int64_t)row * m.ss + 8 * g;
#pragma unroll
    for (int c = 0; c < D / 16; ++c) {
        f32x4 x = f32x4{}, y = f32x4{};
        if (row < rows) {
            x = __builtin_bit_cast(f32x4, load16(p + 16 * c));
            y = __builtin_bit_cast(f32x4, load16(p + 16 * c + 4));
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            f[c].v[e] = neg ? -x[e] : x[e];
            f[c].v[4 + e] = neg ? -y[e] : y[e];
        }
    }
}

// Per-lane LDS byte addresses of the fragment reads of a stream's tiles
// (TileGeom<float, D>'s swizzle), so that every read is one of these plus a
// compile-time constant.  The swizzle of row r is a function of r % 16, and of
// two tiles or rows 16 apart only constants differ:
//   row[]   row (lane % 32), 16-byte chunk x = 4c + 2g + h: one address per
//           x / 2 % 4 and h (at d = 128 chunks 16 apart differ by 256 bytes)
//   col[]   column lane % 32 at row 4g + e (+ 8): one address per e; 8 rows
//           further the chunk's bit 3 flips, which is bit 0 of the 32-column
//           block.  At d = 32 (8 chunks per row, swizzle r / 2 % 8) one per
//           e / 2 and run of 8 rows.
template <int D>
struct F32Lane {
    using G = TileGeom<float, D>;
    static constexpr int NX = D == 32 ? 4 : 8;
    uint32_t row[NX], col[4];
    FBL_DEV void init(uint32_t base, int lane) {
        const int g = lane >> 5, c32 = lane & 31;
#pragma unroll
        for (int x = 0; x < NX; ++x)
            row[x] = base + 4u * (uint32_t)G::off(c32, 16 * (x >> 1) + 8 * g + 4 * (x & 1));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int r = D == 32 ? 4 * g + 2 * (k & 1) + 8 * (k >> 1) : 4 * g + k;
            col[k] = base + 4u * (uint32_t)G::off(r, c32);
        }
    }
    // elements 16c + 8g .. +7 of row (lane % 32) of the tile `off` bytes on
    FBL_DEV void row_frag(Frag<float>& f, uint32_t off, int c) const {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 x = *(const FBL_LDS f32x4*)(uintptr_t)(row[(2 * c + h) % NX] + (off + 128u * NX * (2 * c / NX) / 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) f.v[4 * h + e] = x[e];
        }
    }
    // column 32t + (lane % 32) at rows 16cc + 4g + [0..3] and 8 rows further
    FBL_DEV void col_frag(Frag<float>& f, uint32_t off, int cc, int t) const {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int run = e >> 2, j = e & 3;
            if constexpr (D == 32)
                f.v[e] = *(const FBL_LDS float*)(uintptr_t)(col[(j >> 1) + 2 * run] + (off + 4u * D * (16 * cc + (j & 1))));
            else
                f.v[e] = *(const FBL_LDS float*)(uintptr_t)(col[j] + (off + 4u * D * (16 * cc + 8 * run) + 128u * (t ^ run)));
        }
    }
};

// acc += tile rows . f over d: accumulator rows = the tile's rows, columns = the lane's row.
template <int D>
FBL_DEV void row_product(f32x16& acc, const F32Lane<D>& la, uint32_t off, const Frag<float>* f) {
#pragma unroll
    for (int c = 0; c < D / 16; ++c) {
        Frag<float> t;
        la.row_frag(t, off, c);
        mma(acc, t, f[c]);
    }
}

// acc[t] += tile^T . x over the tile's 32 rows, x in accumulator order (its
// rows = the tile's rows): accumulator rows = d, columns = the lane's row.
template <int D>
FBL_DEV void col_product(f32x16* acc, const F32Lane<D>& la, uint32_t off, const f32x16& x) {
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
        Frag<float> xf;
#pragma unroll
        for (int e = 0; e < 8; ++e) xf.v[e] = x[8 * cc + e];
#pragma unroll
        for (int t = 0; t < D / 32; ++t) {
            Frag<float> tf;
            la.col_frag(tf, off, cc, t);
            mma(acc[t], tf, xf);
        }
    }
}

// Partial results through LDS: slot w holds one wavefront's 32 x D result as
// [quad][lane] x 16 bytes.
template <int D>
FBL_DEV void park(unsigned char* lds, int slot, const f32x16* acc, int lane) {
#pragma unroll
    for (int i = 0; i < F32Attn<D>::QUADS; ++i)
        *(FBL_LDS f32x4*)(lds + slot * F32Attn<D>::TB + (i * 64 + lane) * 16) =
            f32x4{acc[i / 4][4 * (i % 4)], acc[i / 4][4 * (i % 4) + 1], acc[i / 4][4 * (i % 4) + 2],
                  acc[i / 4][4 * (i % 4) + 3]};
}
template <int D>
FBL_DEV f32x4 parked(const unsigned char* lds, int slot, int i, int lane) {
    return *(const FBL_LDS f32x4*)(lds + slot * F32Attn<D>::TB + (i * 64 + lane) * 16);
}

// ---------------------------------------------------------------- forward
template <int D>
__global__ __launch_bounds__(256, F32Attn<D>::OCC) void attn_fwd_f32(FwdArgs a) {
    using C = F32Attn<D>;
    extern __shared__ __attribute__((aligned(1024))) unsigned char fwd_smem[];
    const uint32_t lds = lds_addr(fwd_smem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int st = wave;  // one stream per wavefront
    const int g = lane >> 5, c32 = lane & 31;
    const int S = a.S, Skv = a.Skv;
    const int nqb = (S + 31) / 32;
    int rank, bh;
    if (!rank_major_item(workgroup_id(), nqb, a.Hq * a.B, rank, bh)) return;
    const int h = bh % a.Hq, b = bh / a.Hq;
    // causal: the last query blocks see the most keys; start them first
    const int qb = a.mask.causal ? (nqb - 1 - rank) : rank;
    const int hk = h / (a.Hq / a.Hkv);
    int kv_end = Skv;
    if (a.mask.kv_len) kv_end = min(max(a.mask.kv_len[b], 0), Skv);
    const int qw0 = qb * 32;
    const int qi = qw0 + c32;  // this lane's query (column of S^T)
    int k_hi = kv_end;
    if (a.mask.causal) k_hi = min(k_hi, (qb + 1) * 32);
    const int nkb = (k_hi + 31) / 32;

    // the softmax FMA below needs a non-negative scale: fold the sign into Q
    const bool neg = a.scale_log2 < 0.f;
    const float c = neg ? -a.scale_log2 : a.scale_log2;
    Frag<float> qf[C::NC];
    row_operands<D>(qf, a.q, a.mq, b, h, qi, S, g, neg);

    const Rsrc rk = head_rsrc<D>(a.k, a.mk, b, hk, Skv), rv = head_rsrc<D>(a.v, a.mv, b, hk, Skv);
    const uint32_t kbytes = (uint32_t)(a.mk.ss * 4), vbytes = (uint32_t)(a.mv.ss * 4);
    typename C::Dma dk, dv;
    dk.init(kbytes, 0, lane);
    dv.init(vbytes, 0, lane);
    const uint32_t tk = lds + st * C::SB, tv = tk + C::TB;
    auto issue_k = [&](int j) { if (j < nkb) dk.issue(tk, rk, (uint32_t)(j * 32) * kbytes, 0); };
    auto issue_v = [&](int j) { if (j < nkb) dv.issue(tv, rv, (uint32_t)(j * 32) * vbytes, 0); };

    f32x16 o[C::ND];
#pragma unroll
    for (int t = 0; t < C::ND; ++t) o[t] = f32x16{};
    float m = -INFINITY;  // running maximum (log2 units), equal in both lane halves
    float l = 0.f;        // this lane half's share of the running sum

    F32Lane<D> la;
    la.init(lds + st * C::SB, lane);
    // One key tile.  Its K rows are done with after S, its V rows after O += P V:
    // each buffer is refilled with the stream's next tile right then, and has
    // the other half of the step to arrive.
    auto block = [&](auto mask_c, int j) {
        constexpr bool MASK = decltype(mask_c)::value;
        const int k0 = j * 32;
        wait_tile<C::LOADS>();  // K has landed; V may be in flight
        f32x16 s = f32x16{};
        row_product<D>(s, la, 0, qf);
        wait_lds();
        issue_k(j + C::NS);
        if constexpr (MASK) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = k0 + acc_row(r, g);
                if (key >= kv_end || (a.mask.causal && key > qi)) s[r] = -INFINITY;
            }
        }
        float mx = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
        mx = fmaxf(mx, other_half(mx)) * c;
        if (__any(mx > m + kRescaleSlack)) {
            const float m_new = fmaxf(m, mx);
            const float alpha = (m_new == -INFINITY) ? 1.f : fast_exp2(m - m_new);  // 0 when m was -inf
            l *= alpha;
#pragma unroll
            for (int t = 0; t < C::ND; ++t) o[t] *= alpha;
            m = m_new;
        }
        const float nm = (m == -INFINITY) ? 0.f : -m;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float p = fast_exp2(__builtin_fmaf(s[r], c, nm));
            if constexpr (MASK) {
                if (s[r] == -INFINITY) p = 0.f;
            }
            s[r] = p;
            l += p;
        }
        if (j + C::NS < nkb) wait_tile<C::LOADS>();
        else wait_tile<0>();
        col_product<D>(o, la, C::TB, s);
        wait_lds();
        issue_v(j + C::NS);
    };

    issue_k(st);
    issue_v(st);
    for (int j = st; j < nkb; j += C::NS) {
        if (j * 32 + 32 > kv_end || (a.mask.causal && j * 32 + 31 > qw0)) block(std::true_type{}, j);
        else block(std::false_type{}, j);
    }
    l += other_half(l);

    // Combine the streams in a fixed order; every wavefront takes its share of the columns.
    __syncthreads();
    park<D>(fwd_smem, wave, o, lane);
    float* ml = reinterpret_cast<float*>(fwd_smem + 4 * C::TB);  // [wave][m, l][32]
    if (g == 0) {
        ml[wave * 64 + c32] = m;
        ml[wave * 64 + 32 + c32] = l;
    }
    __syncthreads();
    float mm = -INFINITY, f[C::NS], lsum = 0.f;
#pragma unroll
    for (int w = 0; w < C::NS; ++w) mm = fmaxf(mm, ml[w * 64 + c32]);
#pragma unroll
    for (int w = 0; w < C::NS; ++w) {
        const float mw = ml[w * 64 + c32];
        f[w] = mw == -INFINITY ? 0.f : fast_exp2(mw - mm);
        lsum += f[w] * ml[w * 64 + 32 + c32];
    }
    if (qi < S) {
        const float inv = (lsum > 0.f) ? 1.f / lsum : 0.f;
        float* orow = static_cast<float*>(a.o) + a.mo.head_base(b, h) + (int64_t)qi * a.mo.ss;
#pragma unroll
        for (int i = 0; i < C::QUADS / C::NS; ++i) {
            const int q = i * C::NS + st;
            f32x4 x = f32x4{};
#pragma unroll
            for (int w = 0; w < C::NS; ++w) x += f[w] * parked<D>(fwd_smem, w, q, lane);
            *reinterpret_cast<f32x4*>(orow + 32 * (q / 4) + 8 * (q % 4) + 4 * g) = x * inv;
        }
        if (g == 0 && st == 0)
            a.lse[((int64_t)b * a.Hq + h) * S + qi] = (lsum > 0.f) ? (mm + __log2f(lsum)) * kLn2 : -INFINITY;
    }
}

// ------------------------------------------------------- backward: dK, dV
template <int D>
__global__ __launch_bounds__(256, F32Attn<D>::OCC) void attn_bwd_kv_f32(BwdArgs a) {
    using C = F32Attn<D>;
    extern __shared__ __attribute__((aligned(1024))) unsigned char kv_smem[];
    const uint32_t lds = lds_addr(kv_smem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int st = wave;
    const int g = lane >> 5, c32 = lane & 31;
    const int S = a.S, Skv = a.Skv;
    const int nkb = (Skv + 31) / 32;
    // causal: the first key blocks see the most queries and start first
    int kblk, bh;
    if (!rank_major_item(workgroup_id(), nkb, a.Hkv * a.B, kblk, bh)) return;
    const int hk = bh % a.Hkv, b = bh / a.Hkv;
    const int G_ = a.Hq / a.Hkv;
    int kv_end = Skv;
    if (a.mask.kv_len) kv_end = min(max(a.mask.kv_len[b], 0), Skv);
    const int kw0 = kblk * 32;
    const int key = kw0 + c32;  // this lane's key (column of S)

    // K rows in registers, V rows (the same for every stream) in LDS: both in
    // registers leave none for two wavefronts per SIMD at d = 64 and spill at 128
    Frag<float> kf[C::NC];
    row_operands<D>(kf, a.k, a.mk, b, hk, key, Skv, g, false);
    DmaPlan<float, D, 32, C::NS> pv;
    pv.init((uint32_t)(a.mv.ss * 4), wave, lane);
    pv.issue(lds + C::OWN, head_rsrc<D>(a.v, a.mv, b, hk, Skv), (uint32_t)(kw0 * a.mv.ss * 4), wave);

    // the blocks of 32 queries of every query head of the group, dealt to the streams
    const int qb0 = a.mask.causal ? kblk : 0;
    const int per_head = (S + 31) / 32 - qb0;
    const int n_blk = kw0 < kv_end ? G_ * per_head : 0;
    const uint32_t qbytes = (uint32_t)(a.mq.ss * 4), obytes = (uint32_t)(a.mdo.ss * 4);
    typename C::Dma pq, po;
    pq.init(qbytes, 0, lane);
    po.init(obytes, 0, lane);
    const uint32_t tq = lds + st * C::SB, to = tq + C::TB, ts = lds + C::STATS + st * 512;
    auto issue_q = [&](int i) {
        if (i >= n_blk) return;
        const int h = hk * G_ + i / per_head, q0 = (qb0 + i % per_head) * 32;
        pq.issue(tq, head_rsrc<D>(a.q, a.mq, b, h, S), (uint32_t)q0 * qbytes, 0);
    };
    auto issue_do = [&](int i) {  // and the block's row statistics (lanes past the row read zeros)
        if (i >= n_blk) return;
        const int h = hk * G_ + i / per_head, q0 = (qb0 + i % per_head) * 32;
        po.issue(to, head_rsrc<D>(a.dout, a.mdo, b, h, S), (uint32_t)q0 * obytes, 0);
        const float* row = a.stats + 2 * ((int64_t)b * a.Hq + h) * S;
        dma4(make_rsrc(row, (uint32_t)(S * 4)), ts, (uint32_t)lane * 4u, (uint32_t)q0 * 4u);
        dma4(make_rsrc(row + S, (uint32_t)(S * 4)), ts + 256, (uint32_t)lane * 4u, (uint32_t)q0 * 4u);
    };

    // dK^T and dV^T: accumulator rows = d, columns = keys
    f32x16 dk[C::ND], dv[C::ND];
#pragma unroll
    for (int t = 0; t < C::ND; ++t) dk[t] = dv[t] = f32x16{};

    F32Lane<D> la;
    la.init(lds + st * C::SB, lane);
    F32Lane<D> lown;
    lown.init(lds + C::OWN, lane);
    const float* stats = reinterpret_cast<const float*>(kv_smem + C::STATS + st * 512);
    // One block of queries.  dO is done with after dV, Q after dK: each buffer is
    // refilled right then; the next block's dP comes first, so that each load
    // has at least one product to arrive under.
    auto block = [&](auto mask_c, int i, int q0) {
        constexpr bool MASK = decltype(mask_c)::value;
        // S = Q K_w^T and dP = dO V_w^T: lane <-> key, in-lane query acc_row
        f32x16 s = f32x16{}, dp = f32x16{};
        wait_tile<C::LOADS>();  // dO and the statistics have landed; Q may be in flight
#pragma unroll
        for (int c = 0; c < C::NC; ++c) {
            Frag<float> of, vf;
            la.row_frag(of, C::TB, c);
            lown.row_frag(vf, 0, c);
            mma(dp, of, vf);
        }
        wait_tile<0>();
        row_product<D>(s, la, 0, kf);
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const f32x4 l4 = *(const FBL_LDS f32x4*)(stats + 8 * rr + 4 * g);
            const f32x4 d4 = *(const FBL_LDS f32x4*)(stats + 64 + 8 * rr + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 4 * rr + e;
                float p = fast_exp2(__builtin_fmaf(s[r], a.scale_log2, -l4[e]));
                if constexpr (MASK) {
                    if (key >= kv_end || (a.mask.causal && key > q0 + acc_row(r, g))) p = 0.f;
                }
                s[r] = p;
                dp[r] = p * (dp[r] - d4[e]);
            }
        }
        col_product<D>(dv, la, C::TB, s);
        wait_lds();
        issue_do(i + C::NS);
        col_product<D>(dk, la, 0, dp);
        wait_lds();
        issue_q(i + C::NS);
    };

    wait_tile<0>();
    __syncthreads();  // the V rows are in LDS
    issue_do(st);
    issue_q(st);
    for (int i = st; i < n_blk; i += C::NS) {
        const int q0 = (qb0 + i % per_head) * 32;
        if (kw0 + 32 > kv_end || (a.mask.causal && kw0 + 31 > q0)) block(std::true_type{}, i, q0);
        else block(std::false_type{}, i, q0);
    }

    // sum over the streams; every wavefront takes its share of the columns
    __syncthreads();
    park<D>(kv_smem, wave, dk, lane);
    park<D>(kv_smem, 4 + wave, dv, lane);
    __syncthreads();
    if (key < Skv) {
        float* dkrow = static_cast<float*>(a.dk) + a.mdk.head_base(b, hk) + (int64_t)key * a.mdk.ss;
        float* dvrow = static_cast<float*>(a.dv) + a.mdv.head_base(b, hk) + (int64_t)key * a.mdv.ss;
#pragma unroll
        for (int i = 0; i < C::QUADS / C::NS; ++i) {
            const int q = i * C::NS + st, col = 32 * (q / 4) + 8 * (q % 4) + 4 * g;
            f32x4 x = f32x4{}, y = f32x4{};
#pragma unroll
            for (int w = 0; w < C::NS; ++w) {
                x += parked<D>(kv_smem, w, q, lane);
                y += parked<D>(kv_smem, 4 + w, q, lane);
            }
            *reinterpret_cast<f32x4*>(dkrow + col) = x * a.scale;
            *reinterpret_cast<f32x4*>(dvrow + col) = y;
        }
    }
}

// ----------------------------------------------------------- backward: dQ
template <int D>
__global__ __launch_bounds__(256, F32Attn<D>::OCC) void attn_bwd_q_f32(BwdArgs a) {
    using C = F32Attn<D>;
    extern __shared__ __attribute__((aligned(1024))) unsigned char q_smem[];
    const uint32_t lds = lds_addr(q_smem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int st = wave;
    const int g = lane >> 5, c32 = lane & 31;
    const int S = a.S, Skv = a.Skv;
    const int nqb = (S + 31) / 32;
    int rank, bh;
    if (!rank_major_item(workgroup_id(), nqb, a.Hq * a.B, rank, bh)) return;
    const int h = bh % a.Hq, b = bh / a.Hq;
    const int qb = a.mask.causal ? (nqb - 1 - rank) : rank;
    const int hk = h / (a.Hq / a.Hkv);
    int kv_end = Skv;
    if (a.mask.kv_len) kv_end = min(max(a.mask.kv_len[b], 0), Skv);
    const int qw0 = qb * 32;
    const int qi = qw0 + c32;  // this lane's query (column of S^T)
    int k_hi = kv_end;
    if (a.mask.causal) k_hi = min(k_hi, (qb + 1) * 32);
    const int nkb = (k_hi + 31) / 32;

    Frag<float> qf[C::NC], of[C::NC];
    row_operands<D>(qf, a.q, a.mq, b, h, qi, S, g, false);
    row_operands<D>(of, a.dout, a.mdo, b, h, qi, S, g, false);
    float lse2 = INFINITY, drow = 0.f;  // this lane's query row statistics
    if (qi < S) {
        const float* row = a.stats + 2 * ((int64_t)b * a.Hq + h) * S;
        lse2 = row[qi];
        drow = row[S + qi];
    }

    const Rsrc rk = head_rsrc<D>(a.k, a.mk, b, hk, Skv), rv = head_rsrc<D>(a.v, a.mv, b, hk, Skv);
    const uint32_t kbytes = (uint32_t)(a.mk.ss * 4), vbytes = (uint32_t)(a.mv.ss * 4);
    typename C::Dma pk, pv;
    pk.init(kbytes, 0, lane);
    pv.init(vbytes, 0, lane);
    const uint32_t tk = lds + st * C::SB, tv = tk + C::TB;
    auto issue_k = [&](int j) { if (j < nkb) pk.issue(tk, rk, (uint32_t)(j * 32) * kbytes, 0); };
    auto issue_v = [&](int j) { if (j < nkb) pv.issue(tv, rv, (uint32_t)(j * 32) * vbytes, 0); };

    f32x16 dq[C::ND];  // dQ^T: rows = d, columns = queries
#pragma unroll
    for (int t = 0; t < C::ND; ++t) dq[t] = f32x16{};

    F32Lane<D> la;
    la.init(lds + st * C::SB, lane);
    // One key tile.  Its V rows are done with after dP, its K rows after dQ.
    auto block = [&](auto mask_c, int j) {
        constexpr bool MASK = decltype(mask_c)::value;
        const int k0 = j * 32;
        // S^T = K Q^T and dP^T = V dO^T: lane <-> query, in-lane key acc_row
        f32x16 s = f32x16{}, dp = f32x16{};
        wait_tile<C::LOADS>();  // V has landed; K may be in flight
        row_product<D>(dp, la, C::TB, of);
        wait_lds();
        issue_v(j + C::NS);
        if (j + C::NS < nkb) wait_tile<C::LOADS>();
        else wait_tile<0>();
        row_product<D>(s, la, 0, qf);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float p = fast_exp2(__builtin_fmaf(s[r], a.scale_log2, -lse2));
            if constexpr (MASK) {
                const int key = k0 + acc_row(r, g);
                if (key >= kv_end || (a.mask.causal && key > qi)) p = 0.f;
            }
            dp[r] = p * (dp[r] - drow);
        }
        col_product<D>(dq, la, 0, dp);
        wait_lds();
        issue_k(j + C::NS);
    };

    issue_v(st);
    issue_k(st);
    for (int j = st; j < nkb; j += C::NS) {
        if (j * 32 + 32 > kv_end || (a.mask.causal && j * 32 + 31 > qw0)) block(std::true_type{}, j);
        else block(std::false_type{}, j);
    }

    __syncthreads();
    park<D>(q_smem, wave, dq, lane);
    __syncthreads();
    if (qi < S) {
        float* dqrow = static_cast<float*>(a.dq) + a.mdq.head_base(b, h) + (int64_t)qi * a.mdq.ss;
#pragma unroll
        for (int i = 0; i < C::QUADS / C::NS; ++i) {
            const int q = i * C::NS + st;
            f32x4 x = f32x4{};
#pragma unroll
            for (int w = 0; w < C::NS; ++w) x += parked<D>(q_smem, w, q, lane);
            *reinterpret_cast<f32x4*>(dqrow + 32 * (q / 4) + 8 * (q % 4) + 4 * g) = x * a.scale;
        }
    }
}

}  // namespace

template <int D>
hipError_t launch_attn_fwd_f32(const FwdArgs& a, hipStream_t stream) {
    using C = F32Attn<D>;
    const hipError_t e = ensure_dynamic_lds<&attn_fwd_f32<D>>(C::BYTES);
    if (e != hipSuccess) return e;
    const int n = rank_major_grid((a.S + 32 - 1) / 32, a.Hq * a.B);
    hipLaunchKernelGGL((attn_fwd_f32<D>), grid_of(n), dim3(256), C::BYTES, stream, a);
    return hipGetLastError();
}

template <int D>
hipError_t launch_attn_bwd_kv_f32(const BwdArgs& a, hipStream_t stream) {
    using C = F32Attn<D>;
    const hipError_t e = ensure_dynamic_lds<&attn_bwd_kv_f32<D>>(C::KV_BYTES);
    if (e != hipSuccess) return e;
    const int n = rank_major_grid((a.Skv + 32 - 1) / 32, a.Hkv * a.B);
    hipLaunchKernelGGL((attn_bwd_kv_f32<D>), grid_of(n), dim3(256), C::KV_BYTES, stream, a);
    return hipGetLastError();
}

template <int D>
hipError_t launch_attn_bwd_q_f32(const BwdArgs& a, hipStream_t stream) {
    using C = F32Attn<D>;
    const hipError_t e = ensure_dynamic_lds<&attn_bwd_q_f32<D>>(C::BYTES);
    if (e != hipSuccess) return e;
    const int n = rank_major_grid((a.S + 32 - 1) / 32, a.Hq * a.B);
    hipLaunchKernelGGL((attn_bwd_q_f32<D>), grid_of(n), dim3(256), C::BYTES, stream, a);
    return hipGetLastError();
}

#define FBL_ATTN_F32(D)                                                      \
    template hipError_t launch_attn_fwd_f32<D>(const FwdArgs&, hipStream_t); \
    template hipError_t launch_attn_bwd_kv_f32<D>(const BwdArgs&, hipStream_t); \
    template hipError_t launch_attn_bwd_q_f32<D>(const BwdArgs&, hipStream_t);
FBL_ATTN_F32(32)
FBL_ATTN_F32(64)
FBL_ATTN_F32(128)
#undef FBL_ATTN_F32

}  // namespace fbl
