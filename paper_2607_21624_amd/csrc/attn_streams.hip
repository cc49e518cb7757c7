// attn_streams.hip -- attention forward and backward in 32-row workgroups on
// token-major tensors, gfx950: the fp32 calls (but for short walks of many rows,
// attn_rows_f32.hip), and the bf16 calls too small for the larger tiles of
// attn_fwd_bf16.hip, attn_bwd_kv.hip and attn_bwd_dq.hip.
//
// Kernels of one shape: attn_fwd_streams (O, LSE), a kv pass (dK, dV) and a q
// pass (dQ, recomputing S and dP).  attn_bwd_streams runs both passes as one
// launch, each workgroup forming the row statistics it needs from O, dO and the
// LSE; attn_bwd_kv_f32 and attn_bwd_q_f32 run them apart.  A workgroup of 4 wavefronts
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
//
// One launch for the whole backward: statistics, kv and dQ passes of 4.8 + 32.5 +
// 26.2 us in their own launches (the shape above) become 45: no gaps, and the dQ
// workgroups fill the CUs that the longest kv chains leave.  What a small call
// waits for is latency -- its loads, then a chain of products with barriers -- so the
// more workgroups the better: B8 S128 H12 d64 bf16 ran 96 workgroups of two serial
// steps each in 16.1 us, now 768 of one in 9.3; B1 S64 H2 d32 fp32 13.4 -> 7.1.  bf16
// products are 16 times shorter than fp32's and hide little, so three workgroups
// share a CU where the state fits 168 registers (d <= 64: the workgroup's K and V
// rows in LDS, 13.7 us with two and the rows in registers).  Masks are one
// comparison per score on one path: two paths per step cost the registers more
// (spills) than the comparisons.
#include <type_traits>

#include "cdna4.hpp"
#include "kernels.hpp"
#include "stage.hpp"
#include "tokmap.hpp"

namespace fbl {

namespace {

constexpr float kRescaleSlack = 8.0f;  // log2 of the largest unnormalised probability

template <typename T, int D>
struct Streams {
    static constexpr int ES = (int)sizeof(T);
    static constexpr int NC = D / 16;              // 16-deep chunks over the head dim
    static constexpr int ND = D / 32;              // 32-wide column blocks
    static constexpr int NS = 4;                   // streams: one wavefront each
    static constexpr int TB = 32 * D * ES;         // bytes of one tile
    static constexpr int SB = 2 * TB;              // bytes of a stream: a tile of each of two tensors
    static constexpr int PB = 32 * D * 4;          // bytes of one parked 32 x D result
    static constexpr int BYTES = NS * SB;
    static constexpr int FWD_BYTES = BYTES > NS * PB + 1024 ? BYTES : NS * PB + 1024;
    // kv pass: fp32 parks dK and dV side by side, bf16 (whose tiles take half
    // of that) one after the other
    static constexpr bool PARK2 = BYTES >= 2 * NS * PB;
    static constexpr int STATS = BYTES;            // kv pass: [stream][lse2, D][64 floats]
    // kv pass: the workgroup's V and K rows, the same for every stream, where
    // registers are what limits the wavefronts of a SIMD
    static constexpr bool OWN_V = ES == 4 || D < 128, OWN_K = ES == 2 && D < 128;
    static constexpr int OWN = STATS + NS * 512;
    static constexpr int KV_BYTES = OWN + (OWN_V ? TB : 0) + (OWN_K ? TB : 0);
    static constexpr bool HOLD_O = ES == 2;        // the next block's O rows in registers
    static constexpr int QUADS = 4 * ND;           // f32x4 per lane of a 32 x D result
    // workgroups per CU (registers, LDS)
    static constexpr int OCC = D == 128 ? 1 : ES == 2 ? 3 : 2;
    static constexpr int FWD_OCC = D == 128 ? (ES == 2 ? 2 : 1) : ES == 2 ? 3 : 2;
    static constexpr int LOADS = TB / 1024;        // DMA loads of one tile
    static_assert(KV_BYTES * OCC <= 160 * 1024, "LDS of the workgroups of a CU");
    static_assert(BYTES >= NS * PB, "the parked results of one product fit the streams' tiles");
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

template <typename T, int D>
FBL_DEV Rsrc head_rsrc(const void* base, const TokMap& m, int b, int h, int rows) {
    Rsrc r = make_rsrc(static_cast<const T*>(base) + m.head_base(b, h),
                       (uint32_t)(((int64_t)(rows - 1) * m.ss + D) * (int)sizeof(T)));
    // (uniform, but its head may come from a division, which the vector ALUs do)
    r[0] = __builtin_amdgcn_readfirstlane(r[0]);
    r[1] = __builtin_amdgcn_readfirstlane(r[1]);
    r[2] = __builtin_amdgcn_readfirstlane(r[2]);
    return r;
}

// DMA of a 32-row tile by one wavefront.  A row's chunk order repeats after 16
// rows (TileGeom::swz), so the offsets of the first 16 rows serve both halves.
template <typename T, int D>
struct StreamDma {
    using G = TileGeom<T, D>;
    static constexpr int HALF = Streams<T, D>::LOADS / 2;
    uint32_t voff[HALF];
    FBL_DEV void init(uint32_t row_bytes, int lane) {
#pragma unroll
        for (int j = 0; j < HALF; ++j) {
            const int q = j * 64 + lane, r = q / G::CPR;
            voff[j] = (uint32_t)r * row_bytes + (uint32_t)((q % G::CPR) ^ G::swz(r)) * 16u;
        }
    }
    FBL_DEV void issue(uint32_t tile, Rsrc rs, uint32_t row0_bytes, uint32_t row_bytes) const {
#pragma unroll
        for (int j = 0; j < HALF; ++j) {
            if (j == 0) dma16<true>(rs, tile, voff[0], row0_bytes);
            else dma16<false>(rs, tile + j * 1024u, voff[j], row0_bytes);
        }
        uint32_t half = 16 * row_bytes;
        asm volatile("" : "+s"(half));  // added at each use, not kept in as many registers again
#pragma unroll
        for (int j = 0; j < HALF; ++j) dma16<true>(rs, tile + (HALF + j) * 1024u, voff[j] + half, row0_bytes);
    }
};

// Row `row` of a head as MFMA operands: lane <-> row, in-lane d = 16c + 8g + e.
template <typename T, int D>
FBL_DEV void row_operands(Frag<T>* f, const void* base, const TokMap& m, int b, int h, int row, int rows, int g,
                          bool neg) {
    const T* p = static_cast<const T*>(base) + m.head_base(b, h) + (int64_t)row * m.ss + 8 * g;
#pragma unroll
    for (int c = 0; c < D / 16; ++c) {
        if constexpr (sizeof(T) == 2) {
            uint4 x = uint4{0u, 0u, 0u, 0u};
            if (row < rows) x = load16(p + 16 * c);
            if (neg) { x.x ^= 0x80008000u; x.y ^= 0x80008000u; x.z ^= 0x80008000u; x.w ^= 0x80008000u; }
            f[c].v = __builtin_bit_cast(bf16x8, x);
        } else {
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
template <typename T, int D>
struct StreamLane;

template <int D>
struct StreamLane<float, D> {
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
    FBL_DEV void row_frag(Frag<float>& f, uint32_t off, int c) const { row_frag_at(f, 0, off, c); }
    FBL_DEV void row_frag_at(Frag<float>& f, uint32_t moved, uint32_t off, int c) const {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 x = *(const FBL_LDS f32x4*)(uintptr_t)(row[(2 * c + h) % NX] + moved +
                                                              (off + 128u * NX * (2 * c / NX) / 4));
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

// bf16: the addresses of stage.hpp; transposed reads for the columns.
template <int D>
struct StreamLane<bf16, D> {
    LaneOffsets<D> lo;
    FBL_DEV void init(uint32_t base, int lane) { lo.init(base, lane); }
    FBL_DEV void row_frag(Frag<bf16>& f, uint32_t off, int c) const { f.v = lds_b128(lo.row[c], off); }
    FBL_DEV void row_frag_at(Frag<bf16>& f, uint32_t moved, uint32_t off, int c) const {
        f.v = lds_b128(lo.row[c] + moved, off);
    }
    FBL_DEV void col_frag(Frag<bf16>& f, uint32_t off, int cc, int t) const {
        const bf16x4 x = lds_tr(lo.tr[t][0], off + 32u * D * cc), y = lds_tr(lo.tr[t][1], off + 32u * D * cc);
        f.v = bf16x8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
    }
};

// acc += tile rows . f over d: accumulator rows = the tile's rows, columns = the lane's row.
template <typename T, int D>
FBL_DEV void row_product(f32x16& acc, const StreamLane<T, D>& la, uint32_t off, const Frag<T>* f) {
#pragma unroll
    for (int c = 0; c < D / 16; ++c) {
        Frag<T> t;
        la.row_frag(t, off, c);
        mma(acc, t, f[c]);
    }
}

// acc[t] += tile^T . x over the tile's 32 rows, x in accumulator order (its
// rows = the tile's rows): accumulator rows = d, columns = the lane's row.
template <typename T, int D>
FBL_DEV void col_product(f32x16* acc, const StreamLane<T, D>& la, uint32_t off, const f32x16& x) {
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
        Frag<T> xf;
        float xv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) xv[e] = x[8 * cc + e];
        pack_frag(xf, xv);
#pragma unroll
        for (int t = 0; t < D / 32; ++t) {
            Frag<T> tf;
            la.col_frag(tf, off, cc, t);
            mma(acc[t], tf, xf);
        }
        if constexpr (sizeof(T) == 2) __builtin_amdgcn_sched_barrier(0);
    }
}

// Partial results through LDS: slot w holds one wavefront's 32 x D result as
// [quad][lane] x 16 bytes.
template <typename T, int D>
FBL_DEV void park(unsigned char* lds, int slot, const f32x16* acc, int lane) {
#pragma unroll
    for (int i = 0; i < Streams<T, D>::QUADS; ++i)
        *(FBL_LDS f32x4*)(lds + slot * Streams<T, D>::PB + (i * 64 + lane) * 16) =
            f32x4{acc[i / 4][4 * (i % 4)], acc[i / 4][4 * (i % 4) + 1], acc[i / 4][4 * (i % 4) + 2],
                  acc[i / 4][4 * (i % 4) + 3]};
}
template <typename T, int D>
FBL_DEV f32x4 parked(const unsigned char* lds, int slot, int i, int lane) {
    return *(const FBL_LDS f32x4*)(lds + slot * Streams<T, D>::PB + (i * 64 + lane) * 16);
}

// ---------------------------------------------------------------- forward
template <typename T, int D>
__global__ __launch_bounds__(256, (Streams<T, D>::FWD_OCC)) void attn_fwd_streams(FwdArgs a) {
    using C = Streams<T, D>;
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
    Frag<T> qf[C::NC];
    row_operands<T, D>(qf, a.q, a.mq, b, h, qi, S, g, neg);

    const Rsrc rk = head_rsrc<T, D>(a.k, a.mk, b, hk, Skv), rv = head_rsrc<T, D>(a.v, a.mv, b, hk, Skv);
    const uint32_t kbytes = (uint32_t)(a.mk.ss * C::ES), vbytes = (uint32_t)(a.mv.ss * C::ES);
    StreamDma<T, D> dk, dv;
    dk.init(kbytes, lane);
    dv.init(vbytes, lane);
    const uint32_t tk = lds + st * C::SB, tv = tk + C::TB;
    auto issue_k = [&](int j) { if (j < nkb) dk.issue(tk, rk, (uint32_t)(j * 32) * kbytes, kbytes); };
    auto issue_v = [&](int j) { if (j < nkb) dv.issue(tv, rv, (uint32_t)(j * 32) * vbytes, vbytes); };

    f32x16 o[C::ND];
#pragma unroll
    for (int t = 0; t < C::ND; ++t) o[t] = f32x16{};
    float m = -INFINITY;  // running maximum (log2 units), equal in both lane halves
    float l = 0.f;        // this lane half's share of the running sum

    StreamLane<T, D> la;
    la.init(lds + st * C::SB, lane);
    // One key tile.  Its K rows are done with after S, its V rows after O += P V:
    // each buffer is refilled with the stream's next tile right then, and has
    // the other half of the step to arrive.
    auto block = [&](auto mask_c, int j) {
        constexpr bool MASK = decltype(mask_c)::value;
        const int k0 = j * 32;
        wait_tile<C::LOADS>();  // K has landed; V may be in flight
        f32x16 s = f32x16{};
        row_product<T, D>(s, la, 0, qf);
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
        col_product<T, D>(o, la, C::TB, s);
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
    park<T, D>(fwd_smem, wave, o, lane);
    float* ml = reinterpret_cast<float*>(fwd_smem + C::NS * C::PB);  // [wave][m, l][32]
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
        T* orow = static_cast<T*>(a.o) + a.mo.head_base(b, h) + (int64_t)qi * a.mo.ss;
#pragma unroll
        for (int i = 0; i < C::QUADS / C::NS; ++i) {
            const int q = i * C::NS + st;
            f32x4 x = f32x4{};
#pragma unroll
            for (int w = 0; w < C::NS; ++w) x += f[w] * parked<T, D>(fwd_smem, w, q, lane);
            x *= inv;
            store4(orow + 32 * (q / 4) + 8 * (q % 4) + 4 * g, x[0], x[1], x[2], x[3]);
        }
        if (g == 0 && st == 0)
            a.lse[((int64_t)b * a.Hq + h) * S + qi] = (lsum > 0.f) ? (mm + __log2f(lsum)) * kLn2 : -INFINITY;
    }
}

// ------------------------------------------------------- backward: dK, dV
// Key/value-major pass of workgroup `id`.  INLINE: the row statistics are formed
// here from O, dO and the forward's LSE; else they are read from the workspace.
template <typename T, int D, bool INLINE>
FBL_DEV void kv_pass(const BwdArgs& a, int id, unsigned char* kv_smem) {
    using C = Streams<T, D>;
    const uint32_t lds = lds_addr(kv_smem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int st = wave;
    const int g = lane >> 5, c32 = lane & 31;
    const int S = a.S, Skv = a.Skv;
    const int nkb = (Skv + 31) / 32;
    // causal: the first key blocks see the most queries and start first
    int kblk, bh;
    if (!rank_major_item(id, nkb, a.Hkv * a.B, kblk, bh)) return;
    const int hk = bh % a.Hkv, b = bh / a.Hkv;
    const int G_ = a.Hq / a.Hkv;
    int kv_end = Skv;
    if (a.mask.kv_len) kv_end = min(max(a.mask.kv_len[b], 0), Skv);
    const int kw0 = kblk * 32;
    const int key = kw0 + c32;  // this lane's key (column of S)

    Frag<T> kreg[C::OWN_K ? 1 : C::NC], vreg[C::OWN_V ? 1 : C::NC];
    auto stage_own = [&](const void* base, const TokMap& m, uint32_t tile) {
        DmaPlan<T, D, 32, C::NS> p;
        p.init((uint32_t)(m.ss * C::ES), wave, lane);
        p.issue(tile, head_rsrc<T, D>(base, m, b, hk, Skv), (uint32_t)(kw0 * m.ss * C::ES), wave);
    };
    if constexpr (C::OWN_V) stage_own(a.v, a.mv, lds + C::OWN);
    else row_operands<T, D>(vreg, a.v, a.mv, b, hk, key, Skv, g, false);
    if constexpr (C::OWN_K) stage_own(a.k, a.mk, lds + C::OWN + C::TB);
    else row_operands<T, D>(kreg, a.k, a.mk, b, hk, key, Skv, g, false);

    // the blocks of 32 queries of every query head of the group, dealt to the streams
    const int qb0 = a.mask.causal ? kblk : 0;
    const int per_head = (S + 31) / 32 - qb0;
    const int n_blk = kw0 < kv_end ? G_ * per_head : 0;
    const uint32_t qbytes = (uint32_t)(a.mq.ss * C::ES), obytes = (uint32_t)(a.mdo.ss * C::ES);
    StreamDma<T, D> pq, po;
    pq.init(qbytes, lane);
    po.init(obytes, lane);
    const uint32_t tq = lds + st * C::SB, to = tq + C::TB, ts = lds + C::STATS + st * 512;
    // (the division runs on the vector ALUs; the loads need its result in scalar registers)
    auto head_of = [&](int i) { return hk * G_ + __builtin_amdgcn_readfirstlane(i / per_head); };
    auto query_of = [&](int i) { return __builtin_amdgcn_readfirstlane((qb0 + i % per_head) * 32); };
    auto issue_q = [&](int i) {
        if (i >= n_blk) return;
        const int h = head_of(i), q0 = query_of(i);
        pq.issue(tq, head_rsrc<T, D>(a.q, a.mq, b, h, S), (uint32_t)q0 * qbytes, qbytes);
    };
    // INLINE: the O row of query c32 of the next block (bf16; fp32 has no registers
    // for it and reads it chunk by chunk in the step) and its LSE
    constexpr bool kHoldO = INLINE && C::HOLD_O;
    Frag<T> orow[kHoldO ? C::NC : 1];
    float lse = 0.f;
    auto issue_do = [&](int i) {  // and the block's row statistics (lanes past the row read zeros) or what forms them
        if (i >= n_blk) return;
        const int h = head_of(i), q0 = query_of(i);
        if constexpr (INLINE) {
            if constexpr (kHoldO) row_operands<T, D>(orow, a.o, a.mo, b, h, q0 + c32, S, g, false);
            lse = q0 + c32 < S ? a.lse[((int64_t)b * a.Hq + h) * S + q0 + c32] : -INFINITY;
        }
        po.issue(to, head_rsrc<T, D>(a.dout, a.mdo, b, h, S), (uint32_t)q0 * obytes, obytes);
        if constexpr (!INLINE) {
            const float* row = a.stats + 2 * ((int64_t)b * a.Hq + h) * S;
            dma4(make_rsrc(row, (uint32_t)(S * 4)), ts, (uint32_t)lane * 4u, (uint32_t)q0 * 4u);
            dma4(make_rsrc(row + S, (uint32_t)(S * 4)), ts + 256, (uint32_t)lane * 4u, (uint32_t)q0 * 4u);
        }
    };

    // dK^T and dV^T: accumulator rows = d, columns = keys
    f32x16 dk[C::ND], dv[C::ND];
#pragma unroll
    for (int t = 0; t < C::ND; ++t) dk[t] = dv[t] = f32x16{};

    StreamLane<T, D> la;
    la.init(lds + st * C::SB, lane);
    float* stats = reinterpret_cast<float*>(kv_smem + C::STATS + st * 512);
    // One block of queries.  dO is done with after dV, Q after dK: each buffer is
    // refilled right then; the next block's dP comes first, so that each load
    // has at least one product to arrive under.
    const int q_min = key >= kv_end ? INT32_MAX : a.mask.causal ? key : 0;  // the first query that sees the key
    auto block = [&](int i, int q0) {
        const int row_min = q_min - q0;  // of the block's rows
        uint32_t own = C::OWN - st * C::SB;  // from the stream's tiles to the workgroup's rows
        asm volatile("" : "+s"(own));  // (added at each use: no second set of addresses in registers)
        // S = Q K_w^T and dP = dO V_w^T: lane <-> key, in-lane query acc_row
        f32x16 s = f32x16{}, dp = f32x16{};
        // dO and the statistics have landed; Q may be in flight.  (INLINE, bf16: until the second
        // dP product only.  The O rows and the LSE are plain loads, and the compiler, which does
        // not count the tiles' loads behind them, waits there for all.)
        wait_tile<C::LOADS>();
        float dsum = 0.f;
        const bool q_ok = q0 + c32 < S;
        const T* optr = static_cast<const T*>(a.o) + a.mo.head_base(b, head_of(i)) + (int64_t)min(q0 + c32, S - 1) * a.mo.ss + 8 * g;
#pragma unroll
        for (int c = 0; c < C::NC; ++c) {
            Frag<T> of, vf;
            la.row_frag(of, C::TB, c);
            if constexpr (C::OWN_V) la.row_frag_at(vf, own, 0, c);
            else vf = vreg[c];
            mma(dp, of, vf);
            if constexpr (INLINE) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if constexpr (kHoldO) dsum += (float)of.v[e] * (float)orow[c].v[e];
                    else dsum += (float)of.v[e] * (float)optr[16 * c + e];
                }
                if constexpr (kHoldO) __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (INLINE) {  // query c32: LSE in log2 units (+inf: empty row) from half 0, D from half 1
            dsum += other_half(dsum);
            if (!q_ok) dsum = 0.f;  // (fp32 read a neighbour's O there)
            const float lse2 = lse == -INFINITY ? INFINITY : lse * kLog2e;
            *(FBL_LDS float*)(stats + 64 * g + c32) = g ? dsum : lse2;
            wait_lds();
        }
        wait_tile<0>();
#pragma unroll
        for (int c = 0; c < C::NC; ++c) {
            Frag<T> qf, kf;
            la.row_frag(qf, 0, c);
            if constexpr (C::OWN_K) la.row_frag_at(kf, own, C::TB, c);
            else kf = kreg[c];
            mma(s, qf, kf);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const f32x4 l4 = *(const FBL_LDS f32x4*)(stats + 8 * rr + 4 * g);
            const f32x4 d4 = *(const FBL_LDS f32x4*)(stats + 64 + 8 * rr + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 4 * rr + e;
                float p = fast_exp2(__builtin_fmaf(s[r], a.scale_log2, -l4[e]));
                if (acc_row(r, g) < row_min) p = 0.f;
                s[r] = p;
                dp[r] = masked_ds(p, dp[r] - d4[e]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        col_product<T, D>(dv, la, C::TB, s);
        wait_lds();
        issue_do(i + C::NS);
        col_product<T, D>(dk, la, 0, dp);
        wait_lds();
        issue_q(i + C::NS);
    };

    issue_do(st);
    issue_q(st);
    if constexpr (C::OWN_V) {
        wait_tile<0>();
        __syncthreads();  // the workgroup's rows are in LDS
    }
    for (int i = st; i < n_blk; i += C::NS) block(i, query_of(i));

    // sum over the streams; every wavefront takes its share of the columns
    // (the lane's place is formed again: kept across the loop it costs two registers there is no room for)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int ln = tid & 63, own_key = kw0 + (ln & 31);
    auto store_share = [&](int slot, void* out, const TokMap& m, float f) {
        if (own_key >= Skv) return;
        T* row = static_cast<T*>(out) + m.head_base(b, hk) + (int64_t)own_key * m.ss;
#pragma unroll
        for (int i = 0; i < C::QUADS / C::NS; ++i) {
            const int q = i * C::NS + st;
            f32x4 x = f32x4{};
#pragma unroll
            for (int w = 0; w < C::NS; ++w) x += parked<T, D>(kv_smem, slot + w, q, ln);
            x *= f;
            if (own_key >= kv_end) x = f32x4{};  // no part in the sums, whatever dO and Q hold
            store4(row + 32 * (q / 4) + 8 * (q % 4) + 4 * (ln >> 5), x[0], x[1], x[2], x[3]);
        }
    };
    __syncthreads();
    park<T, D>(kv_smem, wave, dk, ln);
    if constexpr (C::PARK2) park<T, D>(kv_smem, 4 + wave, dv, ln);
    __syncthreads();
    store_share(0, a.dk, a.mdk, a.scale);
    if constexpr (!C::PARK2) {
        __syncthreads();
        park<T, D>(kv_smem, wave, dv, ln);
        __syncthreads();
    }
    store_share(C::PARK2 ? 4 : 0, a.dv, a.mdv, 1.f);
}

// ----------------------------------------------------------- backward: dQ
template <typename T, int D, bool INLINE>
FBL_DEV void q_pass(const BwdArgs& a, int id, unsigned char* q_smem) {
    using C = Streams<T, D>;
    const uint32_t lds = lds_addr(q_smem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int st = wave;
    const int g = lane >> 5, c32 = lane & 31;
    const int S = a.S, Skv = a.Skv;
    const int nqb = (S + 31) / 32;
    int rank, bh;
    if (!rank_major_item(id, nqb, a.Hq * a.B, rank, bh)) return;
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

    Frag<T> qf[C::NC], of[C::NC];
    row_operands<T, D>(qf, a.q, a.mq, b, h, qi, S, g, false);
    row_operands<T, D>(of, a.dout, a.mdo, b, h, qi, S, g, false);
    float lse2 = INFINITY, drow = 0.f;  // this lane's query row statistics
    if constexpr (INLINE) {
        Frag<T> orow[C::NC];
        row_operands<T, D>(orow, a.o, a.mo, b, h, qi, S, g, false);
        const float lse = qi < S ? a.lse[((int64_t)b * a.Hq + h) * S + qi] : -INFINITY;
#pragma unroll
        for (int c = 0; c < C::NC; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) drow += (float)of[c].v[e] * (float)orow[c].v[e];
        __builtin_amdgcn_sched_barrier(0);
        drow += other_half(drow);
        lse2 = lse == -INFINITY ? INFINITY : lse * kLog2e;
    } else if (qi < S) {
        const float* row = a.stats + 2 * ((int64_t)b * a.Hq + h) * S;
        lse2 = row[qi];
        drow = row[S + qi];
    }

    const Rsrc rk = head_rsrc<T, D>(a.k, a.mk, b, hk, Skv), rv = head_rsrc<T, D>(a.v, a.mv, b, hk, Skv);
    const uint32_t kbytes = (uint32_t)(a.mk.ss * C::ES), vbytes = (uint32_t)(a.mv.ss * C::ES);
    StreamDma<T, D> pk, pv;
    pk.init(kbytes, lane);
    pv.init(vbytes, lane);
    const uint32_t tk = lds + st * C::SB, tv = tk + C::TB;
    auto issue_k = [&](int j) { if (j < nkb) pk.issue(tk, rk, (uint32_t)(j * 32) * kbytes, kbytes); };
    auto issue_v = [&](int j) { if (j < nkb) pv.issue(tv, rv, (uint32_t)(j * 32) * vbytes, vbytes); };

    f32x16 dq[C::ND];  // dQ^T: rows = d, columns = queries
#pragma unroll
    for (int t = 0; t < C::ND; ++t) dq[t] = f32x16{};

    StreamLane<T, D> la;
    la.init(lds + st * C::SB, lane);
    // One key tile.  Its V rows are done with after dP, its K rows after dQ.
    const int q_end = a.mask.causal ? min(kv_end, qi + 1) : kv_end;  // the first key the query does not see
    auto block = [&](int j) {
        const int row_end = q_end - j * 32;  // of the tile's rows
        // S^T = K Q^T and dP^T = V dO^T: lane <-> query, in-lane key acc_row
        f32x16 s = f32x16{}, dp = f32x16{};
        wait_tile<C::LOADS>();  // V has landed; K may be in flight
        row_product<T, D>(dp, la, C::TB, of);
        wait_lds();
        issue_v(j + C::NS);
        if (j + C::NS < nkb) wait_tile<C::LOADS>();
        else wait_tile<0>();
        row_product<T, D>(s, la, 0, qf);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float p = fast_exp2(__builtin_fmaf(s[r], a.scale_log2, -lse2));
            if (acc_row(r, g) >= row_end) p = 0.f;
            dp[r] = masked_ds(p, dp[r] - drow);
        }
        col_product<T, D>(dq, la, 0, dp);
        wait_lds();
        issue_k(j + C::NS);
    };

    issue_v(st);
    issue_k(st);
    for (int j = st; j < nkb; j += C::NS) block(j);

    __syncthreads();
    park<T, D>(q_smem, wave, dq, lane);
    __syncthreads();
    if (qi < S) {
        T* dqrow = static_cast<T*>(a.dq) + a.mdq.head_base(b, h) + (int64_t)qi * a.mdq.ss;
#pragma unroll
        for (int i = 0; i < C::QUADS / C::NS; ++i) {
            const int q = i * C::NS + st;
            f32x4 x = f32x4{};
#pragma unroll
            for (int w = 0; w < C::NS; ++w) x += parked<T, D>(q_smem, w, q, lane);
            x *= a.scale;
            store4(dqrow + 32 * (q / 4) + 8 * (q % 4) + 4 * g, x[0], x[1], x[2], x[3]);
        }
    }
}

template <int D>
__global__ __launch_bounds__(256, (Streams<float, D>::OCC)) void attn_bwd_kv_f32(BwdArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char bwd_smem[];
    kv_pass<float, D, false>(a, workgroup_id(), bwd_smem);
}
template <int D>
__global__ __launch_bounds__(256, (Streams<float, D>::OCC)) void attn_bwd_q_f32(BwdArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char bwd_smem[];
    q_pass<float, D, false>(a, workgroup_id(), bwd_smem);
}

// ----------------------------------------------------- one-launch backward
template <typename T, int D>
__global__ __launch_bounds__(256, (Streams<T, D>::OCC)) void attn_bwd_streams(BwdArgs a, int n_kv) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char bwd_smem[];
    const int id = workgroup_id();
    if (id < n_kv) kv_pass<T, D, true>(a, id, bwd_smem);
    else q_pass<T, D, true>(a, id - n_kv, bwd_smem);
}

}  // namespace

template <typename T, int D>
hipError_t launch_attn_fwd_streams(const FwdArgs& a, hipStream_t stream) {
    using C = Streams<T, D>;
    const hipError_t e = ensure_dynamic_lds<&attn_fwd_streams<T, D>>(C::FWD_BYTES);
    if (e != hipSuccess) return e;
    const int n = rank_major_grid((a.S + 32 - 1) / 32, a.Hq * a.B);
    hipLaunchKernelGGL((attn_fwd_streams<T, D>), grid_of(n), dim3(256), C::FWD_BYTES, stream, a);
    return hipGetLastError();
}

template <int D>
hipError_t launch_attn_bwd_kv_f32(const BwdArgs& a, hipStream_t stream) {
    using C = Streams<float, D>;
    const hipError_t e = ensure_dynamic_lds<&attn_bwd_kv_f32<D>>(C::KV_BYTES);
    if (e != hipSuccess) return e;
    const int n = rank_major_grid((a.Skv + 32 - 1) / 32, a.Hkv * a.B);
    hipLaunchKernelGGL((attn_bwd_kv_f32<D>), grid_of(n), dim3(256), C::KV_BYTES, stream, a);
    return hipGetLastError();
}

template <int D>
hipError_t launch_attn_bwd_q_f32(const BwdArgs& a, hipStream_t stream) {
    using C = Streams<float, D>;
    const hipError_t e = ensure_dynamic_lds<&attn_bwd_q_f32<D>>(C::BYTES);
    if (e != hipSuccess) return e;
    const int n = rank_major_grid((a.S + 32 - 1) / 32, a.Hq * a.B);
    hipLaunchKernelGGL((attn_bwd_q_f32<D>), grid_of(n), dim3(256), C::BYTES, stream, a);
    return hipGetLastError();
}

template <typename T, int D>
hipError_t launch_attn_bwd_streams(const BwdArgs& a, hipStream_t stream) {
    using C = Streams<T, D>;
    constexpr int lds = C::KV_BYTES > C::BYTES ? C::KV_BYTES : C::BYTES;
    const hipError_t e = ensure_dynamic_lds<&attn_bwd_streams<T, D>>(lds);
    if (e != hipSuccess) return e;
    const int n_kv = rank_major_grid((a.Skv + 32 - 1) / 32, a.Hkv * a.B);
    const int n = n_kv + rank_major_grid((a.S + 32 - 1) / 32, a.Hq * a.B);
    hipLaunchKernelGGL((attn_bwd_streams<T, D>), grid_of(n), dim3(256), lds, stream, a, n_kv);
    return hipGetLastError();
}

#define FBL_ATTN_STREAMS(T, D)                                                      \
    template hipError_t launch_attn_fwd_streams<T, D>(const FwdArgs&, hipStream_t); \
    template hipError_t launch_attn_bwd_streams<T, D>(const BwdArgs&, hipStream_t);
#define FBL_ATTN_F32(D)                                                             \
    FBL_ATTN_STREAMS(float, D)                                                      \
    template hipError_t launch_attn_bwd_kv_f32<D>(const BwdArgs&, hipStream_t);     \
    template hipError_t launch_attn_bwd_q_f32<D>(const BwdArgs&, hipStream_t);
FBL_ATTN_F32(32)
FBL_ATTN_F32(64)
FBL_ATTN_F32(128)
FBL_ATTN_STREAMS(bf16, 32)
FBL_ATTN_STREAMS(bf16, 64)
FBL_ATTN_STREAMS(bf16, 128)
#undef FBL_ATTN_F32
#undef FBL_ATTN_STREAMS

}  // namespace fbl
