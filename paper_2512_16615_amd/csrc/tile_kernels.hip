// Attention forward, dQ and dK/dV in fp32 arithmetic on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32): any block
// size, d = 16 .. 128, both I/O types.  The fp32 path, and the path of the bf16 shapes the bf16 MFMA kernels do not take.
//
// Same tile algebra as the bf16 kernels, one 16 x 16 score tile at a time.  Of v_mfma_f32_16x16x4_f32 (lane = 16 g + i) an A
// operand is row i, contraction slot g; a B operand column i, slot g; the result column i, rows 4g .. 4g+3.
//   First product (scores): both operands are rows of a tensor and contract over channels, whose order is free as long as
//     both sides agree: step 4m + e takes channel 16m + 4g + e, so a lane reads 16-byte pieces of its row.
//   Second product (values, gradients): it contracts over the 16 rows of the tile.  Step r takes row 4g + r in slot g, and
//     the probability of that row is register r of the lane's own score tile, so nothing moves between lanes.  The other
//     operand is E consecutive channels of row 4g + r per lane, 16 lanes covering 16 E channels of a row.
// No LDS tile is needed: the second read of a row comes from L1.  What bounds these kernels is the matrix pipe (32 cycles an
// instruction: 512 per product of a 16 x 16 x 64 tile, against about 100 cycles of L1 for its rows); the one-row-per-wave
// kernels they replaced spent their time in shuffles and dependent row loads.  16 heads x 4096 tokens, d = 64, fp32, M = 272.
#include "mfma_common.h"

namespace llsa {

// ---- I/O types: 4 (or E) consecutive channels as fp32
template <int E> struct FVec { float v[E]; };
template <int E> __device__ __forceinline__ FVec<E> ld_e(const float *p) {
    FVec<E> r;
    if constexpr (E == 4) { const f32x4 x = *reinterpret_cast<const f32x4 *>(p); for (int i = 0; i < 4; ++i) r.v[i] = x[i]; }
    else if constexpr (E == 2) { const float2 x = *reinterpret_cast<const float2 *>(p); r.v[0] = x.x; r.v[1] = x.y; }
    else r.v[0] = p[0];
    return r;
}
template <int E> __device__ __forceinline__ FVec<E> ld_e(const uint16_t *p) {
    FVec<E> r;
    if constexpr (E == 4) {
        const u32x2 x = *reinterpret_cast<const u32x2 *>(p);
        for (int i = 0; i < 2; ++i) { r.v[2 * i] = __uint_as_float(x[i] << 16); r.v[2 * i + 1] = __uint_as_float(x[i] & 0xffff0000u); }
    } else if constexpr (E == 2) {
        const uint32_t x = *reinterpret_cast<const uint32_t *>(p);
        r.v[0] = __uint_as_float(x << 16); r.v[1] = __uint_as_float(x & 0xffff0000u);
    } else r.v[0] = __uint_as_float((uint32_t)p[0] << 16);
    return r;
}
template <int E> __device__ __forceinline__ void st_e(float *p, const FVec<E> &x) {
    if constexpr (E == 4) *reinterpret_cast<f32x4 *>(p) = f32x4{x.v[0], x.v[1], x.v[2], x.v[3]};
    else for (int i = 0; i < E; ++i) p[i] = x.v[i];
}
template <int E> __device__ __forceinline__ void st_e(uint16_t *p, const FVec<E> &x) {
    if constexpr (E == 4) *reinterpret_cast<u32x2 *>(p) = u32x2{pack_bf16(x.v[0], x.v[1]), pack_bf16(x.v[2], x.v[3])};
    else for (int i = 0; i < E; ++i) p[i] = (uint16_t)pack_bf16(x.v[i], 0.f);
}

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <int D> struct TShape {
    static constexpr int KS = D / 4;                    // matrix instructions over the channels
    static constexpr int E = D >= 64 ? 4 : D / 16;      // channels per lane and row piece of the second product
    static constexpr int H = D / (16 * E);              // row pieces
    static constexpr int NT = D / 16;                   // 16-channel accumulator tiles: tile E h + e, row i = channel 16 E h + E i + e
};

// a row as an operand of the first product
template <int D> struct RowOp { float x[D / 4]; };
template <class T, int D> __device__ __forceinline__ RowOp<D> row_op(const T *row, int g) {
    RowOp<D> r;
#pragma unroll
    for (int m = 0; m < D / 16; ++m) {
        const FVec<4> v = ld_e<4>(row + 16 * m + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) r.x[4 * m + e] = v.v[e];
    }
    return r;
}
template <int D> __device__ __forceinline__ f32x4 row_product(const RowOp<D> &a, const RowOp<D> &b) {
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D / 4; ++s) c = mfma4(a.x[s], b.x[s], c);
    return c;
}
// the lane's pieces of tile rows 4g + r (r = 0 .. 3) as an operand of the second product
template <int D> struct ColOp { FVec<TShape<D>::E> x[4][TShape<D>::H]; };
template <class T, int D> __device__ __forceinline__ void col_op(ColOp<D> &c, int r, const T *row, int i16) {
    using S = TShape<D>;
#pragma unroll
    for (int h = 0; h < S::H; ++h) c.x[r][h] = ld_e<S::E>(row + 16 * S::E * h + S::E * i16);
}
template <int D> __device__ __forceinline__ void col_product(f32x4 (&acc)[D / 16], const ColOp<D> &c, const f32x4 &p) {
    using S = TShape<D>;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int h = 0; h < S::H; ++h)
#pragma unroll
            for (int e = 0; e < S::E; ++e) acc[S::E * h + e] = mfma4(c.x[r][h].v[e], p[r], acc[S::E * h + e]);
}
// the lane's results of a second product: channels 16 E h + E (4g + r) .. + E - 1 of column i16, handed out as vectors
template <int D, class Emit> __device__ __forceinline__ void col_emit(const f32x4 (&acc)[D / 16], int g, Emit emit) {
    using S = TShape<D>;
#pragma unroll
    for (int h = 0; h < S::H; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            FVec<S::E> v;
#pragma unroll
            for (int e = 0; e < S::E; ++e) v.v[e] = acc[S::E * h + e][r];
            emit(16 * S::E * h + S::E * (4 * g + r), v);
        }
}

// Logits, maxima and logsumexps are in natural units: scale and weight folded into base-2 units for the bare hardware
// exponential (each factor rounded on its own, at the size of the whole exponent) put dQ 1.05 to 1.35 times and the logsumexp
// 1.05 to 1.4 times as far from a 64-bit computation.

// exp(x) to about a unit: x log2(e) in two parts, the hardware's 2^t of the rounded one, the rest to first order.  (Below -104
// the result is 0; a NaN stays one.)  Forward with it and with expf: one head of 256 tokens 8.8 : 9.2 us, 16 x 4096 62.9 : 65.5.
__device__ __forceinline__ float exp_nat(float x) {
    constexpr float kHi = 1.44269504f, kLo = (float)(1.4426950408889634 - (double)kHi);
    x = x < -104.f ? -104.f : x;
    const float t = x * kHi, rest = fmaf(x, kLo, fmaf(x, kHi, -t)), p = __builtin_amdgcn_exp2f(t);
    return fmaf(p, rest * kLn2, p);
}

// 64 positions of a query block's gathered list (Alg. 1, enrichment loop): addresses of the tokens' key and value rows, log of
// the weight (-inf past the end of the list, whose rows repeat the last one).
struct ListTable {
    uint64_t k[64], v[64];
    float bias[64];
};
template <class T>
__device__ __forceinline__ void list_fill(ListTable &tab, const LevelTable &t, int64_t bh, unsigned blk, int pos0, int len, int lane, int d) {
    const int pos = min(pos0 + lane, len - 1);
    uint64_t kp = 0, vp = 0;
    float b = 0.f;
    unsigned row = blk;                                     // row of I^(l): blk / B^l
    for (int l = 0; l < t.nlev; ++l) {                      // wave-uniform loop over the levels in the list
        const int s0 = pick(t.seg, l), s1 = pick(t.seg, l + 1);
        if (pos >= s0 && pos < s1) {
            const unsigned off = (unsigned)(pos - s0);
            int64_t tok = off;
            if (l < t.L) {
                const unsigned k = off / (unsigned)t.B;
                tok = (int64_t)pick(t.I, l)[(bh * pick(t.rows, l) + row) * pick(t.Kl, l) + k] * t.B + (off - k * t.B);
            }
            const int64_t o = (bh * pick(t.n, l) + tok) * d * (int)sizeof(T);
            kp = reinterpret_cast<uint64_t>(pick(t.K, l)) + o;
            vp = reinterpret_cast<uint64_t>(pick(t.V, l)) + o;
            b = pick(t.bias, l);
        }
        row /= (unsigned)t.B;
    }
    tab.k[lane] = kp;
    tab.v[lane] = vp;
    tab.bias[lane] = pos0 + lane < len ? b : -INFINITY;
}

// The query tile of a wave: up to 16 consecutive queries of one block of B (a block is `tpb` tiles).
struct QTile {
    int64_t bh, row;             // head; first query row of the tile, over all heads
    unsigned blk;                // query block inside the head
    int nq;                      // queries in the tile
};
__device__ __forceinline__ QTile query_tile(int64_t tile, int64_t per_head, int tpb, int B, int64_t N) {
    QTile q;
    q.bh = tile / per_head;
    const unsigned in = (unsigned)(tile - q.bh * per_head);
    q.blk = in / (unsigned)tpb;
    const int first = 16 * (int)(in - q.blk * tpb);
    q.nq = min(16, B - first);
    q.row = q.bh * N + (int64_t)q.blk * B + first;
    return q;
}

// ------------------------------------------------------------------------------------------------ forward
template <class T, int D>
__global__ void __launch_bounds__(256) tile_fwd_kernel(LevelTable t, const T *__restrict__ Q, T *__restrict__ O,
                                                        float *__restrict__ LSE, int64_t N, int tpb, int64_t per_head, int64_t total) {
    using S = TShape<D>;
    __shared__ __attribute__((aligned(16))) ListTable tabs[4];
    const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tile = xcd_contiguous(blockIdx.x, gridDim.x) * 4 + wave;
    if (tile >= total) return;                              // the waves of a workgroup never wait for each other
    const QTile qt = query_tile(tile, per_head, tpb, t.B, N);
    const int64_t row = qt.row + min(i16, qt.nq - 1);
    ListTable &tab = tabs[wave];
    const RowOp<D> q = row_op<T, D>(Q + row * D, g);
    const int len = t.seg[t.nlev];
    f32x4 acc[S::NT];
#pragma unroll
    for (int n = 0; n < S::NT; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, lsum = 0.f;                        // running maximum; this lane's share of the row sum
    for (int c0 = 0; c0 < len; c0 += 64) {
        __builtin_amdgcn_wave_barrier();                    // one wave's LDS operations stay in order
        list_fill<T>(tab, t, qt.bh, qt.blk, c0, len, lane, D);
        __builtin_amdgcn_wave_barrier();
        const int c1 = min(64, len - c0);
        for (int c = 0; c < c1; c += 16) {
            const RowOp<D> k = row_op<T, D>(reinterpret_cast<const T *>(tab.k[c + i16]), g);
            ColOp<D> v;
#pragma unroll
            for (int r = 0; r < 4; ++r) col_op<T, D>(v, r, reinterpret_cast<const T *>(tab.v[c + 4 * g + r]), i16);
            f32x4 s = row_product<D>(k, q);
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[r] = fmaf(s[r], t.scale, tab.bias[c + 4 * g + r]);
                mx = fmaxf(mx, s[r]);
            }
            mx = rows_max(mx);
            if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {
                const float m_new = fmaxf(m, mx), alpha = exp_nat(m - m_new);
                lsum *= alpha;
#pragma unroll
                for (int n = 0; n < S::NT; ++n)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[n][r] *= alpha;
                m = m_new;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) s[r] = exp_nat(s[r] - m);
            lsum += (s[0] + s[1]) + (s[2] + s[3]);
            col_product<D>(acc, v, s);
        }
    }
    lsum = rows_sum(lsum);
    if (i16 >= qt.nq) return;
    const float inv = 1.f / lsum;
    col_emit<D>(acc, g, [&](int ch, FVec<S::E> x) {
#pragma unroll
        for (int e = 0; e < S::E; ++e) {                    // x / lsum: the product and one correction (not of an infinity)
            const float q = x.v[e] * inv, c = fmaf(fmaf(-q, lsum, x.v[e]), inv, q);
            x.v[e] = c == c ? c : q;
        }
        st_e<S::E>(O + row * D + ch, x);
    });
    if (g == 0) LSE[row] = fmaf(__builtin_amdgcn_logf(lsum), kLn2, m);
}

// ----------------------------------------------------------------------------------------------------- dQ
// Same walk; P from the saved logsumexp.  Also produces D = rowsum(dO o O) of its queries for the key-major kernel.  (expf at
// d = 128: as exact, and around exp_nat the compiler schedules that loop worse, 2 heads x 4096 tokens 104 against 137 us.)
template <class T, int D>
__global__ void __launch_bounds__(256) tile_dq_kernel(LevelTable t, const T *__restrict__ Q, const T *__restrict__ O,
                                                       const T *__restrict__ dO, const float *__restrict__ LSE, float *__restrict__ Dsum,
                                                       T *__restrict__ dQ, int64_t N, int tpb, int64_t per_head, int64_t total) {
    using S = TShape<D>;
    __shared__ __attribute__((aligned(16))) ListTable tabs[4];
    const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tile = xcd_contiguous(blockIdx.x, gridDim.x) * 4 + wave;
    if (tile >= total) return;
    const QTile qt = query_tile(tile, per_head, tpb, t.B, N);
    const int64_t row = qt.row + min(i16, qt.nq - 1);
    ListTable &tab = tabs[wave];
    const RowOp<D> q = row_op<T, D>(Q + row * D, g), go = row_op<T, D>(dO + row * D, g);
    float delta = 0.f;
    {
        const RowOp<D> o = row_op<T, D>(O + row * D, g);
#pragma unroll
        for (int s = 0; s < S::KS; ++s) delta = fmaf(go.x[s], o.x[s], delta);
        delta = rows_sum(delta);
        if (g == 0 && i16 < qt.nq) Dsum[row] = delta;
    }
    const float lse = LSE[row];
    const int len = t.seg[t.nlev];
    f32x4 acc[S::NT];
#pragma unroll
    for (int n = 0; n < S::NT; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < len; c0 += 64) {
        __builtin_amdgcn_wave_barrier();
        list_fill<T>(tab, t, qt.bh, qt.blk, c0, len, lane, D);
        __builtin_amdgcn_wave_barrier();
        const int c1 = min(64, len - c0);
        for (int c = 0; c < c1; c += 16) {
            const RowOp<D> k = row_op<T, D>(reinterpret_cast<const T *>(tab.k[c + i16]), g);
            const RowOp<D> v = row_op<T, D>(reinterpret_cast<const T *>(tab.v[c + i16]), g);
            ColOp<D> kc;
#pragma unroll
            for (int r = 0; r < 4; ++r) col_op<T, D>(kc, r, reinterpret_cast<const T *>(tab.k[c + 4 * g + r]), i16);
            f32x4 s = row_product<D>(k, q);
            const f32x4 dp = row_product<D>(v, go);
#pragma unroll
            for (int r = 0; r < 4; ++r) {                   // past the end of the list: weight -inf, P = 0
                const float x = fmaf(s[r], t.scale, tab.bias[c + 4 * g + r]) - lse;
                s[r] = (D == 128 ? expf(x) : exp_nat(x)) * (dp[r] - delta);
            }
            col_product<D>(acc, kc, s);
        }
    }
    if (i16 >= qt.nq) return;
    col_emit<D>(acc, g, [&](int ch, FVec<S::E> x) {
#pragma unroll
        for (int e = 0; e < S::E; ++e) x.v[e] *= t.scale;
        st_e<S::E>(dQ + row * D + ch, x);
    });
}

// ------------------------------------------------------------------------------------------------- dK, dV
// Key-major (Sec. 4.3), every level in one launch: a workgroup of four waves takes one tile of up to 16 keys of a level and a
// share of the queries that attend to it (the fine queries under the query blocks of Alg. 2's list; every query at a dense
// level), dealt to the waves 16 at a time; the waves' sums are added through LDS in wave order.  Shares (`splits`) exist so
// that a level of few keys, whose lists are long, still fills the chip.
struct DkvTileLevel {
    const void *K, *V;
    const int32_t *C, *Iq;       // null when dense
    float *partK, *partV;        // [splits][bh * n][D] fp32
    int64_t n, slab;             // tokens per head; floats of one slab
    unsigned wg0;                // first workgroup of the level
    unsigned tiles, span;        // key tiles per head; fine queries under one listed query block
    int rows, Kl, tpb, splits;
    float bias;
};
struct DkvTileArgs {
    DkvTileLevel lv[kMaxL + 1];
    int nlev, B;
    int64_t N;
    float scale;
};

template <class T, int D>
__global__ void __launch_bounds__(256) tile_dkv_kernel(DkvTileArgs a, const T *__restrict__ Q, const T *__restrict__ dO,
                                                        const float *__restrict__ LSE, const float *__restrict__ Dsum) {
    using S = TShape<D>;
    constexpr int SLOTS = 2 * S::NT;
    __shared__ __attribute__((aligned(16))) float red[4 * SLOTS * 64 * 4 > 4 * 48 ? 4 * SLOTS * 64 * 4 : 4 * 48];
    const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int l = 0;                                              // levels are laid out from the coarsest (longest lists) down
    for (int x = 1; x < a.nlev; ++x) l = blockIdx.x < a.lv[x - 1].wg0 ? x : l;
    const DkvTileLevel &L = a.lv[l];
    const unsigned id = blockIdx.x - L.wg0;
    const unsigned kt = id / (unsigned)L.splits;
    const int split = (int)(id - kt * L.splits);
    const int64_t bh = kt / L.tiles;
    const unsigned in = kt - (unsigned)bh * L.tiles, blk = in / (unsigned)L.tpb;
    const bool dense = L.C == nullptr;
    // a tile of a listed block of B keys, or 16 tokens of a dense level (tpb = 1)
    const int first = 16 * (int)(in - blk * L.tpb);
    const int64_t key0 = dense ? (int64_t)in * 16 : (int64_t)blk * a.B + first;
    const int nk = dense ? (int)min((int64_t)16, L.n - key0) : min(16, a.B - first);
    const int64_t krow = bh * L.n + key0 + min(i16, nk - 1);

    const int32_t *lst = nullptr;
    unsigned qcount = (unsigned)a.N;
    if (!dense) {
        const int32_t *Crow = L.C + bh * (L.rows + 1) + blk;
        lst = L.Iq + bh * L.rows * L.Kl + Crow[0];
        qcount = (unsigned)(Crow[1] - Crow[0]) * L.span;    // a query lists a key at most once: no more than N
    }
    const unsigned chunks = (qcount + 15) >> 4;
    const unsigned c_beg = (unsigned)((uint64_t)chunks * split / L.splits), c_end = (unsigned)((uint64_t)chunks * (split + 1) / L.splits);

    f32x4 accK[S::NT], accV[S::NT];
#pragma unroll
    for (int n = 0; n < S::NT; ++n) { accK[n] = f32x4{0.f, 0.f, 0.f, 0.f}; accV[n] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    if (c_beg + wave < c_end) {
        const RowOp<D> k = row_op<T, D>(static_cast<const T *>(L.K) + krow * D, g);
        const RowOp<D> v = row_op<T, D>(static_cast<const T *>(L.V) + krow * D, g);
        float *st = red + wave * 48;                        // the tile's 16 query rows | LSE | D
        for (unsigned c = c_beg + wave; c < c_end; c += 4) {
            const unsigned p = 16 * c + i16, pc = min(p, qcount - 1);
            unsigned qi = pc;
            if (!dense) {
                const unsigned e = pc / L.span;
                qi = (unsigned)lst[e] * L.span + (pc - e * L.span);
            }
            const int64_t qrow = bh * a.N + qi;
            const RowOp<D> qo = row_op<T, D>(Q + qrow * D, g), go = row_op<T, D>(dO + qrow * D, g);
            __builtin_amdgcn_wave_barrier();
            if (g == 0) {                                   // past the end of the list: LSE inf, P = 0
                st[i16] = __uint_as_float(qi);
                st[16 + i16] = p < qcount ? LSE[qrow] : INFINITY;
                st[32 + i16] = Dsum[qrow];
            }
            __builtin_amdgcn_wave_barrier();
            const f32x4 qx = *reinterpret_cast<const f32x4 *>(st + 4 * g), lse = *reinterpret_cast<const f32x4 *>(st + 16 + 4 * g),
                        dl = *reinterpret_cast<const f32x4 *>(st + 32 + 4 * g);
            ColOp<D> qc, gc;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t o = (bh * a.N + __float_as_uint(qx[r])) * D;
                col_op<T, D>(qc, r, Q + o, i16);
                col_op<T, D>(gc, r, dO + o, i16);
            }
            f32x4 s = row_product<D>(qo, k), dp = row_product<D>(go, v);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[r] = exp_nat(fmaf(s[r], a.scale, L.bias) - lse[r]);
                dp[r] = s[r] * (dp[r] - dl[r]);
            }
            col_product<D>(accV, gc, s);
            col_product<D>(accK, qc, dp);
        }
    }
    __syncthreads();                                        // everyone is done with the tables
#pragma unroll
    for (int n = 0; n < S::NT; ++n) {
        *reinterpret_cast<f32x4 *>(red + ((wave * SLOTS + n) * 64 + lane) * 4) = accK[n];
        *reinterpret_cast<f32x4 *>(red + ((wave * SLOTS + S::NT + n) * 64 + lane) * 4) = accV[n];
    }
    __syncthreads();
    // wave 0 and 1 write dK, wave 2 and 3 dV; half of the row pieces' rows each
    auto slot = [&](int s) {
        f32x4 sum = *reinterpret_cast<const f32x4 *>(red + (s * 64 + lane) * 4);
#pragma unroll
        for (int w = 1; w < 4; ++w) sum += *reinterpret_cast<const f32x4 *>(red + ((w * SLOTS + s) * 64 + lane) * 4);
        return sum;
    };
    const bool isV = wave >= 2;
    float *dst = (isV ? L.partV : L.partK) + split * L.slab + krow * D;
    const float w = isV ? 1.f : a.scale;
    for (int h = 0; h < S::H; ++h) {
        if (S::H > 1 ? (h & 1) != (wave & 1) : (wave & 1) != 0) continue;
        f32x4 t4[S::E];
#pragma unroll
        for (int e = 0; e < S::E; ++e) t4[e] = slot((isV ? S::NT : 0) + S::E * h + e);
        if (i16 >= nk) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            FVec<S::E> x;
#pragma unroll
            for (int e = 0; e < S::E; ++e) x.v[e] = t4[e][r] * w;
            st_e<S::E>(dst + 16 * S::E * h + S::E * (4 * g + r), x);
        }
    }
}

// The levels' partials folded down (adjoint of mean pooling): a level-0 token's gradient is its own sum plus 1/B of its
// level-1 ancestor's total, which holds 1/B of the level-2 ancestor's, and so on.  One workgroup per level-1 token: its total
// (every share of every ancestor, added in a fixed order by 256 / (D / 2) groups of threads), then the token's B children.
struct DkvFoldArgs {
    const float *partK[kMaxL + 1], *partV[kMaxL + 1];
    int64_t n[kMaxL + 1], slab[kMaxL + 1];
    int splits[kMaxL + 1];
    int nlev, B;                 // levels 0 .. nlev - 1
};
template <class T, int D>
__global__ void __launch_bounds__(256) tile_dkv_fold_kernel(DkvFoldArgs a, T *dK, T *dV) {
    constexpr int SL = 2 * D / 4, GR = 256 / SL;
    __shared__ __attribute__((aligned(16))) f32x4 sum[GR][SL];
    const int tid = threadIdx.x, slot = tid % SL, grp = tid / SL;
    const unsigned n1 = (unsigned)(a.n[0] / a.B);
    const int64_t bh = blockIdx.x / n1;
    unsigned tok = blockIdx.x - (unsigned)bh * n1;
    const bool isV = slot >= SL / 2;
    const int c = (slot % (SL / 2)) * 4;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const float inv = 1.f / (float)a.B;
    float w = inv;
    int turn = 0;
    for (int l = 1; l < a.nlev; ++l) {
        const float *src = (isV ? a.partV[l] : a.partK[l]) + (bh * a.n[l] + tok) * D + c;
        for (int s = 0; s < a.splits[l]; ++s, ++turn)
            if (turn % GR == grp) acc += *reinterpret_cast<const f32x4 *>(src + s * a.slab[l]) * w;
        tok /= (unsigned)a.B;
        w *= inv;
    }
    sum[grp][slot] = acc;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * a.B;        // the token's first child, over all heads
    f32x4 par = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < GR; ++x) par += sum[x][slot];
    for (int r = grp; r < a.B; r += GR) {
        const int64_t o = (first + r) * D + c;
        const f32x4 x = *reinterpret_cast<const f32x4 *>((isV ? a.partV[0] : a.partK[0]) + o) + par;
        st_e<4>((isV ? dV : dK) + o, FVec<4>{{x[0], x[1], x[2], x[3]}});
    }
}

// ------------------------------------------------------------------------------------------------- launches
template <class F> static hipError_t by_shape(const Plan &p, F f) {
#define LLSA_BY_D(T)                                                          \
    switch (p.d) {                                                            \
        case 16: f(T{}, std::integral_constant<int, 16>{}); break;            \
        case 32: f(T{}, std::integral_constant<int, 32>{}); break;            \
        case 64: f(T{}, std::integral_constant<int, 64>{}); break;            \
        default: f(T{}, std::integral_constant<int, 128>{}); break;           \
    }
    if (p.elt == 4) { LLSA_BY_D(float) } else { LLSA_BY_D(uint16_t) }
#undef LLSA_BY_D
    return hipGetLastError();
}

hipError_t launch_attn_fwd_tile(const Plan &p, const LevelTable &t, const void *Q, void *O, float *LSE, hipStream_t s) {
    const int tpb = (p.B + 15) / 16;
    const int64_t per_head = p.n[1] * tpb, total = p.bh * per_head;
    return by_shape(p, [&](auto ty, auto d) {
        using T = decltype(ty);
        tile_fwd_kernel<T, d.value><<<(unsigned)((total + 3) / 4), 256, 0, s>>>(t, (const T *)Q, (T *)O, LSE, p.N, tpb, per_head, total);
    });
}

hipError_t launch_dq_tile(const Plan &p, const LevelTable &t, const void *Q, const void *O, const void *dO, const float *LSE,
                          float *D, void *dQ, hipStream_t s) {
    const int tpb = (p.B + 15) / 16;
    const int64_t per_head = p.n[1] * tpb, total = p.bh * per_head;
    return by_shape(p, [&](auto ty, auto d) {
        using T = decltype(ty);
        tile_dq_kernel<T, d.value><<<(unsigned)((total + 3) / 4), 256, 0, s>>>(t, (const T *)Q, (const T *)O, (const T *)dO, LSE, D,
                                                                              (T *)dQ, p.N, tpb, per_head, total);
    });
}

// shares of level l's query lists, key tiles per head, tiles per listed block
static void dkv_tile_shape(const Plan &p, int l, int *splits, int64_t *tiles, int *tpb) {
    const bool dense = l == p.L;
    *tpb = dense ? 1 : (p.B + 15) / 16;
    *tiles = dense ? (p.n[l] + 15) / 16 : p.n[l + 1] * *tpb;
    // level 0's lists are short (K blocks of queries on average) and its result is not summed again.  Above it: enough
    // workgroups for eight on every CU, each with at least two chunks of 16 queries a wave.
    const int64_t chunks = (dense ? p.N : (int64_t)p.Kl[l] * (p.N / p.n[l + 1])) / 16;
    int64_t s = (2048 + p.bh * *tiles - 1) / (p.bh * *tiles);
    if (s > chunks / 8) s = chunks / 8;
    if (s < 1 || l == 0) s = 1;
    if (s > 64) s = 64;
    *splits = (int)s;
}

// bytes of the partial sums of levels 1 .. Le (and of level 0 where the I/O type cannot hold them)
size_t dkv_tile_bytes(const Plan &p) {
    size_t b = 0;
    for (int l = p.elt == 4 ? 1 : 0; l <= p.Le; ++l) {
        int splits, tpb;
        int64_t tiles;
        dkv_tile_shape(p, l, &splits, &tiles, &tpb);
        b += 2 * (size_t)p.bh * p.n[l] * p.d * sizeof(float) * splits;
    }
    return b;
}

// the arguments of both launches; returns the workgroups of the first
static int64_t dkv_tile_args(const Plan &p, const LevelTable &t, void *ws, void *dK, void *dV, DkvTileArgs &a, DkvFoldArgs &f) {
    char *w = static_cast<char *>(ws);
    float *part = reinterpret_cast<float *>(w + p.part_off);
    a.B = f.B = p.B;
    a.N = p.N;
    a.scale = p.scale;
    a.nlev = f.nlev = p.Le + 1;
    int64_t wg = 0;
    for (int l = p.Le; l >= 0; --l) {
        DkvTileLevel &L = a.lv[l];
        const bool dense = l == p.L;
        int64_t tiles;
        dkv_tile_shape(p, l, &L.splits, &tiles, &L.tpb);
        L.tiles = (unsigned)tiles;
        L.K = t.K[l]; L.V = t.V[l];
        L.C = dense ? nullptr : reinterpret_cast<const int32_t *>(w + p.C_off[l]);
        L.Iq = dense ? nullptr : reinterpret_cast<const int32_t *>(w + p.Iq_off[l]);
        L.n = p.n[l];
        L.slab = (int64_t)p.bh * p.n[l] * p.d;
        L.rows = dense ? 0 : (int)p.n[l + 1];
        L.Kl = dense ? 0 : p.Kl[l];
        L.span = dense ? 1 : (unsigned)(p.N / p.n[l + 1]);
        L.bias = t.bias[l];
        if (l == 0 && p.elt == 4) { L.partK = static_cast<float *>(dK); L.partV = static_cast<float *>(dV); }
        else {
            L.partK = part;
            L.partV = part + L.slab * L.splits;
            part += 2 * L.slab * L.splits;
        }
        L.wg0 = (unsigned)wg;
        wg += p.bh * tiles * L.splits;
        f.partK[l] = L.partK; f.partV[l] = L.partV;
        f.n[l] = L.n; f.slab[l] = L.slab; f.splits[l] = L.splits;
    }
    return wg;
}

hipError_t launch_dkv_tile(const Plan &p, const LevelTable &t, const void *Q, const void *dO, const float *LSE, const float *D,
                           void *ws, void *dK, void *dV, hipStream_t s) {
    DkvTileArgs a;
    DkvFoldArgs f;
    const int64_t wg = dkv_tile_args(p, t, ws, dK, dV, a, f);
    if (wg >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    return by_shape(p, [&](auto ty, auto d) {
        using T = decltype(ty);
        tile_dkv_kernel<T, d.value><<<(unsigned)wg, 256, 0, s>>>(a, (const T *)Q, (const T *)dO, LSE, D);
    });
}

bool dkv_tile_folds(const Plan &p) { return p.Le >= 1 || p.elt != 4; }   // fp32 without coarse levels: the sums are the result

hipError_t launch_dkv_tile_fold(const Plan &p, const LevelTable &t, void *ws, void *dK, void *dV, hipStream_t s) {
    DkvTileArgs a;
    DkvFoldArgs f;
    dkv_tile_args(p, t, ws, dK, dV, a, f);
    return by_shape(p, [&](auto ty, auto d) {
        using T = decltype(ty);
        tile_dkv_fold_kernel<T, d.value><<<(unsigned)(p.bh * p.n[1]), 256, 0, s>>>(f, (T *)dK, (T *)dV);
    });
}

}  // namespace llsa
