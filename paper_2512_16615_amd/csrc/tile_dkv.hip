// dK, dV in fp32 arithmetic, every level in one launch, any block size, d = 16 .. 128: fp32 tensors on the fp32 matrix
// instruction (layout: tile_kernels.hip), bf16 tensors on the bf16 one with P and dS in three exact parts (tile_bf16.hip).
//
// Key-major (Sec. 4.3): the unit is a tile of up to 16 keys of a level against the queries that attend to it (the fine queries
// under the query blocks of Alg. 2's list; every query at a dense level), 16 (fp32) or 32 (bf16) at a time.  Q and dO rows of a
// chunk go through the wave's LDS once and are read from there row-wise (scores) and by columns (gradients); the next chunk's
// rows fly during the math, the list entry behind them one chunk further ahead.  Bound: the start of a workgroup (key rows, list
// offsets, entry, query rows, each waiting for the one before) and the sum of its waves, for lists of some 8 chunks; fp32 also the
// matrix pipe.  16 heads, operands straight from memory before: fp32 x 4096 tokens 176 -> 130 us, bf16 x 2704 tokens 126 -> 42.
// A workgroup of four waves takes one tile and a share of its list (`splits`, so that a level of few keys, whose lists are long,
// still fills the chip), dealt to the waves chunk by chunk; their sums are added through LDS in wave order.  (One level-0 tile per
// wave, without that sum: 50 against 44 us at 16 heads x 2704 tokens in bf16, and with few tiles up to twice as long.)
#include "tile_f32.h"

namespace llsa {

struct DkvTileLevel {
    const void *K, *V;
    const int32_t *C, *Iq;       // null when dense
    float *partK, *partV;        // [splits][bh * n][D] fp32
    int64_t n, slab;             // tokens per head; floats of one slab
    unsigned wg0;                // first workgroup of the level
    FastDiv tiles, span, tpb, splits;   // key tiles per head; fine queries under a listed query block; tiles per block; shares
    int rows, Kl;
    float bias;
};
struct DkvTileArgs {
    DkvTileLevel lv[kMaxL + 1];
    int nlev, B;
    int64_t N;
    float scale;
};

// ---- fp32 tensors
template <int D> struct MathF32 {
    using T = float;
    using S = TShape<D>;
    static constexpr int TQ = 16, CH = D / 4, RPR = 64 / CH, R = 16 / RPR;   // queries, 16-byte chunks a row, rows a round, rounds
    static constexpr int ROWB = 4 * D, BUF = 2 * TQ * ROWB;
    static constexpr bool PARTS = false, AHEAD = D < 128;   // 64 more registers for the next chunk's rows would spill
    static constexpr int NT = D / 16, GS = S::E, NG = S::H, E = S::E;    // sums come in NG groups of GS accumulators
    using RT = RowTile<D>;
    static __device__ __forceinline__ int at(int r, int c) { return RT::at(r, c); }
    struct Keys {
        RowOp<D> k, v;
        __device__ __forceinline__ void load(const T *kr, const T *vr, int g) { k = row_op<D>(kr, g); v = row_op<D>(vr, g); }
    };
    template <bool Exact, class Next>
    static __device__ __forceinline__ void tile(const char *buf, const float *st, const Keys &key, f32x4 (&accK)[NT], f32x4 (&accV)[NT],
                                                float scale, float bias, unsigned, int i16, int g, Next next) {
        f32x4 s = row_product<D>(RT::row(buf, i16, g), key.k);
        f32x4 dp = row_product<D>(RT::row(buf + TQ * ROWB, i16, g), key.v);
        const f32x4 lse = *reinterpret_cast<const f32x4 *>(st + 4 * g), dl = *reinterpret_cast<const f32x4 *>(st + TQ + 4 * g);
        next();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r] = exp_nat(fmaf(s[r], scale, bias) - lse[r]);
            dp[r] = s[r] * (dp[r] - dl[r]);
        }
        col_product<D>(accV, RT::col(buf + TQ * ROWB, i16, g), s);
        col_product<D>(accK, RT::col(buf, i16, g), dp);
    }
    // group h of a tensor's sums: E channels at a time of key i16
    template <class Emit> static __device__ __forceinline__ void emit(const f32x4 (&t)[GS], int h, int g, Emit f) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            FVec<E> x;
#pragma unroll
            for (int e = 0; e < E; ++e) x.v[e] = t[e][r];
            f(16 * E * h + E * (4 * g + r), x);
        }
    }
};

// ---- bf16 tensors
template <int D> struct MathBF16 {
    using T = uint16_t;
    static constexpr int TQ = 32, CH = D / 8, RPR = 64 / CH, R = 32 / RPR;
    static constexpr int ROWB = 2 * D, BUF = 2 * TQ * ROWB;
    static constexpr bool PARTS = true, AHEAD = true;
    static constexpr int KS = (D + 31) / 32, NT = D / 16, GS = 1, NG = NT, E = 4;
    static __device__ __forceinline__ int at(int r, int c) { return r * ROWB + ((c ^ swz_key<D>(r)) << 4); }
    // d = 16 fills half of the 32 contraction slots, the others are zero
    static __device__ __forceinline__ bf16x8 half(bf16x8 x, int g) {
        if constexpr (D == 16) return g < 2 ? x : bf16x8{};
        else return x;
    }
    struct Keys {
        bf16x8 k[KS], v[KS];
        __device__ __forceinline__ void load(const T *kr, const T *vr, int g) {
            const int c = D == 16 ? 8 * (g & 1) : 8 * g;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) { k[ks] = half(ld_bf16x8(kr + c + 32 * ks), g); v[ks] = half(ld_bf16x8(vr + c + 32 * ks), g); }
        }
    };
    // rows: how many of the 32 queries exist.  Exact: P and dS as they are on the fp32 matrix instruction (inputs that are not finite)
    template <bool Exact, class Next>
    static __device__ __forceinline__ void tile(const char *buf, const float *st, const Keys &key, f32x4 (&accK)[NT], f32x4 (&accV)[NT],
                                                float scale, float bias, unsigned rows, int i16, int g, Next next) {
        const char *gbuf = buf + TQ * ROWB;
        const TileOffsets<D> o = tile_offsets<D>(16 * g + i16);
        f32x4 s[2], dp[2], lse[2], dl[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            s[h] = f32x4{0.f, 0.f, 0.f, 0.f};
            dp[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                s[h] = mfma16(half(ld_bf16x8(buf + 16 * h * ROWB + o.row[ks]), g), key.k[ks], s[h]);
                dp[h] = mfma16(half(ld_bf16x8(gbuf + 16 * h * ROWB + o.row[ks]), g), key.v[ks], dp[h]);
            }
            lse[h] = *reinterpret_cast<const f32x4 *>(st + 16 * h + 4 * g);
            dl[h] = *reinterpret_cast<const f32x4 *>(st + TQ + 16 * h + 4 * g);
        }
        next();
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[h][r] = exp_nat(fmaf(s[h][r], scale, bias) - lse[h][r]);
                dp[h][r] = s[h][r] * (dp[h][r] - dl[h][r]);
            }
        Parts3 p, ds;
        if constexpr (!Exact) p = split8(s[0], s[1]), ds = split8(dp[0], dp[1]);
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            const bf16x8 tg = lds_tr_pair(gbuf + o.tr[n], gbuf + 16 * ROWB + o.tr[n]);
            const bf16x8 tq = lds_tr_pair(buf + o.tr[n], buf + 16 * ROWB + o.tr[n]);
            if constexpr (Exact) {
                accV[n] = product_fp32(tg, s, (int)min(rows, 32u), g, accV[n]);
                accK[n] = product_fp32(tq, dp, (int)min(rows, 32u), g, accK[n]);
            } else
#pragma unroll
                for (int i = 2; i >= 0; --i) {
                    accV[n] = mfma16(tg, p.p[i], accV[n]);
                    accK[n] = mfma16(tq, ds.p[i], accK[n]);
                }
        }
    }
    template <class Emit> static __device__ __forceinline__ void emit(const f32x4 (&t)[GS], int h, int g, Emit f) {
        f(16 * h + 4 * g, FVec<4>{{t[0][0], t[0][1], t[0][2], t[0][3]}});
    }
};

// One key tile's queries: `lst` null for every query of the head, else listed blocks of L.span queries.
struct QueryList { const int32_t *lst; unsigned count; };
__device__ __forceinline__ QueryList query_list(const DkvTileLevel &L, int64_t bh, unsigned blk, int64_t N) {
    QueryList q = {nullptr, (unsigned)N};
    if (L.C) {
        const int32_t *Crow = L.C + bh * (L.rows + 1) + blk;
        q.lst = L.Iq + bh * L.rows * L.Kl + Crow[0];
        q.count = (unsigned)(Crow[1] - Crow[0]) * L.span.d; // a query lists a key at most once: no more than N
    }
    return q;
}

// Chunks c_beg, c_beg + step, ... < c_end of a list against one key tile: their sums accK / accV.
template <class M, bool Exact>
__device__ __forceinline__ void accumulate(const DkvTileArgs &a, const typename M::T *Q, const typename M::T *dO, const float *LSE,
                                           const float *Dsum, int64_t bh, const QueryList &ql, FastDiv span, float bias, unsigned c_beg,
                                           unsigned step, unsigned c_end, const typename M::Keys &key, f32x4 (&accK)[M::NT],
                                           f32x4 (&accV)[M::NT], char *buf, float *st, int lane) {
    constexpr int TQ = M::TQ;
#pragma unroll
    for (int n = 0; n < M::NT; ++n) { accK[n] = f32x4{0.f, 0.f, 0.f, 0.f}; accV[n] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    if (c_beg >= c_end) return;
    const char *Qb = reinterpret_cast<const char *>(Q) + bh * a.N * M::ROWB, *Gb = reinterpret_cast<const char *>(dO) + bh * a.N * M::ROWB;
    const float *stat_src = (lane & TQ ? Dsum : LSE) + bh * a.N;
    // the query at position lane % TQ of chunk c (past the end of the list: its last one)
    auto query = [&](unsigned c) -> unsigned {
        const unsigned p = min(TQ * c + (lane & (TQ - 1)), ql.count - 1);
        if (!ql.lst) return p;
        const unsigned e = span(p);
        return (unsigned)ql.lst[e] * span.d + (p - e * span.d);
    };
    u32x4 q[M::R], go[M::R];
    float stat;
    auto load = [&](unsigned qi, unsigned c) {
        stat = stat_src[qi];
        if (!(lane & TQ) && TQ * c + (lane & (TQ - 1)) >= ql.count) stat = INFINITY;   // past the end: LSE inf, P = 0
#pragma unroll
        for (int u = 0; u < M::R; ++u) {
            const uint64_t off = (uint64_t)(unsigned)__shfl((int)qi, lane / M::CH + M::RPR * u) * M::ROWB + (lane % M::CH) * 16;
            q[u] = *reinterpret_cast<const u32x4 *>(Qb + off);
            go[u] = *reinterpret_cast<const u32x4 *>(Gb + off);
        }
    };
    unsigned qi = query(c_beg);
    if (M::AHEAD) {
        load(qi, c_beg);
        qi = query(min(c_beg + step, c_end - 1));
    }
    for (unsigned c = c_beg; c < c_end; c += step) {
        if (!M::AHEAD) {
            load(qi, c);
            qi = query(min(c + step, c_end - 1));
        }
        __builtin_amdgcn_wave_barrier();                    // one wave's LDS operations stay in order
#pragma unroll
        for (int u = 0; u < M::R; ++u) {
            const int off = M::at(lane / M::CH + M::RPR * u, lane % M::CH);
            *reinterpret_cast<u32x4 *>(buf + off) = q[u];
            *reinterpret_cast<u32x4 *>(buf + TQ * M::ROWB + off) = go[u];
        }
        if (lane < 2 * TQ) st[lane] = stat;
        __builtin_amdgcn_wave_barrier();
        M::template tile<Exact>(buf, st, key, accK, accV, a.scale, bias, ql.count - TQ * c, lane & 15, lane >> 4, [&]() {
            if (M::AHEAD && c + step < c_end) {
                load(qi, c + step);
                qi = query(min(c + 2 * step, c_end - 1));
            }
        });
    }
}

template <class M, int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : 3)))
tile_dkv_kernel(DkvTileArgs a, const typename M::T *__restrict__ Q, const typename M::T *__restrict__ dO, const float *__restrict__ LSE,
                const float *__restrict__ Dsum) {
    using T = typename M::T;
    constexpr int NT = M::NT, SLOTS = 2 * NT, RED = 4 * SLOTS * 64 * 16, WBUF = M::BUF + 256;
    __shared__ __attribute__((aligned(16))) char lds[RED > 4 * WBUF ? RED : 4 * WBUF];
    const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char *buf = lds + wave * WBUF;
    float *st = reinterpret_cast<float *>(buf + M::BUF);
    float *red = reinterpret_cast<float *>(lds);
    int l = 0;                                              // levels are laid out from the coarsest (longest lists) down
    for (int x = 1; x < a.nlev; ++x) l = blockIdx.x < a.lv[x - 1].wg0 ? x : l;
    const DkvTileLevel &L = a.lv[l];
    const unsigned id = blockIdx.x - L.wg0;

    f32x4 accK[NT], accV[NT];
    const unsigned kt = L.splits(id), split = id - kt * L.splits.d;
    // a tile of a listed block of B keys, or 16 tokens of a dense level (tpb = 1)
    const int64_t bh = L.tiles(kt);
    const unsigned in = kt - (unsigned)bh * L.tiles.d, blk = L.tpb(in);
    const int first = 16 * (int)(in - blk * L.tpb.d);
    const int64_t key0 = L.C ? (int64_t)blk * a.B + first : (int64_t)in * 16;
    const int nk = L.C ? min(16, a.B - first) : (int)min((int64_t)16, L.n - key0);
    const int64_t krow = bh * L.n + key0 + min(i16, nk - 1);
    const QueryList ql = query_list(L, bh, blk, a.N);
    const unsigned chunks = (ql.count + M::TQ - 1) / M::TQ;
    const unsigned c_beg = (unsigned)((uint64_t)chunks * split / L.splits.d), c_end = (unsigned)((uint64_t)chunks * (split + 1) / L.splits.d);
    typename M::Keys key;
    if (c_beg + wave < c_end) key.load(static_cast<const T *>(L.K) + krow * D, static_cast<const T *>(L.V) + krow * D, g);
    accumulate<M, false>(a, Q, dO, LSE, Dsum, bh, ql, L.span, L.bias, c_beg + wave, 4, c_end, key, accK, accV, buf, st, lane);
    if constexpr (M::PARTS)                                 // an input is not finite (tile_bf16.hip says why)
        if (any_nan(accK) || any_nan(accV))
            accumulate<M, true>(a, Q, dO, LSE, Dsum, bh, ql, L.span, L.bias, c_beg + wave, 4, c_end, key, accK, accV, buf, st, lane);
    // the four waves' sums in wave order; wave w finishes groups w, w + 4, ... of [dK | dV]
    __syncthreads();                                        // everyone is done with the tile buffers
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        *reinterpret_cast<f32x4 *>(red + ((wave * SLOTS + n) * 64 + lane) * 4) = accK[n];
        *reinterpret_cast<f32x4 *>(red + ((wave * SLOTS + NT + n) * 64 + lane) * 4) = accV[n];
    }
    __syncthreads();
    for (int grp = wave; grp < 2 * M::NG; grp += 4) {
        f32x4 x[M::GS];
#pragma unroll
        for (int e = 0; e < M::GS; ++e) {
            const float *src = red + ((grp * M::GS + e) * 64 + lane) * 4;
            x[e] = *reinterpret_cast<const f32x4 *>(src);
#pragma unroll
            for (int w = 1; w < 4; ++w) x[e] += *reinterpret_cast<const f32x4 *>(src + w * SLOTS * 256);
        }
        if (i16 >= nk) continue;
        const bool isV = grp >= M::NG;
        float *dst = (isV ? L.partV : L.partK) + split * L.slab + krow * D;
        const float w = isV ? 1.f : a.scale;
        M::emit(x, grp % M::NG, g, [&](int ch, FVec<M::E> v) {
#pragma unroll
            for (int e = 0; e < M::E; ++e) v.v[e] *= w;
            st_e<M::E>(dst + ch, v);
        });
    }
}

// The levels' partials folded down (adjoint of mean pooling): a level-0 token's gradient is its own sum plus 1/B of its
// level-1 ancestor's total, which holds 1/B of the level-2 ancestor's, and so on.  One workgroup per level-1 token: its total
// (every share of every ancestor, added in a fixed order by 256 / (D / 2) groups of threads), then the token's B children.
__device__ __forceinline__ void st_fold(float *p, const FVec<4> &x) { st_e<4>(p, x); }
__device__ __forceinline__ void st_fold(uint16_t *p, const FVec<4> &x) { st_e(p, x); }
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
    const int64_t first = (int64_t)blockIdx.x * a.B;        // the token's first child, over all heads
    const float *own = isV ? a.partV[0] : a.partK[0];
    f32x4 x0[2];                                            // the first children's own sums fly meanwhile
#pragma unroll
    for (int u = 0; u < 2; ++u) x0[u] = *reinterpret_cast<const f32x4 *>(own + (first + min(grp + GR * u, a.B - 1)) * D + c);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const float inv = 1.f / (float)a.B;
    float w = inv;
    int turn = 0;                                           // shares are dealt to the groups in turn
    for (int l = 1; l < a.nlev; ++l) {
        const float *src = (isV ? a.partV[l] : a.partK[l]) + (bh * a.n[l] + tok) * D + c;
        const int splits = a.splits[l];
#pragma unroll 4
        for (int s = (grp + GR - turn % GR) % GR; s < splits; s += GR) acc += *reinterpret_cast<const f32x4 *>(src + s * a.slab[l]) * w;
        turn += splits;
        tok /= (unsigned)a.B;
        w *= inv;
    }
    sum[grp][slot] = acc;
    __syncthreads();
    f32x4 par = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < GR; ++x) par += sum[x][slot];
    for (int r = grp, u = 0; r < a.B; r += GR, ++u) {
        const int64_t o = (first + r) * D + c;
        const f32x4 x = (u == 0 ? x0[0] : u == 1 ? x0[1] : *reinterpret_cast<const f32x4 *>(own + o)) + par;
        st_fold((isV ? dV : dK) + o, FVec<4>{{x[0], x[1], x[2], x[3]}});
    }
}

// ------------------------------------------------------------------------------------------------- launches
template <class F> static hipError_t by_shape(const Plan &p, F f) {
    auto by_d = [&](auto ty) {
        switch (p.d) {
            case 16: f(ty, std::integral_constant<int, 16>{}); break;
            case 32: f(ty, std::integral_constant<int, 32>{}); break;
            case 64: f(ty, std::integral_constant<int, 64>{}); break;
            default: f(ty, std::integral_constant<int, 128>{}); break;
        }
    };
    if (p.elt == 4) by_d(float{});
    else by_d(uint16_t{});
    return hipGetLastError();
}

// shares of level l's query lists, key tiles per head, tiles per listed block
static void dkv_tile_shape(const Plan &p, int l, int *splits, int64_t *tiles, int *tpb) {
    const bool dense = l == p.L;
    *tpb = dense ? 1 : (p.B + 15) / 16;
    *tiles = dense ? (p.n[l] + 15) / 16 : p.n[l + 1] * *tpb;
    // level 0's lists are short (K blocks of queries on average) and its result is not summed again.  Above it: enough workgroups
    // to fill the chip, each with at least two chunks a wave.  bf16 in chunks of 32 at four workgroups per CU: every further share
    // is another start-up, another sum of four waves and another slab to fold (16 heads x 2704 tokens, 12 shares 44 + 14 us, 5
    // 42 + 11).  fp32 in chunks of 16 at eight: fewer, longer sums are faster too (n = 4096: 160 -> 143 us) but less exact (dV 1.04
    // times as far from a 64-bit computation).
    const int64_t chunks = (dense ? p.N : (int64_t)p.Kl[l] * (p.N / p.n[l + 1])) / (p.elt == 2 ? 32 : 16), wgs = p.elt == 2 ? 1024 : 2048;
    int64_t s = (wgs + p.bh * *tiles - 1) / (p.bh * *tiles);
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
        int splits, tpb;
        dkv_tile_shape(p, l, &splits, &tiles, &tpb);
        L.splits = FastDiv(splits);
        L.tpb = FastDiv(tpb);
        L.tiles = FastDiv(tiles);
        L.K = t.K[l]; L.V = t.V[l];
        L.C = dense ? nullptr : reinterpret_cast<const int32_t *>(w + p.C_off[l]);
        L.Iq = dense ? nullptr : reinterpret_cast<const int32_t *>(w + p.Iq_off[l]);
        L.n = p.n[l];
        L.slab = (int64_t)p.bh * p.n[l] * p.d;
        L.rows = dense ? 0 : (int)p.n[l + 1];
        L.Kl = dense ? 0 : p.Kl[l];
        L.span = FastDiv(dense ? 1 : p.N / p.n[l + 1]);
        L.bias = t.bias[l];
        if (l == 0 && p.elt == 4) { L.partK = static_cast<float *>(dK); L.partV = static_cast<float *>(dV); }
        else {
            L.partK = part;
            L.partV = part + L.slab * splits;
            part += 2 * L.slab * splits;
        }
        L.wg0 = (unsigned)wg;
        wg += p.bh * tiles * splits;
        f.partK[l] = L.partK; f.partV[l] = L.partV;
        f.n[l] = L.n; f.slab[l] = L.slab; f.splits[l] = splits;
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
        using M = std::conditional_t<std::is_same<T, float>::value, MathF32<d.value>, MathBF16<d.value>>;
        tile_dkv_kernel<M, d.value><<<(unsigned)wg, 256, 0, s>>>(a, (const T *)Q, (const T *)dO, LSE, D);
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
