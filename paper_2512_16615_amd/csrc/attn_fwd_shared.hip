// Attention forward over the gathered lists on bf16 MFMA, variant that shares the coarse levels
// (B = 16, 32 or 64, d = 64 or 128, N a multiple of 256, at most 64 level-0 tiles of 16 tokens per list).
//
// 256 consecutive queries (B = 16: the 16 fine query blocks under one level-1 query block) use the same lists at
// every level >= 1 (Alg. 1, enrichment loop: block i reads row i / B^l of I^(l)), i.e. the same coarse key/value
// tokens.  One workgroup of 4 or 8 waves owns such a group or half of one; every wave owns one or two of its
// 16-query tiles.
//   Phase A (levels >= 1): the workgroup stages each tile of two 16-token blocks (K and V rows) once in
//     LDS, double-buffered; every wave reads the K operand once and multiplies it with both of its query
//     blocks, likewise the transposed V operand, so the gather traffic of the coarse tokens is paid once
//     per 128 or 256 queries instead of once per 16.
//   Phase B (level 0): each wave walks the level-0 tiles of each of its query tiles' lists; their K and V rows are
//     fetched as whole cache lines and reach the operand layouts through the wave's private LDS tiles.
// Score tiles are computed transposed (S^T = K Q^T) so that the accumulator layout (4 keys x 1 query per
// lane) is the B operand of O^T += V^T P^T; see mfma_common.h for the register layouts.
#include <type_traits>

#include "mfma_common.h"

namespace llsa {

typedef const __attribute__((address_space(1))) u32x4 *gvec_ptr;
__device__ __forceinline__ u32x4 gload16(const char *base, unsigned off) {
    return *reinterpret_cast<gvec_ptr>(reinterpret_cast<const __attribute__((address_space(1))) char *>(
        reinterpret_cast<uintptr_t>(base)) + off);
}
constexpr float kMaxSum = 4096.f;   // a query's softmax reference is raised only when a tile's probabilities exceed this

// NB = fine query tiles per wave (1 or 2), NW = waves per workgroup (4 or 8); a workgroup owns NW * NB consecutive
// tiles, all siblings.  GW = waves whose tiles make up a block of 32 or 64 queries and share a level-0 list (0: B = 16)
template <int D, int NB, int NW, int GW>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2))) attn_fwd_shared_kernel(ListArgs args, const uint16_t *__restrict__ Q,
                                                               uint16_t *__restrict__ O, float *__restrict__ LSE,
                                                               int64_t N, FastDiv groups) {
    constexpr int KS = D / 32, NT = D / 16, STRIDE = D * 2 + 32, PARTS = D / 8, TILE = 32 * STRIDE;
    constexpr int NTHR = 64 * NW;
    constexpr int RND = (2 * 32 * PARTS) / NTHR;        // staging rounds of the workgroup per shared tile (K and V)
    constexpr int VCH = D / 16, KPU = 64 / PARTS;       // private V staging of one wave (phase B)
    // Phase B: per wave a K tile (row-wise reads: rows 32 bytes apart in the banks) and a V tile (transposed reads only:
    // 16 bytes of padding do).  Phase A's two double-buffered [K | V] tiles live in the first 4 TILE bytes of the same
    // memory; a workgroup barrier separates the phases.
    constexpr int VSTRIDE = D * 2 + 16, VTILE = 32 * VSTRIDE;
    __shared__ __attribute__((aligned(16))) char lds[NW * (TILE + VTILE)];
    static_assert(4 * TILE <= NW * (TILE + VTILE), "phase A's buffers must fit");
    auto sh = [&](int buf, int which) { return lds + (buf * 2 + which) * TILE; };

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const unsigned wg = xcd_contiguous32(blockIdx.x, gridDim.x);
    const int64_t bh = groups(wg), blk0 = (wg - (unsigned)bh * groups.d) * (NW * NB);   // groups.d workgroups per head
    auto tile_of = [&](int b) { return blk0 + NB * wave + b; };
    (void)args;                                                       // read through the pointer: fields of a level by scalar loads
    const list_args_ptr t = kernel_list_args();
    const float sc2 = t->scale * kLog2e;

    bf16x8 qop[NB][KS];
    f32x4 acc[NB][NT];
    float m[NB], lsum[NB];                                            // reference; this lane's share of the row sum
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const uint16_t *qrow = Q + (bh * N + tile_of(b) * 16 + i16) * D + g * 8;
#pragma unroll
        for (int s = 0; s < KS; ++s) qop[b][s] = ld_bf16x8(qrow + 32 * s);
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[b][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        m[b] = -INFINITY;
        lsum[b] = 0.f;
    }

    using StrideA = std::integral_constant<int, STRIDE>;
    using StrideB = std::integral_constant<int, VSTRIDE>;
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    // Softmax update of query block b for one tile (s0 / s1: raw S^T of the two halves; b0 / b1: log2 weights of their levels,
    // -inf for an absent half): the probabilities as the B operand of O^T += V^T P^T.  The reference m[b] of a query is not
    // its exact maximum, and the usual tile does not even look for one: it takes the exponentials against the reference as
    // it is and checks their sum, which a later row sum needs anyway.  Only if that exceeds kMaxSum in some lane (or is inf
    // or nan; always in the first tile, where the reference is -inf) is the maximum found, the accumulators rescaled and
    // the exponentials taken again.  Probabilities up to 2^12 cost fp32 sums and bf16 operands no precision.  Scale, level
    // weight and reference are folded into the one multiply-add in front of the exponential.  31 vector instructions per
    // 16 x 32 tile where finding the maximum first took 52.
    auto probs = [&](auto bsel, f32x4 s0, f32x4 s1, int c0, int c1, float b0, float b1) -> bf16x8 {
        constexpr int b = decltype(bsel)::value;
        f32x4 s[2] = {s0, s1}, p[2];
        if (c0 < 16 || c1 < 16) {                                     // ragged block: mask
            const int c[2] = {c0, c1};
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (4 * g + r >= c[h]) s[h][r] = -INFINITY;
        }
        float sum;
        auto exps = [&]() {
            const float cb[2] = {b0 - m[b], b1 - m[b]};
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r) p[h][r] = __builtin_amdgcn_exp2f(fmaf(s[h][r], sc2, cb[h]));
            sum = ((p[0][0] + p[0][1]) + (p[0][2] + p[0][3])) + ((p[1][0] + p[1][1]) + (p[1][2] + p[1][3]));
        };
        exps();
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(sum <= kMaxSum)) != 0, 0)) {
            float z = -INFINITY;                                      // this lane's largest logit (log2 units)
#pragma unroll
            for (int r = 0; r < 4; ++r) z = fmaxf(z, fmaxf(fmaf(s[0][r], sc2, b0), fmaf(s[1][r], sc2, b1)));
            const float m_new = fmaxf(m[b], rows_max(z));
            const float alpha = __builtin_amdgcn_exp2f(m[b] - m_new);
            lsum[b] *= alpha;
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[b][n][r] *= alpha;
            m[b] = m_new;
            exps();
        }
        lsum[b] += sum;
        return pack8(p[0], p[1]);
    };
    // O^T += V^T P^T with the V tile at `vt` (row-major, VS bytes per key row)
    auto pv = [&](auto bsel, const bf16x8 pop, const char *vt, auto vstride) {
        constexpr int b = decltype(bsel)::value;
        constexpr int VS = decltype(vstride)::value;
        const char *base = vt + (4 * g + (i16 >> 2)) * VS + (i16 & 3) * 8;
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[b][n] = mfma16(lds_tr_pair(base + n * 32, base + 16 * VS + n * 32), pop, acc[b][n]);
    };
    // One tile of 32 staged keys against all query tiles of the wave: every K operand and every transposed V operand is read
    // from LDS once.
    auto shared_tile = [&](const char *kt, const char *vt, auto vstride, int c0, int c1, float b0, float b1) {
        constexpr int VS = decltype(vstride)::value;
        bf16x8 kop[2][KS];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                kop[h][ks] = *reinterpret_cast<const bf16x8 *>(kt + (h * 16 + i16) * STRIDE + g * 16 + ks * 64);
        f32x4 s[NB][2];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                s[b][h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) s[b][h] = mfma16(kop[h][ks], qop[b][ks], s[b][h]);
            }
        if constexpr (NB > 1) {                                       // both tiles' P first, then one transposing read of V for both
            const bf16x8 p0 = probs(B0{}, s[0][0], s[0][1], c0, c1, b0, b1);
            const bf16x8 p1 = probs(B1{}, s[NB - 1][0], s[NB - 1][1], c0, c1, b0, b1);
            const char *base = vt + (4 * g + (i16 >> 2)) * VS + (i16 & 3) * 8;
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const bf16x8 vtr = lds_tr_pair(base + n * 32, base + 16 * VS + n * 32);
                acc[0][n] = mfma16(vtr, p0, acc[0][n]);
                acc[NB - 1][n] = mfma16(vtr, p1, acc[NB - 1][n]);
            }
        } else {
            pv(B0{}, probs(B0{}, s[0][0], s[0][1], c0, c1, b0, b1), vt, vstride);
        }
    };

    // The level-0 lists of this wave's NB query blocks, fetched now so that phase B does not wait for them:
    // lane LL b + j holds the first token of 16-token tile j of query tile b's list (at most LL tiles; a listed block of B
    // tokens is B / 16 consecutive tiles, and B / 16 consecutive query tiles share a row of I^(0): one list for all if GW > 0).
    constexpr int LL = GW > 0 ? 64 : 64 / NB;
    const int nb0 = t->lev[0].end;                                        // level-0 tiles (the list always holds level 0)
    int tok0 = 0;
    {
        const int b = lane / LL, j = lane % LL;
        if (j < nb0) {
            const int64_t row = tile_of(b) >> t->ls;
            tok0 = (t->lev[0].I[(bh * t->lev[0].rows + row) * t->lev[0].Kl + (j >> t->ls)] << t->lb) + ((j & ((1 << t->ls) - 1)) << 4);
        }
    }

    // ------------------------------------------------------------------ phase A: shared coarse levels
    const int nbc = t->lev[t->nlev - 1].end - nb0;                    // coarse tiles of the list
    if (nbc > 0) {
        CoarseTable ctab;                                              // lane j: coarse block 64 * chunk + j
        ctab.fill<D>(t, bh, (unsigned)blk0, 0, lane);
        // Staging round r of this wave: 64 consecutive 16-byte chunks of the [K | V] tile, i.e. 64 / PARTS key rows of
        // one half of K or of V, the same choice for the whole wave.
        // (One round: the first half of the waves stages K, the other V; more: the first half of the rounds stages K.)
        u32x4 sreg[RND];
        int s_half[RND];
        unsigned s_off[RND];
#pragma unroll
        for (int r = 0; r < RND; ++r) {
            const int key0 = ((64 * wave + NTHR * r) % (32 * PARTS)) / PARTS;   // the wave's first key row in round r
            s_half[r] = key0 >> 4;
            s_off[r] = (unsigned)((((key0 & 15) + lane / PARTS) * D + (lane % PARTS) * 8) * 2);
        }
        const bool v_wave = RND == 1 && wave >= NW / 2;
        uint64_t sptr = v_wave ? ctab.vptr : ctab.kptr;               // d = 64: the tensor this wave stages
        const int ntile = (nbc + 1) >> 1;                             // only the last tile may be ragged or lack its second half
        auto load_shared = [&](int u) {                               // coarse blocks 2u, 2u + 1 -> registers
            if (u > 0 && ((2 * u) & 63) == 0) {
                ctab.fill<D>(t, bh, (unsigned)blk0, (2 * u) >> 6, lane);
                sptr = v_wave ? ctab.vptr : ctab.kptr;
            }
#pragma unroll
            for (int r = 0; r < RND; ++r) {
                const bool have = 2 * u + s_half[r] < nbc;
                const int j = (have ? 2 * u + s_half[r] : 2 * u) & 63;
                const char *src = RND == 1 ? BlockTable::rl_ptr(sptr, j) : (r < RND / 2 ? ctab.K(j) : ctab.V(j));
                unsigned off = s_off[r];
                if (u + 1 == ntile) {
                    const int cnt = have ? ctab.count(j) : 0;
                    if (cnt < 16) {                                   // ragged or absent block: re-read its last valid row
                        const int row = min((int)(off / (D * 2)), max(cnt, 1) - 1);
                        off = (unsigned)(row * D * 2) + off % (D * 2);
                    }
                }
                sreg[r] = gload16(src, off);
            }
        };
        auto store_shared = [&](int buf) {
#pragma unroll
            for (int r = 0; r < RND; ++r) {
                const int cc = tid + NTHR * r, which = cc / (32 * PARTS), c = cc % (32 * PARTS);
                *reinterpret_cast<u32x4 *>(sh(buf, which) + (c / PARTS) * STRIDE + (c % PARTS) * 16) = sreg[r];
            }
        };
        load_shared(0);
        for (int u = 0; u < ntile; ++u) {
            const int buf = u & 1;
            store_shared(buf);
            // per-half fields of this tile, before the table may be refilled for the next one
            int cnt[2] = {16, 16};
            float bias2[2] = {ctab.bias((2 * u) & 63), ctab.bias((2 * u + 1) & 63)};
            if (u + 1 == ntile) {
                cnt[0] = ctab.count((2 * u) & 63);
                if (2 * u + 1 < nbc) cnt[1] = ctab.count((2 * u + 1) & 63);
                else bias2[1] = -INFINITY;                            // an absent half: probabilities 0
            }
            __syncthreads();                                          // tile u visible; buffer buf^1 free again
            if (u + 1 < ntile) load_shared(u + 1);
            shared_tile(sh(buf, 0), sh(buf, 1), StrideA{}, cnt[0], cnt[1], bias2[0], bias2[1]);
        }
    }

    if constexpr (GW > 0) {
        // -------------------------------------------------------------- phase B, blocks of 32 or 64 tokens
        // The B queries of a block use one level-0 list: the GW waves that hold them stage its tiles together, as phase A does
        // for the whole workgroup, double-buffered per group (GW = 1: a wave alone, whose LDS operations stay in order).  A
        // list is whole blocks of B >= 32 tokens: no half of a tile is ever absent.  16 heads x 65536 tokens in blocks of 64, K = 8:
        // 512 -> 365 us.
        constexpr int R = 2 * 32 * PARTS / (64 * GW), BUF = TILE + VTILE, NBUF = GW > 1 ? 2 : 1;
        static_assert((NW / GW) * NBUF * BUF <= NW * (TILE + VTILE), "the groups' buffers must fit");
        __syncthreads();                                              // phase A's buffers are free
        const int wg_in = wave % GW;
        char *base = lds + (wave / GW) * (NBUF * BUF);
        const int64_t head = bh * N;
        const char *K0 = static_cast<const char *>(t->lev[0].K), *V0 = static_cast<const char *>(t->lev[0].V);
        u32x4 sreg[R];
        auto load_group = [&](int u) {                                // 64 chunks a round: rows of one half of K or of V
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int c0 = 64 * (wg_in + GW * r), key0 = (c0 % (32 * PARTS)) / PARTS;
                const char *src = c0 >= 32 * PARTS ? V0 : K0;
                const int64_t row = head + __builtin_amdgcn_readlane(tok0, 2 * u + (key0 >> 4));
                sreg[r] = gload16(src + row * (D * 2), (unsigned)((((key0 & 15) + lane / PARTS) * D + (lane % PARTS) * 8) * 2));
            }
        };
        load_group(0);
        for (int u = 0; 2 * u < nb0; ++u) {
            char *buf = base + (u % NBUF) * BUF;
            if constexpr (GW == 1) __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int c0 = 64 * (wg_in + GW * r), row = (c0 % (32 * PARTS)) / PARTS + lane / PARTS;
                char *dst = c0 >= 32 * PARTS ? buf + TILE + row * VSTRIDE : buf + row * STRIDE;
                *reinterpret_cast<u32x4 *>(dst + (lane % PARTS) * 16) = sreg[r];
            }
            if constexpr (GW > 1) __syncthreads();
            else __builtin_amdgcn_wave_barrier();
            if (2 * u + 2 < nb0) load_group(u + 1);
            shared_tile(buf, buf + TILE, StrideB{}, 16, 16, 0.f, 0.f);
        }
    } else {
    // ------------------------------------------------------------------ phase B: own level-0 blocks
    // K and V rows are fetched with 8 consecutive lanes per 128-byte row (whole cache lines per instruction: loading
    // the MFMA operand layout straight from memory, 16 rows x half a line per instruction, caps the gather rate at a
    // third of what the L2 delivers) and reach the operand layouts through the wave's own LDS tiles.
    __syncthreads();                                                  // phase A's buffers are free
    char *my_k = lds + wave * (TILE + VTILE), *my_v = my_k + TILE;
    unsigned voff[VCH];
#pragma unroll
    for (int u = 0; u < VCH; ++u) voff[u] = (unsigned)((((lane / PARTS + KPU * u) & 15) * D + (lane % PARTS) * 8) * 2);

    // The tiles of the wave's NB query blocks form one stream: the next tile's rows are in flight during the
    // current tile's math, also across the border between the two blocks (tok0: fetched before phase A).
    u32x4 kreg[VCH], vreg[VCH];
    const char *K0 = static_cast<const char *>(t->lev[0].K), *V0 = static_cast<const char *>(t->lev[0].V);
    auto load_tile = [&](int b, int j0) {
        int64_t off[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j = (j0 + h < nb0) ? j0 + h : j0;               // an absent second half re-reads the first
            off[h] = (bh * N + __builtin_amdgcn_readlane(tok0, LL * b + j)) * (D * 2);
        }
#pragma unroll
        for (int u = 0; u < VCH; ++u) {
            kreg[u] = gload16(K0 + off[(KPU * u) >> 4], voff[u]);
            vreg[u] = gload16(V0 + off[(KPU * u) >> 4], voff[u]);
        }
    };
    auto phase_b = [&](auto bsel) {
        constexpr int b = decltype(bsel)::value;
        for (int j0 = 0; j0 < nb0; j0 += 2) {
            __builtin_amdgcn_wave_barrier();                          // one wave's LDS operations stay in order
#pragma unroll
            for (int u = 0; u < VCH; ++u) {
                *reinterpret_cast<u32x4 *>(my_k + (lane / PARTS + KPU * u) * STRIDE + (lane % PARTS) * 16) = kreg[u];
                *reinterpret_cast<u32x4 *>(my_v + (lane / PARTS + KPU * u) * VSTRIDE + (lane % PARTS) * 16) = vreg[u];
            }
            __builtin_amdgcn_wave_barrier();
            if (j0 + 2 < nb0) load_tile(b, j0 + 2);                   // the registers are free again: next tile's rows
            else if (b + 1 < NB) load_tile(b + 1, 0);                 // fly during all of this tile's math
            f32x4 s[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                s[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    s[h] = mfma16(*reinterpret_cast<const bf16x8 *>(my_k + (h * 16 + i16) * STRIDE + g * 16 + ks * 64), qop[b][ks], s[h]);
            }
            // level-0 blocks are always full; an absent second half has weight 0
            pv(bsel, probs(bsel, s[0], s[1], 16, 16, 0.f, j0 + 1 < nb0 ? 0.f : -INFINITY), my_v, StrideB{});
        }
    };
    load_tile(0, 0);
    phase_b(B0{});
    if constexpr (NB > 1) phase_b(B1{});
    }

    // ------------------------------------------------------------------ epilogue
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const float l = rows_sum(lsum[b]);
        const float inv = 1.f / l;
        const int64_t row = bh * N + tile_of(b) * 16 + i16;
        uint16_t *orow = O + row * D + 4 * g;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            u32x2 w;
            w[0] = pack_bf16(acc[b][n][0] * inv, acc[b][n][1] * inv);
            w[1] = pack_bf16(acc[b][n][2] * inv, acc[b][n][3] * inv);
            *reinterpret_cast<u32x2 *>(orow + n * 16) = w;
        }
        if (g == 0) LSE[row] = (m[b] + __builtin_amdgcn_logf(l)) * kLn2;
    }
}

hipError_t launch_attn_fwd_shared(const Plan &p, const LevelTable &t, const void *Q, void *O, float *LSE,
                                  hipStream_t s) {
    const FastDiv groups(p.N / 128);
    const unsigned wgs = (unsigned)p.bh * groups.d;
    const ListArgs a = make_list_args(t);
    const uint16_t *q = (const uint16_t *)Q;
    uint16_t *o = (uint16_t *)O;
    const int ls = p.lb - 4;
    auto go = [&](auto d, auto nb, auto gw) {
        constexpr int NB = decltype(nb)::value, NW = 8 / NB;
        attn_fwd_shared_kernel<decltype(d)::value, NB, NW, decltype(gw)::value><<<wgs, 64 * NW, 0, s>>>(a, q, o, LSE, p.N, groups);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using D64 = std::integral_constant<int, 64>;
    using D128 = std::integral_constant<int, 128>;
    // Two query tiles per wave read every coarse operand from LDS once for both: half the LDS reads, which bound d = 128
    // (16 heads x 262144 tokens, K = 16: 1977 -> 1512 us; 4096 tokens: 33.9 -> 30.1).  At d = 64 they pay from four
    // workgroups per CU on (131072 queries: 33.6 -> 30.4 us); with fewer, eight waves with a tile each hide more of the
    // latency (65536 queries: 18.2 against 18.9, 32768: 12.6 against 14.1).  Both tiles' level-0 lists have to fit one register.
    if (ls == 1) {
        if (p.d == 64) go(D64{}, I2{}, I1{});
        else go(D128{}, I2{}, I1{});
    } else if (ls == 2) {
        if (p.d == 64) go(D64{}, I2{}, I2{});
        else go(D128{}, I2{}, I2{});
    } else if (p.d == 64) {
        if (p.Kl[0] <= 32 && wgs >= 1024) go(D64{}, I2{}, I0{});
        else go(D64{}, I1{}, I0{});
    } else {
        if (p.Kl[0] <= 32) go(D128{}, I2{}, I0{});
        else go(D128{}, I1{}, I0{});
    }
    return hipGetLastError();
}

}  // namespace llsa
