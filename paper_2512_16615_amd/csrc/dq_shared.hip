// dQ on bf16 MFMA, variant that shares the coarse levels (B = 16, 32 or 64, d = 64 or 128, at most
// 64 level-0 tiles per list); see attn_fwd_shared.hip for the decomposition (a workgroup of 4 or 8 waves owns
// 128 consecutive queries, which use the same lists at every level >= 1, every wave one or two 16-query tiles; the coarse
// key/value tiles are staged once per workgroup in LDS, the level-0 tiles are walked per query tile).
// Per tile and query block:  S^T = K Q^T, dP^T = V dO^T  ->  dS^T = P^T o (dP^T - D)  ->  dQ^T += K^T dS^T,
// with K read from LDS both row-wise (first product) and transposed (last product).
// The kernel also produces D = rowsum(dO o O) for its queries and stores it for the key-major kernels.
#include <type_traits>

#include "mfma_common.h"

namespace llsa {

typedef const __attribute__((address_space(1))) u32x4 *gvec_ptr_t;
__device__ __forceinline__ u32x4 gload16b(const char *base, unsigned off) {
    return *reinterpret_cast<gvec_ptr_t>(reinterpret_cast<const __attribute__((address_space(1))) char *>(
        reinterpret_cast<uintptr_t>(base)) + off);
}
__device__ __forceinline__ bf16x8 to_bf16x8(u32x4 v) {
    union { u32x4 u; bf16x8 b; } c;
    c.u = v;
    return c.b;
}
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// NB = fine query tiles per wave (1 or 2), NW = waves; a workgroup owns NW * NB consecutive tiles, all siblings.  GW = waves
// whose tiles make up a block of 32 or 64 queries and share a level-0 list (0: B = 16; 1: one wave holds the whole block).
// Three waves per SIMD leave two tiles at d = 64 the registers they need (four spill: 572 against 477 us at 65536 tokens in
// blocks of 64; two: 480).
template <int D, int NB, int NW, int GW>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 64 ? (NB == 2 ? 3 : 4) : 2)))
dq_shared_kernel(ListArgs args, const uint16_t *__restrict__ Q, const uint16_t *__restrict__ O,
                 const uint16_t *__restrict__ dO, const float *__restrict__ LSE, float *__restrict__ Dsum,
                 uint16_t *__restrict__ dQ, int64_t N, FastDiv groups) {
    constexpr int KS = D / 32, NT = D / 16, STRIDE = D * 2 + 32, PARTS = D / 8, TILE = 32 * STRIDE;
    constexpr int NTHR = 64 * NW, RND = (2 * 32 * PARTS) / NTHR, VCH = D / 16, KPU = 64 / PARTS;
    // Phase B: per wave a K tile (row-wise and transposed reads) and a V tile (row-wise reads only; 16 bytes of
    // padding keep it smaller).  Phase A's two double-buffered [K | V] tiles live in the first 4 TILE bytes of the
    // same memory; a workgroup barrier separates the phases.
    constexpr int VSTRIDE = D * 2 + 16, VTILE = 32 * VSTRIDE;
    __shared__ __attribute__((aligned(16))) char lds[NW * (TILE + VTILE)];
    static_assert(4 * TILE <= NW * (TILE + VTILE), "phase A's buffers must fit");
    auto sh = [&](int buf, int which) { return lds + (buf * 2 + which) * TILE; };

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int64_t nblk = N >> 4;                                      // query tiles per head
    const unsigned wg = xcd_contiguous32(blockIdx.x, gridDim.x);
    const int64_t bh = groups(wg), blk0 = (wg - (unsigned)bh * groups.d) * (NW * NB);   // groups.d workgroups per head
    // a spare wave of a head's last workgroup works on the head's last tile without storing it
    auto tile_of = [&](int b) { return min(blk0 + NB * wave + b, nblk - 1); };
    (void)args;                                                       // read through the pointer: fields of a level by scalar loads
    const list_args_ptr t = kernel_list_args();
    const float sc2 = t->scale * kLog2e;

    bf16x8 qop[NB][KS], gop[NB][KS];
    f32x4 acc[NB][NT];
    float lse2[NB];
    f32x4 ndelta[NB];                                                 // -D in every register: what dP^T's sums start from
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int64_t qrow = bh * N + tile_of(b) * 16 + i16;
        float dl = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            qop[b][s] = ld_bf16x8(Q + qrow * D + g * 8 + 32 * s);
            const u32x4 gw = *reinterpret_cast<const u32x4 *>(dO + qrow * D + g * 8 + 32 * s);
            const u32x4 ow = *reinterpret_cast<const u32x4 *>(O + qrow * D + g * 8 + 32 * s);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dl = fmaf(bf_lo(gw[e]), bf_lo(ow[e]), dl);
                dl = fmaf(bf_hi(gw[e]), bf_hi(ow[e]), dl);
            }
            gop[b][s] = to_bf16x8(gw);
        }
        dl = rows_sum(dl);
        ndelta[b] = f32x4{-dl, -dl, -dl, -dl};
        if (g == 0 && blk0 + NB * wave + b < nblk) Dsum[qrow] = dl;
        lse2[b] = LSE[qrow] * kLog2e;
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[b][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // dS^T of query tile b for one tile of keys (dp: dP^T - D); a half of weight -inf is absent
    auto ds_of = [&](auto bsel, f32x4 s0, f32x4 s1, f32x4 dp0, f32x4 dp1, int c0, int c1, float b0, float b1) -> bf16x8 {
        constexpr int b = decltype(bsel)::value;
        f32x4 s[2] = {s0, s1};
        const f32x4 dp[2] = {dp0, dp1};
        const float c2[2] = {b0 - lse2[b], b1 - lse2[b]};
        const int c[2] = {c0, c1};
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float p = __builtin_amdgcn_exp2f(fmaf(s[h][r], sc2, c2[h]));
                s[h][r] = p * dp[h][r];
            }
        if (c[0] < 16 || c[1] < 16) {                                 // rows past the end of a ragged block contribute nothing
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (4 * g + r >= c[h]) s[h][r] = 0.f;
        }
        return pack8(s[0], s[1]);
    };
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    // Scores, dP - D and dQ^T += K^T dS^T of query tiles b0 .. b0 + n - 1 for one tile of 32 staged keys (V rows VS bytes apart):
    // every LDS read serves all of them.
    auto tile = [&](auto first, auto count, const char *kt, const char *vt, auto vstride, int c0, int c1, float w0, float w1) {
        constexpr int b0 = decltype(first)::value, n = decltype(count)::value, VS = decltype(vstride)::value;
        f32x4 s[n][2], dp[n][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const char *krow = kt + (h * 16 + i16) * STRIDE + g * 16, *vrow = vt + (h * 16 + i16) * VS + g * 16;
#pragma unroll
            for (int b = 0; b < n; ++b) { s[b][h] = f32x4{0.f, 0.f, 0.f, 0.f}; dp[b][h] = ndelta[b0 + b]; }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 k = *reinterpret_cast<const bf16x8 *>(krow + ks * 64), v = *reinterpret_cast<const bf16x8 *>(vrow + ks * 64);
#pragma unroll
                for (int b = 0; b < n; ++b) {
                    s[b][h] = mfma16(k, qop[b0 + b][ks], s[b][h]);
                    dp[b][h] = mfma16(v, gop[b0 + b][ks], dp[b][h]);
                }
            }
        }
        bf16x8 ds[n];
        ds[0] = ds_of(first, s[0][0], s[0][1], dp[0][0], dp[0][1], c0, c1, w0, w1);
        if constexpr (n > 1) ds[n - 1] = ds_of(B1{}, s[n - 1][0], s[n - 1][1], dp[n - 1][0], dp[n - 1][1], c0, c1, w0, w1);
        const char *base = kt + (4 * g + (i16 >> 2)) * STRIDE + (i16 & 3) * 8;
#pragma unroll
        for (int x = 0; x < NT; ++x) {
            const bf16x8 ktr = lds_tr_pair(base + x * 32, base + 16 * STRIDE + x * 32);
#pragma unroll
            for (int b = 0; b < n; ++b) acc[b0 + b][x] = mfma16(ktr, ds[b], acc[b0 + b][x]);
        }
    };
    using One = std::integral_constant<int, 1>;
    using All = std::integral_constant<int, NB>;
    using StrideA = std::integral_constant<int, STRIDE>;
    using StrideB = std::integral_constant<int, VSTRIDE>;

    // The level-0 lists of this wave's NB query blocks, fetched now so that phase B does not wait for them:
    // lane LL b + j holds the first token of 16-token tile j of query tile b's list (as in the forward kernel).
    constexpr int LL = GW > 0 ? 64 : 64 / NB;
    const int nb0 = t->lev[0].end;
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
        CoarseTable ctab;
        ctab.fill<D>(t, bh, (unsigned)blk0, 0, lane);
        // Staging round r of this wave: 64 consecutive 16-byte chunks of the [K | V] tile, i.e. 64 / PARTS key rows of
        // one half of K or of V, the same choice for the whole wave (one round: the first half of the waves stages K, the
        // other V; more: the first half of the rounds stages K).
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
        auto load_shared = [&](int u) {
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
                sreg[r] = gload16b(src, off);
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
            int cnt[2] = {16, 16};
            float bias2[2] = {ctab.bias((2 * u) & 63), ctab.bias((2 * u + 1) & 63)};
            if (u + 1 == ntile) {
                cnt[0] = ctab.count((2 * u) & 63);
                if (2 * u + 1 < nbc) cnt[1] = ctab.count((2 * u + 1) & 63);
                else bias2[1] = -INFINITY;                            // an absent half: P = 0
            }
            __syncthreads();
            if (u + 1 < ntile) load_shared(u + 1);
            tile(B0{}, All{}, sh(buf, 0), sh(buf, 1), StrideA{}, cnt[0], cnt[1], bias2[0], bias2[1]);
        }
    }

    if constexpr (GW > 0) {
        // -------------------------------------------------------------- phase B, blocks of 32 or 64 tokens
        // The GW waves that hold the B queries of a block stage the tiles of their one level-0 list together, double-buffered
        // per group, as in the forward kernel (16 heads x 65536 tokens in blocks of 64, K = 8: 677 -> 554 us).
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
                sreg[r] = gload16b(src + row * (D * 2), (unsigned)((((key0 & 15) + lane / PARTS) * D + (lane % PARTS) * 8) * 2));
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
            tile(B0{}, All{}, buf, buf + TILE, StrideB{}, 16, 16, 0.f, 0.f);
        }
    } else {
    // ------------------------------------------------------------------ phase B: own level-0 blocks
    // K and V rows are fetched with 8 consecutive lanes per 128-byte row (whole cache lines per instruction: loading
    // the MFMA operand layout straight from memory, 16 rows x half a line per instruction, caps the gather rate at a
    // third of what the L2 delivers) and reach the operand layouts through the wave's own LDS tiles.
    __syncthreads();                                                  // phase A's buffers are free
    char *my = lds + wave * (TILE + VTILE), *my_v = my + TILE;
    const char *K0 = static_cast<const char *>(t->lev[0].K), *V0 = static_cast<const char *>(t->lev[0].V);
    unsigned voff[VCH];
#pragma unroll
    for (int u = 0; u < VCH; ++u) voff[u] = (unsigned)((((lane / PARTS + KPU * u) & 15) * D + (lane % PARTS) * 8) * 2);

    auto phase_b = [&](auto bsel) {
        constexpr int b = decltype(bsel)::value;
        u32x4 kreg[VCH], vreg[VCH];
        auto load_tile = [&](int j0) {
            int64_t off[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = (j0 + h < nb0) ? j0 + h : j0;           // an absent second half re-reads the first
                off[h] = (bh * N + __builtin_amdgcn_readlane(tok0, LL * b + j)) * (D * 2);
            }
#pragma unroll
            for (int u = 0; u < VCH; ++u) {
                kreg[u] = gload16b(K0 + off[(KPU * u) >> 4], voff[u]);
                vreg[u] = gload16b(V0 + off[(KPU * u) >> 4], voff[u]);
            }
        };
        load_tile(0);
        for (int j0 = 0; j0 < nb0; j0 += 2) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < VCH; ++u) {
                *reinterpret_cast<u32x4 *>(my + (lane / PARTS + KPU * u) * STRIDE + (lane % PARTS) * 16) = kreg[u];
                *reinterpret_cast<u32x4 *>(my_v + (lane / PARTS + KPU * u) * VSTRIDE + (lane % PARTS) * 16) = vreg[u];
            }
            __builtin_amdgcn_wave_barrier();
            if (j0 + 2 < nb0) load_tile(j0 + 2);                      // the registers are free again
            tile(bsel, One{}, my, my_v, StrideB{}, 16, 16, 0.f, j0 + 1 < nb0 ? 0.f : -INFINITY);
        }
    };
    phase_b(B0{});
    if constexpr (NB > 1) phase_b(B1{});
    }

#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (blk0 + NB * wave + b >= nblk) break;
        uint16_t *orow = dQ + (bh * N + (blk0 + NB * wave + b) * 16 + i16) * D + 4 * g;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            u32x2 w;
            w[0] = pack_bf16(acc[b][n][0] * t->scale, acc[b][n][1] * t->scale);
            w[1] = pack_bf16(acc[b][n][2] * t->scale, acc[b][n][3] * t->scale);
            *reinterpret_cast<u32x2 *>(orow + n * 16) = w;
        }
    }
}

hipError_t launch_dq_shared(const Plan &p, const LevelTable &t, const void *Q, const void *O, const void *dO,
                            const float *LSE, float *D, void *dQ, hipStream_t s) {
    const FastDiv groups((p.N + 127) / 128);
    const unsigned wgs = (unsigned)p.bh * groups.d;
    const ListArgs a = make_list_args(t);
    const int ls = p.lb - 4;
    auto go = [&](auto d, auto nb, auto gw) {
        constexpr int NB = decltype(nb)::value, NW = 8 / NB;
        dq_shared_kernel<decltype(d)::value, NB, NW, decltype(gw)::value><<<wgs, 64 * NW, 0, s>>>(
            a, (const uint16_t *)Q, (const uint16_t *)O, (const uint16_t *)dO, LSE, D, (uint16_t *)dQ, p.N, groups);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    auto by_block = [&](auto d, auto nb) {
        constexpr int NB = decltype(nb)::value;
        if (ls == 0) go(d, nb, I0{});
        else if (ls == 1) go(d, nb, std::integral_constant<int, 2 / NB>{});
        else go(d, nb, std::integral_constant<int, 4 / NB>{});
    };
    // Two query tiles per wave read every staged operand from LDS once for both (16 heads, d = 128 x 262144 tokens, K = 16:
    // 2240 -> 1819 us; d = 64 x 65536 tokens: 320 -> 293 us, in blocks of 64: 550 -> 477).  At d = 64 they pay from four
    // workgroups per CU on (262144 queries: 73.8 -> 69.8 us; 131072: equal); with fewer, eight waves with a tile each hide
    // more of the latency (65536 queries: 19.9 against 21.0 us).  Both tiles' level-0 lists have to fit one register, and
    // blocks of 32 tokens at d = 128 keep one tile: with two, the wave's registers spill.
    const bool fit = ls > 0 || p.Kl[0] <= 32;
    if (p.d == 128) {
        using D128 = std::integral_constant<int, 128>;
        if (fit && ls == 0) go(D128{}, I2{}, I0{});
        else if (ls == 2) go(D128{}, I2{}, I2{});
        else if (ls == 1) go(D128{}, I1{}, I2{});
        else go(D128{}, I1{}, I0{});
    } else {
        if (fit && wgs >= 1024) by_block(std::integral_constant<int, 64>{}, I2{});
        else by_block(std::integral_constant<int, 64>{}, I1{});
    }
    return hipGetLastError();
}

}  // namespace llsa
