// dQ on bf16 MFMA, variant that shares the coarse levels (B = 16, 32 or 64, d = 64 or 128, at most
// 64 level-0 tiles per list); see attn_fwd_shared.hip for the decomposition (a workgroup of 4 or 8 waves owns
// 128 consecutive queries, which use the same lists at every level >= 1, every wave one or two 16-query tiles; the coarse
// key/value tiles are staged once per workgroup in LDS, the level-0 tiles are walked per query tile).
// Per tile and query block:  S^T = K Q^T, dP^T = V dO^T  ->  dS^T = P^T o (dP^T - D)  ->  dQ^T += K^T dS^T,
// with K read from LDS both row-wise (first product) and transposed (last product).
// Rows go from memory straight into LDS, as in the forward kernel (16 heads x 65536 tokens, d = 64: 269 -> 249 us; 8 x 65536, d = 128,
// K = 16: 447 -> 383).  The ring's places known at compile time and level 0's first rows asked for beside the last coarse tile, as there: kernel in a
// step, us, 16 x 65536 272.1 -> 267.0 (Gaussian 304.6 -> 297.2), 16 x 4096 20.8 -> 19.8, 32 x 16384 132.1 -> 129.5, 8 x 65536, d = 128, K = 16
// 405.4 -> 392.1, 8 x 262144 1594 -> 1526.
// The kernel also produces D = rowsum(dO o O) for its queries and stores it for the key-major kernels.
#include <type_traits>

#include "csc_small.h"
#include "dkv_group.h"

namespace llsa {

__device__ __forceinline__ u32x4 from_bf16x8(bf16x8 v) {
    union { u32x4 u; bf16x8 b; } c;
    c.b = v;
    return c.u;
}
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// NB = fine query tiles per wave (1 or 2), NW = waves; a workgroup owns NW * NB consecutive tiles, all siblings.  GW = waves
// whose tiles make up a block of 32 or 64 queries and share a level-0 list (0: B = 16; 1: one wave holds the whole block).
// Three waves per SIMD leave two tiles at d = 64 the registers they need (four spill: 572 against 477 us at 65536 tokens in
// blocks of 64; two: 480; with rows straight into LDS 294 against 249 at 65536 tokens in blocks of 16).
// Along: nothing, or the grouped dK / dV kernel's work (with DENSE, its dense level) in workgroups of this launch's.
struct NothingAlong {};
template <bool DENSE> struct WithGroup { GroupAlong g; };
template <int D, int NB, int NW, int GW, class Along>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 64 ? (NB == 2 ? 3 : 4) : 2)))
dq_shared_kernel(ListArgs args, const uint16_t *__restrict__ Q, const uint16_t *__restrict__ O,
                 const uint16_t *__restrict__ dO, const float *__restrict__ LSE, float *__restrict__ Dsum,
                 uint16_t *__restrict__ dQ, int64_t N, FastDiv groups, CscSmall csc, Along along) {
    constexpr int KS = D / 32, NT = D / 16, ROWB = 2 * D, HALF = 16 * ROWB, TILE = 2 * HALF;   // 16 rows, 32 rows
    constexpr int CPH = HALF / 1024;                    // load_lds steps of 16 rows
    constexpr int CPW = 4 * CPH / NW;                   // of a [K | V] tile that the workgroup shares, per wave
    constexpr int RING = 4, NBUF = GW > 1 ? 2 : 1;      // phase A's tiles; phase B's tiles per group of waves
    constexpr int OWN = (GW > 0 ? NW / GW : NW) * NBUF; // phase B's places
    constexpr int PLACES = (OWN > RING - 1 ? OWN : RING - 1) + 1;     // one that phase A still reads when phase B's first rows are asked for
    __shared__ __attribute__((aligned(16))) char lds[PLACES * 2 * TILE];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int64_t nblk = N >> 4;                                      // query tiles per head
    // the first workgroups make the key-major lists, which nothing here reads
    static_assert(sizeof(lds) >= kCscSmallLds, "");
    if (blockIdx.x < csc.wgs) {
        csc_small<64 * NW>(csc, blockIdx.x, reinterpret_cast<uint32_t *>(lds));
        return;
    }
    unsigned front = csc.wgs;
    if constexpr (!std::is_same<Along, NothingAlong>::value) {
        const GroupAlong &ga = along.g;
        if (blockIdx.x < front + ga.wgs) {
            const unsigned R = xcd_contiguous32(blockIdx.x - front, ga.wgs);
            static_assert(sizeof(lds) >= kGroupLds<D>, "");
            if (R < ga.groups) group_body<D, NW, std::is_same<Along, WithGroup<true>>::value, true>(ga.t, ga.a, R, lds, O);
            return;
        }
        front += ga.wgs;
    }
    const unsigned wg = xcd_contiguous32(blockIdx.x - front, gridDim.x - front);
    const int64_t bh = groups(wg), blk0 = (wg - (unsigned)bh * groups.d) * (NW * NB);   // groups.d workgroups per head
    // a spare wave of a head's last workgroup works on the head's last tile without storing it
    auto tile_of = [&](int b) { return min(blk0 + NB * wave + b, nblk - 1); };
    (void)args;                                                       // read through the pointer: fields of a level by scalar loads
    const list_args_ptr t = kernel_list_args();
    const float sc2 = t->scale * kLog2e;
    const TileOffsets<D> o = tile_offsets<D>(lane);
    const RowSource<D> src(lane);

    // The lists first: everything else waits for them, and loads come back in the order in which they were asked for.
    // Level 0, of this wave's NB query blocks: lane LL b + j holds the first token of 16-token tile j of query tile b's list (as in the
    // forward kernel).
    constexpr int LL = GW > 0 ? 64 : 64 / NB;
    const int nb0 = t->lev[0].end;                                        // level-0 tiles
    const int nbc = t->lev[t->nlev - 1].end - nb0;                    // coarse tiles of the list
    const int j0_ = min(lane % LL, nb0 - 1);                              // a tile past the end is never asked for
    const int raw0 = t->lev[0].I[(bh * t->lev[0].rows + (tile_of(min(lane / LL, NB - 1)) >> t->ls)) * t->lev[0].Kl + (j0_ >> t->ls)];
    CoarseTable ctab;                                                  // lane j: coarse block 64 * chunk + j, of the tile issued last
    ctab.ask<D>(t, bh, (unsigned)blk0, 0, lane);

    bf16x8 qop[NB][KS], gop[NB][KS];
    u32x4 orow[NB][KS];
    f32x4 acc[NB][NT];
    float lse2[NB];
    f32x4 ndelta[NB];                                                 // -D in every register: what dP^T's sums start from
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int64_t qrow = bh * N + tile_of(b) * 16 + i16;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            qop[b][s] = ld_bf16x8(Q + qrow * D + g * 8 + 32 * s);
            gop[b][s] = ld_bf16x8(dO + qrow * D + g * 8 + 32 * s);
            orow[b][s] = *reinterpret_cast<const u32x4 *>(O + qrow * D + g * 8 + 32 * s);
        }
        lse2[b] = LSE[qrow];
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[b][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // D of the wave's queries.  Asked for behind the first tiles: the wait for its rows is one for those tiles too, since the compiler counts only the
    // loads that it knows of (in front of the tiles: 16 x 4096 tokens 96.0 and 96.8 us a step, 4 x 77056 550 and 546, even elsewhere).
    auto deltas = [&]() {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            float dl = 0.f;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const u32x4 gw = from_bf16x8(gop[b][s]), ow = orow[b][s];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    dl = fmaf(bf_lo(gw[e]), bf_lo(ow[e]), dl);
                    dl = fmaf(bf_hi(gw[e]), bf_hi(ow[e]), dl);
                }
            }
            dl = rows_sum(dl);
            ndelta[b] = f32x4{-dl, -dl, -dl, -dl};
            if (g == 0 && blk0 + NB * wave + b < nblk) Dsum[bh * N + tile_of(b) * 16 + i16] = dl;
            lse2[b] *= kLog2e;
        }
    };

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
    // Scores, dP - D and dQ^T += K^T dS^T of query tiles first .. first + count - 1 for one tile of 32 keys in LDS: every read
    // serves all of them.  alone: the tile is in the wave's own place, K's transposed operands are read before the scores are worked on, and
    // `have_read` is called when LDS holds nothing more of the tile that is wanted.
    auto tile = [&](auto first, auto count, auto alone, const char *kt, const char *vt, int c0, int c1, float w0, float w1, auto have_read) {
        constexpr int b0 = decltype(first)::value, n = decltype(count)::value;
        constexpr bool E = decltype(alone)::value;
        f32x4 s[n][2], dp[n][2];
        bf16x8 ktr[E ? NT : 1];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int b = 0; b < n; ++b) { s[b][h] = f32x4{0.f, 0.f, 0.f, 0.f}; dp[b][h] = ndelta[b0 + b]; }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 k = ld_bf16x8(kt + h * HALF + o.row[ks]), v = ld_bf16x8(vt + h * HALF + o.row[ks]);
#pragma unroll
                for (int b = 0; b < n; ++b) {
                    s[b][h] = mfma16(k, qop[b0 + b][ks], s[b][h]);
                    dp[b][h] = mfma16(v, gop[b0 + b][ks], dp[b][h]);
                }
            }
        }
        if constexpr (E) {
#pragma unroll
            for (int x = 0; x < NT; ++x) ktr[x] = lds_tr_pair(kt + o.tr[x], kt + HALF + o.tr[x]);
            have_read();
        }
        bf16x8 ds[n];
        ds[0] = ds_of(first, s[0][0], s[0][1], dp[0][0], dp[0][1], c0, c1, w0, w1);
        if constexpr (n > 1) ds[n - 1] = ds_of(B1{}, s[n - 1][0], s[n - 1][1], dp[n - 1][0], dp[n - 1][1], c0, c1, w0, w1);
#pragma unroll
        for (int x = 0; x < NT; ++x) {
            const bf16x8 k = E ? ktr[E ? x : 0] : lds_tr_pair(kt + o.tr[x], kt + HALF + o.tr[x]);
#pragma unroll
            for (int b = 0; b < n; ++b) acc[b0 + b][x] = mfma16(k, ds[b], acc[b0 + b][x]);
        }
    };
    using One = std::integral_constant<int, 1>;
    using All = std::integral_constant<int, NB>;
    using Alone = std::true_type;
    using Shared = std::false_type;
    auto nothing = []() {};

    const unsigned lds0 = lds_address(lds);
    const int ntile = (nbc + 1) >> 1;                                 // of the coarse levels
    // lane LL b + j: tile j's K rows; V's rows stand to_v0 further on
    const uint64_t row0 = reinterpret_cast<uint64_t>(t->lev[0].K) + (uint64_t)(bh * N + ((int64_t)raw0 << t->lb) + ((j0_ & ((1 << t->ls) - 1)) << 4)) * ROWB;
    const uint64_t to_v0 = reinterpret_cast<uint64_t>(t->lev[0].V) - reinterpret_cast<uint64_t>(t->lev[0].K);
    if (nbc > 0) ctab.finish<D>(t);

    // ------------------------------------------------------------------ phase B's loads: level 0
    // half h of the K rows (to_v = 0) or V rows of tile j0 of the list that begins at lane l0
    auto load_half = [&](uint64_t to_v, int l0, int j0, int h, unsigned dst) {
        const int j = j0 + h < nb0 ? j0 + h : j0;                     // an absent second half re-reads the first
        load_lds<CPH>(reinterpret_cast<uint64_t>(BlockTable::rl_ptr(row0, l0 + j)) + to_v, src.v0, src.v1, dst + h * HALF);
    };
    // place x of phase B: not the one of phase A's last tile, which other waves may still be reading
    const int keep = (ntile + RING - 1) % RING;
    auto place = [&](int x) { return (unsigned)(x < keep ? x : x + 1) * (2 * TILE); };
    constexpr int SHARE = GW > 0 ? GW : 1;                            // waves that bring in a list's tiles together
    const int own = GW > 1 ? wave / SHARE * NBUF : wave;
    const unsigned place0 = place(own), place1 = place(own + NBUF - 1);
    auto issue_b = [&](int u) {                                       // GW > 1: the wave's share of tile u
        const unsigned dst = lds0 + (u & 1 ? place1 : place0);
#pragma unroll
        for (int x = 0; x < 4 / SHARE; ++x) {
            const int part = wave % SHARE * (4 / SHARE) + x;          // K, K, V, V: its halves
            load_half(part < 2 ? 0 : to_v0, 0, 2 * u, part & 1, dst + (part >> 1) * TILE);
        }
    };
    auto load_rows = [&](uint64_t to_v, int l0, int j0, unsigned to) {
        load_half(to_v, l0, j0, 0, lds0 + place0 + to);
        load_half(to_v, l0, j0, 1, lds0 + place0 + to);
    };
    auto begin_b = [&]() {
        if constexpr (GW > 1) issue_b(0);
        else {
            load_rows(0, 0, 0, 0);
            load_rows(to_v0, 0, 0, TILE);
        }
    };

    // ------------------------------------------------------------------ phase A: shared coarse levels
    if (nbc > 0) {
        const bool v_wave = wave >= NW / 2;                           // this wave brings in V rows
        uint64_t rows = v_wave ? +ctab.vptr : +ctab.kptr;
        float w_now = ctab.bias2, w_next = w_now;                     // the weights, of the tile worked on
        int c0 = 16, c1 = 16;                                         // rows of the last tile's halves (only it may be ragged or lack its second half)
        // this wave's share of a tile: load_lds steps of one half of K or of V
        const int part = wave * CPW / CPH, sub = wave * CPW % CPH, half = part & 1;
        auto issue = [&](int u, int to) {                             // coarse blocks 2u, 2u + 1, to place `to`
            if (u > 0 && ((2 * u) & 63) == 0) {
                list_args_ptr t2 = t;
                asm volatile("" : "+s"(t2));                          // the levels' fields are not kept for this
                ctab.fill<D>(t2, bh, (unsigned)blk0, (2 * u) >> 6, lane);
                rows = v_wave ? +ctab.vptr : +ctab.kptr;
                w_next = ctab.bias2;
            }
            const int j = (2 * u + half < nbc ? 2 * u + half : 2 * u) & 63;
            const uint64_t base = reinterpret_cast<uint64_t>(BlockTable::rl_ptr(rows, j));
            const unsigned dst = lds0 + to * (2 * TILE) + wave * CPW * 1024;
            if (u + 1 == ntile) {
                const int n0 = ctab.count((2 * u) & 63), n1 = 2 * u + 1 < nbc ? ctab.count((2 * u + 1) & 63) : 16;
                const int cnt = ctab.count(j);
                c0 = n0;
                c1 = n1;
                if (cnt < 16) {                                       // rows past a ragged end repeat the last one
#pragma unroll
                    for (int x = 0; x < CPW; ++x) {
                        const int r = (sub + x) * (512 / D) + lane / (D / 8);
                        const unsigned v = (unsigned)(min(r, cnt - 1) * ROWB + (((lane % (D / 8)) ^ swz_key<D>(r)) << 4));
                        load_lds<1>(base, v, v, dst + x * 1024);
                    }
                    return;
                }
            }
            load_lds<CPW>(base + sub * 1024, src.v0, src.v1, dst);
        };
        auto weight = [&](int j) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w_now), j & 63)); };
#pragma unroll
        for (int u = 0; u < RING - 1; ++u)
            if (u < ntile) issue(u, u);
        deltas();
        // All tiles but the last, in a loop that is unrolled over the ring: the places are known, no half is short.
        auto turn = [&](int u, auto at) {
            constexpr int x = decltype(at)::value;
            // tile u is there, and tile u - 1, whose place tile u + 3 takes, has been read by every wave
            if (u + 2 < ntile) vm_wait_barrier<2 * CPW>();
            else vm_wait_barrier<CPW>();
            if (u + RING - 1 < ntile) issue(u + RING - 1, (x + RING - 1) % RING);
            if (x == 0 && ((2 * u) & 63) == 0) w_now = w_next;        // (a chunk of 64 blocks begins at place 0)
            const char *kt = lds + x * (2 * TILE);
            tile(B0{}, All{}, Shared{}, kt, kt + TILE, 16, 16, weight(2 * u), weight(2 * u + 1), nothing);
        };
        int u = 0;
        for (; u + RING < ntile; u += RING) {
            turn(u, std::integral_constant<int, 0>());
            turn(u + 1, std::integral_constant<int, 1>());
            turn(u + 2, std::integral_constant<int, 2>());
            turn(u + 3, std::integral_constant<int, 3>());
        }
        if (u + 1 < ntile) { turn(u, std::integral_constant<int, 0>()); ++u; }
        if (u + 1 < ntile) { turn(u, std::integral_constant<int, 1>()); ++u; }
        if (u + 1 < ntile) { turn(u, std::integral_constant<int, 2>()); ++u; }
        vm_wait_barrier<0>();
        begin_b();                                                    // only the last tile's place is in use any more
        if (((2 * u) & 63) == 0) w_now = w_next;
        const char *kt = lds + (u % RING) * (2 * TILE);
        // an absent half: P = 0
        tile(B0{}, All{}, Shared{}, kt, kt + TILE, c0, c1, weight(2 * u), 2 * u + 1 < nbc ? weight(2 * u + 1) : -INFINITY, nothing);
    } else {
        begin_b();
        deltas();
    }

    // ------------------------------------------------------------------ phase B: level 0
    if constexpr (GW > 1) {
        // Blocks of 32 or 64 tokens: the B queries of a block use one level-0 list, whose tiles the GW waves that hold them bring in
        // together, double-buffered.  A list is whole blocks of B >= 32 tokens: no half of a tile is ever absent.
        for (int u = 0; 2 * u < nb0; ++u) {
            vm_wait_barrier<0>();
            if (2 * u + 2 < nb0) issue_b(u + 1);
            const char *kt = lds + (u & 1 ? place1 : place0);
            tile(B0{}, All{}, Shared{}, kt, kt + TILE, 16, 16, 0.f, 0.f, nothing);
        }
    } else {
        // Every wave alone: the tiles of its query tiles (GW = 1: of all of them at once) form one stream.  The next tile's rows are
        // asked for as soon as the current one's have been read, so they fly during all of its math.
        const char *my = lds + place0;
        auto walk = [&](auto first, auto count, bool end) {
            const int l0 = LL * decltype(first)::value;
            for (int j0 = 0; j0 < nb0; j0 += 2) {
                const bool here = j0 + 2 < nb0;
                const int nl = here ? l0 : l0 + LL, nj = here ? j0 + 2 : 0;
                vm_wait<0>();
                // level-0 blocks are always full; an absent second half has weight 0
                tile(first, count, Alone{}, my, my + TILE, 16, 16, 0.f, j0 + 1 < nb0 ? 0.f : -INFINITY, [&]() {
                    if (!here && end) return;
                    load_rows(0, nl, nj, 0);
                    load_rows(to_v0, nl, nj, TILE);
                });
            }
        };
        if constexpr (GW == 1) walk(B0{}, All{}, true);
        else {
            walk(B0{}, One{}, NB == 1);
            if constexpr (NB > 1) walk(B1{}, One{}, true);
        }
    }

#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (blk0 + NB * wave + b >= nblk) break;
        auto out = [&](int n) {
            return u32x2{pack_bf16(acc[b][n][0] * t->scale, acc[b][n][1] * t->scale), pack_bf16(acc[b][n][2] * t->scale, acc[b][n][3] * t->scale)};
        };
#pragma unroll
        for (int n = 0; n < NT; n += 2) store_pair(dQ + (bh * N + (blk0 + NB * wave + b) * 16 + i16) * D, n, g, out(n), out(n + 1));
    }
}

static unsigned dq_groups(const Plan &p) { return (unsigned)p.bh * (unsigned)((p.N + 127) / 128); }
// where this launch has one query tile a wave, in workgroups of the grouped kernel's size
bool dq_takes_group(const Plan &p) { return dq_takes_lists(p) && p.d == 64 && p.B == 16 && !(p.Kl[0] <= 32 && dq_groups(p) >= 1024); }

hipError_t launch_dq_shared(const Plan &p, const LevelTable &t, const void *Q, const void *O, const void *dO,
                            const float *LSE, float *D, void *dQ, const CscSmall &csc, const GroupAlong *group, hipStream_t s) {
    const FastDiv groups((p.N + 127) / 128);
    const unsigned wgs = dq_groups(p);
    const ListArgs a = make_list_args(t);
    const int ls = p.lb - 4;
    auto launch = [&](auto d, auto nb, auto gw, auto along, unsigned more) {
        constexpr int NB = decltype(nb)::value, NW = 8 / NB;
        dq_shared_kernel<decltype(d)::value, NB, NW, decltype(gw)::value, decltype(along)><<<wgs + csc.wgs + more, 64 * NW, 0, s>>>(
            a, (const uint16_t *)Q, (const uint16_t *)O, (const uint16_t *)dO, LSE, D, (uint16_t *)dQ, p.N, groups, csc, along);
    };
    auto go = [&](auto d, auto nb, auto gw) { launch(d, nb, gw, NothingAlong{}, 0u); };
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
    if (group) {
        using D64 = std::integral_constant<int, 64>;
        if (group->dense) launch(D64{}, I1{}, I0{}, WithGroup<true>{*group}, group->wgs);
        else launch(D64{}, I1{}, I0{}, WithGroup<false>{*group}, group->wgs);
    } else if (p.d == 128) {
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
