// Attention forward over the gathered lists on bf16 MFMA, variant that shares the coarse levels
// (B = 16, 32 or 64, d = 64 or 128, N a multiple of 256, at most 64 level-0 tiles of 16 tokens per list).
//
// 256 consecutive queries (B = 16: the 16 fine query blocks under one level-1 query block) use the same lists at
// every level >= 1 (Alg. 1, enrichment loop: block i reads row i / B^l of I^(l)), i.e. the same coarse key/value
// tokens.  One workgroup of 4 or 8 waves owns such a group or half of one; every wave owns one or two of its
// 16-query tiles.
//   Phase A (levels >= 1): the workgroup brings each tile of two 16-token blocks (K and V rows) once into
//     LDS, in a ring of four; every wave reads the K operand once and multiplies it with both of its query
//     blocks, likewise the transposed V operand, so the gather traffic of the coarse tokens is paid once
//     per 128 or 256 queries instead of once per 16.
//   Phase B (level 0): each wave walks the level-0 tiles of each of its query tiles' lists; their K and V rows are
//     fetched as whole cache lines and reach the operand layouts through the wave's private LDS tiles.
// All rows go from memory straight into LDS (load_lds): through registers and LDS writes the writes alone held the LDS for a third
// (d = 64) to half (d = 128) of the kernel's time.  16 heads x 65536 tokens, d = 64, K = 8: 204 -> 195 us; 8 x 65536, d = 128, K = 16:
// 362 -> 328; 8 x 262144: 1510 -> 1390.  Not so for Gaussian inputs, whose rows come from all over the head, from 32768 tokens on and for
// blocks of 64 with K <= 4 at 65536: the forward call takes 1 to 2 % longer (16 heads x 65536, Gaussian 348 -> 352 us), asking for K rows before
// V's operands are read changes nothing.  What is left, d = 64: 21 % of the matrix pipe, half of the vector issue slots; level 0 by
// itself (Le = 0) takes 162 us as before, at a third of the rate its gathers reach without any arithmetic.
// The ring's places are known at compile time (the loop is unrolled over it, the last tile, the only one that may be short, stands behind it), no wait
// of the compiler's own drains it, level 0's first rows are asked for beside the last coarse tile (one more place in LDS: 40 KB at d = 64, as much as
// four workgroups a CU leave each), and at level 0 K's place is filled again while V's is still read.  Kernel in a step, before and now, us: 16 heads x
// 65536 tokens 213.6 -> 209.0 (Gaussian 242.5 -> 232.3), in blocks of 64 372.6 -> 353.7, 32 x 16384 95.6 -> 91.4, 8 x 65536, d = 128, K = 16
// 346.7 -> 328.9, 8 x 262144 1413 -> 1311; the forward call of 16 x 4096 tokens 29.5 -> 28.6.  What it spends its time on, by clocks in its waves at
// 16 x 65536 (48000 cycles a wave): start to first tile 12000, a coarse tile 2500 (barrier 300, asking for the next tile 400, scores 450,
// exponentials 650, second product 400), a level-0 tile 1450.  Without the math of level 0 the launch takes 193 us, without its loads 177.
// Score tiles are computed transposed (S^T = K Q^T) so that the accumulator layout (4 keys x 1 query per
// lane) is the B operand of O^T += V^T P^T; see mfma_common.h for the register layouts.
#include <type_traits>

#include "mfma_common.h"

namespace llsa {

constexpr float kMaxSum = 4096.f;   // a query's softmax reference is raised only when a tile's probabilities exceed this

// Selection of the lists by the workgroup that walks them (d = 64, B = 16, K <= 8, small problems): the 8 level-1 tokens of its query tiles share their
// candidates, and the launch that it saves costs more than the work, which two workgroups to a level-2 token then do twice.  A wave a query: the candidates'
// rows through LDS, a score per lane by plain multiply-adds, the K-th best of two a lane by comparisons and counts (no sorted lists, whose registers
// the attention has no room for).  Bound: a chain of loads (parent's picks, their rows) and of 32 steps per list.
// Forward call, a launch of its own and here, us: 4 heads x 1024 tokens 19.3 and 15.3, 2 x 4096 20.7 and 16.9, 16 x 4096 28.1 and 25.9, 24 x 4096 37.5 and 35.5,
// 30 x 4096 42.4 and 42.1, 8 x 8192, L = 3 36.3 and 34.2, 2 x 16384 30.4 and 27.3; step of 16 x 4096 92.2 and 88.7.  (Two bits a step: 16 x 4096 27.1.)
struct SelectHere {
    const char *Q1, *K1, *Q2, *K2;   // pooled levels 1 and 2
    int32_t *I0, *I1;                // I^(0), written here; I^(1), read (SEL = 1) or, level 2 being the coarsest one, written (SEL = 2)
    int32_t n1, n2, K0, K1n;         // tokens per head; picks of I^(0) and of I^(1)
};
constexpr int kSelPicks = 8;         // of either list at most: 128 candidates, two a lane

// A score as the fp32 multiply-add chain over channels 0 .. 63 that the selection's contract states (select_mfma.hip), and as a number whose order as an
// unsigned integer is the order of scores (-0 ties with +0).  q: the query's row, the same in every lane; k: 16 bytes u of the candidate's
template <class K> __device__ __forceinline__ uint32_t score_key(uint64_t q, K k) {
    const auto *qw = reinterpret_cast<const __attribute__((address_space(4))) uint32_t *>(q);
    float acc = 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const u32x4 w = k(u);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t x = qw[4 * u + i];
            acc = fmaf(__uint_as_float(x << 16), __uint_as_float(w[i] << 16), acc);
            acc = fmaf(__uint_as_float(x & 0xffff0000u), __uint_as_float(w[i] & 0xffff0000u), acc);
        }
    }
    const uint32_t u = __float_as_uint(acc + 0.f);
    return u ^ (uint32_t)(((int32_t)u >> 31) | (int32_t)0x80000000);
}
// Which of the candidates 64 x + lane < count (at least K of them) are the K best, lower positions first among equals: the K-th largest key bit by bit, each
// bit a comparison and a count.
template <int PER> __device__ __forceinline__ void best(uint32_t (&key)[PER], int count, int K, int lane, uint64_t (&win)[PER]) {
    uint64_t there[PER];
#pragma unroll
    for (int x = 0; x < PER; ++x) {
        there[x] = __builtin_amdgcn_ballot_w64(64 * x + lane < count);
        key[x] = 64 * x + lane < count ? key[x] : 0u;                 // below every number that is compared with
    }
    uint32_t kth = 0;
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t t = kth | 1u << bit;
        int n = 0;
#pragma unroll
        for (int x = 0; x < PER; ++x) n += __popcll(__builtin_amdgcn_ballot_w64(key[x] >= t));
        kth = n >= K ? t : kth;
    }
    int left = K;
#pragma unroll
    for (int x = 0; x < PER; ++x) {
        win[x] = __builtin_amdgcn_ballot_w64(key[x] > kth) & there[x];
        left -= __popcll(win[x]);
    }
#pragma unroll
    for (int x = 0; x < PER; ++x) {
        uint64_t e = __builtin_amdgcn_ballot_w64(key[x] == kth) & there[x];
        for (; left > 0 && e; --left) {
            win[x] |= e & -e;
            e &= e - 1;
        }
    }
}

// NB = fine query tiles per wave (1 or 2), NW = waves per workgroup (4 or 8); a workgroup owns NW * NB consecutive
// tiles, all siblings.  GW = waves whose tiles make up a block of 32 or 64 queries and share a level-0 list (0: B = 16).  SEL: the lists of level 0 (1), of
// level 1 too (2), are selected here
template <int D, int NB, int NW, int GW, int SEL>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2))) attn_fwd_shared_kernel(ListArgs args, const uint16_t *__restrict__ Q,
                                                               uint16_t *__restrict__ O, float *__restrict__ LSE,
                                                               int64_t N, FastDiv groups, SelectHere sel) {
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
    const unsigned wg = xcd_contiguous32(blockIdx.x, gridDim.x);
    const int64_t bh = groups(wg), blk0 = (wg - (unsigned)bh * groups.d) * (NW * NB);   // groups.d workgroups per head
    auto tile_of = [&](int b) { return blk0 + NB * wave + b; };
    (void)args;                                                       // read through the pointer: fields of a level by scalar loads
    const list_args_ptr t = kernel_list_args();
    const float sc2 = t->scale * kLog2e;
    const TileOffsets<D> o = tile_offsets<D>(lane);
    const RowSource<D> src(lane);

    // The lists first: everything else waits for them, and loads come back in the order in which they were asked for.
    // Level 0, of this wave's NB query blocks: lane LL b + j holds the first token of 16-token tile j of query tile b's list (at most LL
    // tiles; a listed block of B tokens is B / 16 consecutive tiles, and B / 16 consecutive query tiles share a row of I^(0): one list for
    // all if GW > 0).
    constexpr int LL = GW > 0 ? 64 : 64 / NB;
    const int nb0 = t->lev[0].end;                                        // level-0 tiles (the list always holds level 0)
    const int nbc = t->lev[t->nlev - 1].end - nb0;                    // coarse tiles of the list
    const int j0_ = min(lane % LL, nb0 - 1);                              // a tile past the end is never asked for
    bf16x8 qop[NB][KS];
    auto ask_query = [&](int b) {
        const uint16_t *qrow = Q + (bh * N + tile_of(b) * 16 + i16) * D + g * 8;
#pragma unroll
        for (int s = 0; s < KS; ++s) qop[b][s] = ld_bf16x8(qrow + 32 * s);
    };
    int raw0;
    CoarseTable ctab;                                                  // lane j: coarse block 64 * chunk + j, of the tile issued last
    if constexpr (SEL > 0) {
        static_assert(D == 64 && NB == 1 && NW == kSelPicks && GW == 0, "a wave a pick's candidates, a wave a query");
        constexpr int STRIDE = 2 * D + 16;
        char *rows = lds + RING * 2 * TILE;                           // (phase A's ring is in front of it)
        static_assert(sizeof(lds) >= RING * 2 * TILE + 16 * kSelPicks * STRIDE, "");
        __shared__ int32_t pick_sh[NW][kSelPicks], list_sh[NW][kSelPicks];   // every wave's own copy of the parent's picks; its list
        ask_query(0);
        const int64_t tok1 = bh * sel.n1 + blk0, tok2 = bh * sel.n2 + (blk0 >> 4);   // the group's first level-1 token; its level-2 token
        if constexpr (SEL == 2) {                                     // every wave for itself: nothing to wait for
            const char *krow = sel.K2 + (bh * sel.n2 + min(lane, sel.n2 - 1)) * (2 * D);
            u32x4 kreg[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) kreg[u] = gload<u32x4>(krow + 16 * u);
            uint32_t key[1] = {score_key(reinterpret_cast<uint64_t>(sel.Q2) + tok2 * (2 * D), [&](int u) { return kreg[u]; })};
            uint64_t win[1];
            best<1>(key, sel.n2, sel.K1n, lane, win);
            if ((win[0] >> lane) & 1) {
                const int rank = __popcll(win[0] & ((1ull << lane) - 1));
                pick_sh[wave][rank] = lane;
                if (wave == 0 && (blk0 & 15) == 0) sel.I1[tok2 * sel.K1n + rank] = lane;
            }
        } else if (lane < sel.K1n) pick_sh[wave][lane] = sel.I1[tok2 * sel.K1n + lane];
        __builtin_amdgcn_wave_barrier();                              // one wave's LDS operations stay in order
        if (wave < sel.K1n) {                                         // the 16 candidates under the wave's pick
            const char *from = sel.K1 + (bh * sel.n1 + (int64_t)__builtin_amdgcn_readfirstlane(pick_sh[wave][wave]) * 16) * (2 * D);
#pragma unroll
            for (int u = 0; u < 2; ++u)
                *reinterpret_cast<u32x4 *>(rows + (16 * wave + 8 * u + lane / 8) * STRIDE + lane % 8 * 16) = gload<u32x4>(from + 1024 * u + 16 * lane);
        }
        __syncthreads();
        uint32_t key[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            key[x] = 0;
            if (x == 0 || sel.K1n > 4) key[x] = score_key(reinterpret_cast<uint64_t>(sel.Q1) + (tok1 + wave) * (2 * D),
                               [&](int u) { return *reinterpret_cast<const u32x4 *>(rows + (64 * x + lane) * STRIDE + 16 * u); });
        }
        uint64_t win[2];
        best<2>(key, 16 * sel.K1n, sel.K0, lane, win);
#pragma unroll
        for (int x = 0; x < 2; ++x)
            if ((win[x] >> lane) & 1) {
                const int rank = (x ? __popcll(win[0]) : 0) + __popcll(win[x] & ((1ull << lane) - 1));
                const int id = pick_sh[wave][4 * x + (lane >> 4)] * 16 + (lane & 15);
                list_sh[wave][rank] = id;
                sel.I0[(tok1 + wave) * sel.K0 + rank] = id;
            }
        __builtin_amdgcn_wave_barrier();
        raw0 = list_sh[wave][j0_];
        ctab.ask<D>(t, bh, (unsigned)blk0, 0, lane);
        if (SEL == 2 && nbc > 0 && ctab.n < 0) ctab.raw = pick_sh[wave][ctab.k];   // (level 1: the only coarse level with lists)
        if (nbc == 0) __syncthreads();                                       // phase B's places are where the candidates were
    } else {
        raw0 = t->lev[0].I[(bh * t->lev[0].rows + (tile_of(min(lane / LL, NB - 1)) >> t->ls)) * t->lev[0].Kl + (j0_ >> t->ls)];
        ctab.ask<D>(t, bh, (unsigned)blk0, 0, lane);
    }
    f32x4 acc[NB][NT];
    float m[NB], lsum[NB];                                            // reference; this lane's share of the row sum
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if constexpr (SEL == 0) ask_query(b);
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[b][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        m[b] = -INFINITY;
        lsum[b] = 0.f;
    }

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
    // Query tiles first .. first + count - 1 of the wave against one tile of 32 keys in LDS; every operand is read once for all of
    // them.  alone: the tile is in the wave's own place.  `k_read` is called when LDS holds nothing more of K's rows that is wanted,
    // `v_wanted` before V's are read, and `v_read` when all of them have been.
    auto tile = [&](auto first, auto count, auto alone, const char *kt, const char *vt, int c0, int c1, float w0, float w1, auto k_read,
                    auto v_wanted, auto v_read) {
        constexpr int b0 = decltype(first)::value, n = decltype(count)::value;
        constexpr bool E = decltype(alone)::value;
        f32x4 s[n][2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 kop = ld_bf16x8(kt + h * HALF + o.row[ks]);
#pragma unroll
                for (int b = 0; b < n; ++b) s[b][h] = mfma16(kop, qop[b0 + b][ks], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[b][h]);
            }
        k_read();
        bf16x8 p[n];
        p[0] = probs(first, s[0][0], s[0][1], c0, c1, w0, w1);
        if constexpr (n > 1) p[n - 1] = probs(B1{}, s[n - 1][0], s[n - 1][1], c0, c1, w0, w1);
        v_wanted();
        bf16x8 vtr[E ? NT : 1];
        if constexpr (E) {
#pragma unroll
            for (int x = 0; x < NT; ++x) vtr[x] = lds_tr_pair(vt + o.tr[x], vt + HALF + o.tr[x]);
            v_read();
        }
#pragma unroll
        for (int x = 0; x < NT; ++x) {
            const bf16x8 v = E ? vtr[E ? x : 0] : lds_tr_pair(vt + o.tr[x], vt + HALF + o.tr[x]);
#pragma unroll
            for (int b = 0; b < n; ++b) acc[b0 + b][x] = mfma16(v, p[b], acc[b0 + b][x]);
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
    // The compiler counts the loads that it knows of: unless Q's rows are waited for here, it waits for them in front of every tile's first
    // products, and with them for all tiles on their way.
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qop[b][s]));

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
        // All tiles but the last, in a loop that is unrolled over the ring: the places are known, no half is short.
        auto turn = [&](int u, auto at) {
            constexpr int x = decltype(at)::value;
            // tile u is there, and tile u - 1, whose place tile u + 3 takes, has been read by every wave
            if (u + 2 < ntile) vm_wait_barrier<2 * CPW>();
            else vm_wait_barrier<CPW>();
            if (u + RING - 1 < ntile) issue(u + RING - 1, (x + RING - 1) % RING);
            if (x == 0 && ((2 * u) & 63) == 0) w_now = w_next;        // (a chunk of 64 blocks begins at place 0)
            const char *kt = lds + x * (2 * TILE);
            tile(B0{}, All{}, Shared{}, kt, kt + TILE, 16, 16, weight(2 * u), weight(2 * u + 1), nothing, nothing, nothing);
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
        // an absent half: probabilities 0
        tile(B0{}, All{}, Shared{}, kt, kt + TILE, c0, c1, weight(2 * u), 2 * u + 1 < nbc ? weight(2 * u + 1) : -INFINITY, nothing, nothing, nothing);
    } else {
        begin_b();
    }

    // ------------------------------------------------------------------ phase B: level 0
    if constexpr (GW > 1) {
        // Blocks of 32 or 64 tokens: the B queries of a block use one level-0 list, whose tiles the GW waves that hold them bring in
        // together, double-buffered.  A list is whole blocks of B >= 32 tokens: no half of a tile is ever absent.
        for (int u = 0; 2 * u < nb0; ++u) {
            vm_wait_barrier<0>();
            if (2 * u + 2 < nb0) issue_b(u + 1);
            const char *kt = lds + (u & 1 ? place1 : place0);
            tile(B0{}, All{}, Shared{}, kt, kt + TILE, 16, 16, 0.f, 0.f, nothing, nothing, nothing);
        }
    } else {
        // Every wave alone: the tiles of its query tiles (GW = 1: of all of them at once) form one stream.  The next tile's K rows are asked
        // for as soon as this tile's have been read, its V rows likewise: K's fly during the exponentials and the second product, V's
        // during the second product, the next tile's first one and its exponentials.
        const char *my = lds + place0;
        auto walk = [&](auto first, auto count, bool end) {
            const int l0 = LL * decltype(first)::value;
            for (int j0 = 0; j0 < nb0; j0 += 2) {
                const bool here = j0 + 2 < nb0, more = here || !end;
                const int nl = here ? l0 : l0 + LL, nj = here ? j0 + 2 : 0;
                vm_wait<2 * CPH>();
                // level-0 blocks are always full; an absent second half has weight 0
                tile(first, count, Alone{}, my, my + TILE, 16, 16, 0.f, j0 + 1 < nb0 ? 0.f : -INFINITY,
                     [&]() { if (more) load_rows(0, nl, nj, 0); },
                     [&]() { if (more) vm_wait<2 * CPH>(); else vm_wait<0>(); },
                     [&]() { if (more) load_rows(to_v0, nl, nj, TILE); });
            }
        };
        if constexpr (GW == 1) walk(B0{}, All{}, true);
        else {
            walk(B0{}, One{}, NB == 1);
            if constexpr (NB > 1) walk(B1{}, One{}, true);
        }
    }

    // ------------------------------------------------------------------ epilogue
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const float l = rows_sum(lsum[b]);
        const float inv = 1.f / l;
        const int64_t row = bh * N + tile_of(b) * 16 + i16;
        auto out = [&](int n) { return u32x2{pack_bf16(acc[b][n][0] * inv, acc[b][n][1] * inv), pack_bf16(acc[b][n][2] * inv, acc[b][n][3] * inv)}; };
#pragma unroll
        for (int n = 0; n < NT; n += 2) store_pair(O + row * D, n, g, out(n), out(n + 1));
        if (g == 0) LSE[row] = (m[b] + __builtin_amdgcn_logf(l)) * kLn2;
    }
}

static unsigned attn_groups(const Plan &p) { return (unsigned)p.bh * (unsigned)(p.N / 128); }
// Two query tiles per wave read every coarse operand from LDS once for both: half the LDS reads, which bound d = 128
// (16 heads x 262144 tokens, K = 16: 1977 -> 1512 us; 4096 tokens: 33.9 -> 30.1).  At d = 64 they pay from four
// workgroups per CU on (131072 queries: 33.6 -> 30.4 us); with fewer, eight waves with a tile each hide more of the
// latency (65536 queries: 18.2 against 18.9, 32768: 12.6 against 14.1).  Both tiles' level-0 lists have to fit one register.
static bool two_tiles(const Plan &p) { return p.B > 16 || (p.Kl[0] <= 32 && (p.d == 128 || attn_groups(p) >= 1024)); }

// Are the lists of level 0 (1), of level 1 too (2), selected by the attention's own launch?
int attn_selects(const Plan &p) {
    if (!p.fast || p.desc.kernel_path != 0 || p.B != 16 || p.d != 64 || p.L < 2 || p.N % 256 != 0) return 0;
    if (p.Kl[0] > kSelPicks || p.Kl[1] > kSelPicks || two_tiles(p)) return 0;
    return p.L > 2 ? 1 : p.n[2] <= 64 ? 2 : 0;
}

hipError_t launch_attn_fwd_shared(const Plan &p, const LevelTable &t, const void *Q, void *O, float *LSE, const AttnSelect *select, hipStream_t s) {
    const FastDiv groups(p.N / 128);
    const unsigned wgs = attn_groups(p);
    const ListArgs a = make_list_args(t);
    const uint16_t *q = (const uint16_t *)Q;
    uint16_t *o = (uint16_t *)O;
    const int ls = p.lb - 4;
    SelectHere sel = {};
    if (select) {
        const char *w = static_cast<const char *>(select->workspace);
        sel = {w + p.pyr_off[0][1], w + p.pyr_off[1][1], w + p.pyr_off[0][2], w + p.pyr_off[1][2], select->I0, select->I1,
               (int32_t)p.n[1], (int32_t)p.n[2], p.Kl[0], p.Kl[1]};
    }
    auto kernel = [&](auto d, auto nb, auto gw, auto how) {
        constexpr int NB = decltype(nb)::value, NW = 8 / NB;
        attn_fwd_shared_kernel<decltype(d)::value, NB, NW, decltype(gw)::value, decltype(how)::value><<<wgs, 64 * NW, 0, s>>>(a, q, o, LSE, p.N, groups, sel);
    };
    auto go = [&](auto d, auto nb, auto gw) { kernel(d, nb, gw, std::integral_constant<int, 0>{}); };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using D64 = std::integral_constant<int, 64>;
    using D128 = std::integral_constant<int, 128>;
    if (select) {
        if (attn_selects(p) == 1) kernel(D64{}, I1{}, I0{}, I1{});
        else kernel(D64{}, I1{}, I0{}, I2{});
    } else if (ls == 1) {
        if (p.d == 64) go(D64{}, I2{}, I1{});
        else go(D128{}, I2{}, I1{});
    } else if (ls == 2) {
        if (p.d == 64) go(D64{}, I2{}, I2{});
        else go(D128{}, I2{}, I2{});
    } else if (p.d == 64) {
        if (two_tiles(p)) go(D64{}, I2{}, I0{});
        else go(D64{}, I1{}, I0{});
    } else {
        if (two_tiles(p)) go(D128{}, I2{}, I0{});
        else go(D128{}, I1{}, I0{});
    }
    return hipGetLastError();
}

}  // namespace llsa
