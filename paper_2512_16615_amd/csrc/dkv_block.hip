// dK, dV of a key block of several 16-key tiles on bf16 MFMA, Sec. 4.3: blocks of 32 and 64 keys at every level with lists, and
// wide dense levels (any block size), four tiles at a time.
//
// All tiles of a block use one query list, so a tile of 32 queries (Q and dO rows, LSE, D) is brought into LDS once for the SW waves that
// together hold the block, each a share of the rows, and every wave runs it against its own TPW key tiles, whose K / V operands and sums stay
// in registers.  The 4 / SW groups of a workgroup take the list's tiles in turn and are added up through LDS in order.  A block of level 0 is
// finished here (the parent token's share added, one rounding); levels >= 1 write fp32 sums, one slab per share of the list, for
// dkv_reduce_kernel.
// Rows go straight into LDS, into a ring of places that the loop is unrolled over: a place is asked for again as soon as the barrier says
// that every wave is done with it.  Before, two tiles were in flight in registers and stored to LDS: those registers are waves now, and the
// stores took as long as a third of the reads.  us (profiled, before -> now): 16 heads x 65536 tokens in blocks of 64, K = 8, level 1
// 392 -> 325, level 0 459 -> 412; in blocks of 32 306 -> 260 and 450 -> 357; 8 heads, d = 128, blocks of 64, K = 4 280 -> 192 and 421 -> 315.
// (With the place worked out at run time, which is an addition for every LDS read, 412 and 436.)
// Bound, by counters at 16 x 65536 in blocks of 64 (share of a SIMD's cycles; 25 % would be all of the LDS that four share): level 1 issue, vector
// ALU 45 % and MFMA 43 %, LDS 10; level 0 waits for gathered rows, 47 % of a wave's life, vector ALU 46 %, MFMA 33, scalar 20, LDS 14 (16 KB read per
// 32 x 16 score tile at TPW = 1, half of that at 2).  (224 us each at the rate of a large matrix product.)  TPW = 1 at level 1 and 2 at
// level 0 each take about 1.1 times as long.
#include <type_traits>

#include "dkv_common.h"

namespace llsa {

// Waves a SIMD: what the registers have room for.  Tiles of a group in LDS, the one in hand and those on their way: three where that costs no
// wave and the lists are long (level 1 in blocks of 64: 325 us, with four 350; d = 128 and three waves 192, with two waves and four tiles 216).
// Steps with two and with three: level 0 in blocks of 64 at d = 64 1704 and 1717 us; with two everywhere 0.4 to 1.5 % slower than as it is.
// Level 0 in blocks of 32: two tiles and four waves 357 us, three and three 402.
template <int D, int TPW, int SW> struct BlockShape {
    static constexpr int WAVES = D == 64 ? (TPW == 2 ? 3 : SW == 4 ? 5 : 4) : SW == 4 ? 3 : 2;
    static constexpr int RING = (D == 64 ? TPW == 2 : SW == 4) ? 3 : 2;
};

template <int D, int TPW, int SW>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(BlockShape<D, TPW, SW>::WAVES))) dkv_block_kernel(DkvArgs a) {
    using S = GShape<D>;
    constexpr int TPB = TPW * SW, P = 4 / SW;              // key tiles of the block; groups of waves
    constexpr int RING = BlockShape<D, TPW, SW>::RING;     // tiles of a group in LDS: one in use, one or more on their way
    constexpr int HALF = 32 * S::ROWB, BUF = 2 * HALF;     // a tile: Q rows | dO rows
    static_assert(RING == 2 || RING == 3, "");
    static_assert(SW == 2 || SW == 4, "the waves of a group meet at the workgroup's barrier; each brings rows of Q or of dO");
    constexpr int SHARE = BUF / SW, LOADS = SHARE / 1024;  // a wave's part of a tile
    constexpr int SLOTS = 2 * S::NT * TPW;                 // f32x4 sums per lane
    constexpr int RED = (P - 1) * SW * SLOTS * 64 * 16;
    __shared__ __attribute__((aligned(16))) char lds[P * RING * BUF > RED ? P * RING * BUF : RED];
    __shared__ __attribute__((aligned(16))) float st_sh[P][RING][64];   // LSE [32] | D [32]

    const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave / SW, wig = wave % SW;
    // order: head, share, key block; where lists are shared out, one XCD after the other
    const unsigned wgid = a.splits > 1 ? xcd_contiguous32(blockIdx.x, gridDim.x) : blockIdx.x;
    const unsigned hs = a.blocks(wgid), blk = wgid - hs * a.blocks.d, bh = a.split_of(hs), split = hs - bh * (unsigned)a.splits;
    const int ntile = (int)((a.n_l + 15) >> 4);
    const TileOffsets<D> o = tile_offsets<D>(lane);

    BlockAcc<D> key[TPW];
#pragma unroll
    for (int x = 0; x < TPW; ++x) {
        const int j = (int)blk * TPB + wig * TPW + x;      // key tile (past the end of a dense level: its last one, not stored)
        const int64_t row = (int64_t)bh * a.n_l + 16 * min(j, ntile - 1);
        const int cnt = (int)min((int64_t)16, a.n_l - 16 * min(j, ntile - 1));
        key[x].load(reinterpret_cast<const char *>(a.Kl + row * D), reinterpret_cast<const char *>(a.Vl + row * D), cnt, a.bias2, lane);
        key[x].clear();
    }
    const int32_t *lst = nullptr;
    unsigned groups = (unsigned)(a.N >> 4);                // 16-query groups of the list
    if (!a.dense) {
        const int32_t *Crow = a.C + bh * (a.rows + 1) + blk;
        const int32_t beg = Crow[0];
        groups = (unsigned)(Crow[1] - beg) << a.span_shift;
        lst = a.Iq + bh * a.rows * a.Kl_cnt + beg;
    }
    // tiles of 32 consecutive queries: a listed block has at least two groups, and N is a multiple of 64, so no tile is short
    const unsigned tiles = (groups + 1) >> 1, entries = groups >> a.span_shift;
    const unsigned t_beg = (unsigned)((uint64_t)tiles * split / a.splits), t_end = (unsigned)((uint64_t)tiles * (split + 1) / a.splits);
    const unsigned span_mask = (1u << a.span_shift) - 1;

    int ecache = 0;                                        // lane e: list entry 64 * echunk + e
    unsigned echunk = ~0u;
    const RowSource<D> src(lane);
    const unsigned row_in = (unsigned)(wig % (SW / 2)) * (SHARE / S::ROWB);   // the wave's rows of the tile: of Q, in the group's second half of dO
    const uint64_t rows = reinterpret_cast<uint64_t>(wig < SW / 2 ? a.Q : a.dO) + ((uint64_t)bh * a.N + row_in) * S::ROWB;
    const float *stats = ((lane & 32) ? a.Dsum : a.LSE) + (int64_t)bh * a.N + (lane & 31);
    const unsigned ring = lds_address(lds) + (unsigned)grp * RING * BUF + (unsigned)wig * SHARE, st_ring = lds_address(st_sh[grp]);
    auto load = [&](unsigned t, unsigned b) {
        unsigned q0 = 32 * t;
        if (!a.dense) {
            const unsigned e = (2 * t) >> a.span_shift;
            if ((e >> 6) != echunk) {
                echunk = e >> 6;
                ecache = 64 * echunk + lane < entries ? lst[64 * echunk + lane] : 0;
                asm volatile("" : "+v"(ecache));           // waited for here: at its use the compiler would wait for every tile on its way, every time
            }
            q0 = 16 * (((unsigned)__builtin_amdgcn_readlane(ecache, (int)(e & 63)) << a.span_shift) + ((2 * t) & span_mask));
        }
        const uint64_t from = rows + (uint64_t)q0 * S::ROWB;
        constexpr int N = LOADS < 4 ? LOADS : 4;
#pragma unroll
        for (int r = 0; r < LOADS; r += N) load_lds<N>(from + 1024 * r, src.v0, src.v1, ring + b * BUF + 1024 * r);
        if (wig == 0) load_lds_dword(stats + q0, st_ring + 256 * b);
    };
    auto wait = [&](auto ahead) {                          // all but the group's last `ahead` tiles have come, in every wave
        constexpr int n = decltype(ahead)::value;
        if (wig == 0) vm_wait_barrier<n * (LOADS + 1)>();
        else vm_wait_barrier<n * LOADS>();
    };
    const unsigned turns = (t_end - t_beg + P - 1) / P;    // the same number for every wave
    unsigned t = t_beg + grp;
#pragma unroll
    for (int x = 0; x < TPW; ++x)                          // the keys have come before the first tile is asked for (see ecache)
#pragma unroll
        for (int ks = 0; ks < S::KS; ++ks) asm volatile("" : "+v"(key[x].kop[ks]), "+v"(key[x].vop[ks]));
#pragma unroll
    for (int b = 0; b < RING - 1; ++b)
        if (t + b * P < t_end) load(t + b * P, b);
    auto turn = [&](auto place) {
        constexpr int cur = decltype(place)::value;
        if (RING == 3 && t + P < t_end) wait(std::integral_constant<int, 1>());
        else wait(std::integral_constant<int, 0>());
        // no wave reads the tile before this one any more: its place is the next one's
        if (t + (RING - 1) * P < t_end) load(t + (RING - 1) * P, cur == 0 ? RING - 1 : cur - 1);
        if (t < t_end) {
            const char *buf = lds + (grp * RING + cur) * BUF;
            group_tile<D, TPW, true>(buf, buf + HALF, st_sh[grp][cur], st_sh[grp][cur] + 32, 0, o, key, a.sc2, g);
        }
        t += P;
    };
    for (unsigned i = 0; i < turns; i += RING) {
        turn(std::integral_constant<int, 0>());
        if (i + 1 < turns) turn(std::integral_constant<int, 1>());
        if (RING == 3 && i + 2 < turns) turn(std::integral_constant<int, RING - 1>());
    }

    if constexpr (P > 1) {                                 // the groups' sums, in group order
        float *red = reinterpret_cast<float *>(lds);
        __syncthreads();
        if (grp > 0) {
            float *dst = red + (((grp - 1) * SW + wig) * SLOTS * 64 + lane) * 4;
#pragma unroll
            for (int x = 0; x < TPW; ++x)
#pragma unroll
                for (int n = 0; n < S::NT; ++n) {
                    *reinterpret_cast<f32x4 *>(dst + (2 * S::NT * x + n) * 256) = key[x].accK[n];
                    *reinterpret_cast<f32x4 *>(dst + (2 * S::NT * x + S::NT + n) * 256) = key[x].accV[n];
                }
        }
        __syncthreads();
        if (grp > 0) return;
#pragma unroll
        for (int p = 1; p < P; ++p) {
            const float *src = red + (((p - 1) * SW + wig) * SLOTS * 64 + lane) * 4;
#pragma unroll
            for (int x = 0; x < TPW; ++x)
#pragma unroll
                for (int n = 0; n < S::NT; ++n) {
                    key[x].accK[n] += *reinterpret_cast<const f32x4 *>(src + (2 * S::NT * x + n) * 256);
                    key[x].accV[n] += *reinterpret_cast<const f32x4 *>(src + (2 * S::NT * x + S::NT + n) * 256);
                }
        }
    }
    const float wV = __builtin_amdgcn_exp2f(a.bias2), wK = wV * a.scale;   // the level's weight, left out of the tiles' P
#pragma unroll
    for (int x = 0; x < TPW; ++x) {
        const int j = (int)blk * TPB + wig * TPW + x;
        if (j >= ntile || 16 * j + i16 >= a.n_l) continue;
        const int64_t row = ((int64_t)bh * a.n_l + 16 * j + i16) * D;
        if (a.dK) {                                        // level 0: whole tiles, all lanes are here
            auto value = [&](f32x4 sum, const float *par, int n) {
                if (par) sum += *reinterpret_cast<const f32x4 *>(par + ((int64_t)bh * a.blocks.d + blk) * D + n * 16 + 4 * g) * a.inv_B;
                return u32x2{pack_bf16(sum[0], sum[1]), pack_bf16(sum[2], sum[3])};
            };
#pragma unroll
            for (int n = 0; n < S::NT; n += 2) {
                store_pair(a.dK + row, n, g, value(key[x].accK[n] * wK, a.parK, n), value(key[x].accK[n + 1] * wK, a.parK, n + 1));
                store_pair(a.dV + row, n, g, value(key[x].accV[n] * wV, a.parV, n), value(key[x].accV[n + 1] * wV, a.parV, n + 1));
            }
        } else {
#pragma unroll
            for (int n = 0; n < S::NT; ++n) {
                *reinterpret_cast<f32x4 *>(a.partK + split * a.slab + row + n * 16 + 4 * g) = key[x].accK[n] * wK;
                *reinterpret_cast<f32x4 *>(a.partV + split * a.slab + row + n * 16 + 4 * g) = key[x].accV[n] * wV;
            }
        }
    }
}

// Key tiles of a block of level l, or 0 if the level is left to the one-tile kernels: lists of 16-key blocks, and dense levels
// of one or two tiles, where a workgroup's four waves would mostly hold nothing.
int dkv_block_tiles(const Plan &p, int l) {
    if (l == p.L) return p.n[l] > 32 ? 4 : 0;
    return p.B / 16 > 1 ? p.B / 16 : 0;
}

int dkv_block_splits(const Plan &p, int l) {
    const int tpb = dkv_block_tiles(p, l);
    const int64_t blocks = p.bh * (((p.n[l] + 15) / 16 + tpb - 1) / tpb);
    const int64_t tiles = (l == p.L ? p.N : (int64_t)p.Kl[l] * (p.N / p.n[l + 1])) / 32;   // average list
    int64_t s = (2048 + blocks - 1) / blocks;              // eight workgroups per CU, each with at least 8 tiles
    if (s > tiles / 8) s = tiles / 8;
    if (s < 1 || l == 0) s = 1;
    if (s > 64) s = 64;
    return (int)s;
}

hipError_t launch_dkv_block(const Plan &p, int l, DkvArgs &a, hipStream_t s) {
    const int tpb = dkv_block_tiles(p, l);
    a.blocks = FastDiv(((p.n[l] + 15) / 16 + tpb - 1) / tpb);
    a.split_of = FastDiv(a.splits);
    const unsigned grid = (unsigned)p.bh * a.blocks.d * (unsigned)a.splits;
    if (p.d == 64) {
        // coarse levels (long lists, evenly shared out) are bound by LDS reads, level 0 by waiting for its gathered rows
        if (tpb == 4 && l > 0) dkv_block_kernel<64, 2, 2><<<grid, 256, 0, s>>>(a);
        else if (tpb == 4) dkv_block_kernel<64, 1, 4><<<grid, 256, 0, s>>>(a);
        else dkv_block_kernel<64, 1, 2><<<grid, 256, 0, s>>>(a);
    } else {
        if (tpb == 4) dkv_block_kernel<128, 1, 4><<<grid, 256, 0, s>>>(a);
        else dkv_block_kernel<128, 1, 2><<<grid, 256, 0, s>>>(a);
    }
    return hipGetLastError();
}

}  // namespace llsa
