// dK, dV of a key block of several 16-key tiles on bf16 MFMA, Sec. 4.3: blocks of 32 and 64 keys at every level with lists, and
// wide dense levels (any block size), four tiles at a time.
//
// All tiles of a block use one query list, so its waves stage each tile of 32 queries (Q and dO rows, LSE, D) once in LDS,
// double-buffered, and every wave runs it against its own TPW key tiles, whose K / V operands and sums stay in registers.
// SW waves share a staged tile and together hold the block; the 4 / SW groups of a workgroup take the list's tiles in
// turn and are added up through LDS in order.  Two tiles per group are in flight in registers.  A block of level 0 is finished here (the parent token's share added, one
// rounding); levels >= 1 write fp32 sums, one slab per share of the list, for dkv_reduce_kernel.
// Bound: LDS reads (16 KB per 32 x 16 score tile at TPW = 1, half of that at 2) and the latency of the gathered rows; 16 heads
// x 65536 tokens in blocks of 64, K = 8: level 1 340 us, level 0 423 us (profiled; 224 us each at the rate of a large matrix product).  Relative to that, when written:
// level 1 with TPW = 1 1.12 times as long, level 0 with TPW = 2 1.11 times; with one tile in flight 1.34 and 1.23; the kernels
// of dkv_mfma.hip, which these replace here and which staged every query tile once per key tile, 1.53 and 1.54.  (Blocks of 32 at
// d = 64: two tiles a wave would be a wave alone with 255 registers and spills.)
#include <type_traits>

#include "dkv_common.h"

namespace llsa {

template <int D, int TPW, int SW>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 && TPW == 1 ? 3 : 2))) dkv_block_kernel(DkvArgs a) {
    using S = GShape<D>;
    constexpr int TPB = TPW * SW, P = 4 / SW;              // key tiles of the block; groups of waves
    constexpr int HALF = 32 * S::ROWB, BUF = 2 * HALF;     // one staged tile: Q rows | dO rows
    static_assert(SW > 1, "the waves of a group meet at the workgroup's barrier");
    constexpr int R = 2 * 32 * S::CH / (64 * SW);          // 16-byte chunks per thread
    constexpr int SLOTS = 2 * S::NT * TPW;                 // f32x4 sums per lane
    constexpr int RED = (P - 1) * SW * SLOTS * 64 * 16;
    __shared__ __attribute__((aligned(16))) char lds[P * 2 * BUF > RED ? P * 2 * BUF : RED];
    __shared__ __attribute__((aligned(16))) float st_sh[P][2][64];   // -LSE log2(e) [32] | -D [32]

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
    // tiles of 32 consecutive queries: a listed block has at least two groups, so only a dense level's last tile can be short
    const unsigned tiles = (groups + 1) >> 1, entries = groups >> a.span_shift;
    const unsigned t_beg = (unsigned)((uint64_t)tiles * split / a.splits), t_end = (unsigned)((uint64_t)tiles * (split + 1) / a.splits);
    const unsigned span_mask = (1u << a.span_shift) - 1;

    int ecache = 0;                                        // lane e: list entry 64 * echunk + e
    unsigned echunk = ~0u;
    struct Staged { u32x4 r[R]; float stat; };
    Staged even, odd;                                      // two tiles are in flight: one is not enough for the latency of L2 misses
    auto load = [&](Staged &x, unsigned t) {
        unsigned q0 = 32 * t;
        if (!a.dense) {
            const unsigned e = (2 * t) >> a.span_shift;
            if ((e >> 6) != echunk) {
                echunk = e >> 6;
                ecache = 64 * echunk + lane < entries ? lst[64 * echunk + lane] : 0;
            }
            q0 = 16 * (((unsigned)__builtin_amdgcn_readlane(ecache, (int)(e & 63)) << a.span_shift) + ((2 * t) & span_mask));
        }
        const int64_t row0 = (int64_t)bh * a.N + q0;
        const int last = (int)min((int64_t)32, a.N - q0) - 1;           // rows past the head's end re-read its last one
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int c = 64 * (wig + SW * r) + lane;      // chunk of [Q rows | dO rows]; one of the two for the whole wave
            const int row = (c % (32 * S::CH)) / S::CH;
            const uint16_t *src = 64 * (wig + SW * r) >= 32 * S::CH ? a.dO : a.Q;
            x.r[r] = *reinterpret_cast<const u32x4 *>(src + (row0 + min(row, last)) * D + (c % S::CH) * 8);
        }
        {
            const int q = lane & 31;
            const float v = (lane & 32 ? a.Dsum : a.LSE)[row0 + min(q, last)];
            x.stat = lane & 32 ? -v : q > last ? -INFINITY : v * -kLog2e;   // an absent query: P = 0
        }
    };
    auto store = [&](const Staged &x, int b) {
        char *buf = lds + (grp * 2 + b) * BUF;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int c = 64 * (wig + SW * r) + lane, row = (c % (32 * S::CH)) / S::CH;
            *reinterpret_cast<u32x4 *>(buf + (64 * (wig + SW * r) >= 32 * S::CH ? HALF : 0) + swz<D>(row, c % S::CH)) = x.r[r];
        }
        if (wig == 0) st_sh[grp][b][lane] = x.stat;
    };
    const unsigned turns = (t_end - t_beg + P - 1) / P;    // the same number for every wave, rounded up to pairs
    unsigned t = t_beg + grp;
    auto turn = [&](Staged &x, int b) {
        const bool have = t < t_end;
        if (have) store(x, b);
        __syncthreads();
        load(x, min(t + 2 * P, t_end - 1));                // flies during this turn's math and the next one's
        if (have) {
            const char *buf = lds + (grp * 2 + b) * BUF;
            group_tile<D, TPW>(buf, buf + HALF, st_sh[grp][b], st_sh[grp][b] + 32, 0, o, key, a.sc2, g);
        }
        t += P;
    };
    // (loads behind a condition would make every wait one for all loads: past the end they repeat the last tile)
    if (turns > 0) {
        load(even, min(t, t_end - 1));
        load(odd, min(t + P, t_end - 1));
    }
    for (unsigned i = 0; i < turns; i += 2) {
        turn(even, 0);
        turn(odd, 1);
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
        const int64_t row = ((int64_t)bh * a.n_l + 16 * j + i16) * D + 4 * g;
#pragma unroll
        for (int n = 0; n < S::NT; ++n) {
            f32x4 k = key[x].accK[n] * wK, v = key[x].accV[n] * wV;
            if (a.dK) {                                    // level 0
                if (a.parK) {
                    const int64_t par = ((int64_t)bh * a.blocks.d + blk) * D + n * 16 + 4 * g;
                    k += *reinterpret_cast<const f32x4 *>(a.parK + par) * a.inv_B;
                    v += *reinterpret_cast<const f32x4 *>(a.parV + par) * a.inv_B;
                }
                *reinterpret_cast<u32x2 *>(a.dK + row + n * 16) = u32x2{pack_bf16(k[0], k[1]), pack_bf16(k[2], k[3])};
                *reinterpret_cast<u32x2 *>(a.dV + row + n * 16) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
            } else {
                *reinterpret_cast<f32x4 *>(a.partK + split * a.slab + row + n * 16) = k;
                *reinterpret_cast<f32x4 *>(a.partV + split * a.slab + row + n * 16) = v;
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
