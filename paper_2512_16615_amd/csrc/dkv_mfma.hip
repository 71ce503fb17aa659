// dK, dV of the gathered-list attention on bf16 MFMA (d = 64 or 128), Sec. 4.3: key-major over the transposed lists of Alg. 2
// where blocks have 16 keys, or over every query at a dense level of at most 32 tokens (any block size; dkv_block.hip has the
// lists of larger blocks and the wider dense levels), with no mask and no floating-point atomics.
// With P = exp(z - LSE), dP = dO V^T, dS = P o (dP - D):  dK = scale dS^T Q,  dV = P^T dO.
//
// The unit of work is a tile of 16 level-l keys, a listed block or a piece of a dense level.  The
// queries that attend to it are the fine queries under the level-l query blocks listed for its block, walked in
// groups of 16 consecutive queries; a tile of the loop is two groups.  Per tile a wave
// computes
//   S = Q K^T, dP = dO V^T   (lane: 4 queries x 1 key)  ->  P, dS  ->
//   dV^T += dO^T P,  dK^T += Q^T dS   (A = the Q / dO tile read transposed from LDS, B = P / dS).
// Two kernels:
//   dkv_coarse_kernel (levels >= 1): one workgroup of 4 waves per (key block, split); the tiles of its
//     share are dealt round-robin to the waves, whose accumulators are summed through LDS in wave order;
//     fp32 partial sums go to one slab per split and a second kernel adds the slabs in split order (and
//     the share of the level above, the adjoint of mean pooling).
//   dkv_fine_kernel (level 0): lists are short (K on average) and very different, from none to hundreds, so single waves take them from a
//     row of tiles (fine_tiles.h), several short lists or a piece of a long one each; the epilogue adds the parent token's share and
//     rounds once to bf16.
// Every sum has a fixed order, so results do not depend on timing.
#include "dkv_common.h"
#include "fine_tiles.h"

namespace llsa {

template <int D> struct DkvShape {
    static constexpr int KS = D / 32, NT = D / 16, HALF = 32 * D, TILE = 2 * HALF;   // bytes of 16 and of 32 rows
    static constexpr int CPH = HALF / 1024;                 // load_lds steps of 16 rows
    static constexpr int WAVE = 2 * TILE + 256;             // LDS of a wave: Q rows | dO rows | LSE [32], D [32]
};

// Tiles t_first, t_first + t_step, ... < t_end of one key block's query list, accumulated into accK / accV.
// lst: the block's listed query-block rows (null when dense); groups: 16-query groups in the list.
// Rows go from memory straight into the wave's LDS.  Every operand of a tile is read before its exponentials, so that the next
// tile's rows, for which there is only this one place, fly during the rest.  Measured when level 0 walked its lists in this loop too: through
// registers 317 us at 16 x 65536 tokens, K = 8, this way 309 (a second place in LDS was worth a wave less per SIMD).
template <int D>
__device__ __forceinline__ void dkv_tile_loop(const DkvArgs &a, int64_t bh, const int32_t *lst, int64_t groups,
                                              int64_t t_first, int64_t t_step, int64_t t_end,
                                              const bf16x8 (&kop)[D / 32], const bf16x8 (&vop)[D / 32],
                                              f32x4 (&accK)[D / 16], f32x4 (&accV)[D / 16], char *qt, int lane) {
    using S = DkvShape<D>;
    const int i16 = lane & 15, g = lane >> 4;
    const int64_t span_mask = ((int64_t)1 << a.span_shift) - 1;
    const int64_t entries = groups >> a.span_shift;
    const TileOffsets<D> o = tile_offsets<D>(lane);
    const RowSource<D> src(lane);
    char *gt = qt + S::TILE;
    float *st = reinterpret_cast<float *>(gt + S::TILE);
    const unsigned dst = lds_address(qt);

    // the list entries, 64 at a time in one register (lane e: entry 64 * chunk + e)
    int ecache = 0;
    int64_t echunk = -1;
    auto entry = [&](int64_t e) -> int64_t {
        if ((e >> 6) != echunk) {
            echunk = e >> 6;
            const int64_t idx = echunk * 64 + lane;
            ecache = idx < entries ? lst[idx] : 0;
        }
        return __builtin_amdgcn_readlane(ecache, (int)(e & 63));
    };

    float stat = 0.f;                                       // lane x: LSE (x < 32) or D (x >= 32) of tile query x % 32
    int valid1 = 0;                                         // does the tile on its way have its second group?
    auto load_tile = [&](int64_t tile) {
        valid1 = 2 * tile + 1 < groups;
        int64_t row0[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t gi = (h == 0 || valid1) ? 2 * tile + h : 2 * tile;   // an absent group re-reads the first
            const int64_t q0 = a.dense ? gi * 16 : ((entry(gi >> a.span_shift) << a.span_shift) + (gi & span_mask)) * 16;
            row0[h] = bh * a.N + q0;
        }
        stat = ((lane & 32) ? a.Dsum : a.LSE)[((lane & 16) ? row0[1] : row0[0]) + i16];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            load_lds<S::CPH>(reinterpret_cast<uint64_t>(a.Q + row0[h] * D), src.v0, src.v1, dst + h * S::HALF);
            load_lds<S::CPH>(reinterpret_cast<uint64_t>(a.dO + row0[h] * D), src.v0, src.v1, dst + S::TILE + h * S::HALF);
        }
    };

    int64_t tile = t_first;
    if (tile < t_end) load_tile(tile);
    while (tile < t_end) {
        st[lane] = stat;                                    // one wave's LDS operations stay in order
        vm_wait<0>();
        f32x4 s[2], dp[2], l2[2], dl[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            s[h] = f32x4{0.f, 0.f, 0.f, 0.f};
            dp[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < S::KS; ++ks) {
                s[h] = mfma16(ld_bf16x8(qt + h * S::HALF + o.row[ks]), kop[ks], s[h]);
                dp[h] = mfma16(ld_bf16x8(gt + h * S::HALF + o.row[ks]), vop[ks], dp[h]);
            }
        }
        bf16x8 tg[S::NT], tq[S::NT];
#pragma unroll
        for (int n = 0; n < S::NT; ++n) {
            tg[n] = lds_tr_pair(gt + o.tr[n], gt + S::HALF + o.tr[n]);
            tq[n] = lds_tr_pair(qt + o.tr[n], qt + S::HALF + o.tr[n]);
        }
        const int v1 = valid1;
        const int64_t next = tile + t_step;
        if (next < t_end) load_tile(next);

#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // this lane's 4 queries: rows 4g .. 4g+3 (the next tile's are written at the head of the loop)
            l2[h] = *reinterpret_cast<const f32x4 *>(st + 16 * h + 4 * g);
            dl[h] = *reinterpret_cast<const f32x4 *>(st + 32 + 16 * h + 4 * g);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float p = __builtin_amdgcn_exp2f(fmaf(s[h][r], a.sc2, fmaf(l2[h][r], -kLog2e, a.bias2)));
                s[h][r] = p;
                dp[h][r] = p * (dp[h][r] - dl[h][r]);
            }
        }
        if (!v1) {                                          // the list ends with a single group
            s[1] = f32x4{0.f, 0.f, 0.f, 0.f};
            dp[1] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        const bf16x8 pop = pack8(s[0], s[1]), dsop = pack8(dp[0], dp[1]);
#pragma unroll
        for (int n = 0; n < S::NT; ++n) {
            accV[n] = mfma16(tg[n], pop, accV[n]);
            accK[n] = mfma16(tq[n], dsop, accK[n]);
        }
        tile = next;
    }
}

// Sum of the four waves' accumulators in wave order through LDS; wave w ends up owning slots w, w + 4, ...
// (slot = which * NT + n, which: 0 = dK, 1 = dV) and hands each finished slot to `emit(slot, sum)`.
template <int D, class Emit>
__device__ __forceinline__ void dkv_reduce_waves(float *red, int wave, int lane, const f32x4 (&accK)[D / 16],
                                                 const f32x4 (&accV)[D / 16], Emit emit) {
    constexpr int NT = D / 16, SLOTS = 2 * NT;
    __syncthreads();                                        // everyone is done with the tile buffers
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        *reinterpret_cast<f32x4 *>(red + ((wave * SLOTS + n) * 64 + lane) * 4) = accK[n];
        *reinterpret_cast<f32x4 *>(red + ((wave * SLOTS + NT + n) * 64 + lane) * 4) = accV[n];
    }
    __syncthreads();
    for (int slot = wave; slot < SLOTS; slot += 4) {
        f32x4 sum = *reinterpret_cast<const f32x4 *>(red + ((0 * SLOTS + slot) * 64 + lane) * 4);
#pragma unroll
        for (int w = 1; w < 4; ++w) {
            const f32x4 x = *reinterpret_cast<const f32x4 *>(red + ((w * SLOTS + slot) * 64 + lane) * 4);
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[r] += x[r];
        }
        emit(slot, sum);
    }
}

template <int D>
__device__ __forceinline__ void dkv_load_keys(const DkvArgs &a, int64_t row, int lane, bf16x8 (&kop)[D / 32],
                                              bf16x8 (&vop)[D / 32]) {
    const int g = lane >> 4;
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
        kop[s] = ld_bf16x8(a.Kl + row * D + g * 8 + 32 * s);
        vop[s] = ld_bf16x8(a.Vl + row * D + g * 8 + 32 * s);
    }
}

// ----------------------------------------------------------------------------------------- levels >= 1
template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2))) dkv_coarse_kernel(DkvArgs a) {
    using S = DkvShape<D>;
    __shared__ __attribute__((aligned(16))) char lds[4][S::WAVE];
    static_assert(4 * 2 * S::NT * 64 * 16 <= 4 * 2 * S::TILE, "reduction buffer must fit in the tile buffers");

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int64_t nkb = (a.n_l + 15) >> 4;                 // key blocks per head
    const int64_t wgid = xcd_contiguous(blockIdx.x, gridDim.x);   // neighbouring key blocks share query tiles in L2
    const int64_t kbf = wgid / a.splits;                   // flat key block
    const int split = (int)(wgid % a.splits);
    const int64_t bh = kbf / nkb, j = kbf % nkb;
    const int cntk = (int)min((int64_t)16, a.n_l - j * 16);

    bf16x8 kop[S::KS], vop[S::KS];                          // B operands (columns = keys), held throughout
    dkv_load_keys<D>(a, bh * a.n_l + j * 16 + min(i16, cntk - 1), lane, kop, vop);
    const int32_t *lst = nullptr;
    int64_t groups;
    if (a.dense) {
        groups = a.N >> 4;
    } else {
        const int32_t *Crow = a.C + bh * (a.rows + 1) + j;
        const int32_t beg = Crow[0], end = Crow[1];
        lst = a.Iq + bh * a.rows * a.Kl_cnt + beg;
        groups = (int64_t)(end - beg) << a.span_shift;
    }
    const int64_t tiles = (groups + 1) >> 1;
    const int64_t t_beg = tiles * split / a.splits, t_end = tiles * (split + 1) / a.splits;

    f32x4 accK[S::NT], accV[S::NT];
#pragma unroll
    for (int n = 0; n < S::NT; ++n) { accK[n] = f32x4{0.f, 0.f, 0.f, 0.f}; accV[n] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    dkv_tile_loop<D>(a, bh, lst, groups, t_beg + wave, 4, t_end, kop, vop, accK, accV, lds[wave], lane);

    dkv_reduce_waves<D>(reinterpret_cast<float *>(&lds[0][0]), wave, lane, accK, accV, [&](int slot, f32x4 sum) {
        const bool isV = slot >= S::NT;
        const int n = isV ? slot - S::NT : slot;
        if (i16 >= cntk) return;                            // rows past the end of a ragged coarsest level
        if (!isV)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[r] *= a.scale;
        float *dst = (isV ? a.partV : a.partK) + (int64_t)split * a.slab;
        *reinterpret_cast<f32x4 *>(dst + (bh * a.n_l + j * 16 + i16) * D + n * 16 + 4 * g) = sum;
    });
}

// ---------------------------------------------------------------------------------------------- level 0
// A wave by itself: the lists that begin in its few places of the head's row of tiles, one after the other without a stop (the next list's
// rows, keys and parent row are on their way while the one in hand is finished), or a piece of a list that is cut.  No wave waits for
// another.  Rows, logsumexps, D and the parents' gradients all go straight into LDS.  XCDs take whole stretches of heads, whose rows stay in
// their L2 (0.97 GB fetched from beyond at 16 x 65536 tokens; dealt round 340 us, 1.4 GB).
// A workgroup of four waves per four key blocks, the short lists by one wave each and the long ones by all four afterwards, with a barrier
// between, took 295 us at 16 x 65536 tokens (now 254; Gaussian 325, 318), 150 at 32 x 16384 (133), 26 at 16 x 4096 (21), 1580 at 8 x 262144
// with d = 128 and K = 16 (1610; a step with the one and the other 6759 and 6742, Gaussian 10027 and 9711); with constant keys, whose lists hold every query, a step of 4 x 65536 takes 559 us instead of 1226.
// What bounds it: a wave's chain (1700 cycles a tile alone on its SIMD: 320 in LDS reads, 170 + 430 in products and softmax, 530 in asking
// for the next rows), three waves a SIMD (with four the registers do not suffice: 300 us), and under load the requests, which take 1280
// cycles a tile then.  Not faster: reading all operands in front of the first product, rows from one place only (243 of then 273 us), waves
// that draw their work from a counter (27 ns a draw, one after the other: 630 us).
constexpr int kEmpty = 8;                                   // the key blocks that nothing lists, of this many, are one wave's work
struct FineArgs {
    const FineTile *tiles;
    int32_t *arrived;
    float *part;
    unsigned T, places, slots;                              // of a head: key blocks, places, slots of pieces
    int lc, pack;                                           // log2 of the tiles of a piece; a wave takes the lists and pieces that begin in `pack` places
    FastDiv packs, others;                                  // of a head: waves for tiles, waves for key blocks that nothing lists
    FastDiv span;                                           // waves of a part of the launch: of a head, or of all of them (fine_one_part)
    unsigned walks, dealt;                                  // waves for tiles, which come first in a part; waves that are dealt to the XCDs
    int stretch;                                            // log2 of the consecutive waves that an XCD takes at a time; -1: an eighth of all
};
__device__ __forceinline__ unsigned xcd_stretches(unsigned w, unsigned total, int ls) {
    if (ls < 0) return xcd_contiguous32(w, total);
    const unsigned r = w & ((8u << ls) - 1), w0 = w - r;
    return w0 + (8u << ls) <= total ? w0 + ((r & 7) << ls) + (r >> 3) : w;
}

template <int D>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2))) dkv_fine_kernel(DkvArgs a, FineArgs f) {
    using S = DkvShape<D>;
    __shared__ __attribute__((aligned(16))) char qt[S::WAVE];         // Q rows | dO rows | LSE [32], D [32]
    __shared__ __attribute__((aligned(16))) float par_sh[2][2 * D];   // the parent token's dK | dV: of the list in hand, of the next
    char *gt = qt + S::TILE;
    float *st = reinterpret_cast<float *>(gt + S::TILE);

    const int lane = threadIdx.x, i16 = lane & 15, g = lane >> 4;
    const bool has_par = a.parK != nullptr;
    const unsigned id = blockIdx.x < f.dealt ? xcd_stretches(blockIdx.x, f.dealt, f.stretch) : blockIdx.x;
    const unsigned part = f.span(id), in = id - part * f.span.d;
    const bool walk = in < f.walks;
    const unsigned w = walk ? in : in - f.walks, head = walk ? f.packs(w) : f.others(w), v = w - head * (walk ? f.packs.d : f.others.d);
    const unsigned bh = part + head;                        // one head to a part, or one part
    const int64_t key0 = (int64_t)bh * f.T;
    const int32_t *C = a.C + (int64_t)bh * (f.T + 1);

    if (!walk) {                                            // key blocks that nothing lists: the parent's share in every row
        const unsigned j0 = kEmpty * v;
        const int c0 = C[min(j0 + lane, f.T)], c1 = C[min(j0 + lane + 1, f.T)];
        uint64_t m = __ballot(lane < kEmpty && j0 + lane < f.T && c0 == c1);
        constexpr int CH = D / 8, RPI = 64 / CH;            // 16-byte chunks of a row, rows per store
        const int c = lane % CH;
        while (m) {                                         // two at a time, so that their loads fly together
            int64_t key[2];
            f32x4 par[2][4];
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const int b = m ? (int)__builtin_ctzll(m) : -1;
                key[x] = b < 0 ? -1 : key0 + j0 + b;
                if (b >= 0) m &= m - 1;
                const int64_t at = max(key[x], key[0]) * D + 8 * c;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    par[x][q] = has_par ? *reinterpret_cast<const f32x4 *>((q < 2 ? a.parK : a.parV) + at + 4 * (q & 1)) * a.inv_B : f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                if (key[x] < 0) break;
                const int64_t row = key[x] * 16 + lane / CH;
                const bf16x8 k = pack8(par[x][0], par[x][1]), w = pack8(par[x][2], par[x][3]);
#pragma unroll
                for (int r = 0; r < 16; r += RPI) {
                    *reinterpret_cast<bf16x8 *>(a.dK + (row + r) * D + 8 * c) = k;
                    *reinterpret_cast<bf16x8 *>(a.dV + (row + r) * D + 8 * c) = w;
                }
            }
        }
        return;
    }

    // The wave's places, 32 at a time: lane 2t the key word of place base + t, lane 2t + 1 its entry word; then the entries themselves,
    // lane 2t + x entry x (-1: there is none)
    const int p0 = f.pack * (int)v;
    int base = p0, word = 0, entry = 0;
    uint64_t starts = 0, gaps = 0;
    auto window = [&]() {
        const int32_t *src = reinterpret_cast<const int32_t *>(f.tiles + (int64_t)bh * f.places + base);
        word = base + (lane >> 1) < (int)f.places ? src[lane] : kGap;
        starts = __ballot(!(lane & 1) && word >= 0);
        gaps = __ballot(!(lane & 1) && word == kGap);
        const int w = __shfl(word, lane | 1, 64), e = w < 0 ? ~w : w;
        const bool there = !((gaps >> (lane & ~1)) & 1) && !(w < 0 && (lane & 1));
        entry = there ? a.Iq[(int64_t)bh * f.T * a.Kl_cnt + e + (lane & 1)] : -1;
    };
    window();
    if (!(starts & ((1ull << 2 * f.pack) - 1))) return;      // nothing begins here
    const int first = p0 + ((int)__builtin_ctzll(starts) >> 1);

    const TileOffsets<D> o = tile_offsets<D>(lane);
    const RowSource<D> src(lane);
    const unsigned dst = lds_address(qt), par_at = lds_address(par_sh);
    const uint64_t Qh = reinterpret_cast<uint64_t>(a.Q + (int64_t)bh * a.N * D), Gh = reinterpret_cast<uint64_t>(a.dO + (int64_t)bh * a.N * D);
    const float *stats = ((lane & 32) ? a.Dsum : a.LSE) + (int64_t)bh * a.N + i16;
    const unsigned koff = (unsigned)(i16 * D + g * 8) * 2;
    bf16x8 kop[S::KS], vop[S::KS];
    f32x4 accK[S::NT], accV[S::NT];
    int key = 0, next_key = 0, began = 0, turn = 0;         // key words; the place where the list or piece in hand begins
    bool both = false;                                      // does the tile on its way have its second entry?
    auto begins = [&](int t) { return (starts >> 2 * (t - base)) & 1; };
    auto load_tile = [&](int t) {
        const int e0 = __builtin_amdgcn_readlane(entry, 2 * (t - base)), e1 = __builtin_amdgcn_readlane(entry, 2 * (t - base) + 1);
        both = e1 >= 0;
        const int e[2] = {e0, both ? e1 : e0};              // an absent second one re-reads the first
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            load_lds<S::CPH>(Qh + (uint64_t)(unsigned)e[x] * (32 * D), src.v0, src.v1, dst + x * S::HALF);
            load_lds<S::CPH>(Gh + (uint64_t)(unsigned)e[x] * (32 * D), src.v0, src.v1, dst + S::TILE + x * S::HALF);
        }
        load_lds_dword(stats + 16 * ((lane & 16) ? e[1] : e[0]), dst + 2 * S::TILE);
        if (begins(t)) {                                    // the key block's rows, the parent's gradient
            next_key = __builtin_amdgcn_readlane(word, 2 * (t - base));
            const int64_t k = key0 + (next_key & (kPiece - 1));
            const char *kb = reinterpret_cast<const char *>(a.Kl) + k * (32 * D), *vb = reinterpret_cast<const char *>(a.Vl) + k * (32 * D);
#pragma unroll
            for (int ks = 0; ks < S::KS; ++ks) {
                kop[ks] = ld_bf16x8(kb + koff + 64 * ks);
                vop[ks] = ld_bf16x8(vb + koff + 64 * ks);
            }
            turn ^= 1;
            if (has_par)
#pragma unroll
                for (int x = 0; x < D / 64; ++x) {
                    load_lds_dword(a.parK + k * D + 64 * x + lane, par_at + 8 * D * turn + 256 * x);
                    load_lds_dword(a.parV + k * D + 64 * x + lane, par_at + 8 * D * turn + 4 * D + 256 * x);
                }
        }
    };
    // scale dK, add the parent token's share (adjoint of mean pooling), round once
    auto value = [&](int n, f32x4 sum, const float *par) {
        if (has_par) {
            const f32x4 x = *reinterpret_cast<const f32x4 *>(par + 16 * n + 4 * g);
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[r] += x[r] * a.inv_B;
        }
        return u32x2{pack_bf16(sum[0], sum[1]), pack_bf16(sum[2], sum[3])};
    };
    load_tile(first);
    int t = first, follows = 1;                             // follows: 0 nothing, 1 another tile of this list, 2 another list
    while (follows) {
        vm_wait<0>();
        if (begins(t)) {
            key = next_key;
            began = t;
#pragma unroll
            for (int n = 0; n < S::NT; ++n) { accK[n] = f32x4{0.f, 0.f, 0.f, 0.f}; accV[n] = f32x4{0.f, 0.f, 0.f, 0.f}; }
        }
        f32x4 s[2], dp[2], l2[2], dl[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            s[x] = f32x4{0.f, 0.f, 0.f, 0.f};
            dp[x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < S::KS; ++ks) {
                s[x] = mfma16(ld_bf16x8(qt + x * S::HALF + o.row[ks]), kop[ks], s[x]);
                dp[x] = mfma16(ld_bf16x8(gt + x * S::HALF + o.row[ks]), vop[ks], dp[x]);
            }
        }
#pragma unroll
        for (int x = 0; x < 2; ++x) {                       // this lane's 4 queries: rows 4g .. 4g+3
            l2[x] = *reinterpret_cast<const f32x4 *>(st + 16 * x + 4 * g);
            dl[x] = *reinterpret_cast<const f32x4 *>(st + 32 + 16 * x + 4 * g);
        }
        bf16x8 tg[S::NT], tq[S::NT];
#pragma unroll
        for (int n = 0; n < S::NT; ++n) {
            tg[n] = lds_tr_pair(gt + o.tr[n], gt + S::HALF + o.tr[n]);
            tq[n] = lds_tr_pair(qt + o.tr[n], qt + S::HALF + o.tr[n]);
        }
        const bool two = both;
        // what follows: places without a tile are passed over, lists that begin behind the wave's places are another wave's
        int next = t + 1;
        if (next - base == 32) {                            // (a list or piece longer than the window)
            base = next;
            window();
        }
        if ((gaps >> 2 * (next - base)) & 1) {              // the list ends here; the window reaches beyond the wave's places
            const uint64_t tiles = (~gaps & 0x5555555555555555ull) >> 2 * (next - base);
            next = tiles ? next + ((int)__builtin_ctzll(tiles) >> 1) : (int)f.places;
        }
        follows = next >= (int)f.places ? 0 : !begins(next) ? 1 : next < p0 + f.pack ? 2 : 0;
        if (follows) load_tile(next);
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float p = __builtin_amdgcn_exp2f(fmaf(s[x][r], a.sc2, fmaf(l2[x][r], -kLog2e, a.bias2)));
                s[x][r] = p;
                dp[x][r] = p * (dp[x][r] - dl[x][r]);
            }
        if (!two) {
            s[1] = f32x4{0.f, 0.f, 0.f, 0.f};
            dp[1] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        const bf16x8 pop = pack8(s[0], s[1]), dsop = pack8(dp[0], dp[1]);
#pragma unroll
        for (int n = 0; n < S::NT; ++n) {
            accV[n] = mfma16(tg[n], pop, accV[n]);
            accK[n] = mfma16(tq[n], dsop, accK[n]);
        }
        t = next;
        if (follows == 1) continue;
        const float *par = par_sh[follows ? turn ^ 1 : turn];
        const unsigned j = (unsigned)key & (kPiece - 1);
        if (key & kPiece) {
            // A piece: its sums to memory, past the caches that other XCDs do not see; the wave that finds itself the last of the list adds
            // all of them up, in order.
            // What orders it is the machine, not the atomics' own order: device-scope stores are written through and acknowledged when every XCD
            // would see them, so behind vmcnt(0) they come before this wave's count; a wave's loads are issued behind the count that it has
            // got back, and at device scope they pass its own XCD's caches by.  The two asm statements keep the compiler to that order.  With
            // acquire and release at the counter, which write back and invalidate an XCD's whole L2 for every piece: 8 x 262144
            // tokens, d = 128, K = 16 6679 -> 7014 us a step, 8 x 65536, K = 12 1482 -> 1505.
            auto slot = [&](int place) { return f.part + ((int64_t)bh * f.slots + piece_slot(place, f.lc)) * (32 * D) + lane; };   // [register][lane]
            float *p = slot(began);
#pragma unroll
            for (int n = 0; n < S::NT; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    __hip_atomic_store(p + 64 * (4 * n + r), accK[n][r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(p + 64 * (4 * n + r) + 16 * D, accV[n][r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            const int start = __builtin_amdgcn_readfirstlane(C[j]), len = __builtin_amdgcn_readfirstlane(C[j + 1]) - start;
            const int t0 = tile_place(start, (int)j), np = piece_count((len + 1) >> 1, f.lc);
            vm_wait<0>();
            int before = 0;
            if (lane == 0) before = __hip_atomic_fetch_add(f.arrived + (int64_t)bh * f.slots + piece_slot(t0, f.lc), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (__builtin_amdgcn_readfirstlane(before) != np - 1) continue;
            asm volatile("" ::: "memory");
#pragma unroll
            for (int n = 0; n < S::NT; ++n) { accK[n] = f32x4{0.f, 0.f, 0.f, 0.f}; accV[n] = f32x4{0.f, 0.f, 0.f, 0.f}; }
            for (int q = 0; q < np; ++q) {
                const float *y = slot(t0 + (q << f.lc));
                auto add = [&](f32x4 (&acc)[S::NT], const float *from) {
                    f32x4 x[S::NT];                         // all asked for before the first is added
#pragma unroll
                    for (int n = 0; n < S::NT; ++n)
#pragma unroll
                        for (int r = 0; r < 4; ++r) x[n][r] = __hip_atomic_load(from + 64 * (4 * n + r), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int n = 0; n < S::NT; ++n) acc[n] += x[n];
                };
                add(accK, y);
                add(accV, y + 16 * D);
            }
        }
#pragma unroll
        for (int n = 0; n < S::NT; n += 2) {
            store_pair(a.dK + ((key0 + j) * 16 + i16) * D, n, g, value(n, accK[n] * a.scale, par), value(n + 1, accK[n + 1] * a.scale, par));
            store_pair(a.dV + ((key0 + j) * 16 + i16) * D, n, g, value(n, accV[n], par + D), value(n + 1, accV[n + 1], par + D));
        }
    }
}

// Adds the split slabs of one coarse level in split order and, if there is a coarser level above it,
// that level's share (adjoint of mean pooling, 1/B of the parent token): dst[t] = sum_s part[s][t]
// (+ up[t / B] / B).  dst is the level's fp32 gradient buffer.  One thread per 4 consecutive floats,
// eight slabs in flight: a short launch is one chain of loads (4 heads x 65536 tokens, B = 32: a step 396 -> 370 us with the gather's).
__global__ void __launch_bounds__(256) dkv_reduce_kernel(const float *partK, const float *partV, float *dstK,
                                                          float *dstV, const float *upK, const float *upV,
                                                          int64_t total4, int64_t slab, int splits, int d, int lb,
                                                          float inv_B) {
    const int64_t i4 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i4 >= total4) return;
    const int64_t i = i4 * 4;
    f32x4 k = {0.f, 0.f, 0.f, 0.f}, v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int s = 0; s < splits; ++s) {
        k += *reinterpret_cast<const f32x4 *>(partK + s * slab + i);
        v += *reinterpret_cast<const f32x4 *>(partV + s * slab + i);
    }
    if (upK) {
        const int64_t tok = i / d, c = i % d;
        k += *reinterpret_cast<const f32x4 *>(upK + (tok >> lb) * d + c) * inv_B;
        v += *reinterpret_cast<const f32x4 *>(upV + (tok >> lb) * d + c) * inv_B;
    }
    *reinterpret_cast<f32x4 *>(dstK + i) = k;
    *reinterpret_cast<f32x4 *>(dstV + i) = v;
}

int dkv_splits(const Plan &p, int l) {
    if (l == 0) return 1;
    if (dkv_block_tiles(p, l)) return dkv_block_splits(p, l);
    // aim for a few thousand workgroups per level; a workgroup should still see several tiles
    const int64_t key_blocks = (int64_t)p.bh * ((p.n[l] + 15) / 16);
    const int64_t tiles_per_block = (l == p.L) ? p.N / 32 : (int64_t)p.K * (p.N / p.n[l + 1]) / 32;  // average
    int64_t s = (4096 + key_blocks - 1) / key_blocks;
    if (s > tiles_per_block / 8) s = tiles_per_block / 8;
    if (s < 1) s = 1;
    if (s > 64) s = 64;
    return (int)s;
}

bool dkv_by_tiles(const Plan &p) { return p.fast && p.B == 16; }

// Tiles of a piece and places of a wave, by the tiles for each wave that the chip holds.  A cut list's sums go to memory and back, 16 KB a piece
// (d = 128: 32), so pieces are as long as the launch's end allows: its last waves run alone while they finish one.  us at pieces of 8 / 16 / 32 / 64
// tiles: 8 x 16384 tokens 34 / 35 (12 tiles a wave), 16 x 4096, K = 16 31.6 / 33.9 (11), 32 x 4096 33.7 / 35.0 (12), d = 128, 4 x 16384 38.2 / 40.6 (9), 8 x 12288
// 47.5 / 51 (13); 63 x 4096 60.8 / 57.4 (24), 32 x 16384 147 / 135 (48) and, another time, - / 133 / 138 / 141; 16 x 65536 - / 266 / 254 / 263; steps at d = 128,
// 2 x 65536, K = 8 363 / 374 / 399 (18 tiles a wave, pieces from 16 on), 4 x 65536
// 596 / 609 / 629 (36), 8 x 65536 1088 / 1074 / 1089 (72), 8 x 65536, K = 16 1665 / 1642 / 1667 (136), 8 x 131072, K = 16 3657 / 3586 / 3571 (272),
// 8 x 262144, K = 16 6984 / 6883 / 6876 (544).
static int64_t fine_tiles(const Plan &p) { return p.bh * tile_places(p.n[1], p.n[1] * p.Kl[0]); }
static int64_t fine_share(const Plan &p) { return (fine_tiles(p) - 1) / (p.d == 128 ? 2048 : 3072) + 1; }   // two and three waves a SIMD
int fine_piece_log2(const Plan &p) {
    const int64_t share = fine_share(p);
    return share <= 16 ? 3 : share <= 64 ? 4 : p.d == 64 || share <= 256 ? 5 : 6;
}
// Places: a wave starts with a chain of loads (its places, their entries, the first rows), which several lists share, but with little to do each, a wave
// less is worth more.  us at 2 / 3 / 4 / 6 / 8 places (tiles a wave): 2 x 4096 tokens 12.9 / 13.7 / 13.9, 4 x 1024 10.4 / 10.5 / 11.6 (one or less),
// 16 x 4096 23.6 / 22.7 / 23.2, 8 x 8192 22.7 / 21.7 / 22.7, Gaussian 22.4 / 22.5 / 22.3, 8 x 8192, K = 4 18.6 / 18.4 / 18.2, Gaussian 19.0 / 18.4 / 17.4 (4 to
// 6), 5 x 16384 28.3 / 26.6 / 27.8 (8), d = 128, 8 x 4096 26.0 / 24.3 / 25.6 (5), 32 x 4096 35.9 / 35.0 / 33.7 / 34.8 (12), 16 x 16384 - / 56.3 / 55.0 / 56.0 /
// 55.9, Gaussian 62.8 / 61.8 / 62.8 / 65.4, 4 x 65536 - / 56.4 / 56.4 / 56.1 / 56.1, Gaussian 73.6 / 75.2 / 78.6 / 82.2 (24), 20 x 16384 - / 74.0 / 73.3 / 71.2 /
// 72.5, Gaussian 93.7 / 91.0 / 90.1 / 89.8 (30), 6 x 65536 - / 98.9 / 96.9 / 95.5 / 94.5, Gaussian 111.1 / 110.2 / 112.8 / 116.6 (36), 6 x 65536, K = 12
// - / - / 132.5 / 126.8 / 125.9 (53).
// Shapes of one share differ by as much as the widths do; the lines lie where the mean over them turns.  Four against three: even over eight shapes of 3 to
// 6 tiles a wave (-6 to +7 %), +2 % at 8.  Six against four, smooth and Gaussian: +1 and +3 % at 18, 0 and +2 at 22 to 24 (seven shapes), -4 and +1 at 30 to 36.
// More only where the waves have enough to do for their end not to matter (steps with 4 and 8: 4 x 110592 tokens, K = 4, Gaussian
// 460 and 474 us, smooth 439 and 447; 16 x 65536 1082 and 1070; d = 128, 4 x 131072, K = 8 Gaussian 1353 and
// 1368, 8 x 65536 1104 and 1098, both 147456 places).
static int fine_pack(const Plan &p) {
    const int64_t share = fine_share(p);
    return share <= 2 ? 2 : share <= 8 ? 3 : share <= 24 ? 4 : fine_tiles(p) > 64 * 3072 ? 8 : p.d == 64 ? 6 : 4;
}
// Whole stretches of heads keep rows that neighbouring blocks share in an XCD's L2 (dealt in stretches of 32 to 512 waves 16 x 65536 tokens, K = 8,
// 1 to 7 % slower, 8 x 262144 at d = 128, K = 16 6 to 12).  With lists of few blocks there is less to share, and where a head's Q and dO are
// more than 16 MB, eight XCDs in as many places are more than the cache behind L2 holds.  Steps, whole and in stretches of 64 waves, K = 4:
// 8 x 131072 955 and 939 us, Gaussian 995 and 975, 2 x 262144 Gaussian 649 and 639, 4 x 110592 446 and 450, Gaussian 468 and 461; but 4 x 65536
// (16 MB) 291 and 304.
static int fine_stretch(const Plan &p) { return p.Kl[0] <= 4 && p.N * p.d * 4 > 16 << 20 ? 6 : -1; }
// A head's waves for tiles stand before its waves for key blocks that nothing lists, which are much shorter.  Where an XCD's eighth is whole heads
// that is the same for every XCD; where it is not, some have more of the long ones than others: all heads' waves for tiles come first then and
// are dealt by themselves.  Steps, K = 8, a head at a time and like this: 4 x 262144 Gaussian 1446 and 1412 us, smooth 1178 and 1162, 6 x 196608
// Gaussian 1671 and 1619, 6 x 249856 Gaussian 2087 and 2028, 12 x 65536 887 and 882, 3 x 65536 306 and 301.  With whole heads it costs: 32 x 16384
// 533 and 538, in stretches 8 x 131072, K = 4 909 and 936.
static bool fine_one_part(const Plan &p) { return p.bh % 8 != 0 && fine_stretch(p) < 0; }

// level0_alone: level 0's own gradient only, without the share of its parent tokens (the pooled levels' gradients)
hipError_t launch_dkv_mfma(const Plan &p, const LevelTable &t, int l, const void *Q, const void *dO, const float *LSE,
                           const float *D, void *ws, void *dK, void *dV, hipStream_t s, bool level0_alone) {
    char *w = static_cast<char *>(ws);
    DkvArgs a;
    const int64_t key_blocks = (int64_t)p.bh * ((p.n[l] + 15) / 16);
    a.Q = (const uint16_t *)Q; a.dO = (const uint16_t *)dO;
    a.Kl = (const uint16_t *)t.K[l]; a.Vl = (const uint16_t *)t.V[l];
    a.LSE = LSE; a.Dsum = D;
    a.dense = (l == p.L);
    a.C = a.dense ? nullptr : (const int32_t *)(w + p.C_off[l]);
    a.Iq = a.dense ? nullptr : (const int32_t *)(w + p.Iq_off[l]);
    a.splits = dkv_splits(p, l);
    a.slab = key_blocks * 16 * p.d;
    a.partK = (float *)(w + p.part_off);
    a.partV = a.partK + (size_t)a.splits * a.slab;
    const bool has_parent = (l == 0 && p.Le >= 1 && !level0_alone);
    a.parK = has_parent ? (const float *)(w + p.dKacc_off[1]) : nullptr;
    a.parV = has_parent ? (const float *)(w + p.dVacc_off[1]) : nullptr;
    a.dK = (uint16_t *)dK; a.dV = (uint16_t *)dV;
    a.N = p.N; a.n_l = p.n[l];
    a.rows = a.dense ? 0 : p.n[l + 1];
    a.span_shift = a.dense ? 0 : p.lb * (l + 1) - 4;
    a.inv_B = 1.f / (float)p.B;
    a.Kl_cnt = a.dense ? 0 : p.Kl[l];
    a.sc2 = p.scale * kLog2e; a.bias2 = t.bias[l] * kLog2e; a.scale = p.scale;
    const bool block = dkv_block_tiles(p, l) > 0;
    if (block) {
        if (l > 0) a.dK = a.dV = nullptr;
        const hipError_t e = launch_dkv_block(p, l, a, s);
        if (l == 0 || e != hipSuccess) return e;
    } else if (l == 0) {
        const int64_t T = p.n[1], E = T * p.Kl[0];
        FineArgs f;
        f.tiles = (const FineTile *)(w + p.tiles_off);
        f.arrived = (int32_t *)(w + p.arrived_off);
        f.part = (float *)(w + p.piece_off);
        f.T = (unsigned)T;
        f.places = (unsigned)tile_places(T, E);
        f.lc = fine_piece_log2(p);
        f.slots = (unsigned)piece_slots(T, E, f.lc);
        f.pack = fine_pack(p);
        f.stretch = fine_stretch(p);
        f.packs = FastDiv((f.places + f.pack - 1) / f.pack);
        f.others = FastDiv((T + kEmpty - 1) / kEmpty);
        const unsigned heads = fine_one_part(p) ? (unsigned)p.bh : 1u, wgs = (unsigned)p.bh * (f.packs.d + f.others.d);
        f.walks = heads * f.packs.d;
        f.span = FastDiv(heads * (f.packs.d + f.others.d));
        f.dealt = fine_one_part(p) ? f.walks : wgs;
        if (p.d == 64) dkv_fine_kernel<64><<<wgs, 64, 0, s>>>(a, f);
        else dkv_fine_kernel<128><<<wgs, 64, 0, s>>>(a, f);
        return hipGetLastError();
    }
    if (!block) {
        dim3 grid((unsigned)(key_blocks * a.splits));
        if (p.d == 64) dkv_coarse_kernel<64><<<grid, 256, 0, s>>>(a);
        else dkv_coarse_kernel<128><<<grid, 256, 0, s>>>(a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // fold the slabs (and the level above) into this level's fp32 gradient
    const int64_t total4 = (int64_t)p.bh * p.n[l] * p.d / 4;
    const bool has_up = l < p.Le;
    dkv_reduce_kernel<<<(unsigned)((total4 + 255) / 256), 256, 0, s>>>(
        a.partK, a.partV, (float *)(w + p.dKacc_off[l]), (float *)(w + p.dVacc_off[l]),
        has_up ? (const float *)(w + p.dKacc_off[l + 1]) : nullptr, has_up ? (const float *)(w + p.dVacc_off[l + 1]) : nullptr,
        total4, a.slab, a.splits, p.d, p.lb, 1.f / (float)p.B);
    return hipGetLastError();
}

}  // namespace llsa
