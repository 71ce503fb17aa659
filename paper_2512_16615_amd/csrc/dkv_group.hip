// dK, dV of the coarse levels (l >= 1) on bf16 MFMA, grouped by query block (B = 16, d = 64 or 128, N % 256 == 0).
//
// The 256 fine queries under one level-1 query block R attend to the same coarse key blocks (Alg. 1,
// enrichment loop: fine block i reads row i / B^l of I^(l)).  Key-major processing (Sec. 4.3) re-reads the
// Q / dO rows of R once per listed key block; here a workgroup stages them once in LDS and its waves run
// the key-major tile loop over the 8 query tiles of R against R's coarse key blocks:
//   S = Q K^T, dP = dO V^T (lane: 4 queries x 1 key) -> P, dS -> dV^T += dO^T P, dK^T += Q^T dS.
// That yields, per (query group, coarse block of its list), the block's gradient restricted to the group's
// queries: a fp32 partial of 2 x 16 x d values.  Three kernels produce the partials:
//   dkv_group_kernel: one R per workgroup of 8 waves; a wave takes one list block at a time of the levels it is given;
//   dkv_chain_kernel: level 1 with at most 16 listed blocks.  The same tile loop, but a workgroup walks several
//     neighbouring R and a key block listed by a run of them keeps its sums in registers: one partial per run;
//   dkv_upper_kernel: levels >= 2 only.  The 16 level-1 blocks under one level-2 query block list the same
//     key blocks at every level >= 2, so a workgroup of 8 waves walks G of them (G divides 16; the next one's
//     rows are prefetched into registers; d = 128: dkv_upper_ring_kernel) and keeps its accumulators in registers meanwhile: every wave owns
//     one or two of the listed blocks (d = 128: one), and (d = 64) the single block of a coarsest level of at most 16 tokens is shared:
//     wave w takes query tile w of every R and the 8 waves' sums are added through LDS at the end.  G times fewer partials,
//     and no idle rounds when the number of key blocks is not a multiple of the waves.  The blocks of a larger dense level
//     are owned by waves like listed ones (N = 65536 with 256 coarsest tokens: without this, every level-1 query block
//     wrote 24 partials, 805 MB, and the coarse stage took 593 us instead of 335).
// The partials are then added up in a fixed order:
//   1. levels l >= 2: the query groups under one level-l query block list the same key blocks, so their
//      partials are summed up to 16 at a time (slab_reduce_kernel) until one partial per level-l query
//      block is left; the coarsest enriched level (every query attends to it) is summed down to one
//      partial per head;
//   2. per level, top-down, every key block gathers the partials of the query blocks that listed it
//      (Alg. 2's key-major lists, ascending), adds the share of its parent token (adjoint of mean
//      pooling) and writes the level's fp32 gradient (dkv_gather_kernel).
// No floating-point atomics; every sum has a fixed order.
#include "dkv_group.h"

namespace llsa {

template <int D, int NW, bool DENSE>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2))) dkv_group_kernel(LevelTable t, GroupArgs a) {
    __shared__ __attribute__((aligned(16))) char lds[kGroupLds<D>];
    group_body<D, NW, DENSE, false>(t, a, xcd_contiguous(blockIdx.x, gridDim.x), lds, nullptr);
}

// Tiles of 32 queries (Q rows | dO rows, LSE and D) on their way from memory straight into a ring of RING places in LDS, each of a workgroup's NW
// waves bringing a share of the rows.  All RING - 1 tiles behind the one in hand are always asked for (past the end the caller names a
// tile again), so that a wave knows how many of its loads may still be out.
template <int D, int NW, int RING> struct TileRing {
    static constexpr int HALF = 32 * GShape<D>::ROWB, BUF = 2 * HALF, SHARE = BUF / NW, LOADS = SHARE / 1024;
    uint64_t from;
    const float *stats;
    unsigned rows_at, stats_at;
    RowSource<D> src;
    int wave;
    // lds: [RING][BUF]; st: [RING][64]; q0: first query row of what the workgroup walks
    __device__ __forceinline__ TileRing(const GroupArgs &a, int64_t q0, const char *lds, const float *st, int wave_, int lane) : src(lane), wave(wave_) {
        from = reinterpret_cast<uint64_t>(wave < NW / 2 ? a.Q : a.dO) + (uint64_t)(q0 + (wave % (NW / 2)) * (SHARE / GShape<D>::ROWB)) * GShape<D>::ROWB;
        stats = ((lane & 32) ? a.Dsum : a.LSE) + q0 + (lane & 31);
        rows_at = lds_address(lds) + (unsigned)wave * SHARE;
        stats_at = lds_address(st);
    }
    __device__ __forceinline__ void load(int64_t q, int place) const {   // the tile q queries behind the first
        load_lds<LOADS>(from + (uint64_t)q * GShape<D>::ROWB, src.v0, src.v1, rows_at + place * BUF);
        if (wave == 0) load_lds_dword(stats + q, stats_at + 256 * place);
    }
    // the next tile is there, and no wave reads the one before it any more
    __device__ __forceinline__ void wait() const {
        if (wave == 0) vm_wait_barrier<(RING - 2) * (LOADS + 1)>();
        else vm_wait_barrier<(RING - 2) * LOADS>();
    }
};
// keys that the compiler waits for here: at their use it would wait for every tile on its way, each time
template <int D> __device__ __forceinline__ void keys_come(BlockAcc<D> &b) {
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) asm volatile("" : "+v"(b.kop[ks]), "+v"(b.vop[ks]));
}

constexpr int kChain = 8, kChainRow = 16;                              // query blocks of a chain, listed blocks of a row at most

// Level 1 alone, rows of I^(1) with at most NW * NB * P entries.  Neighbouring level-1 query blocks list mostly the same
// level-1 key blocks (for spatially smooth inputs a block stays listed over many consecutive rows), and a partial per
// (query block, listed block) then carries the same key block's sums to memory again and again.  Here a workgroup
// walks GC level-1 query blocks, GS apart, and keeps one listed block per register slot, as dkv_group_kernel does
// for a single query block.  From one query block R to the next, a slot whose key block is listed again goes on
// accumulating; a slot whose block is not listed by R + GS writes its partial to the place of (R, the block's
// position in R's row) and takes one of the blocks that are new in R + GS (both rows have Kl distinct entries,
// so as many slots come free as blocks are new; slots from Kl on compute on block 0 and are never stored).  A partial therefore covers a run of query blocks of
// one chain that all list the key block, and sits where the last of them would have put its own; the gather skips
// a lister whose successor in the same chain lists the block too.  Same arithmetic per tile, fewer partials.
// P workgroups share the slots of a row of more than NW * NB entries; each walks the same rows and keeps the same books.
// The tiles stream through a ring in LDS that runs on from query block to query block; the rows of I^(1) are looked up once, since a load of the
// compiler's in the walk would be waited for together with every tile on its way.  Bound, by counters (share of a SIMD's cycles; 25 % would be
// all of the LDS that four share): d = 64 a tile's chain at two waves a SIMD, vector ALU 36 %, MFMA 32, LDS 7, a wave waits 34 % of its life; d = 128
// LDS reads, 19 %, and issue, vector ALU 42, MFMA 46, at three waves.  With all 256 rows staged in LDS by way of registers, kernel, us: 16 heads
// x 65536 tokens 107 -> 99, 8 x 65536, d = 128 133 -> 118, 8 x 262144, d = 128, K = 16 800 -> 611; steps, 32 x 16384 527 -> 510.  (d = 64 with three waves a SIMD spills 6 registers: 103; two places 101.)
template <int D, int NW, int NB, int P>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW == 8 || NB == 2 ? 2 : D == 128 ? 3 : 4))) dkv_chain_kernel(LevelTable t, GroupArgs a) {
    using S = GShape<D>;
    constexpr int SL = NW * NB * P, RING = NW == 4 && D == 128 ? 2 : 4;
    using Ring = TileRing<D, NW, RING>;
    __shared__ __attribute__((aligned(16))) char lds[RING * Ring::BUF];
    __shared__ __attribute__((aligned(16))) float st_sh[RING][64];    // LSE [32] | D [32]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4;
    const int64_t per_head = a.NR / a.GC;
    const int64_t wg = xcd_contiguous(blockIdx.x, gridDim.x), chain = wg / P, bh = chain / per_head, c = chain % per_head;
    const int64_t R0 = c / a.GS * (a.GS * a.GC) + c % a.GS;           // the chain: R0, R0 + GS, ...
    const int slot0 = NB * (NW * (int)(wg % P) + wave);               // this wave's first slot
    const int Kl = t.Kl[1];
    const TileOffsets<D> o = tile_offsets<D>(lane);
    const int32_t *I1 = t.I[1] + (bh * a.NR + R0) * Kl;               // I^(1) has one row per level-1 query block
    const char *K1 = static_cast<const char *>(t.K[1]) + bh * t.n[1] * D * 2;
    const char *V1 = static_cast<const char *>(t.V[1]) + bh * t.n[1] * D * 2;
    const float bias2 = t.bias[1] * kLog2e;
    float *slab1 = a.slab + a.lvl_off[1] + (bh * a.NR + R0) * Kl * S::UNIT;
    const int64_t far = (int64_t)a.GS * Kl;                           // from a row of the chain to the next

    // the chain's rows of I^(1): entry e = row * Kl + place in lane e % 64 of word e / 64
    int rows[kChain * kChainRow / 64];
#pragma unroll
    for (int x = 0; x < kChain * kChainRow / 64; ++x) {
        const int e = 64 * x + lane;
        rows[x] = e < a.GC * Kl ? I1[e / Kl * far + e % Kl] : -1;
    }
    auto row = [&](int r) {                                           // lane p: entry p of row r, -1 from Kl on
        const int e = r * Kl + min(lane, Kl - 1);
        int v = __shfl(rows[0], e & 63, 64);
#pragma unroll
        for (int x = 1; x < kChain * kChainRow / 64; ++x) {
            const int y = __shfl(rows[x], e & 63, 64);
            v = e >> 6 == x ? y : v;
        }
        return lane < Kl ? v : -1;
    };
    int sblk = row(0), spos = lane;                                   // lane s < Kl: the block slot s holds, its place in the row
    BlockAcc<D> blk[NB];                                              // this wave's slots slot0 ...
    auto take = [&](int b, int id) {
        const int64_t at = (int64_t)max(id, 0) * 16 * D * 2;
        blk[b].load(K1 + at, V1 + at, 16, bias2, lane);
        blk[b].clear();
        keys_come(blk[b]);
    };
#pragma unroll
    for (int b = 0; b < NB; ++b) take(b, __builtin_amdgcn_readlane(sblk, slot0 + b));

    const Ring ring(a, bh * a.N + R0 * 256, lds, &st_sh[0][0], wave, lane);
    const int last = 8 * a.GC - 1;
    auto load = [&](int tile, int place) {                            // tile: 8 * row of the chain + its eighth
        tile = min(tile, last);
        ring.load((int64_t)(tile >> 3) * a.GS * 256 + 32 * (tile & 7), place);
    };
#pragma unroll
    for (int x = 0; x < RING - 1; ++x) load(x, x);
    for (int r = 0; r < a.GC; ++r) {
        if (r > 0) {
            const int nb = row(r);
            bool keep = false, fresh = lane < Kl;                  // (slots without a block keep it: -1 on both sides)
            int npos = 0;
#pragma unroll
            for (int x = 0; x < SL; ++x) {
                if (sblk == __builtin_amdgcn_readlane(nb, x)) { keep = true; npos = x; }
                if (nb == __builtin_amdgcn_readlane(sblk, x)) fresh = false;
            }
            const uint64_t kept = __ballot(keep), freed = __ballot(lane < Kl && !keep), news = __ballot(fresh);
            // the k-th slot that comes free takes the k-th new entry of the row
            const int k = __popcll(freed & ((1ull << lane) - 1));
            uint64_t m = news;
#pragma unroll
            for (int x = 0; x < SL; ++x) m = (x < k) ? (m & (m - 1)) : m;
            const int from = m ? (int)__builtin_ctzll(m) : 0;
            const int nid = __shfl(nb, from, 64);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int s = slot0 + b;
                if (!((kept >> s) & 1)) {                             // wave-uniform
                    const int oldpos = __builtin_amdgcn_readlane(spos, s);
                    store_partial(slab1 + ((r - 1) * far + oldpos) * S::UNIT, blk[b], a.scale, lane);
                    take(b, __builtin_amdgcn_readlane(nid, s));
                }
            }
            sblk = keep ? sblk : nid;
            spos = keep ? npos : from;
        }
        for (int u = 0; u < 8; u += RING)
#pragma unroll
            for (int x = 0; x < RING; ++x) {
                ring.wait();
                load(8 * r + u + x + RING - 1, (x + RING - 1) % RING);
                const char *buf = lds + x * Ring::BUF;
                group_tile<D, NB, true>(buf, buf + Ring::HALF, st_sh[x], st_sh[x] + 32, 0, o, blk, a.sc2, g);
            }
    }
    vm_wait<0>();                                                     // nothing may still come into LDS that is another workgroup's by then
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (slot0 + b >= Kl) continue;
        const int pos = __builtin_amdgcn_readlane(spos, slot0 + b);
        store_partial(slab1 + ((a.GC - 1) * far + pos) * S::UNIT, blk[b], a.scale, lane);
    }
}

// d = 128, where a workgroup of eight waves that holds all 256 rows of Q and dO has a CU to itself, two waves a SIMD: workgroups of four, three on
// a CU, with the tiles in a ring of two places.  A wave owns a listed block.  Bound, by counters: LDS reads, 18 %
// of a SIMD's cycles of the 25 that four have of one LDS, MFMA 43, vector ALU 31, and the barriers, waits of 56 % of a wave's life.  us, before ->
// now: 8 heads x 262144 tokens, K = 16 (20 listed blocks and a dense one) 1066 -> 876 (with four places, two workgroups a CU, 1055), 8 x 65536, K = 8 104 -> 98; steps 6997 -> 6698 and
// 1184 -> 1168 with the chain kernel's ring, 2 x 131072, K = 4 574 -> 526, Gaussian 568 -> 520.
template <int D, int NW>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(3))) dkv_upper_ring_kernel(LevelTable t, GroupArgs a) {
    constexpr int RING = 2;
    using Ring = TileRing<D, NW, RING>;
    __shared__ __attribute__((aligned(16))) char lds[RING * Ring::BUF];
    __shared__ __attribute__((aligned(16))) float st_sh[RING][64];    // LSE [32] | D [32]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4;
    const int64_t per_head = a.NR / a.G;
    const unsigned ngrp = gridDim.x / (unsigned)a.passes, c0 = blockIdx.x / (8u * a.passes) * 8u;   // eight groups, pass by pass
    const unsigned width = min(8u, ngrp - c0), rem = blockIdx.x - c0 * a.passes;
    const int jb = (int)(rem / width) * NW + wave;                    // this wave's listed block
    const int64_t grp = c0 + rem % width;                             // query group: G consecutive level-1 query blocks
    const int64_t bh = grp / per_head, R0 = (grp % per_head) * a.G;
    const TileOffsets<D> o = tile_offsets<D>(lane);
    const int nlev = min(t.nlev, a.lev_end);
    const int u_begin = t.bseg[2];                                    // first listed block of level 2
    const bool have = jb < a.nbs;
    BlockAcc<D> blk[1];
    {
        BlockTable ctab;                                              // lane j: listed block u_begin + 64 * (jb / 64) + j
        ctab.fill(t, bh, R0 * 16, u_begin, have ? jb >> 6 : 0, lane, D, nlev);
        blk[0].load(have ? ctab.K(jb & 63) : nullptr, ctab.V(jb & 63), ctab.count(jb & 63), ctab.bias(jb & 63), lane);
        blk[0].clear();
        keys_come(blk[0]);
    }
    const Ring ring(a, bh * a.N + R0 * 256, lds, &st_sh[0][0], wave, lane);
    const int last = 8 * a.G - 1;
#pragma unroll
    for (int x = 0; x < RING - 1; ++x) ring.load(32 * x, x);
    for (int u = 0; u <= last; u += RING)
#pragma unroll
        for (int x = 0; x < RING; ++x) {
            ring.wait();
            ring.load(32 * (int64_t)min(u + x + RING - 1, last), (x + RING - 1) % RING);
            const char *buf = lds + x * Ring::BUF;
            if (have) group_tile<D, 1, true>(buf, buf + Ring::HALF, st_sh[x], st_sh[x] + 32, 0, o, blk, a.sc2, g);
        }
    vm_wait<0>();                                                     // nothing may still come into LDS that is another workgroup's by then
    if (have) store_partial(partial_ptr<D>(t, a, nlev, u_begin + jb, grp), blk[0], a.scale, lane);
}

// d = 64.  SS = listed blocks a wave owns (block wave of the workgroup's share, + 8, ...): a workgroup takes 8 SS of them, and where a
// query group has more, a.passes workgroups take a share each.  All of them read the group's rows: they run at about the same
// time, eight ids apart and so on one XCD, for the rows to come from memory once (as launches of their own, three passes at 8 x 262144
// tokens, d = 128, which this kernel served then, read 1.07 GB each, and the coarse levels' dK / dV took 2185 us instead of 2098).
// DENSE: may this instantiation take the shared dense block (the first pass does).
template <int SS, bool DENSE>
__global__ void __launch_bounds__(512) dkv_upper_kernel(LevelTable t, GroupArgs a) {
    constexpr int D = 64;
    using S = GShape<D>;
    __shared__ __attribute__((aligned(16))) char lds[2 * 256 * S::ROWB];   // Q rows | dO rows; the final reduction reuses it
    __shared__ __attribute__((aligned(16))) float st[512];
    char *qs = lds, *gs = lds + 256 * S::ROWB;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4;
    const int64_t per_head = a.NR / a.G;
    const unsigned ngrp = gridDim.x / (unsigned)a.passes, c0 = blockIdx.x / (8u * a.passes) * 8u;   // eight groups, pass by pass
    const unsigned width = min(8u, ngrp - c0), rem = blockIdx.x - c0 * a.passes;
    const int pass = (int)(rem / width), first = pass * 8 * SS;       // first listed block of this workgroup
    const int64_t grp = c0 + rem % width;                             // query group: G consecutive level-1 query blocks
    const int64_t bh = grp / per_head, R0 = (grp % per_head) * a.G;
    const TileOffsets<D> o = tile_offsets<D>(lane);

    const int nlev = min(t.nlev, a.lev_end);
    const int u_begin = t.bseg[2];                                    // first listed block of level 2
    const bool dense = DENSE && a.nbd > 0 && pass == 0;
    BlockAcc<D> sp[SS][1], dn[DENSE ? 1 : 1];                         // this wave's sparse blocks; the dense block
    {
        BlockTable ctab;                                              // lane j: listed block u_begin + 64 * chunk + j
        int chunk = -1;
#pragma unroll
        for (int s = 0; s < SS; ++s) {
            const int jb = first + wave + 8 * s;
            const bool have = jb < a.nbs;
            if (have && (jb >> 6) != chunk) { chunk = jb >> 6; ctab.fill(t, bh, R0 * 16, u_begin, chunk, lane, D, nlev); }
            sp[s][0].load(have ? ctab.K(jb & 63) : nullptr, ctab.V(jb & 63), ctab.count(jb & 63), ctab.bias(jb & 63), lane);
            sp[s][0].clear();
        }
        if (dense) {
            if ((a.nbs >> 6) != chunk) ctab.fill(t, bh, R0 * 16, u_begin, a.nbs >> 6, lane, D, nlev);
            dn[0].load(ctab.K(a.nbs & 63), ctab.V(a.nbs & 63), ctab.count(a.nbs & 63), ctab.bias(a.nbs & 63), lane);
        } else {
            dn[0].load(nullptr, nullptr, 16, 0.f, lane);
        }
        dn[0].clear();
    }

    StageRegs<D, 512> sr;
    stage_load<D, 512, false>(sr, a, bh * a.N + R0 * 256, tid, nullptr);
    for (int r = 0; r < a.G; ++r) {
        stage_store<D, 512, false>(sr, qs, gs, st, tid);
        __syncthreads();
        if (r + 1 < a.G) stage_load<D, 512, false>(sr, a, bh * a.N + (R0 + r + 1) * 256, tid, nullptr);   // flies during the math
#pragma unroll
        for (int s = 0; s < SS; ++s)
            if (first + wave + 8 * s < a.nbs)
#pragma unroll 1                                                      // unrolled it takes 251 registers: none left beside it
                for (int u = 0; u < 8; ++u) group_tile<D, 1>(qs, gs, st, st + 256, u, o, sp[s], a.sc2, g);
        if (dense) group_tile<D, 1>(qs, gs, st, st + 256, wave, o, dn, a.sc2, g);
        __syncthreads();                                              // everyone is done with this R's rows
    }

#pragma unroll
    for (int s = 0; s < SS; ++s) {
        const int jb = first + wave + 8 * s;
        if (jb < a.nbs) store_partial(partial_ptr<D>(t, a, nlev, u_begin + jb, grp), sp[s][0], a.scale, lane);
    }
    if constexpr (DENSE)
        if (dense) store_shared<D, 8>(partial_ptr<D>(t, a, nlev, u_begin + a.nbs, grp), dn[0], lds, a.scale, wave, lane);
}

// out[h][r][x] = sum_{c < f, f r + c < cnt_in} in[h][f r + c][x], x over `width` floats (one thread per float4)
__global__ void __launch_bounds__(256) slab_reduce_kernel(const float *in, float *out, int64_t cnt_in, int64_t cnt_out,
                                                           int64_t f, int64_t width4, int64_t total4) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total4) return;
    const int64_t x = i % width4, hr = i / width4, r = hr % cnt_out, h = hr / cnt_out;
    const int64_t first = f * r, n = min(f, cnt_in - first);
    const f32x4 *src = reinterpret_cast<const f32x4 *>(in) + (h * cnt_in + first) * width4 + x;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int64_t c = 0; c < n; ++c) acc += src[c * width4];
    reinterpret_cast<f32x4 *>(out)[i] = acc;
}

// One workgroup per key block j of level l: sums the partials of the query blocks that listed j, in list
// order, adds the parent token's share and writes the level's fp32 gradient rows.
// FLY > 1 (no chains): that many partials are asked for before the first of them is added.
struct GatherArgs {
    const float *part;           // [bh][cnt][nblk][UNIT]
    const int32_t *C, *Iq, *I;   // key-major lists and I^(l) (null when dense)
    const float *upK, *upV;      // gradient of level l + 1 or null
    const float *upPart;         // or: the partials of level l + 1, dense in one block, up_cnt <= 16 per head
    int up_cnt;
    float *dstK, *dstV;          // [bh, n_l, D]
    int64_t cnt, n_l, rows;      // listers per head, tokens, rows of I^(l)
    FastDiv nkb;                 // key blocks per head
    int nblk, Kl, dense;
    int chain, apart;            // chain > 1: partials come from the chain kernel, which walked `chain` listers, `apart` apart
};
template <int D, int NT, int FLY>
__global__ void __launch_bounds__(NT) dkv_gather_kernel(GatherArgs a) {
    constexpr int U4 = GShape<D>::UNIT / 4, H4 = U4 / 2, PER = H4 / NT;   // float4 per partial / per half / per thread and half
    const int tid = threadIdx.x;
    const unsigned head = a.nkb(blockIdx.x);
    const int64_t bh = head, j = blockIdx.x - head * a.nkb.d;
    const f32x4 *part = reinterpret_cast<const f32x4 *>(a.part);
    f32x4 k[PER], v[PER];
#pragma unroll
    for (int x = 0; x < PER; ++x) { k[x] = f32x4{0.f, 0.f, 0.f, 0.f}; v[x] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    // The parent token's partials, one to each row of threads (a thread of each row for every four channels), added up behind the lists
    constexpr int ROW = D / 4, UP = FLY > 1 ? 16 : 0;                 // (group_takes_dense: few workgroups)
    __shared__ f32x4 up_sh[2][UP + 1][ROW];                           // dK | dV: the partials, their sum
    const int upr = tid / ROW, upc = tid % ROW;
    f32x4 pk, pv;
    const bool brings = UP && a.upPart && upr < a.up_cnt;
    if (brings) {
        static_assert(UP * ROW <= NT, "a row of threads for every partial");
        const float *p = a.upPart + (bh * a.up_cnt + upr) * GShape<D>::UNIT + j * D + upc * 4;
        pk = *reinterpret_cast<const f32x4 *>(p);
        pv = *reinterpret_cast<const f32x4 *>(p + 16 * D);
    }
    if (a.dense) {
        const f32x4 *p = part + ((bh * a.cnt) * a.nblk + j) * U4;
#pragma unroll
        for (int x = 0; x < PER; ++x) { k[x] = p[tid + NT * x]; v[x] = p[H4 + tid + NT * x]; }
    } else {
        // first every thread resolves one lister (query block row and the position of j in that row's list),
        // NT at a time, then all threads add the partials in list order with independent loads
        __shared__ int64_t unit[NT];
        const int32_t beg = a.C[bh * (a.rows + 1) + j], end = a.C[bh * (a.rows + 1) + j + 1];
        const int32_t *lst = a.Iq + bh * a.rows * a.Kl;
        for (int32_t e0 = beg; e0 < end; e0 += NT) {
            const int32_t m = min(NT, end - e0);
            __syncthreads();
            if (tid < m) {
                const int64_t r = lst[e0 + tid];
                const int32_t *row = a.I + (bh * a.rows + r) * a.Kl;
                int pos = 0;
                constexpr int AT = FLY > 1 ? 8 : 1;                        // asked for at a time
                for (int x0 = 0; x0 < a.Kl; x0 += AT) {
                    int32_t y[AT];
#pragma unroll
                    for (int x = 0; x < AT; ++x) y[x] = row[min(x0 + x, a.Kl - 1)];
#pragma unroll
                    for (int x = 0; x < AT; ++x) pos += (x0 + x < a.Kl && y[x] < (int32_t)j) ? 1 : 0;   // rows are ascending
                }
                int64_t un = ((bh * a.cnt + r) * a.nblk + pos) * U4;
                if (a.chain > 1 && r / a.apart % a.chain != a.chain - 1) {        // carried on by the next lister of the chain?
                    bool cont = false;
                    for (int x = 0; x < a.Kl; ++x) cont |= row[a.apart * a.Kl + x] == (int32_t)j;
                    if (cont) un = -1;
                }
                unit[tid] = un;
            }
            __syncthreads();
            if constexpr (FLY > 1) {                                      // every partial is there
                for (int32_t e = 0; e < m; e += FLY) {
                    f32x4 kk[FLY][PER], vv[FLY][PER];
#pragma unroll
                    for (int f = 0; f < FLY; ++f) {
                        const f32x4 *p = part + unit[min(e + f, m - 1)];
#pragma unroll
                        for (int x = 0; x < PER; ++x) { kk[f][x] = p[tid + NT * x]; vv[f][x] = p[H4 + tid + NT * x]; }
                    }
#pragma unroll
                    for (int f = 0; f < FLY; ++f)
                        if (e + f < m)
#pragma unroll
                            for (int x = 0; x < PER; ++x) { k[x] += kk[f][x]; v[x] += vv[f][x]; }
                }
            } else {
#pragma unroll 4
                for (int32_t e = 0; e < m; ++e) {
                    if (unit[e] < 0) continue;                            // same for every thread
                    const f32x4 *p = part + unit[e];
#pragma unroll
                    for (int x = 0; x < PER; ++x) { k[x] += p[tid + NT * x]; v[x] += p[H4 + tid + NT * x]; }
                }
            }
        }
    }
    if (UP && a.upPart) {
        if (brings) { up_sh[0][upr][upc] = pk; up_sh[1][upr][upc] = pv; }
        __syncthreads();
        if (tid < 2 * ROW) {
            f32x4 sum = {0.f, 0.f, 0.f, 0.f};
            for (int c = 0; c < a.up_cnt; ++c) sum += up_sh[tid / ROW][c][upc];
            up_sh[tid / ROW][UP][upc] = sum;
        }
        __syncthreads();
        pk = up_sh[0][UP][upc];
        pv = up_sh[1][UP][upc];
    }
#pragma unroll
    for (int x = 0; x < PER; ++x) {
        const int e4 = tid + NT * x;                                   // float4 index inside [16 keys][D channels]
        const int64_t tok = j * 16 + e4 / (D / 4);
        if (tok >= a.n_l) continue;
        const int col = (e4 % (D / 4)) * 4;
        f32x4 kk = k[x], vv = v[x];
        if (a.upK) {
            const int64_t up = (bh * ((a.n_l + 15) / 16) + j) * D + col;   // parent token of the block's 16 tokens
            kk += *reinterpret_cast<const f32x4 *>(a.upK + up) * 0.0625f;
            vv += *reinterpret_cast<const f32x4 *>(a.upV + up) * 0.0625f;
        } else if (UP && a.upPart) {                                   // (a thread's rows share its channels)
            kk += pk * 0.0625f;
            vv += pv * 0.0625f;
        }
        *reinterpret_cast<f32x4 *>(a.dstK + (bh * a.n_l + tok) * D + col) = kk;
        *reinterpret_cast<f32x4 *>(a.dstV + (bh * a.n_l + tok) * D + col) = vv;
    }
}

// Level-1 query blocks one workgroup of the upper kernels walks: as many as leave one workgroup per CU (d = 128: for each share of the listed
// blocks; steps of 8 x 65536 tokens, K = 8 and 4, with twice as many workgroups 1172 and 897 us, like this 1142 and 874, with half as many 1180 and 905).
static int query_group(const Plan &p) {
    const int64_t NR = p.N / 256;
    int G = 16;                                             // divides 16, so a group never straddles a level-2 query block
    while (G > 1 && (NR % G != 0 || (int64_t)p.bh * (NR / G) < 256)) G >>= 1;
    return G;
}

// Highest level the grouped kernels take; levels above it go to the split key-major kernel: a wide dense coarsest
// level (every query block would write a partial sum for every one of its key blocks, and summing over all queries
// is what the split kernel does in registers), and at d = 128 a dense level of a problem whose query groups are shorter than four query
// blocks.  There a wave owns a dense block as it does a listed one, often in a share of four waves more, which reads the group's rows
// once more; the split kernel reads all of Q and dO too, in two launches, and leaves no partials of every group to be added.  us a step, in
// the split kernel and in the upper one: groups of one query block, 1 x 65536 tokens, K = 8 300 and 315, 2 x 16384, K = 12 202 and 220; of
// two, 1 x 131072 418 and 422 to 428, 2 x 65536 393 and 398, 8 x 16384 351 and 351; of four, 2 x 131072, L = 4 582 and 553, 16 x 16384, K = 4
// 476 and 458; of more, 8 x 65536, K = 8 1157 and 1104, K = 4 934 and 872, 8 x 262144, K = 16 6900 and 6680, with 8 dense blocks (2 x 524288,
// K = 4) 1982 and 1900, with 16 (1 x 1048576) 2236 and 2095.
int dkv_group_top(const Plan &p) {
    if (p.Le < p.L) return p.Le;
    if ((p.n[p.L] + 15) / 16 > 32) return p.L - 1;
    if (p.d == 128 && (p.L <= 2 || query_group(p) < 4)) return p.L - 1;   // (L <= 2: no listed blocks to go along with)
    return p.Le;
}

// Blocks of levels 2 .. top: owned by waves (nbs: the sparse levels' listed ones and a dense level's, if it has several blocks, a
// wave has nothing else to do meanwhile or, d = 128, no wave has registers for a shared one) and shared by them (nbd: the block of a dense level, when the others fill all waves).
static void upper_blocks(const Plan &p, int *nbs, int *nbd) {
    const int top = dkv_group_top(p);
    *nbs = *nbd = 0;
    for (int l = 2; l <= top; ++l) {
        if (l < p.L) *nbs += p.Kl[l];
        else *nbd = (int)((p.n[l] + 15) / 16);
    }
    if (*nbd > 1 || *nbs % 8 != 0 || p.d == 128) { *nbs += *nbd; *nbd = 0; }
}

// Level-1 query blocks per workgroup of the upper kernel, or 0 if the group has no level >= 2.
static int upper_G(const Plan &p) {
    int nbs, nbd;
    upper_blocks(p, &nbs, &nbd);
    return dkv_group_top(p) < 2 || nbs + nbd == 0 ? 0 : query_group(p);
}

// Level-1 query blocks one workgroup of the chain kernel walks (1: the plain group kernel takes level 1), and how far apart they are.
// Rows of at most 16 level-1 blocks (beyond 8: several workgroups that stage the same rows), level 1 sparse and the only level the kernel
// is given.
// GS: 256 tokens of a square grid in raster order are a row's part from 262144 tokens on, and the query block next to R in the
// list of tokens lies beside it, 256 pixels away; the one below it, which lists 90 % of the same blocks on smooth inputs where
// the next one lists 3 to 11 %, is sqrt(N) / 256 further on.  GS is the power of two below that: it meets the block below on sides of
// 256 2^k and no better one than GS = 1 on others.  In nested-patch order the next block is the nearest, and GS > 1 costs a little.
// Backward, d = 64, K = 8, no chains / GS = 1 / 2 / 4, us: 8 heads x 512^2 raster 1974 / 1953 / 1730 / -, nested 2035 / 1887 / 1916 / -,
// Gaussian 2157 / 2149 / 2131 / -; 4 x 1024^2 raster 4878 / 4769 / 4718 / 4320, nested 4767 / 4429 / 4485 / 4548, Gaussian
// 4607 / 4599 / 4610 / 4595; 8 x 768^2 raster 5522 / 5449 / 5395 / - (GS = 3: 5036).
// Coarse stage, GS = 1 (rows of more than 8 blocks: one workgroup per query block) and as it is: 8 heads x 262144 tokens, K = 16,
// d = 128 2860 -> 2166 us; d = 64, K = 8 800 -> 587; 16 heads x 65536, K = 16 621 -> 425, Gaussian inputs 617 -> 611.
// With chains and without, GS = 1, steps: 16 heads x 65536 tokens, smooth K = 4 958 -> 875 us, K = 6 1105 -> 1017, d = 128 2677 ->
// 2463; Gaussian, which share few blocks: K = 4 970 -> 951, d = 128 2903 -> 2868.
// Measured at 16 heads x 65536 tokens: 8 query blocks per workgroup in 512 workgroups (two per CU) 259 us for the coarse stage,
// 4 in 1024: 275 us, 2: 297 us, 16 in 256 workgroups: 286 us, one query block per workgroup (no carrying): 357 us.
static void chain_shape(const Plan &p, int *GC, int *GS) {
    *GC = *GS = 1;
    if (p.L < 2 || p.Kl[1] > kChainRow) return;
    if (upper_G(p) == 0 && dkv_group_top(p) > 1) return;
    const int64_t NR = p.N / 256;
    int gc = kChain, gs = 1;
    while (gc > 1 && (NR % gc != 0 || (int64_t)p.bh * (NR / gc) < 512)) gc >>= 1;   // at least two workgroups per CU
    while ((int64_t)(2 * gs) * (2 * gs) * 65536 <= p.N && NR % (2 * gs * gc) == 0) gs *= 2;
    *GC = gc;
    *GS = gs;
}

// A dense level 2 of at most 16 tokens, d = 64: the group kernel takes its one block along, and the gather of level 1 adds up the (at most 16)
// partials of a parent token itself: three launches less, which is what there is to save at the size.  16 heads x 4096 tokens: the upper,
// reducing and gathering kernels of that level took 8 + 6 + 3 us, the group kernel takes 18 us with it and without (a step 122.1 ->
// 107.0 us; 2 heads 83.1 -> 72.2).  From 1024 level-1 query blocks on the chain kernel is the better one.
static bool group_takes_dense(const Plan &p) {
    int nbs, nbd, gc, gs;
    upper_blocks(p, &nbs, &nbd);
    chain_shape(p, &gc, &gs);
    return p.d == 64 && p.L == 2 && p.Le == 2 && nbs == 0 && nbd == 1 && gc == 1 && p.N <= 4096;
}

// partial-slab layout: level 1 has one partial per (level-1 query block, list position), levels >= 2 one per
// (query group, list position)
static int64_t slab_layout(const Plan &p, int64_t *lvl_off, int *nblk, int64_t *groups) {
    const int64_t NR = p.N / 256, unit = 2 * 16 * p.d;
    const int G = group_takes_dense(p) ? 0 : upper_G(p);
    int64_t off = 0;
    for (int l = 0; l <= kMaxL; ++l) { lvl_off[l] = 0; nblk[l] = 0; groups[l] = 0; }
    for (int l = 1; l <= dkv_group_top(p); ++l) {
        nblk[l] = l < p.L ? p.Kl[l] : (int)((p.n[l] + 15) / 16);
        groups[l] = (l >= 2 && G) ? NR / G : NR;
        lvl_off[l] = off;
        off += (int64_t)p.bh * groups[l] * nblk[l] * unit;
    }
    return off;
}

// bytes of the partial slab and of each of the two reduction buffers
void dkv_group_sizes(const Plan &p, size_t *slab_bytes, size_t *red_bytes) {
    const int64_t NR = p.N / 256, unit = 2 * 16 * p.d;
    int64_t lvl_off[kMaxL + 1], groups[kMaxL + 1];
    int nblk[kMaxL + 1];
    *slab_bytes = (size_t)slab_layout(p, lvl_off, nblk, groups) * sizeof(float);
    size_t red = 0;
    for (int l = 1; l <= dkv_group_top(p); ++l) {
        const size_t r = (size_t)p.bh * ((NR + 15) / 16) * nblk[l] * unit * sizeof(float);
        if ((l >= 2 || l == p.L) && r > red) red = r;       // levels that get reduced before the gather
    }
    *red_bytes = red;
}

#define GRP_TRY(expr)                     \
    do {                                  \
        const hipError_t e_ = (expr);     \
        if (e_ != hipSuccess) return e_;  \
    } while (0)

// reductions and gather of level l on stream s; `groups` = partials per head the kernels left for the level
static hipError_t finish_level(const Plan &p, const LevelTable &t, const GroupArgs &a, int l, int64_t groups, char *w,
                               hipStream_t s) {
    float *red[2] = {(float *)(w + p.grp_red_off[0]), (float *)(w + p.grp_red_off[1])};
    const int64_t unit = 2 * 16 * p.d;
    const bool dense = (l == p.L);
    const float *cur = a.slab + a.lvl_off[l];
    int64_t cnt = groups;
    const int64_t target = dense ? 1 : p.n[l + 1];          // listers per head: level-l query blocks, or the head
    const int64_t width4 = (int64_t)a.nblk[l] * (unit / 4);
    int flip = 0;
    while (cnt > target) {
        // groups under one lister are consecutive and their number is a power of two (any count when dense)
        const int64_t f = dense ? 16 : (cnt / target < 16 ? cnt / target : 16);
        const int64_t cnt_out = (cnt + f - 1) / f;
        const int64_t total4 = (int64_t)p.bh * cnt_out * width4;
        slab_reduce_kernel<<<dim3((unsigned)((total4 + 255) / 256)), 256, 0, s>>>(cur, red[flip], cnt, cnt_out, f, width4, total4);
        GRP_TRY(hipGetLastError());
        cur = red[flip];
        flip ^= 1;
        cnt = cnt_out;
    }
    GatherArgs ga;
    ga.part = cur;
    ga.dense = dense;
    ga.C = dense ? nullptr : (const int32_t *)(w + p.C_off[l]);
    ga.Iq = dense ? nullptr : (const int32_t *)(w + p.Iq_off[l]);
    ga.I = dense ? nullptr : t.I[l];
    const bool with_dense = l == 1 && group_takes_dense(p), has_up = l < p.Le && !with_dense;
    ga.upPart = with_dense ? a.slab + a.lvl_off[2] : nullptr;
    ga.up_cnt = (int)a.NR;
    ga.upK = has_up ? (const float *)(w + p.dKacc_off[l + 1]) : nullptr;
    ga.upV = has_up ? (const float *)(w + p.dVacc_off[l + 1]) : nullptr;
    ga.dstK = (float *)(w + p.dKacc_off[l]);
    ga.dstV = (float *)(w + p.dVacc_off[l]);
    ga.cnt = cnt; ga.n_l = p.n[l]; ga.nkb = FastDiv((p.n[l] + 15) / 16); ga.rows = dense ? 0 : p.n[l + 1];
    ga.nblk = a.nblk[l]; ga.Kl = dense ? 0 : p.Kl[l];
    ga.chain = l == 1 ? a.GC : 1;
    ga.apart = a.GS;
    const dim3 grid((unsigned)p.bh * ga.nkb.d);
    // Latency-bound (lists -> rows of I -> partials).  Many key blocks: more, smaller workgroups per CU shorten the launch, and few
    // registers let the upper levels' gathers run beside the chain kernel, which leaves no room for larger waves (8 partials in flight
    // there: 6 us more of 1110 a step at 16 heads x 65536 tokens, 2 of 560 at 32 x 16384).  At most 1024, and no chain kernel: the launch
    // is as long as one workgroup's chain of loads, and twice the threads with 8 partials in flight shorten that: 16 heads x 4096
    // tokens 12.0 -> 8.8 us, steps: 100.4 -> 96.7 us, 2 heads 69.0 -> 64.9, 8 x 16384 251 -> 242, 16 x 8192 178.6 -> 176.6.
    // A parent token's partials: one to a row of threads, on their way with the lists, where every thread read all of them, four at a time, in
    // front of the lists: steps of 16 x 4096 84.8 -> 83.1 us (coarse stage alone 27.3 -> 25.2; 2 heads 21.8 -> 19.9, 100 x 3840 92.5 -> 89.2).
    const bool few = (grid.x <= 1024 || with_dense) && a.GC == 1;
    if (p.d == 64) {
        if (few) dkv_gather_kernel<64, 256, 8><<<grid, 256, 0, s>>>(ga);
        else dkv_gather_kernel<64, 128, 1><<<grid, 128, 0, s>>>(ga);
    } else {
        if (few) dkv_gather_kernel<128, 512, 8><<<grid, 512, 0, s>>>(ga);
        else dkv_gather_kernel<128, 256, 1><<<grid, 256, 0, s>>>(ga);
    }
    return hipGetLastError();
}

static hipError_t launch_group_kernel(const Plan &p, const LevelTable &t, const GroupArgs &a, hipStream_t s) {
    if (a.GC > 1) {
        const unsigned wgs = (unsigned)(p.bh * (a.NR / a.GC));
        if (p.d == 128) {
            // workgroups of four waves, three on a CU, where they split a row of more than eight blocks (four of them 611 us, two of eight waves
            // 742 at 8 x 262144 tokens, K = 16); for 5 to 8 blocks one of eight (steps at 8 x 65536 1200 us, two of four 1237)
            if (p.Kl[1] <= 4) dkv_chain_kernel<128, 4, 1, 1><<<wgs, 256, 0, s>>>(t, a);
            else if (p.Kl[1] <= 8) dkv_chain_kernel<128, 8, 1, 1><<<wgs, 512, 0, s>>>(t, a);
            else dkv_chain_kernel<128, 4, 1, 4><<<4 * wgs, 256, 0, s>>>(t, a);
        } else if (p.Kl[1] <= 4) dkv_chain_kernel<64, 4, 1, 1><<<wgs, 256, 0, s>>>(t, a);
        else if (p.Kl[1] <= 8) dkv_chain_kernel<64, 4, 2, 1><<<wgs, 256, 0, s>>>(t, a);
        else dkv_chain_kernel<64, 4, 2, 2><<<2 * wgs, 256, 0, s>>>(t, a);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)(p.bh * a.NR));
    if (group_takes_dense(p)) dkv_group_kernel<64, 8, true><<<grid, 512, 0, s>>>(t, a);
    else if (p.d == 64) dkv_group_kernel<64, 8, false><<<grid, 512, 0, s>>>(t, a);
    else dkv_group_kernel<128, 8, false><<<grid, 512, 0, s>>>(t, a);
    return hipGetLastError();
}

// what the grouped kernels of a backward pass have in common; groups: partials per head that they leave for every level
static GroupArgs group_args(const Plan &p, const void *Q, const void *dO, const float *LSE, const float *D, char *w, int64_t *groups) {
    GroupArgs a;
    a.Q = (const uint16_t *)Q; a.dO = (const uint16_t *)dO; a.LSE = LSE; a.Dsum = D;
    a.slab = (float *)(w + p.grp_slab_off);
    a.N = p.N; a.NR = p.N / 256;
    a.sc2 = p.scale * kLog2e; a.scale = p.scale;
    slab_layout(p, a.lvl_off, a.nblk, groups);
    a.G = group_takes_dense(p) ? 0 : upper_G(p);
    chain_shape(p, &a.GC, &a.GS);
    upper_blocks(p, &a.nbs, &a.nbd);
    a.passes = 1;
    a.lev_end = a.G || group_takes_dense(p) ? 2 : dkv_group_top(p) + 1;
    return a;
}

bool group_along(const Plan &p, const LevelTable &t, const void *Q, const void *dO, const float *LSE, const float *D, void *ws, GroupAlong *along) {
    int64_t groups[kMaxL + 1];
    if (!p.group || p.d != 64) return false;
    along->a = group_args(p, Q, dO, LSE, D, static_cast<char *>(ws), groups);
    if (along->a.GC > 1) return false;
    along->t = t;
    along->groups = (unsigned)(p.bh * along->a.NR);
    along->wgs = (along->groups + 7) & ~7u;                 // workgroups behind them stay on their XCDs
    along->dense = group_takes_dense(p);
    return true;
}

// taken: the grouped kernel's partials are there (group_along)
hipError_t launch_dkv_group(const Plan &p, const LevelTable &t, const void *Q, const void *dO, const float *LSE,
                            const float *D, void *ws, bool taken, hipStream_t s, hipEvent_t lists, hipStream_t side,
                            hipEvent_t upper_done) {
    char *w = static_cast<char *>(ws);
    int64_t groups[kMaxL + 1];
    const GroupArgs a = group_args(p, Q, dO, LSE, D, w, groups);
    const int64_t NR = a.NR;
    const int top = group_takes_dense(p) ? 1 : dkv_group_top(p), G = a.G;   // (the group kernel takes the dense level along)

    // first the kernels that write the partials (they read no list), then, top-down, the reductions and gathers
    // (a level adds the share of the one above)
    if (G) {                                                // levels >= 2 in their own kernel
        GroupArgs up = a;
        up.lev_end = top + 1;
        // d = 64: 16 listed blocks to a workgroup, two a wave, where that fills the passes.  A last pass of 8 or fewer keeps one wave in two
        // busy or less, at the one workgroup a CU that the registers of two blocks allow: 8 to a workgroup then, of which two fit.
        // Backward, 16 / 8 to a workgroup: 8 heads x 589824 tokens (17 blocks) 5264 / 5081 us, Gaussian 5610 / 5320, 16 x 66560 (17)
        // 1198 / 1095, 16 x 69632, K = 16 (18) 1726 / 1588; 8 x 131072 (32) 1215 / 1258, 16 x 33280 (9) 309 / 323.
        const bool rest = up.nbs > 16 && (up.nbs - 1) % 16 < 8;
        // (d = 128: four, dkv_upper_ring_kernel)
        const int share = p.d == 128 ? 4 : up.nbs > 8 && !rest ? 16 : 8;
        up.passes = max(1, (up.nbs + share - 1) / share);
        const dim3 grid((unsigned)(p.bh * (NR / G) * up.passes));
        if (p.d == 128) dkv_upper_ring_kernel<128, 4><<<grid, 256, 0, s>>>(t, up);
        else if (share == 8) dkv_upper_kernel<1, true><<<grid, 512, 0, s>>>(t, up);
        else if (up.nbd == 0) dkv_upper_kernel<2, false><<<grid, 512, 0, s>>>(t, up);
        else dkv_upper_kernel<2, true><<<grid, 512, 0, s>>>(t, up);
        GRP_TRY(hipGetLastError());
    }
    // With a side stream (the one the lists are made on), the small reductions and gathers of levels >= 2 follow the
    // lists there, beside the level-1 kernel, and `lists` is recorded again behind them.
    const bool split = G && side && lists && upper_done && top >= 2;
    if (split) {
        GRP_TRY(hipEventRecord(upper_done, s));
        GRP_TRY(hipStreamWaitEvent(side, upper_done, 0));
        for (int l = top; l >= 2; --l) GRP_TRY(finish_level(p, t, a, l, groups[l], w, side));
        GRP_TRY(hipEventRecord(lists, side));
    }
    if (!taken) GRP_TRY(launch_group_kernel(p, t, a, s));
    if (lists) GRP_TRY(hipStreamWaitEvent(s, lists, 0));
    for (int l = split ? 1 : top; l >= 1; --l) GRP_TRY(finish_level(p, t, a, l, groups[l], w, s));
    return hipSuccess;
}

}  // namespace llsa
