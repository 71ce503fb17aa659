// The grouped dK / dV kernel's work for one level-1 query block (dkv_group.hip describes the method), by a launch of its own or by workgroups of the dQ
// launch.
#pragma once
#include "dkv_common.h"

namespace llsa {

struct GroupArgs {
    const uint16_t *Q, *dO;
    const float *LSE, *Dsum;
    float *slab;                                        // partials, level-major
    int64_t lvl_off[kMaxL + 1];                         // float offset of level l's partials [group][pos][UNIT]
    int nblk[kMaxL + 1];                                // key blocks of level l in a list
    int64_t N, NR;                                      // NR = level-1 query blocks per head
    int lev_end;                                        // levels below lev_end are processed (from 1, or from 2 in the upper kernel)
    int G;                                              // level-1 query blocks per workgroup (upper kernel)
    int GC, GS;                                         // level-1 query blocks a workgroup of the chain kernel walks, how far apart
    int nbs, nbd;                                       // upper kernel: listed blocks the waves own / shared dense block (0 or 1)
    int passes;                                         // upper kernel: workgroups that share the listed blocks of a query group
    float sc2, scale;
};

// The 256 Q and dO rows from row0 on, and their LSE and D, in the registers of NTHR threads (OWN: the rows of O instead of D) ...
template <int D, int NTHR> struct StageRegs {
    static constexpr int PER = 256 * GShape<D>::CH / NTHR;
    u32x4 q[PER], g[PER], o[PER];
    float s[512 / NTHR];
};
template <int D, int NTHR, bool OWN>
__device__ __forceinline__ void stage_load(StageRegs<D, NTHR> &r, const GroupArgs &a, int64_t row0, int tid, const uint16_t *O) {
    const char *qsrc = reinterpret_cast<const char *>(a.Q + row0 * D), *gsrc = reinterpret_cast<const char *>(a.dO + row0 * D);
#pragma unroll
    for (int k = 0; k < StageRegs<D, NTHR>::PER; ++k) {
        r.q[k] = *reinterpret_cast<const u32x4 *>(qsrc + (tid + NTHR * k) * 16);
        r.g[k] = *reinterpret_cast<const u32x4 *>(gsrc + (tid + NTHR * k) * 16);
        if constexpr (OWN) r.o[k] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(O + row0 * D) + (tid + NTHR * k) * 16);
    }
#pragma unroll
    for (int k = 0; k < 512 / NTHR; ++k) {
        const int i = tid + NTHR * k;
        r.s[k] = i < 256 ? a.LSE[row0 + i] : OWN ? 0.f : a.Dsum[row0 + i - 256];
    }
}
__device__ __forceinline__ float dot_chunk(u32x4 g, u32x4 o, float x) {   // x + 8 channels' products, one after the other
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x = fmaf(__uint_as_float(g[e] << 16), __uint_as_float(o[e] << 16), x);
        x = fmaf(__uint_as_float(g[e] & 0xffff0000u), __uint_as_float(o[e] & 0xffff0000u), x);
    }
    return x;
}
// ... and from there into LDS (qs, gs: swizzled rows; st: -LSE log2(e) [256] | -D [256])
template <int D, int NTHR, bool OWN>
__device__ __forceinline__ void stage_store(const StageRegs<D, NTHR> &r, char *qs, char *gs, float *st, int tid) {
    constexpr int CH = GShape<D>::CH;
#pragma unroll
    for (int k = 0; k < StageRegs<D, NTHR>::PER; ++k) {
        const int cc = tid + NTHR * k;
        *reinterpret_cast<u32x4 *>(qs + swz<D>(cc / CH, cc % CH)) = r.q[k];
        *reinterpret_cast<u32x4 *>(gs + swz<D>(cc / CH, cc % CH)) = r.g[k];
        if constexpr (OWN) {
            // lane group g of the dQ kernel sums chunks g and g + 4 of a row in a chain, then the four groups' sums are added pairwise
            static_assert(!OWN || (CH == 8 && NTHR % 64 == 0), "the 8 chunks of a row in 8 lanes");
            const float lo = dot_chunk(r.g[k], r.o[k], 0.f);
            float x = dot_chunk(r.g[k], r.o[k], __shfl_up(lo, 4, 64));   // (lanes of chunks 4 .. 7)
            x += __shfl_xor(x, 1, 64);
            x += __shfl_xor(x, 2, 64);
            if (cc % CH == 4) st[256 + cc / CH] = -x;
        }
    }
    // the forms the tiles take them in
#pragma unroll
    for (int k = 0; k < 512 / NTHR; ++k) {
        const int i = tid + NTHR * k;
        if (i < 256) st[i] = r.s[k] * -kLog2e;
        else if (!OWN) st[i] = -r.s[k];
    }
}

// where the partial of list block jl (counted from the start of the list) of query group `grp` goes
template <int D>
__device__ __forceinline__ float *partial_ptr(const LevelTable &t, const GroupArgs &a, int nlev, int jl, int64_t grp) {
    int l = 1;
#pragma unroll
    for (int x = 2; x <= kMaxL; ++x) l += (x < nlev && jl >= t.bseg[x]) ? 1 : 0;
    const int pos = jl - pick(t.bseg, l);
    return a.slab + pick(a.lvl_off, l) + (grp * pick(a.nblk, l) + pos) * GShape<D>::UNIT;
}

template <int D> __device__ __forceinline__ void store_partial(float *dst, const BlockAcc<D> &b, float scale, int lane) {
    dst += (lane & 15) * D + 4 * (lane >> 4);
    const float w = __builtin_amdgcn_exp2f(b.bias2);        // the level's weight, left out of the tiles' P
    const float ws = w * scale;
#pragma unroll
    for (int n = 0; n < D / 16; ++n) {
        f32x4 k = b.accK[n], v = b.accV[n];
#pragma unroll
        for (int r = 0; r < 4; ++r) { k[r] *= ws; v[r] *= w; }
        *reinterpret_cast<f32x4 *>(dst + n * 16) = k;
        *reinterpret_cast<f32x4 *>(dst + 16 * D + n * 16) = v;
    }
}

// A key block whose query tiles the NW waves of a workgroup share: their sums added in wave order through LDS (no wave reads anything
// else there any more).
template <int D, int NW>
__device__ __forceinline__ void store_shared(float *dst, const BlockAcc<D> &b, char *lds, float scale, int wave, int lane) {
    using S = GShape<D>;
    constexpr int SLOTS = 2 * S::NT;                                  // f32x4 slots per wave: dK tiles, then dV tiles
    float *red = reinterpret_cast<float *>(lds);                      // [wave][slot][lane] f32x4
    static_assert(NW * SLOTS * 64 * 16 <= 2 * 256 * S::ROWB, "the reduction must fit in the staged rows' memory");
#pragma unroll
    for (int n = 0; n < S::NT; ++n) {
        *reinterpret_cast<f32x4 *>(red + ((wave * SLOTS + n) * 64 + lane) * 4) = b.accK[n];
        *reinterpret_cast<f32x4 *>(red + ((wave * SLOTS + S::NT + n) * 64 + lane) * 4) = b.accV[n];
    }
    __syncthreads();
    dst += (lane & 15) * D + 4 * (lane >> 4);
#pragma unroll
    for (int k = 0; k < SLOTS / NW; ++k) {                            // wave w owns slots w, w + NW, ...
        const int slot = wave + NW * k;
        f32x4 sum = *reinterpret_cast<const f32x4 *>(red + (slot * 64 + lane) * 4);
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            const f32x4 x = *reinterpret_cast<const f32x4 *>(red + ((w * SLOTS + slot) * 64 + lane) * 4);
#pragma unroll
            for (int c = 0; c < 4; ++c) sum[c] += x[c];
        }
        const bool isV = slot >= S::NT;
        const float w = __builtin_amdgcn_exp2f(b.bias2) * (isV ? 1.f : scale);   // level weight (and scale for dK)
#pragma unroll
        for (int c = 0; c < 4; ++c) sum[c] *= w;
        *reinterpret_cast<f32x4 *>(dst + (isV ? 16 * D : 0) + (isV ? slot - S::NT : slot) * 16) = sum;
    }
}

// NW waves, a key block each at a time.  DENSE: the single block of a dense level 2 too, its query tiles dealt to the waves
// (group_takes_dense).  Bound: a wave's chain (rows, list, keys, eight tiles one after the other) where workgroups are few, LDS reads where they are
// many.  Two blocks a wave read every LDS operand once for both, but there are half as many waves, of twice the length: coarse stage at d = 64, four
// waves of two blocks and eight of one, us: 16 heads x 4096 tokens 29.3 and 27.3, K = 16 39.0 and 36.0, K = 32 38.6 and 35.4, 4 x 1024 19.4 and 17.5,
// 32 x 4096 39.7 and 37.7, 63 x 4096 67.0 and 62.1, K = 32: 16 x 16384 204 and 200, 16 x 65536 884 and 872.  (With registers for three waves a SIMD,
// one workgroup a CU, 63 x 4096 78.)
// R: the query block, over all heads.  lds: kGroupLds<D> bytes.  O: if D is to be formed here, as the dQ kernel forms it, bit for bit (OWN).
template <int D> constexpr int kGroupLds = 2 * 256 * GShape<D>::ROWB + 512 * 4;
template <int D, int NW, bool DENSE, bool OWN>
__device__ __forceinline__ void group_body(const LevelTable &t, const GroupArgs &a, int64_t R, char *lds, const uint16_t *O) {
    using S = GShape<D>;
    char *qs = lds;                                                   // Q rows of the group, chunk-swizzled | dO rows
    float *st = reinterpret_cast<float *>(lds + 2 * 256 * S::ROWB);   // -LSE log2(e) | -D
    char *gs = qs + 256 * S::ROWB;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4;
    const int64_t bh = R / a.NR, Rh = R % a.NR;
    const int nlev = min(t.nlev, a.lev_end);
    const int c_begin = t.bseg[1], nbc = pick(t.bseg, nlev) - c_begin;
    BlockTable ctab;
    BlockAcc<D> blk[1];
    auto keys = [&](int jb) {
        blk[0].load(jb < nbc ? ctab.K(jb & 63) : nullptr, ctab.V(jb & 63), ctab.count(jb & 63), ctab.bias(jb & 63), lane);
        blk[0].clear();
    };
    // d = 64: the list's blocks are looked up, and the first keys asked for, while the rows are on their way (d = 128, where the rows' registers leave no
    // room for it, 8 x 4096 tokens 40.4 us so and 39.1 behind them)
    StageRegs<D, 64 * NW> sr;
    stage_load<D, 64 * NW, OWN>(sr, a, bh * a.N + Rh * 256, tid, O);
    if constexpr (D == 64) { ctab.fill(t, bh, Rh * 16, c_begin, 0, lane, D, nlev); keys(wave); }
    stage_store<D, 64 * NW, OWN>(sr, qs, gs, st, tid);
    __syncthreads();
    if constexpr (D != 64) { ctab.fill(t, bh, Rh * 16, c_begin, 0, lane, D, nlev); keys(wave); }
    const TileOffsets<D> o = tile_offsets<D>(lane);

    int chunk = 0;
    for (int jb = wave; jb < nbc; jb += NW) {
        if ((jb >> 6) != chunk) { chunk = jb >> 6; ctab.fill(t, bh, Rh * 16, c_begin, chunk, lane, D, nlev); }
        if (jb != wave) keys(jb);
#pragma unroll 1
        for (int u = 0; u < 8; ++u) group_tile<D, 1>(qs, gs, st, st + 256, u, o, blk, a.sc2, g);
        store_partial(partial_ptr<D>(t, a, nlev, jb + c_begin, R), blk[0], a.scale, lane);
    }
    if constexpr (DENSE) {
        BlockAcc<D> dn[1];
        dn[0].load(static_cast<const char *>(t.K[2]) + bh * t.n[2] * S::ROWB, static_cast<const char *>(t.V[2]) + bh * t.n[2] * S::ROWB,
                   (int)t.n[2], t.bias[2] * kLog2e, lane);
        dn[0].clear();
        for (int u = wave; u < 8; u += NW) group_tile<D, 1>(qs, gs, st, st + 256, u, o, dn, a.sc2, g);
        __syncthreads();                                              // everyone is done with the rows
        store_shared<D, NW>(a.slab + a.lvl_off[2] + R * S::UNIT, dn[0], qs, a.scale, wave, lane);
    }
}

// The grouped kernel's work in the dQ launch: its arguments and its workgroups (a multiple of 8), which come first.  Few workgroups, each a wave's chain
// of waits: neither kernel fills the chip, and what the grouped one needs of dQ's, D, it can form itself (O's rows, 8 MB more to read at 16 heads x 4096
// tokens).  The two launches there took 44 us, the one 32; a step 89.3 -> 84.0 us.  Where dQ has two tiles a wave its workgroups have half the
// threads and more registers than this work leaves two workgroups a CU.
struct GroupAlong {
    LevelTable t;
    GroupArgs a;
    unsigned wgs, groups;
    bool dense;
};
bool group_along(const Plan &p, const LevelTable &t, const void *Q, const void *dO, const float *LSE, const float *D, void *ws, GroupAlong *along);

}  // namespace llsa
