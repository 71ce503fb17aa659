// What the key-major dK / dV kernels (Sec. 4.3) share: their arguments, a key block held by a wave, and the tile of 32 queries
// against it.
#pragma once
#include "mfma_common.h"

namespace llsa {

struct DkvArgs {
    const uint16_t *Q, *dO, *Kl, *Vl;     // Kl, Vl: the level's keys / values [bh, n_l, D]
    const float *LSE, *Dsum;
    const int32_t *C, *Iq;                // key-major lists (unused when dense)
    float *partK, *partV;                 // [splits][slab] fp32 (levels >= 1)
    const float *parK, *parV;             // level-1 totals [bh, n_1, D] fp32 or null (level 0)
    uint16_t *dK, *dV;                    // level-0 outputs
    int64_t N, n_l, rows, slab;           // rows = key blocks of this level per head that have lists
    int span_shift;                       // log2 of the 16-query groups per listed query block: log2(B^(level+1) / 16)
    float inv_B;
    int Kl_cnt, dense, splits;
    float sc2, bias2, scale;
    FastDiv blocks, split_of;             // dkv_block_kernel: key blocks per head, shares per block
};

template <int D> struct GShape {
    static constexpr int ROWB = 2 * D;                  // bytes of a staged row
    static constexpr int CH = D / 8;                    // 16-byte chunks per row
    static constexpr int KS = D / 32, NT = D / 16;
    static constexpr int UNIT = 2 * 16 * D;             // floats of one partial: [dK | dV][16 keys][D channels]
};

// staged rows of Q and dO: unpadded, 16-byte chunks XOR-swizzled by row (swz_key)
template <int D> __device__ __forceinline__ int swz(int r, int c) { return r * GShape<D>::ROWB + ((c ^ swz_key<D>(r)) << 4); }

// One key block held by a wave: its K / V rows as B operands, the level's log2 weight, its gradient sums.
// The tiles compute P = exp(z - LSE) without the level's weight B^l (a power of two for the block sizes of this
// path: scaling by it commutes with the bf16 rounding of P and dS); the sums take it when they are written.
template <int D> struct BlockAcc {
    bf16x8 kop[D / 32], vop[D / 32];
    float bias2;
    f32x4 accK[D / 16], accV[D / 16];

    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int n = 0; n < D / 16; ++n) { accK[n] = f32x4{0.f, 0.f, 0.f, 0.f}; accV[n] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    }
    // rows past a ragged end re-read the last row; an absent block (kp = null) gets zero operands
    __device__ __forceinline__ void load(const char *kp, const char *vp, int cnt, float b2, int lane) {
        bias2 = b2;
        const int off = (min(lane & 15, max(cnt, 1) - 1) * D + (lane >> 4) * 8) * 2;
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks) {
            kop[ks] = kp ? ld_bf16x8(kp + off + 64 * ks) : bf16x8{};
            vop[ks] = kp ? ld_bf16x8(vp + off + 64 * ks) : bf16x8{};
        }
    }
};

// queries 32u .. 32u+31 of the staged rows (lse: -LSE log2(e) of the rows, nd: -D) against NB key blocks:
// accK += Q^T dS, accV += dO^T P.  Every LDS operand is read once and used for all NB blocks; the sums of dP start from -D.
// RAW: lse and nd are LSE and D as they are in memory.
template <int D, int NB, bool RAW = false>
__device__ __forceinline__ void group_tile(const char *qs, const char *gs, const float *lse, const float *nd, int u,
                                           const TileOffsets<D> &o, BlockAcc<D> (&blk)[NB], float sc2, int g) {
    using S = GShape<D>;
    f32x4 s[NB][2], dp[NB][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int base = (32 * u + 16 * h) * S::ROWB;
        bf16x8 aq[S::KS], ag[S::KS];
#pragma unroll
        for (int ks = 0; ks < S::KS; ++ks) {
            aq[ks] = *reinterpret_cast<const bf16x8 *>(qs + base + o.row[ks]);
            ag[ks] = *reinterpret_cast<const bf16x8 *>(gs + base + o.row[ks]);
        }
        f32x4 l2 = *reinterpret_cast<const f32x4 *>(lse + 32 * u + 16 * h + 4 * g);
        f32x4 ndl = *reinterpret_cast<const f32x4 *>(nd + 32 * u + 16 * h + 4 * g);
        if constexpr (RAW)
#pragma unroll
            for (int r = 0; r < 4; ++r) { l2[r] *= -kLog2e; ndl[r] = -ndl[r]; }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            s[b][h] = f32x4{0.f, 0.f, 0.f, 0.f};
            dp[b][h] = ndl;
#pragma unroll
            for (int ks = 0; ks < S::KS; ++ks) {
                s[b][h] = mfma16(aq[ks], blk[b].kop[ks], s[b][h]);
                dp[b][h] = mfma16(ag[ks], blk[b].vop[ks], dp[b][h]);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float p = __builtin_amdgcn_exp2f(fmaf(s[b][h][r], sc2, l2[r]));   // without the level's weight
                s[b][h][r] = p;
                dp[b][h][r] = p * dp[b][h][r];
            }
        }
    }
    bf16x8 pop[NB], dsop[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) { pop[b] = pack8(s[b][0], s[b][1]); dsop[b] = pack8(dp[b][0], dp[b][1]); }
    const int b0 = 32 * u * S::ROWB, b1 = b0 + 16 * S::ROWB;
#pragma unroll
    for (int n = 0; n < S::NT; ++n) {
        const bf16x8 tg = lds_tr_pair(gs + b0 + o.tr[n], gs + b1 + o.tr[n]);
        const bf16x8 tq = lds_tr_pair(qs + b0 + o.tr[n], qs + b1 + o.tr[n]);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            blk[b].accV[n] = mfma16(tg, pop[b], blk[b].accV[n]);
            blk[b].accK[n] = mfma16(tq, dsop[b], blk[b].accK[n]);
        }
    }
}

// dkv_block.hip: fills in `blocks` and `split_of` and launches level l (dkv_block_tiles(p, l) > 0)
hipError_t launch_dkv_block(const Plan &p, int l, DkvArgs &a, hipStream_t s);

}  // namespace llsa
