// Attention forward and dQ of fp32 tensors on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32), any block size, d = 16 .. 128,
// and the launches of the tile kernels (bf16 tensors: tile_bf16.hip; dK / dV of both: tile_dkv.hip).
//
// Same tile algebra as the bf16 kernels, one 16 x 16 score tile at a time.  Of v_mfma_f32_16x16x4_f32 (lane = 16 g + i) an A
// operand is row i, contraction slot g; a B operand column i, slot g; the result column i, rows 4g .. 4g+3.
//   First product (scores): both operands are rows of a tensor and contract over channels, whose order is free as long as
//     both sides agree: step 4m + e takes channel 16m + 4g + e, so a lane reads 16-byte pieces of its row.
//   Second product (values, gradients): it contracts over the 16 rows of the tile.  Step r takes row 4g + r in slot g, and
//     the probability of that row is register r of the lane's own score tile, so nothing moves between lanes.  The other
//     operand is E consecutive channels of row 4g + r per lane, 16 lanes covering 16 E channels of a row.
// Rows that are an operand of the first product go through the wave's LDS (RowTile); rows that are one of the second only are
// fetched as they are, 256 bytes of a row per instruction.  The next tile's rows fly during the current one's math; list entries
// are fetched for 64 blocks at a time, when the walk comes to them.  What bounds these kernels is the matrix pipe (32 cycles an instruction: 512 per product of a
// 16 x 16 x 64 tile).  16 heads x 4096 tokens, d = 64, M = 272: forward 62 -> 58 us, dQ 92 -> 75 (29 and 43 us of matrix
// instructions; the forward without any load in its loop takes 50); 2 heads, a wave alone on its SIMD: 32 -> 28, 39 -> 34.
#include <string.h>

#include "csc_small.h"
#include "tile_f32.h"

namespace llsa {

// ------------------------------------------------------------------------------------------------ forward
template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : 4))) tile_fwd_kernel(TokArgs args, const float *__restrict__ Q, float *__restrict__ O,
                                                        float *__restrict__ LSE, int64_t N) {
    using S = TShape<D>;
    using RT = RowTile<D>;
    __shared__ __attribute__((aligned(16))) TokTable tabs[4];
    __shared__ __attribute__((aligned(16))) char rows_sh[4][RT::BYTES];
    const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned tile = xcd_contiguous32(blockIdx.x, gridDim.x) * 4 + wave;
    if (tile >= (unsigned)args.total) return;               // the waves of a workgroup never wait for each other
    const tok_args_ptr t = kernel_tok_args();
    const QTile qt = query_tile(args, tile, N);
    TokWalk<4 * D> walk;
    walk.begin(t, qt.bh, qt.blk, lane);
    const int64_t row = qt.row + min(i16, qt.nq - 1);
    TokTable &tab = tabs[wave];
    char *rt = rows_sh[wave];
    const RowOp<D> q = row_op<D>(Q + row * D, g);
    const int len = args.len, ntile = (len + 15) >> 4;
    const float scale = args.scale;
    f32x4 acc[S::NT];
#pragma unroll
    for (int n = 0; n < S::NT; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, lsum = 0.f;                        // running maximum; this lane's share of the row sum
    walk.put(tab, t, qt.bh, qt.blk, 0, lane);
    __builtin_amdgcn_wave_barrier();                        // one wave's LDS operations stay in order
    u32x4 kreg[RT::R];
    ColOp<D> v;
    auto load_k = [&](int j) {
#pragma unroll
        for (int u = 0; u < RT::R; ++u)
            kreg[u] = gload<u32x4>(tab.k[16 * (j & 3) + lane / RT::CH + RT::RPR * u] + (lane % RT::CH) * 16);
    };
    auto load_v = [&](int j) {
#pragma unroll
        for (int r = 0; r < 4; ++r) col_gload<D>(v, r, tab.v[16 * (j & 3) + 4 * g + r], i16);
    };
    load_k(0);
    load_v(0);
    for (int j = 0; j < ntile; ++j) {
        __builtin_amdgcn_wave_barrier();
        RT::put(rt, lane, kreg);
        __builtin_amdgcn_wave_barrier();
        const f32x4 bias = *reinterpret_cast<const f32x4 *>(&tab.bias[16 * (j & 3) + 4 * g]);
        if (j + 1 < ntile) {                                // the registers are free: the next rows fly during all of the math
            if (!((j + 1) & 3)) {
                __builtin_amdgcn_wave_barrier();
                walk.put(tab, t, qt.bh, qt.blk, 16 * (j + 1), lane);
                __builtin_amdgcn_wave_barrier();
            }
            load_k(j + 1);
        }
        f32x4 s = row_product<D>(RT::row(rt, i16, g), q);
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r] = fmaf(s[r], scale, bias[r]);
            mx = fmaxf(mx, s[r]);
        }
        mx = rows_max(mx);
        if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {
            const float m_new = fmaxf(m, mx), alpha = exp_nat(m - m_new);
            lsum *= alpha;
#pragma unroll
            for (int n = 0; n < S::NT; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[n][r] *= alpha;
            m = m_new;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] = exp_nat(s[r] - m);
        lsum += (s[0] + s[1]) + (s[2] + s[3]);
        col_product<D>(acc, v, s);
        if (j + 1 < ntile) load_v(j + 1);
    }
    lsum = rows_sum(lsum);
    if (i16 >= qt.nq) return;
    const float inv = 1.f / lsum;
    col_emit<D>(acc, g, [&](int ch, FVec<S::E> x) {
#pragma unroll
        for (int e = 0; e < S::E; ++e) {                    // x / lsum: the product and one correction (not of an infinity)
            const float q = x.v[e] * inv, c = fmaf(fmaf(-q, lsum, x.v[e]), inv, q);
            x.v[e] = c == c ? c : q;
        }
        st_e<S::E>(O + row * D + ch, x);
    });
    if (g == 0) LSE[row] = fmaf(__builtin_amdgcn_logf(lsum), kLn2, m);
}

// ----------------------------------------------------------------------------------------------------- dQ
// Same walk; P from the saved logsumexp.  Also produces D = rowsum(dO o O) of its queries for the key-major kernel.  (expf at
// d = 128: as exact, and around exp_nat the compiler schedules that loop worse, 2 heads x 4096 tokens 104 against 137 us.)
template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : 4))) tile_dq_kernel(TokArgs args, const float *__restrict__ Q, const float *__restrict__ O,
                                                       const float *__restrict__ dO, const float *__restrict__ LSE, float *__restrict__ Dsum,
                                                       float *__restrict__ dQ, int64_t N, CscSmall csc) {
    using S = TShape<D>;
    using RT = RowTile<D>;
    __shared__ __attribute__((aligned(16))) TokTable tabs[4];
    __shared__ __attribute__((aligned(16))) char rows_sh[4][2 * RT::BYTES];
    // the first workgroups make the key-major lists, which nothing here reads
    static_assert(sizeof(tabs) >= kCscSmallLds, "");
    if (blockIdx.x < csc.wgs) {
        csc_small<256>(csc, blockIdx.x, reinterpret_cast<uint32_t *>(tabs));
        return;
    }
    const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned tile = xcd_contiguous32(blockIdx.x - csc.wgs, gridDim.x - csc.wgs) * 4 + wave;
    if (tile >= (unsigned)args.total) return;
    const tok_args_ptr t = kernel_tok_args();
    const QTile qt = query_tile(args, tile, N);
    TokWalk<4 * D> walk;
    walk.begin(t, qt.bh, qt.blk, lane);
    const int64_t row = qt.row + min(i16, qt.nq - 1);
    TokTable &tab = tabs[wave];
    char *rt = rows_sh[wave];
    const RowOp<D> q = row_op<D>(Q + row * D, g), go = row_op<D>(dO + row * D, g);
    float delta = 0.f;
    {
        const RowOp<D> o = row_op<D>(O + row * D, g);
#pragma unroll
        for (int s = 0; s < S::KS; ++s) delta = fmaf(go.x[s], o.x[s], delta);
        delta = rows_sum(delta);
        if (g == 0 && i16 < qt.nq) Dsum[row] = delta;
    }
    const float lse = LSE[row], scale = args.scale;
    const int len = args.len, ntile = (len + 15) >> 4;
    f32x4 acc[S::NT];
#pragma unroll
    for (int n = 0; n < S::NT; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    walk.put(tab, t, qt.bh, qt.blk, 0, lane);
    __builtin_amdgcn_wave_barrier();
    u32x4 kreg[RT::R], vreg[RT::R];
    auto load_rows = [&](int j) {
#pragma unroll
        for (int u = 0; u < RT::R; ++u) {
            const int x = 16 * (j & 3) + lane / RT::CH + RT::RPR * u;
            kreg[u] = gload<u32x4>(tab.k[x] + (lane % RT::CH) * 16);
            vreg[u] = gload<u32x4>(tab.v[x] + (lane % RT::CH) * 16);
        }
    };
    load_rows(0);
    for (int j = 0; j < ntile; ++j) {
        __builtin_amdgcn_wave_barrier();
        RT::put(rt, lane, kreg);
        RT::put(rt + RT::BYTES, lane, vreg);
        __builtin_amdgcn_wave_barrier();
        const f32x4 bias = *reinterpret_cast<const f32x4 *>(&tab.bias[16 * (j & 3) + 4 * g]);
        if (j + 1 < ntile) {                                // the registers are free: the next rows fly during all of the math
            if (!((j + 1) & 3)) {
                __builtin_amdgcn_wave_barrier();
                walk.put(tab, t, qt.bh, qt.blk, 16 * (j + 1), lane);
                __builtin_amdgcn_wave_barrier();
            }
            load_rows(j + 1);
        }
        f32x4 s = row_product<D>(RT::row(rt, i16, g), q);
        const f32x4 dp = row_product<D>(RT::row(rt + RT::BYTES, i16, g), go);
#pragma unroll
        for (int r = 0; r < 4; ++r) {                       // past the end of the list: weight -inf, P = 0
            const float x = fmaf(s[r], scale, bias[r]) - lse;
            s[r] = (D == 128 ? expf(x) : exp_nat(x)) * (dp[r] - delta);
        }
        col_product<D>(acc, RT::col(rt, i16, g), s);
    }
    if (i16 >= qt.nq) return;
    col_emit<D>(acc, g, [&](int ch, FVec<S::E> x) {
#pragma unroll
        for (int e = 0; e < S::E; ++e) x.v[e] *= scale;
        st_e<S::E>(dQ + row * D + ch, x);
    });
}

// ------------------------------------------------------------------------------------------------- launches
static TokArgs tok_args(const Plan &p, const LevelTable &t) {
    TokArgs a;
    memset(&a, 0, sizeof(a));
    int first = 0;
    int64_t span = 1;                                       // query blocks that share a row of I^(l): B^l
    for (int l = 0; l <= kMaxL; ++l) {
        TokLevel &v = a.lev[l < t.nlev ? l : t.nlev - 1];
        if (l < t.nlev) {
            v.K = t.K[l];
            v.V = t.V[l];
            v.I = l < t.L ? t.I[l] : nullptr;
            v.span = FastDiv(l < t.L ? span : 1);
            v.n = (int32_t)t.n[l];
            v.rows = (int32_t)t.rows[l];
            v.Kl = t.Kl[l];
            v.first = first;
            v.bias = t.bias[l];
            first += l < t.L ? t.Kl[l] : (int)((t.n[l] + p.B - 1) / p.B);
            span *= p.B;
        }
        a.end[l] = first;
    }
    const int tpb = (p.B + 15) / 16;
    a.B = FastDiv(p.B);
    a.tpb = FastDiv(tpb);
    a.per_head = FastDiv(p.n[1] * tpb);
    a.len = t.seg[t.nlev];
    a.total = (int32_t)(p.bh * p.n[1] * tpb);
    a.scale = t.scale;
    return a;
}
static bool too_many_tiles(const Plan &p) { return p.bh * p.n[1] * ((p.B + 15) / 16) >= ((int64_t)1 << 31); }

template <class F> static hipError_t by_d(int d, F f) {
    switch (d) {
        case 16: f(std::integral_constant<int, 16>{}); break;
        case 32: f(std::integral_constant<int, 32>{}); break;
        case 64: f(std::integral_constant<int, 64>{}); break;
        default: f(std::integral_constant<int, 128>{}); break;
    }
    return hipGetLastError();
}

hipError_t launch_attn_fwd_tile(const Plan &p, const LevelTable &t, const void *Q, void *O, float *LSE, hipStream_t s) {
    if (too_many_tiles(p)) return hipErrorInvalidValue;
    const TokArgs a = tok_args(p, t);
    if (p.elt == 2) return launch_attn_fwd_tile_bf16(p, a, Q, O, LSE, s);
    return by_d(p.d, [&](auto d) {
        tile_fwd_kernel<d.value><<<(a.total + 3) / 4, 256, 0, s>>>(a, (const float *)Q, (float *)O, LSE, p.N);
    });
}

hipError_t launch_dq_tile(const Plan &p, const LevelTable &t, const void *Q, const void *O, const void *dO, const float *LSE,
                          float *D, void *dQ, const CscSmall &csc, hipStream_t s) {
    if (too_many_tiles(p)) return hipErrorInvalidValue;
    const TokArgs a = tok_args(p, t);
    if (p.elt == 2) return launch_dq_tile_bf16(p, a, Q, O, dO, LSE, D, dQ, csc, s);
    return by_d(p.d, [&](auto d) {
        tile_dq_kernel<d.value><<<(a.total + 3) / 4 + csc.wgs, 256, 0, s>>>(a, (const float *)Q, (const float *)O, (const float *)dO, LSE, D,
                                                                 (float *)dQ, p.N, csc);
    });
}

}  // namespace llsa
