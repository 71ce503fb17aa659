// Attention forward and dQ of bf16 tensors in fp32 arithmetic on the bf16 matrix instruction: the bf16 shapes that the bf16 MFMA
// kernels do not take (lengths that are no multiple of 64, other block sizes, d = 16 and 32), any block size, d = 16 .. 128.
//
// Scores and dP are products of bf16 rows, which v_mfma_f32_16x16x32_bf16 forms exactly and sums in fp32.  P and dS are fp32 and
// stay so: each enters its product as three bf16 parts that add up to it exactly (split8), so a product costs three matrix
// instructions of 16 cycles per 32 keys where the fp32 one takes eight of 32.  One wave per tile of up to 16 queries, 32 keys at a
// time; K and V rows are fetched whole (the operand layout straight from memory, 16 rows x half a line per instruction, caps
// gathers at a third of what the L2 delivers: 26 us each for the figures below) and go through the wave's LDS, rows swizzled.
// The next 32 keys' rows are in flight during the current ones' math.  List entries are fetched for 64 blocks at a time, when the walk
// comes to them: a list of more than 64 blocks waits for one load every 64 blocks.
// Bound: the vector instructions (softmax and splitting, about 150 a tile) and the latency of a wave's chain.
// 16 heads x 2704 tokens, d = 64, 297 tokens a list, against the fp32 matrix instruction on operands straight from memory: forward
// 54 -> 23 us, dQ 82 -> 24 us.
#include "csc_small.h"
#include "tile_f32.h"

namespace llsa {

template <int D> struct BShape {
    static constexpr int KS = (D + 31) / 32;            // matrix instructions over the channels
    static constexpr int NT = D / 16, ROWB = 2 * D, PARTS = D / 8;
    static constexpr int KPU = 64 / PARTS, VCH = 32 / KPU;   // staging: rows per round, rounds per 32 rows
};

// Where an input is not finite, a part that is 0 meets an infinite row, or an infinite dS has no parts, and the sum is a NaN where
// the product of fp32 values is an infinity.  So a pass that ends with a NaN in any lane is walked again with the fp32 matrix
// instruction, whose results then stand (finite inputs give no NaN: they pay for looking, 1 % of a tile's vector instructions).

// contraction step ks of a row as an operand; d = 16 fills half of the 32 slots, the others are zero
template <int D> __device__ __forceinline__ bf16x8 row_step(const char *row, int g, int ks) {
    if constexpr (D == 16) return g < 2 ? ld_bf16x8(row + 16 * (g & 1)) : bf16x8{};
    else return ld_bf16x8(row + 16 * g + 64 * ks);
}
template <int D> __device__ __forceinline__ bf16x8 row_zero(bf16x8 x, int g) {
    if constexpr (D == 16) return g < 2 ? x : bf16x8{};
    else return x;
}

// The lane number for a pass: computed from it in the second pass, addresses are not kept in registers throughout the first.
template <bool Exact> __device__ __forceinline__ int pass_lane(int lane) {
    if constexpr (Exact) asm volatile("" : "+v"(lane));
    return lane;
}

// acc += X^T p with the 32 rows of X at `xt` (swizzled), p in three parts, smallest first (Exact: as it is)
template <int D, bool Exact>
__device__ __forceinline__ void add_product(f32x4 (&acc)[D / 16], const char *xt, const TileOffsets<D> &o, const f32x4 (&p)[2], int rows, int g) {
    Parts3 parts;
    if constexpr (!Exact) parts = split8(p[0], p[1]);
#pragma unroll
    for (int n = 0; n < D / 16; ++n) {
        const bf16x8 x = lds_tr_pair(xt + o.tr[n], xt + 32 * D + o.tr[n]);
        if constexpr (Exact) acc[n] = product_fp32(x, p, rows, g, acc[n]);
        else
#pragma unroll
            for (int i = 2; i >= 0; --i) acc[n] = mfma16(x, parts.p[i], acc[n]);
    }
}

template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : 4)))
tile_fwd_bf16_kernel(TokArgs args, const uint16_t *__restrict__ Q, uint16_t *__restrict__ O, float *__restrict__ LSE, int64_t N) {
    using S = BShape<D>;
    constexpr int TILE = 32 * S::ROWB;
    __shared__ __attribute__((aligned(16))) char lds[4][2 * TILE];   // per wave: K rows | V rows
    __shared__ __attribute__((aligned(16))) TokTable tabs[4];
    const int lane0 = threadIdx.x & 63, i16 = lane0 & 15, g = lane0 >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned tile = xcd_contiguous32(blockIdx.x, gridDim.x) * 4 + wave;
    if (tile >= (unsigned)args.total) return;               // the waves of a workgroup never wait for each other
    const tok_args_ptr t = kernel_tok_args();
    const QTile qt = query_tile(args, tile, N);
    TokWalk<S::ROWB> walk;
    walk.begin(t, qt.bh, qt.blk, lane0);
    const int64_t row = qt.row + min(i16, qt.nq - 1);
    char *kt = lds[wave], *vt = kt + TILE;
    TokTable &tab = tabs[wave];

    bf16x8 q[S::KS];
#pragma unroll
    for (int ks = 0; ks < S::KS; ++ks) q[ks] = row_step<D>(reinterpret_cast<const char *>(Q + row * D), g, ks);
    f32x4 acc[S::NT];
    float m, lsum;                                          // running maximum; this lane's share of the row sum
    const int len = args.len, ntile = (len + 31) >> 5;
    const float scale = args.scale;

    auto pass = [&](auto exact) {
        constexpr bool Exact = decltype(exact)::value;
        const int lane = pass_lane<Exact>(lane0), g = lane >> 4;
        const TileOffsets<D> o = tile_offsets<D>(lane);
        m = -INFINITY;
        lsum = 0.f;
#pragma unroll
        for (int n = 0; n < S::NT; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
        walk.put(tab, t, qt.bh, qt.blk, 0, lane);
        u32x4 kreg[S::VCH], vreg[S::VCH];
        auto load = [&](int j) {
#pragma unroll
            for (int u = 0; u < S::VCH; ++u) {
                const int x = 32 * (j & 1) + lane / S::PARTS + S::KPU * u;
                kreg[u] = gload<u32x4>(tab.k[x] + (lane % S::PARTS) * 16);
                vreg[u] = gload<u32x4>(tab.v[x] + (lane % S::PARTS) * 16);
            }
        };
        __builtin_amdgcn_wave_barrier();                        // one wave's LDS operations stay in order
        load(0);
        for (int j = 0; j < ntile; ++j) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < S::VCH; ++u) {
                const int r = lane / S::PARTS + S::KPU * u, off = r * S::ROWB + (((lane % S::PARTS) ^ swz_key<D>(r)) << 4);
                *reinterpret_cast<u32x4 *>(kt + off) = kreg[u];
                *reinterpret_cast<u32x4 *>(vt + off) = vreg[u];
            }
            __builtin_amdgcn_wave_barrier();
            f32x4 bias[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) bias[h] = *reinterpret_cast<const f32x4 *>(&tab.bias[32 * (j & 1) + 16 * h + 4 * g]);
            if (j + 1 < ntile) {                                // the registers are free: the next rows fly during all of the math
                if (j & 1) {
                    __builtin_amdgcn_wave_barrier();
                    walk.put(tab, t, qt.bh, qt.blk, 32 * (j + 1), lane);
                    __builtin_amdgcn_wave_barrier();
                }
                load(j + 1);
            }
            f32x4 s[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                s[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < S::KS; ++ks) s[h] = mfma16(row_zero<D>(ld_bf16x8(kt + 16 * h * S::ROWB + o.row[ks]), g), q[ks], s[h]);
            }
            float mx = -INFINITY;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    s[h][r] = fmaf(s[h][r], scale, bias[h][r]);
                    mx = fmaxf(mx, s[h][r]);
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
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r) s[h][r] = exp_nat(s[h][r] - m);
            lsum += ((s[0][0] + s[0][1]) + (s[0][2] + s[0][3])) + ((s[1][0] + s[1][1]) + (s[1][2] + s[1][3]));
            add_product<D, Exact>(acc, vt, o, s, len - 32 * j, g);
        }
    };
    pass(std::false_type{});
    if (any_nan(acc)) pass(std::true_type{});
    lsum = rows_sum(lsum);
    if (i16 >= qt.nq) return;
    const float inv = 1.f / lsum;
#pragma unroll
    for (int n = 0; n < S::NT; ++n) {
        FVec<4> x;
#pragma unroll
        for (int r = 0; r < 4; ++r) {                       // x / lsum: the product and one correction (not of an infinity)
            const float a = acc[n][r], p = a * inv, c = fmaf(fmaf(-p, lsum, a), inv, p);
            x.v[r] = c == c ? c : p;
        }
        st_e(O + row * D + 16 * n + 4 * g, x);
    }
    if (g == 0) LSE[row] = add_log(m, lsum);
}

// dQ: the same walk, P from the saved logsumexp; K rows are read from LDS row-wise and transposed, V rows row-wise only.  Also
// produces D = rowsum(dO o O) of its queries for the key-major kernel.
template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : 4)))
tile_dq_bf16_kernel(TokArgs args, const uint16_t *__restrict__ Q, const uint16_t *__restrict__ O, const uint16_t *__restrict__ dO,
                    const float *__restrict__ LSE, float *__restrict__ Dsum, uint16_t *__restrict__ dQ, int64_t N, CscSmall csc) {
    using S = BShape<D>;
    constexpr int TILE = 32 * S::ROWB;
    __shared__ __attribute__((aligned(16))) char lds[4][2 * TILE];   // per wave: K rows | V rows
    __shared__ __attribute__((aligned(16))) TokTable tabs[4];
    // the first workgroups make the key-major lists, which nothing here reads
    static_assert(sizeof(tabs) >= kCscSmallLds, "");
    if (blockIdx.x < csc.wgs) {
        csc_small<256>(csc, blockIdx.x, reinterpret_cast<uint32_t *>(tabs));
        return;
    }
    const int lane0 = threadIdx.x & 63, i16 = lane0 & 15, g = lane0 >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned tile = xcd_contiguous32(blockIdx.x - csc.wgs, gridDim.x - csc.wgs) * 4 + wave;
    if (tile >= (unsigned)args.total) return;
    const tok_args_ptr t = kernel_tok_args();
    const QTile qt = query_tile(args, tile, N);
    TokWalk<S::ROWB> walk;
    walk.begin(t, qt.bh, qt.blk, lane0);
    const int64_t row = qt.row + min(i16, qt.nq - 1);
    char *kt = lds[wave], *vt = kt + TILE;
    TokTable &tab = tabs[wave];

    bf16x8 q[S::KS], go[S::KS];
    float delta = 0.f;
#pragma unroll
    for (int ks = 0; ks < S::KS; ++ks) {
        q[ks] = row_step<D>(reinterpret_cast<const char *>(Q + row * D), g, ks);
        go[ks] = row_step<D>(reinterpret_cast<const char *>(dO + row * D), g, ks);
        const bf16x8 ov = row_step<D>(reinterpret_cast<const char *>(O + row * D), g, ks);
#pragma unroll
        for (int x = 0; x < 8; ++x) delta = fmaf((float)go[ks][x], (float)ov[x], delta);
    }
    delta = rows_sum(delta);
    if (g == 0 && i16 < qt.nq) Dsum[row] = delta;
    const float lse = LSE[row], scale = args.scale;
    f32x4 acc[S::NT];
    const int len = args.len, ntile = (len + 31) >> 5;

    auto pass = [&](auto exact) {
        constexpr bool Exact = decltype(exact)::value;
        const int lane = pass_lane<Exact>(lane0), g = lane >> 4;
        const TileOffsets<D> o = tile_offsets<D>(lane);
#pragma unroll
        for (int n = 0; n < S::NT; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
        walk.put(tab, t, qt.bh, qt.blk, 0, lane);
        u32x4 kreg[S::VCH], vreg[S::VCH];
        auto load = [&](int j) {
#pragma unroll
            for (int u = 0; u < S::VCH; ++u) {
                const int x = 32 * (j & 1) + lane / S::PARTS + S::KPU * u;
                kreg[u] = gload<u32x4>(tab.k[x] + (lane % S::PARTS) * 16);
                vreg[u] = gload<u32x4>(tab.v[x] + (lane % S::PARTS) * 16);
            }
        };
        __builtin_amdgcn_wave_barrier();
        load(0);
        for (int j = 0; j < ntile; ++j) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < S::VCH; ++u) {
                const int r = lane / S::PARTS + S::KPU * u, off = r * S::ROWB + (((lane % S::PARTS) ^ swz_key<D>(r)) << 4);
                *reinterpret_cast<u32x4 *>(kt + off) = kreg[u];
                *reinterpret_cast<u32x4 *>(vt + off) = vreg[u];
            }
            __builtin_amdgcn_wave_barrier();
            f32x4 bias[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) bias[h] = *reinterpret_cast<const f32x4 *>(&tab.bias[32 * (j & 1) + 16 * h + 4 * g]);
            if (j + 1 < ntile) {                                // the registers are free: the next rows fly during all of the math
                if (j & 1) {
                    __builtin_amdgcn_wave_barrier();
                    walk.put(tab, t, qt.bh, qt.blk, 32 * (j + 1), lane);
                    __builtin_amdgcn_wave_barrier();
                }
                load(j + 1);
            }
            f32x4 s[2], dp[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                s[h] = f32x4{0.f, 0.f, 0.f, 0.f};
                dp[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < S::KS; ++ks) {
                    s[h] = mfma16(row_zero<D>(ld_bf16x8(kt + 16 * h * S::ROWB + o.row[ks]), g), q[ks], s[h]);
                    dp[h] = mfma16(row_zero<D>(ld_bf16x8(vt + 16 * h * S::ROWB + o.row[ks]), g), go[ks], dp[h]);
                }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r)                     // past the end of the list: weight -inf, P = 0
                    s[h][r] = exp_nat(fmaf(s[h][r], scale, bias[h][r]) - lse) * (dp[h][r] - delta);
            add_product<D, Exact>(acc, kt, o, s, len - 32 * j, g);
        }
    };
    pass(std::false_type{});
    if (any_nan(acc)) pass(std::true_type{});
    if (i16 >= qt.nq) return;
#pragma unroll
    for (int n = 0; n < S::NT; ++n)
        st_e(dQ + row * D + 16 * n + 4 * g, FVec<4>{{acc[n][0] * scale, acc[n][1] * scale, acc[n][2] * scale, acc[n][3] * scale}});
}

template <class F> static hipError_t by_d(int d, F f) {
    switch (d) {
        case 16: f(std::integral_constant<int, 16>{}); break;
        case 32: f(std::integral_constant<int, 32>{}); break;
        case 64: f(std::integral_constant<int, 64>{}); break;
        default: f(std::integral_constant<int, 128>{}); break;
    }
    return hipGetLastError();
}

hipError_t launch_attn_fwd_tile_bf16(const Plan &p, const TokArgs &a, const void *Q, void *O, float *LSE, hipStream_t s) {
    return by_d(p.d, [&](auto d) {
        tile_fwd_bf16_kernel<d.value><<<(a.total + 3) / 4, 256, 0, s>>>(a, (const uint16_t *)Q, (uint16_t *)O, LSE, p.N);
    });
}

hipError_t launch_dq_tile_bf16(const Plan &p, const TokArgs &a, const void *Q, const void *O, const void *dO, const float *LSE,
                               float *D, void *dQ, const CscSmall &csc, hipStream_t s) {
    return by_d(p.d, [&](auto d) {
        tile_dq_bf16_kernel<d.value><<<(a.total + 3) / 4 + csc.wgs, 256, 0, s>>>(a, (const uint16_t *)Q, (const uint16_t *)O, (const uint16_t *)dO,
                                                                     LSE, D, (uint16_t *)dQ, p.N, csc);
    });
}

}  // namespace llsa
