// Hierarchical Top-K selection, one level (Alg. 1, selection loop), for bf16, B in {16, 32, 64} and 16 < K <= 64 (fewer picks:
// select_mfma.hip, whose sorted lists of K entries per query do not fit the registers here).
//
// One workgroup (256 threads) per level-l query block of 16 query tokens.  The candidate key rows (all
// n_L tokens at the coarsest level, the 16 * K_l children of the parent's picks below it) and the 16
// query rows are staged in LDS; lane (row r, column group c) scores candidates c, c + 16, ... of
// row r, so all scores of a row sit in one 16-lane row group and the Top-K runs in registers.
// Scores are fp32 fused-multiply-add chains over channels 0 .. d-1 in order (the same chain on every
// launch shape), ties go to the lower key id, rows are written in ascending id order.
//
// A score and its candidate position become one number of type double, larger = better, no two alike: the score's bits made
// monotonic above the position's complement.  A round of arg-max is then a chain of v_max_f64 (over the 16 lanes of a row by
// DPP), and whatever the scores are, infinities and NaN among them, the winners are different candidates of the list.
// At most 256 candidates (ONE): a single pass with no running list, and the coarsest level can ride along (TOP).
// Bound: the rounds (21 max, 16 compare-and-clear per pick) and, at d = 128, LDS reads.  Forward call, 4 heads x 16384 tokens, K = 64,
// L = 3: 387 -> 253 us with comparisons of (score, id) pairs and lane permutes replaced; 4 x 1024, K = 64, L = 1: 95 -> 62.
#include <type_traits>

#include "mfma_common.h"

namespace llsa {

__device__ __forceinline__ void unpack8(u32x4 w, float *f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(w[i] << 16);
        f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}

constexpr uint32_t kPos = 0x7fffffffu;                      // 31 bits of position
__device__ __forceinline__ double dense_key(float score, uint32_t pos) {
    const uint32_t u = __float_as_uint(score + 0.f);         // -0 ties with +0
    uint32_t o = u ^ (uint32_t)(((int32_t)u >> 31) | (int32_t)0x80000000);
    o = min(max(o, 0x00200000u), 0xffdfffffu);               // NaN only: keeps the double's exponent off 0 and 0x7ff
    return __hiloint2double((int)(o >> 1), (int)((o << 31) | (kPos - pos)));
}
__device__ __forceinline__ int dense_pos(double k) { return (int)(kPos - ((uint32_t)__double2loint(k) & kPos)); }
template <int CTRL> __device__ __forceinline__ double dpp_max(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true);
    return fmax(x, __hiloint2double(hi, lo));
}
__device__ __forceinline__ double row16_max(double x) {      // over the 16 lanes of a row group: row_ror by 8, 4, 2, 1
    return dpp_max<0x121>(dpp_max<0x122>(dpp_max<0x124>(dpp_max<0x128>(x))));
}

// The coarsest level's selection for a launch that runs the level below it as well (TOP).
struct DenseTop {
    const uint16_t *Q, *K;       // Q^(L), K^(L): [bh, n, D]
    int32_t *out;                // I^(L-1): [bh, n, Kp]
    int n;                       // tokens of level L per head (<= 64)
};

// More than 256 candidates pass through LDS 256 at a time, and the row group keeps its K best so far (lane k % 16: the
// k-th best), which compete in the next chunk's rounds as further candidates of the lane.
// TOP: the first wave scores the level-L token above the workgroup's queries against the at most 64 keys of that level (same
// chain, same rule), which yields the row of I^(L-1) it needs as `parent`; the workgroup with the row's first queries writes it out.
template <int D, bool ONE, bool TOP>
__global__ void __launch_bounds__(256) select_dense_kernel(const uint16_t *__restrict__ Ql, const uint16_t *__restrict__ Kl,
                                                            int64_t n_l, const int32_t *__restrict__ parent, int Kp, int C,
                                                            int Kout, int32_t *__restrict__ out, int64_t nblk, int lb, DenseTop top) {
    constexpr int STRIDE = 2 * D + 16, CH = D / 8, MC = 16, KW = 4;
    __shared__ __attribute__((aligned(16))) char kc[256 * STRIDE];
    __shared__ __attribute__((aligned(16))) char qs[16 * STRIDE];

    const int tid = threadIdx.x;
    const int64_t bh = blockIdx.x / nblk, r = blockIdx.x % nblk;
    const uint16_t *Kb = Kl + bh * n_l * D;
    const int Bm1 = (1 << lb) - 1;
    const int32_t *prow = parent ? parent + (bh * (n_l >> lb) + (r >> (lb - 4))) * Kp : nullptr;
    if constexpr (TOP) {
        __shared__ int32_t prow_sh[16];
        if (tid < 64) {
            const int64_t q = r >> (lb - 4);                 // the level-L token above this query block
            const uint16_t *qrow = top.Q + (bh * top.n + q) * D, *krow = top.K + (bh * top.n + min(tid, top.n - 1)) * D;
            float sc = 0.f;
            for (int ch = 0; ch < CH; ++ch) {
                float qf[8], kf[8];
                unpack8(*reinterpret_cast<const u32x4 *>(qrow + ch * 8), qf);
                unpack8(*reinterpret_cast<const u32x4 *>(krow + ch * 8), kf);
#pragma unroll
                for (int e = 0; e < 8; ++e) sc = __builtin_fmaf(qf[e], kf[e], sc);
            }
            double key = tid < top.n ? dense_key(sc, (uint32_t)tid) : 0.0;
            int won = 0;                                     // lane k: the k-th winner
            for (int k = 0; k < Kp; ++k) {
                double b = row16_max(key);
                b = fmax(b, __shfl_xor(b, 16, 64));
                b = fmax(b, __shfl_xor(b, 32, 64));
                key = key == b ? 0.0 : key;
                won = tid == k ? dense_pos(b) : won;
            }
            int rank = 0;                                    // rows are stored in ascending id order
            for (int k = 0; k < Kp; ++k) rank += (__shfl(won, k, 64) < won) ? 1 : 0;
            if (tid < Kp) {
                prow_sh[rank] = won;
                if ((r & ((1 << (lb - 4)) - 1)) == 0) top.out[(bh * top.n + q) * Kp + rank] = won;
            }
        }
        __syncthreads();
        prow = prow_sh;
    }
    auto key_id = [&](int pos) { return prow ? (prow[pos >> lb] << lb) + (pos & Bm1) : pos; };
    for (int c = tid; c < 16 * CH; c += 256) {
        const int u = c / CH, part = c % CH;
        const int64_t i = min(r * 16 + u, n_l - 1);          // rows past a ragged end are computed but not stored
        *reinterpret_cast<u32x4 *>(qs + u * STRIDE + part * 16) =
            *reinterpret_cast<const u32x4 *>(Ql + (bh * n_l + i) * D + part * 8);
    }
    const int cg = tid & 15, row = tid >> 4;
    double best[KW];                                         // lane k % 16 of the row group: k-th best so far
#pragma unroll
    for (int w = 0; w < KW; ++w) best[w] = 0.0;
    for (int c0 = 0; c0 < C; c0 += 256) {
        const int cnt = ONE ? C : min(256, C - c0);
        if (!ONE) __syncthreads();                           // the previous chunk has been scored
        for (int c = tid; c < cnt * CH; c += 256) {
            const int p = c / CH, part = c % CH;
            const int64_t id = key_id(c0 + p);
            *reinterpret_cast<u32x4 *>(kc + p * STRIDE + part * 16) = *reinterpret_cast<const u32x4 *>(Kb + id * D + part * 8);
        }
        __syncthreads();
        float sc[MC];
#pragma unroll
        for (int m = 0; m < MC; ++m) sc[m] = 0.f;
        for (int ch = 0; ch < CH; ++ch) {
            float q[8];
            unpack8(*reinterpret_cast<const u32x4 *>(qs + row * STRIDE + ch * 16), q);
#pragma unroll
            for (int m = 0; m < MC; ++m) {
                float k[8];
                unpack8(*reinterpret_cast<const u32x4 *>(kc + min(cg + 16 * m, cnt - 1) * STRIDE + ch * 16), k);
#pragma unroll
                for (int e = 0; e < 8; ++e) sc[m] = __builtin_fmaf(q[e], k[e], sc[m]);
            }
        }
        double key[MC];
#pragma unroll
        for (int m = 0; m < MC; ++m) key[m] = cg + 16 * m < cnt ? dense_key(sc[m], (uint32_t)(c0 + cg + 16 * m)) : 0.0;
        double old[KW];                                      // this lane's entries of the running list compete too
#pragma unroll
        for (int w = 0; w < KW; ++w) { old[w] = best[w]; best[w] = 0.0; }
        for (int k = 0; k < Kout; ++k) {
            double b = key[0];
#pragma unroll
            for (int m = 1; m < MC; ++m) b = fmax(b, key[m]);
            if (!ONE)
#pragma unroll
                for (int w = 0; w < KW; ++w) b = fmax(b, old[w]);
            b = row16_max(b);
            if (!ONE)
#pragma unroll
                for (int w = 0; w < KW; ++w) old[w] = old[w] == b ? 0.0 : old[w];
#pragma unroll
            for (int m = 0; m < MC; ++m) key[m] = key[m] == b ? 0.0 : key[m];
#pragma unroll
            for (int w = 0; w < KW; ++w) best[w] = k == cg + 16 * w ? b : best[w];
        }
    }
    int pos[KW], rank[KW];                                   // positions ascend with the key id: rank the winners by position
#pragma unroll
    for (int w = 0; w < KW; ++w) { pos[w] = dense_pos(best[w]); rank[w] = 0; }
#pragma unroll
    for (int w2 = 0; w2 < KW; ++w2)
        for (int k = 0; k < 16 && 16 * w2 + k < Kout; ++k) {
            const int other = __shfl(pos[w2], k, 16);
#pragma unroll
            for (int w = 0; w < KW; ++w) rank[w] += (other < pos[w]) ? 1 : 0;
        }
    const int64_t i = r * 16 + row;
#pragma unroll
    for (int w = 0; w < KW; ++w)
        if (cg + 16 * w < Kout && i < n_l) out[(bh * n_l + i) * Kout + rank[w]] = key_id(pos[w]);
}

// true if the kernel covers this level
bool select_dense_ok(const Plan &p, int l) {
    const int64_t C = (l == p.L) ? p.n[l] : (int64_t)p.Kl[l] * p.B;
    // any number of candidates (256 at a time beyond 256); 16 consecutive query tokens share their candidates
    return p.blocks16 && p.Kl[l - 1] <= 64 && p.n[l] < ((int64_t)1 << 30) && C < (1 << 30) &&
           (l == p.L || p.n[l] % 16 == 0);
}

// Level L - 1 here, and level L in the same launch?
bool select_dense_top_ok(const Plan &p) {
    return p.L >= 2 && select_dense_ok(p, p.L - 1) && p.n[p.L] <= 64 && p.Kl[p.L - 1] <= 16 && p.Kl[p.L - 1] * p.B <= 256;
}

hipError_t launch_select_dense(const Plan &p, int l, const void *ws, const int32_t *parent, int32_t *out, hipStream_t s, int32_t *top_out) {
    const char *w = static_cast<const char *>(ws);
    const bool dense = (l == p.L);
    const int64_t nblk = (p.n[l] + 15) / 16;
    const uint16_t *Ql = (const uint16_t *)(w + p.pyr_off[0][l]), *Kl = (const uint16_t *)(w + p.pyr_off[1][l]);
    const int32_t *par = dense ? nullptr : parent;
    const int Kp = dense ? 0 : p.Kl[l], Kout = p.Kl[l - 1], C = dense ? (int)p.n[l] : p.Kl[l] * p.B;
    const DenseTop top = {(const uint16_t *)(w + p.pyr_off[0][p.L]), (const uint16_t *)(w + p.pyr_off[1][p.L]), top_out, (int)p.n[p.L]};
    auto go = [&](auto d, auto one, auto tp) {
        select_dense_kernel<decltype(d)::value, decltype(one)::value, decltype(tp)::value>
            <<<(unsigned)(p.bh * nblk), 256, 0, s>>>(Ql, Kl, p.n[l], par, Kp, C, Kout, out, nblk, p.lb, top);
    };
    auto by_c = [&](auto d) {
        if (top_out) go(d, std::true_type{}, std::true_type{});
        else if (C <= 256) go(d, std::true_type{}, std::false_type{});
        else go(d, std::false_type{}, std::false_type{});
    };
    if (p.d == 64) by_c(std::integral_constant<int, 64>{});
    else by_c(std::integral_constant<int, 128>{});
    return hipGetLastError();
}

}  // namespace llsa
