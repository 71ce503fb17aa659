// The steps around the attention, for any supported shape and both I/O types: pooling, the layer glue fused with it, the
// portable selection, the index transpose, the mask comparator and the index reordering.
#include "csc_small.h"

#include <math.h>
#include <string.h>

namespace llsa {

// ------------------------------------------------------------------------------------------ element types
struct bf16_t { uint16_t v; };

__device__ __forceinline__ float to_f(float x) { return x; }
__device__ __forceinline__ float to_f(bf16_t x) { return __uint_as_float(((uint32_t)x.v) << 16); }

template <class T> __device__ __forceinline__ T from_f(float f);
template <> __device__ __forceinline__ float from_f<float>(float f) { return f; }
template <> __device__ __forceinline__ bf16_t from_f<bf16_t>(float f) {
    // round to nearest even; inf / nan pass through unchanged in their upper half
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) != 0x7f800000u) u += 0x7fffu + ((u >> 16) & 1u);
    bf16_t r; r.v = (uint16_t)(u >> 16);
    return r;
}

template <class T> struct Vec;                       // 16-byte vector of T
template <> struct Vec<float>  { static constexpr int n = 4; };
template <> struct Vec<bf16_t> { static constexpr int n = 8; };

template <class T> __device__ __forceinline__ void load_vec(const T *p, float *out);
template <> __device__ __forceinline__ void load_vec<float>(const float *p, float *out) {
    float4 v = *reinterpret_cast<const float4 *>(p);
    out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
}
template <> __device__ __forceinline__ void load_vec<bf16_t>(const bf16_t *p, float *out) {
    uint4 v = *reinterpret_cast<const uint4 *>(p);
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        out[2 * i] = __uint_as_float(w[i] << 16);
        out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}
template <class T> __device__ __forceinline__ void store_vec(T *p, const float *in);
template <> __device__ __forceinline__ void store_vec<float>(float *p, const float *in) {
    *reinterpret_cast<float4 *>(p) = make_float4(in[0], in[1], in[2], in[3]);
}
template <> __device__ __forceinline__ void store_vec<bf16_t>(bf16_t *p, const float *in) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        w[i] = (uint32_t)from_f<bf16_t>(in[2 * i]).v | ((uint32_t)from_f<bf16_t>(in[2 * i + 1]).v << 16);
    *reinterpret_cast<uint4 *>(p) = make_uint4(w[0], w[1], w[2], w[3]);
}

// ------------------------------------------------------------------------------------------------ pooling
// Alg. 1, compression loop: out[t] = (x[tB] + x[tB+1] + ... + x[tB+B-1]) / B, summed in that order in
// fp32, one IEEE division, one rounding to the I/O type.  The order is part of the contract: the
// selection below is decided on these values, so they must not depend on the launch shape.
//
// A workgroup also pools its own output further (up[0], up[1], ..: the levels above).  Its 256 / (d / VN) output tokens
// are whole groups of B, of B * B, .. as far as B divides them: their rounded values pass through LDS and are summed in
// the same ascending order, so every level is bit for bit what a launch of its own would write.  What bounds these
// kernels beyond level 1 is the launch (3 to 4 us each, one after the other), not the few MB that they read: a training
// step on 256 fp32 tokens at B = 4, three levels in one launch instead of three, 46.4 -> 40.2 us.
constexpr int kPoolUp = kMaxL - 1;
struct PoolArgs { const void *in[3]; void *out[3]; void *up[3][kPoolUp]; int n_up; };

// How many of the levels above `l` a workgroup whose output is level l can make: whole groups only.
static int pool_up_levels(const Plan &p, int l) {
    const int vpr = p.d / (16 / p.elt);
    int n = 0;
    for (int tok = 256 / vpr; l + n < p.L && tok % p.B == 0; tok /= p.B) ++n;
    return n;
}

// s: the mean that this thread holds of (token first + threadIdx.x / vpr, channels cv * VN ..), live where that token
// exists.  lds: 256 * VN floats.  The whole workgroup calls.  `left`: the existing tokens from `first` on.
template <class T>
__device__ __forceinline__ void pool_above(float (&s)[Vec<T>::n], float *lds, void *const *up, int n_up, int64_t first,
                                           int64_t left, int d, int B) {
    constexpr int VN = Vec<T>::n;
    const int vpr = d / VN, tl = threadIdx.x / vpr, cv = threadIdx.x % vpr;
    int live = (int)min((int64_t)(256 / vpr), left);       // a multiple of B for each level that is still to come
    const float Bf = (float)B;
    for (int k = 0; k < n_up; ++k) {
        if (tl < live)
#pragma unroll
            for (int e = 0; e < VN; ++e) lds[threadIdx.x * VN + e] = to_f(from_f<T>(s[e]));   // what was stored, as fp32
        __syncthreads();
        live /= B;
        first /= B;
        if (tl < live) {
#pragma unroll
            for (int e = 0; e < VN; ++e) s[e] = 0.f;
            for (int r = 0; r < B; ++r)
#pragma unroll
                for (int e = 0; e < VN; ++e) s[e] = s[e] + lds[((tl * B + r) * vpr + cv) * VN + e];
#pragma unroll
            for (int e = 0; e < VN; ++e) s[e] = __fdiv_rn(s[e], Bf);
            store_vec<T>(static_cast<T *>(up[k]) + (first + tl) * (int64_t)d + cv * VN, s);
        }
        __syncthreads();                                   // read before the next level overwrites it
    }
}

// One token's mean over its B rows.  BC: block size known at compile time (the row loop is unrolled, so all B loads of a
// thread are in flight at once), or 0 to take it from the argument.  Same order of additions either way.
template <class T, int BC>
__device__ __forceinline__ void pool_rows(const T *in, int d, int B, float (&s)[Vec<T>::n]) {
    constexpr int VN = Vec<T>::n;
    if constexpr (BC != 0) {
        float x[BC][VN];
#pragma unroll
        for (int r = 0; r < BC; ++r) load_vec<T>(in + (int64_t)r * d, x[r]);
#pragma unroll
        for (int r = 0; r < BC; ++r)
#pragma unroll
            for (int e = 0; e < VN; ++e) s[e] = s[e] + x[r][e];
    } else {
        int r0 = 0;
        for (; r0 + 16 <= B; r0 += 16) {                   // 16 rows in flight at a time, added in row order
            float x[16][VN];
#pragma unroll
            for (int r = 0; r < 16; ++r) load_vec<T>(in + (int64_t)(r0 + r) * d, x[r]);
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int e = 0; e < VN; ++e) s[e] = s[e] + x[r][e];
        }
        float x[VN];
        for (int r = r0; r < B; ++r) {
            load_vec<T>(in + (int64_t)r * d, x);
#pragma unroll
            for (int e = 0; e < VN; ++e) s[e] = s[e] + x[e];
        }
    }
    const float Bf = (float)B;
#pragma unroll
    for (int e = 0; e < VN; ++e) s[e] = __fdiv_rn(s[e], Bf);
}

template <class T, int BC>
__global__ void __launch_bounds__(256) pool_kernel(PoolArgs a, int64_t n_out_total, int d, int B_arg) {
    constexpr int VN = Vec<T>::n;
    __shared__ float lds[256 * VN];
    const int B = BC ? BC : B_arg;
    const int vpr = d / VN;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t t = idx / vpr;
    const int cv = (int)(idx % vpr), y = blockIdx.y;
    float s[VN];
#pragma unroll
    for (int e = 0; e < VN; ++e) s[e] = 0.f;
    if (t < n_out_total) {
        pool_rows<T, BC>(static_cast<const T *>(a.in[y]) + (t * B) * (int64_t)d + cv * VN, d, B, s);
        store_vec<T>(static_cast<T *>(a.out[y]) + t * (int64_t)d + cv * VN, s);
    }
    if (a.n_up == 0) return;
    const int64_t first = (int64_t)blockIdx.x * (256 / vpr);
    pool_above<T>(s, lds, a.up[y], a.n_up, first, n_out_total - first, d, B);
}

// Levels `from` .. L of the tensors x0 .. 2 (0 = Q, 1 = K, 2 = V; src: their level 0, used where from is 1).
static hipError_t pool_levels(const Plan &p, const void *const *src, char *w, int from, int x0, hipStream_t s) {
    for (int l = from; l <= p.L;) {
        PoolArgs a{};
        a.n_up = pool_up_levels(p, l);
        for (int x = x0; x < 3; ++x) {
            a.in[x - x0] = (l == 1) ? src[x] : (const void *)(w + p.pyr_off[x][l - 1]);
            a.out[x - x0] = w + p.pyr_off[x][l];
            for (int k = 0; k < a.n_up; ++k) a.up[x - x0][k] = w + p.pyr_off[x][l + 1 + k];
        }
        const int64_t n_out_total = (int64_t)p.bh * p.n[l];
        const int64_t threads = n_out_total * (p.d / (16 / p.elt));
        dim3 grid((unsigned)((threads + 255) / 256), 3 - x0);
        if (p.elt == 4)     pool_kernel<float, 0><<<grid, 256, 0, s>>>(a, n_out_total, p.d, p.B);
        else if (p.B == 16) pool_kernel<bf16_t, 16><<<grid, 256, 0, s>>>(a, n_out_total, p.d, p.B);
        else                pool_kernel<bf16_t, 0><<<grid, 256, 0, s>>>(a, n_out_total, p.d, p.B);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        l += 1 + a.n_up;
    }
    return hipSuccess;
}

hipError_t launch_pool(const Plan &p, const void *Q, const void *K, const void *V, void *ws, bool q_too,
                       hipStream_t s) {
    const void *src[3] = {Q, K, V};
    return pool_levels(p, src, static_cast<char *>(ws), 1, q_too ? 0 : 1, s);
}

// ----------------------------------------------------------------------- layer glue fused with pooling
// QK-Norm and RoPE in front of the layer (Sec. 5.2, "Training Settings") fused with the first step of the
// compression loop of Alg. 1: one pass over the pre-norm tensor writes the level-0 tensor the layer consumes
// and its level-1 mean, so the level-0 tensor is never read back for pooling.
//   y[c]      = x[c] / sqrt(mean_c(x^2) + eps) * gamma[c]                      (per token, over the head dimension)
//   out[2i]   = y[2i] cos[t][i] - y[2i+1] sin[t][i]
//   out[2i+1] = y[2i] sin[t][i] + y[2i+1] cos[t][i]                             (t: token index within the head)
// out is rounded to the I/O type; the level-1 token is pooled from those rounded values exactly as pool_kernel
// does it (ascending fp32 sum, one division, one rounding), so it equals pool_kernel's result on `out` bit for bit.
// One thread per (level-1 token, 16-byte channel vector); the d / VN threads of a token are neighbouring lanes and
// reduce the sum of squares of a row with xor shuffles.  grid.y: 0 = Q, 1 = K, 2 = V, which is only pooled.
// The levels above come from the same workgroup where its tokens are whole groups: 32 x 16384 tokens, d = 64, three
// levels, glue and layer 206 -> 194.5 us, with two launches before the selection where there were four.
struct GlueArgs { const void *in[2]; void *out[2]; const float *gamma[2]; PoolArgs pool; };

template <class T>
__global__ void __launch_bounds__(256) qknorm_rope_pool_kernel(GlueArgs a, const float *__restrict__ cos_t,
                                                               const float *__restrict__ sin_t, float eps,
                                                               int64_t n1_total, int64_t N, int d, int B) {
    constexpr int VN = Vec<T>::n, ROWS = 4;                // rows of one token group in flight at a time
    __shared__ float lds[256 * VN];
    const int vpr = d / VN;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t t1 = idx / vpr;                          // level-1 token, flat over (batch, head)
    const int cv = (int)(idx % vpr);
    const int y = blockIdx.y;
    float s[VN];
#pragma unroll
    for (int e = 0; e < VN; ++e) s[e] = 0.f;
    if (t1 < n1_total) {                                   // whole token groups are in or out together (vpr divides 64)
        if (y == 2) {
            pool_rows<T, 0>(static_cast<const T *>(a.pool.in[2]) + (t1 * B) * (int64_t)d + cv * VN, d, B, s);
        } else {
            const T *in = static_cast<const T *>(a.in[y]) + (t1 * B) * (int64_t)d + cv * VN;
            T *out = static_cast<T *>(a.out[y]) + (t1 * B) * (int64_t)d + cv * VN;
            const int64_t tok0 = (t1 * B) % N;                     // position of the group's first token inside its head
            float gam[VN];
#pragma unroll
            for (int e = 0; e < VN; ++e) gam[e] = a.gamma[y][cv * VN + e];
            const float inv_d = 1.f / (float)d;
            for (int r0 = 0; r0 < B; r0 += ROWS) {
                float x[ROWS][VN], cs[ROWS][VN / 2], sn[ROWS][VN / 2];
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                    const int rr = min(r0 + r, B - 1);             // B need not be a multiple of ROWS: the tail re-reads
                    load_vec<T>(in + (int64_t)rr * d, x[r]);
                    const int64_t tab = (tok0 + rr) * (d / 2) + cv * (VN / 2);
#pragma unroll
                    for (int e = 0; e < VN / 2; ++e) { cs[r][e] = cos_t[tab + e]; sn[r][e] = sin_t[tab + e]; }
                }
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                    float ss = 0.f;
#pragma unroll
                    for (int e = 0; e < VN; ++e) ss = fmaf(x[r][e], x[r][e], ss);
                    for (int o = 1; o < vpr; o <<= 1) ss += __shfl_xor(ss, o, 64);
                    const float rinv = 1.f / sqrtf(fmaf(ss, inv_d, eps));
                    float o8[VN];
#pragma unroll
                    for (int e = 0; e < VN / 2; ++e) {
                        const float y0 = x[r][2 * e] * rinv * gam[2 * e], y1 = x[r][2 * e + 1] * rinv * gam[2 * e + 1];
                        o8[2 * e] = to_f(from_f<T>(y0 * cs[r][e] - y1 * sn[r][e]));
                        o8[2 * e + 1] = to_f(from_f<T>(y0 * sn[r][e] + y1 * cs[r][e]));
                    }
                    if (r0 + r < B) {
                        store_vec<T>(out + (int64_t)(r0 + r) * d, o8);
#pragma unroll
                        for (int e = 0; e < VN; ++e) s[e] = s[e] + o8[e];
                    }
                }
            }
            const float Bf = (float)B;
#pragma unroll
            for (int e = 0; e < VN; ++e) s[e] = __fdiv_rn(s[e], Bf);
        }
        store_vec<T>(static_cast<T *>(a.pool.out[y]) + t1 * (int64_t)d + cv * VN, s);
    }
    if (a.pool.n_up == 0) return;
    const int64_t first = (int64_t)blockIdx.x * (256 / vpr);
    pool_above<T>(s, lds, a.pool.up[y], a.pool.n_up, first, n1_total - first, d, B);
}

// One launch for everything up to the last level that whole groups of a workgroup reach, pool_kernel for the rest.
hipError_t launch_qknorm_rope_pool(const Plan &p, const void *Qpre, const void *Kpre, const void *V,
                                   const float *gamma_q, const float *gamma_k, const float *cos_t, const float *sin_t,
                                   float eps, void *Qout, void *Kout, void *ws, hipStream_t s) {
    char *w = static_cast<char *>(ws);
    GlueArgs g{};
    g.in[0] = Qpre; g.in[1] = Kpre;
    g.out[0] = Qout; g.out[1] = Kout;
    g.gamma[0] = gamma_q; g.gamma[1] = gamma_k;
    g.pool.in[2] = V;
    g.pool.n_up = pool_up_levels(p, 1);
    for (int x = 0; x < 3; ++x) {
        g.pool.out[x] = w + p.pyr_off[x][1];
        for (int k = 0; k < g.pool.n_up; ++k) g.pool.up[x][k] = w + p.pyr_off[x][2 + k];
    }
    const int64_t n1_total = (int64_t)p.bh * p.n[1];
    const int64_t threads = n1_total * (p.d / (16 / p.elt));
    dim3 grid((unsigned)((threads + 255) / 256), 3);
    if (p.elt == 4) qknorm_rope_pool_kernel<float><<<grid, 256, 0, s>>>(g, cos_t, sin_t, eps, n1_total, p.N, p.d, p.B);
    else            qknorm_rope_pool_kernel<bf16_t><<<grid, 256, 0, s>>>(g, cos_t, sin_t, eps, n1_total, p.N, p.d, p.B);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return pool_levels(p, nullptr, w, 2 + g.pool.n_up, 0, s);
}

// ---------------------------------------------------------------------------------------------- selection
// Alg. 1, selection loop, one level: every wave scores one level-l query token against its candidates
// (all n_L tokens at the coarsest level, the K_l*B children of the parent's picks below it) and keeps the
// Kout best.  Scores are fp32 fused-multiply-add chains over channels 0..d-1 in order, so they do not
// depend on the launch shape; ties go to the lower key id; rows are written in ascending id order.  A score is kept as its bits made
// monotonic, 1 at least (0: taken already), so that the winners are different candidates also where scores are infinite or NaN.
template <class T>
__global__ void select_kernel(const T *Ql, const T *Kl, int64_t n_l, int d, int B, const int32_t *parent, int Kp,
                              int Kout, int32_t *out, int C, int64_t nblk) {
    extern __shared__ float smem[];
    const int W = blockDim.x >> 6, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float *qs = smem + wave * d;
    uint32_t *sc = reinterpret_cast<uint32_t *>(smem + W * d) + (size_t)wave * C;
    const int64_t bh = blockIdx.x / nblk, r = blockIdx.x % nblk;
    const T *Kb = Kl + bh * n_l * d;
    const int32_t *prow = parent ? parent + (bh * nblk + r) * Kp : nullptr;
    const int iters = (B + W - 1) / W;
    for (int it = 0; it < iters; ++it) {
        const int u = it * W + wave;
        const int64_t i = r * B + u;
        const bool active = (u < B) && (i < n_l);
        __syncthreads();                                   // previous row's LDS no longer read
        if (active)
            for (int c = lane; c < d; c += 64) qs[c] = to_f(Ql[(bh * n_l + i) * d + c]);
        __syncthreads();
        if (active)
            for (int p = lane; p < C; p += 64) {
                const int64_t id = prow ? (int64_t)prow[p / B] * B + p % B : p;
                const T *k = Kb + id * d;
                float s = 0.f, tmp[Vec<T>::n];
                for (int c = 0; c < d; c += Vec<T>::n) {
                    load_vec<T>(k + c, tmp);
#pragma unroll
                    for (int e = 0; e < Vec<T>::n; ++e) s = __builtin_fmaf(qs[c + e], tmp[e], s);
                }
                const uint32_t b = __float_as_uint(s + 0.f);     // -0 ties with +0
                sc[p] = max(b ^ (uint32_t)(((int32_t)b >> 31) | (int32_t)0x80000000), 1u);
            }
        int mine = 0;                                      // lane k keeps the k-th winner's position
        for (int k = 0; k < Kout; ++k) {
            __syncthreads();
            uint32_t bs = 0;
            int bp = 0x7fffffff;
            if (active)
                for (int p = lane; p < C; p += 64) {
                    const uint32_t v = sc[p];
                    if (v > bs) { bs = v; bp = p; }        // ascending p: strict '>' keeps the lowest position
                }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) {
                const uint32_t os = __shfl_xor(bs, o, 64);
                const int op = __shfl_xor(bp, o, 64);
                if (os > bs || (os == bs && op < bp)) { bs = os; bp = op; }
            }
            if (active && lane == (bp & 63)) sc[bp] = 0;
            if (lane == k) mine = bp;
        }
        if (active) {
            // candidate positions ascend with key id (parent rows are ascending), so rank by position
            int rank = 0;
            for (int k = 0; k < Kout; ++k) rank += (__shfl(mine, k, 64) < mine) ? 1 : 0;
            if (lane < Kout) {
                const int64_t id = prow ? (int64_t)prow[mine / B] * B + mine % B : mine;
                out[(bh * n_l + i) * Kout + rank] = (int32_t)id;
            }
        }
    }
}

hipError_t launch_select(const Plan &p, int l, const void *ws, const int32_t *parent, int32_t *out, hipStream_t s) {
    if (select_mfma_ok(p, l)) return launch_select_mfma(p, l, ws, parent, out, s);
    if (p.desc.kernel_path == 0 && select_dense_ok(p, l)) return launch_select_dense(p, l, ws, parent, out, s);
    const char *w = static_cast<const char *>(ws);
    const bool top = (l == p.L);
    const int C = top ? (int)p.n[l] : p.Kl[l] * p.B;
    const int Kout = p.Kl[l - 1];
    const int64_t nblk = (p.n[l] + p.B - 1) / p.B;
    const int W = C <= 2048 ? 4 : (C <= 4096 ? 2 : 1);
    const size_t lds = (size_t)W * (p.d + C) * sizeof(float);
    dim3 grid((unsigned)(p.bh * nblk));
    const int Kp = top ? 0 : p.Kl[l];
    const void *Ql = w + p.pyr_off[0][l], *Kl = w + p.pyr_off[1][l];
    if (p.elt == 4)
        select_kernel<float><<<grid, W * 64, lds, s>>>((const float *)Ql, (const float *)Kl, p.n[l], p.d, p.B,
                                                       top ? nullptr : parent, Kp, Kout, out, C, nblk);
    else
        select_kernel<bf16_t><<<grid, W * 64, lds, s>>>((const bf16_t *)Ql, (const bf16_t *)Kl, p.n[l], p.d, p.B,
                                                        top ? nullptr : parent, Kp, Kout, out, C, nblk);
    return hipGetLastError();
}

// -------------------------------------------------------------------------------- index transpose (Alg. 2)
// Key-major lists, every list ascending, so that the result (and with it the summation order of dK / dV) is the same on
// every run.  All levels run in the same launches.
struct CscLevel {
    const int32_t *I;            // I^(l) [bh, T, Kl]
    int32_t *cnt, *C, *Iq, *Iq_tmp;
    int64_t T, eph, total, nk;   // keys per head, entries per head, entries, keys
    int Kl;
    uint32_t *cnt8;              // segment path: [bh][group][Tp][kSegPerGroup] bytes
    int32_t *tot;                // [bh][group][Tp]: a group's entries of a key, then where they start
    int Tp, ngrp;                // T rounded up to 4; groups
};
struct CscLevels { CscLevel lv[kMaxL]; };

// Few rows, one launch, no scratch memory (csc_small.h).
__global__ void __launch_bounds__(256) csc_bitmap_kernel(CscSmall a) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[kCscSmallLds / 4];
    csc_small<256>(a, blockIdx.x, lds);
}

// More rows, up to kSegRowsMax, three launches, O(T K) work: rows are taken in segments of 128, and segments in groups of 16.
//   count: per (group of 2048 rows, 1024 keys) the number of entries of every (segment, key), one byte each, counted in LDS,
//     and the group's sum per key;
//   scan: per head, the sums over the groups and then over the keys: C, and where each group's entries of a key start;
//   fill: per (segment, 1024 keys) a bitmap of 128 rows per key in LDS; an entry's place is the start of its group, plus the
//     counts of the group's earlier segments (one 16-byte load, summed bytewise), plus the marked rows below its own.  Level 0's tiles
//     too: in a launch of their own they were 5 to 29 us more on the stream that the level-1 gather waits for (steps, K = 4, Gaussian,
//     8 x 131072 tokens 964 -> 947 us, 4 x 212992 842 -> 836; smooth 8 x 131072 900 -> 888, 4 x 65536, K = 8 353 -> 349).
// Nothing is sorted and every place follows from counts, so the lists are ascending and the same on every run.  The kernels
// stay below 48 registers: that is what the upper-level dK/dV kernel, in whose shadow they run, leaves of a SIMD's 512.
// Each range of 1024 keys reads its rows again, so the time grows with rows^2 for few heads; the sort's grows with the lists,
// which smooth inputs make long.  Either side of the limit, sort against segments, smooth and Gaussian inputs, K = 8: one head of
// 17408 rows 114 : 89 and 50 : 90 us, two of 32768 rows 224 : 247 and 90 : 250, one of 65536 rows 336 : 834 and 127 : 841.
// grid.x: ranges of level 0's heads, then level 1's, ...
struct CscRanges { CscLevel lv[kMaxL]; unsigned wg_end[kMaxL]; };
// Level 0's lists as tiles (fine_tiles.h) from C, by 16 lanes for key block j of head bh.
struct TileRows { FineTile *tiles; int32_t *arrived; int lc; };   // tiles: null if nothing takes them
__device__ __forceinline__ void tiles_of(const TileRows &r, const int32_t *C, int64_t bh, int64_t T, int64_t E, int j, int lane) {
    const int start = C[j], end = C[j + 1];
    const int64_t places = tile_places(T, E);
    write_tiles(r.tiles + bh * places, r.arrived + bh * piece_slots(T, E, r.lc), r.lc, j, start, end - start,
                j + 1 == T ? (int)places : tile_place(end, j + 1), lane, 16);
}
static TileRows tile_rows(const Plan &p, char *w) {
    if (!dkv_by_tiles(p)) return {nullptr, nullptr, 0};
    return {(FineTile *)(w + p.tiles_off), (int32_t *)(w + p.arrived_off), fine_piece_log2(p)};
}
constexpr int kSegRowsMax = 16384, kSegR = 128, kSegPerGroup = 16, kGroupRows = kSegR * kSegPerGroup, kKeyRange = 1024;
// every entry of rows row0 .. row1 - 1 with key - k0 < kKeyRange: f(row, key - k0)
template <class F> __device__ __forceinline__ void range_entries(const int32_t *I, unsigned Kl, unsigned row0, unsigned row1, unsigned k0, F f) {
    const unsigned e1 = row1 * Kl;
    for (unsigned e = row0 * Kl + threadIdx.x; e < e1; e += 4 * 256) {
        int32_t k[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) k[u] = e + 256 * u < e1 ? I[e + 256 * u] : -1;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if ((unsigned)k[u] - k0 < (unsigned)kKeyRange) f((e + 256 * u) / Kl, (unsigned)k[u] - k0);
    }
}
__global__ void __launch_bounds__(256) csc_seg_count_kernel(CscRanges a) {
    __shared__ __attribute__((aligned(16))) uint32_t cnt[kKeyRange * 4];
    int l = 0;
    while (blockIdx.x >= a.wg_end[l]) ++l;
    const CscLevel &L = a.lv[l];
    const unsigned id = blockIdx.x - (l ? a.wg_end[l - 1] : 0), T = (unsigned)L.T, Tp = (unsigned)L.Tp;
    const unsigned ranges = (T + kKeyRange - 1) / kKeyRange, hg = id / ranges, k0 = (id - hg * ranges) * kKeyRange;
    const unsigned bh = hg / (unsigned)L.ngrp, grp = hg - bh * L.ngrp;
    for (unsigned i = threadIdx.x; i < kKeyRange; i += 256) reinterpret_cast<uint4 *>(cnt)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    range_entries(L.I + (int64_t)bh * L.eph, (unsigned)L.Kl, grp * kGroupRows, min(T, (grp + 1) * kGroupRows), k0, [&](unsigned row, unsigned k) {
        const unsigned seg = (row / kSegR) % kSegPerGroup;
        atomicAdd(&cnt[4 * k + (seg >> 2)], 1u << (8 * (seg & 3)));
    });
    __syncthreads();
    for (unsigned i = threadIdx.x; i < kKeyRange && k0 + i < T; i += 256) {
        const uint4 c = reinterpret_cast<const uint4 *>(cnt)[i];
        const int64_t o = (int64_t)hg * Tp + k0 + i;
        reinterpret_cast<uint4 *>(L.cnt8)[o] = c;
        L.tot[o] = (int32_t)__builtin_amdgcn_sad_u8(c.x, 0u, __builtin_amdgcn_sad_u8(c.y, 0u, __builtin_amdgcn_sad_u8(c.z, 0u, __builtin_amdgcn_sad_u8(c.w, 0u, 0u))));
    }
}
__global__ void __launch_bounds__(256) csc_seg_scan_kernel(CscLevels a) {
    __shared__ int32_t wsum[2][4];
    const CscLevel &L = a.lv[blockIdx.y];
    const int64_t bh = blockIdx.x;
    const int T = (int)L.T, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t *Co = L.C + bh * (T + 1), *tot = L.tot + bh * L.ngrp * L.Tp;
    int32_t carry = 0;
    for (int base = 0, turn = 0; base < T; base += 1024, turn ^= 1) {
        const int i0 = base + 4 * threadIdx.x;              // four consecutive keys per thread
        auto group = [&](int g) {                           // a group's entries of the keys
            int4 v = make_int4(0, 0, 0, 0);
            if (i0 < T) v = *reinterpret_cast<const int4 *>(tot + g * L.Tp + i0);
            if (i0 + 1 >= T) v.y = 0;
            if (i0 + 2 >= T) v.z = 0;
            if (i0 + 3 >= T) v.w = 0;
            return v;
        };
        int4 key = make_int4(0, 0, 0, 0);                   // the keys' totals
#pragma unroll 2
        for (int g = 0; g < L.ngrp; ++g) {
            const int4 v = group(g);
            key.x += v.x; key.y += v.y; key.z += v.z; key.w += v.w;
        }
        const int32_t mine = key.x + key.y + key.z + key.w;
        int32_t x = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {                  // inclusive scan of the threads' sums inside the wave
            const int32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[turn][wave] = x;
        __syncthreads();                                    // (two buffers: the next turn may write before this one is read)
        int32_t pre = carry;
        for (int w = 0; w < wave; ++w) pre += wsum[turn][w];
        for (int w = 0; w < 4; ++w) carry += wsum[turn][w];
        int4 at;                                            // where each key's list starts
        at.x = pre + x - mine; at.y = at.x + key.x; at.z = at.y + key.y; at.w = at.z + key.z;
        if (i0 < T) Co[i0] = at.x;
        if (i0 + 1 < T) Co[i0 + 1] = at.y;
        if (i0 + 2 < T) Co[i0 + 2] = at.z;
        if (i0 + 3 < T) Co[i0 + 3] = at.w;
        for (int g = 0; g < L.ngrp; ++g) {
            const int4 v = group(g);
            if (i0 < T) *reinterpret_cast<int4 *>(tot + g * L.Tp + i0) = at;
            at.x += v.x; at.y += v.y; at.z += v.z; at.w += v.w;
        }
    }
    if (threadIdx.x == 0) Co[T] = carry;
}
__global__ void __launch_bounds__(256) csc_seg_fill_kernel(CscRanges a, TileRows out) {
    __shared__ __attribute__((aligned(16))) uint32_t bm[kKeyRange * 4];
    int l = 0;
    while (blockIdx.x >= a.wg_end[l]) ++l;
    const CscLevel &L = a.lv[l];
    const unsigned id = blockIdx.x - (l ? a.wg_end[l - 1] : 0), T = (unsigned)L.T, Tp = (unsigned)L.Tp;
    const unsigned ranges = (T + kKeyRange - 1) / kKeyRange, segs = (T + kSegR - 1) / kSegR;
    const unsigned hs = id / ranges, k0 = (id - hs * ranges) * kKeyRange, bh = hs / segs, seg = hs - bh * segs;
    const int32_t *I = L.I + (int64_t)bh * L.eph;
    for (unsigned i = threadIdx.x; i < kKeyRange; i += 256) reinterpret_cast<uint4 *>(bm)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const unsigned row0 = seg * kSegR, row1 = min(T, row0 + kSegR), grp = seg / kSegPerGroup, s = seg % kSegPerGroup;
    range_entries(I, (unsigned)L.Kl, row0, row1, k0, [&](unsigned row, unsigned k) {
        const unsigned r = row - row0;
        atomicOr(&bm[4 * k + (r >> 5)], 1u << (r & 31));
    });
    __syncthreads();
    const int64_t slab = ((int64_t)bh * L.ngrp + grp) * Tp + k0;
    int32_t *Iq = L.Iq + (int64_t)bh * L.eph;
    range_entries(I, (unsigned)L.Kl, row0, row1, k0, [&](unsigned row, unsigned k) {
        const unsigned r = row - row0;
        const uint4 m = reinterpret_cast<const uint4 *>(bm)[k], c = reinterpret_cast<const uint4 *>(L.cnt8)[slab + k];
        const uint32_t mw[4] = {m.x, m.y, m.z, m.w}, cw[4] = {c.x, c.y, c.z, c.w};
        uint32_t at = (uint32_t)L.tot[slab + k];
#pragma unroll
        for (unsigned w = 0; w < 4; ++w) {                  // bits / bytes below this row / segment
            const uint32_t mb = w < (r >> 5) ? ~0u : w == (r >> 5) ? (1u << (r & 31)) - 1u : 0u;
            const uint32_t cb = w < (s >> 2) ? ~0u : w == (s >> 2) ? (1u << (8 * (s & 3))) - 1u : 0u;
            at += __popc(mw[w] & mb);
            at = __builtin_amdgcn_sad_u8(cw[w] & cb, 0u, at);
        }
        Iq[at] = (int32_t)row;
    });
    if (l == 0 && out.tiles) {                              // the range's keys are shared out among the segments' workgroups
        const unsigned share = (kKeyRange + segs - 1) / segs, end = min(T, k0 + min((seg + 1) * share, (unsigned)kKeyRange));
        for (unsigned j = k0 + seg * share + (threadIdx.x >> 4); j < end; j += 16)
            tiles_of(out, L.C + (int64_t)bh * (T + 1), bh, T, L.eph, (int)j, (int)(threadIdx.x & 15));
    }
}

// Larger levels still: count -> exclusive scan -> fill -> per-key ascending order.  Counting and filling use integer atomics; the
// order they leave inside a key's list depends on timing, so a last pass sorts every list (an entry counts the smaller ones of
// its list; lists of more than 4096 entries: a bitmap of the list's rows).  blockIdx.y selects the level.
__global__ void csc_zero_kernel(CscLevels a) {
    const CscLevel &L = a.lv[blockIdx.y];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < L.nk) L.cnt[i] = 0;
}
__global__ void csc_count_kernel(CscLevels a) {
    const CscLevel &L = a.lv[blockIdx.y];
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= L.total) return;
    const int64_t bh = e / L.eph;
    atomicAdd(&L.cnt[bh * L.T + L.I[e]], 1);
}
// one workgroup per (head, level): C = exclusive scan of cnt (T+1 entries), cnt reset to 0 for the fill pass.
// 256 threads, so that a workgroup finds room on a CU beside the LDS-bound dK/dV kernels it runs in the shadow of
// (with 1024 threads it waited for a whole CU to drain).
constexpr int kScanThreads = 256;
__global__ void __launch_bounds__(kScanThreads) csc_scan_kernel(CscLevels a) {
    constexpr int NW = kScanThreads / 64;
    __shared__ int32_t wsum[NW];
    __shared__ int32_t carry;
    const CscLevel &L = a.lv[blockIdx.y];
    const int64_t bh = blockIdx.x, T = L.T;
    int32_t *cn = L.cnt + bh * T, *Co = L.C + bh * (T + 1);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < T; base += 4 * kScanThreads) {
        // four consecutive keys per thread
        const int64_t i0 = base + 4 * threadIdx.x;
        int32_t v[4], x = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) { v[k] = i0 + k < T ? cn[i0 + k] : 0; x += v[k]; }
        const int32_t mine = x;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {                  // inclusive scan of the threads' sums inside the wave
            const int32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[wave] = x;
        __syncthreads();
        int32_t pre = carry;
        for (int w2 = 0; w2 < wave; ++w2) pre += wsum[w2];
        int32_t run = pre + x - mine;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i0 + k < T) { Co[i0 + k] = run; cn[i0 + k] = 0; }
            run += v[k];
        }
        __syncthreads();
        if (threadIdx.x == kScanThreads - 1) carry = pre + x;
        __syncthreads();
    }
    if (threadIdx.x == 0) Co[T] = carry;
}
__global__ void csc_fill_kernel(CscLevels a) {
    const CscLevel &L = a.lv[blockIdx.y];
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= L.total) return;
    const int64_t bh = e / L.eph, within = e % L.eph;
    const int32_t key = L.I[e];
    const int32_t slot = L.C[bh * (L.T + 1) + key] + atomicAdd(&L.cnt[bh * L.T + key], 1);
    L.Iq_tmp[bh * L.eph + slot] = (int32_t)(within / L.Kl);
}
// one thread per list entry: its rank among the entries of the same key (entries are distinct query rows)
// is its place in the key's ascending list.  The unsorted list is re-read through the caches.
// Lists longer than kLongList are left to csc_sort_long_kernel (this pass costs len reads per entry).
constexpr int kLongList = 4096;
__global__ void __launch_bounds__(256) csc_sort_kernel(CscLevels a) {
    const CscLevel &L = a.lv[blockIdx.y];
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= L.total) return;
    const int64_t bh = e / L.eph, within = e % L.eph;
    const int32_t key = L.I[e], x = (int32_t)(within / L.Kl);
    const int32_t beg = L.C[bh * (L.T + 1) + key], end = L.C[bh * (L.T + 1) + key + 1];
    if (end - beg > kLongList) return;
    const int32_t *src = L.Iq_tmp + bh * L.eph;
    int32_t rank = 0;
    for (int32_t b = beg; b < end; ++b) rank += (src[b] < x) ? 1 : 0;
    L.Iq[bh * L.eph + beg + rank] = x;
}
// Long lists: every lane of a wave looks at one key, and the wave then works through the long lists among its 64
// keys together (usually none): the list's rows are marked in a bitmap of kSegRows rows at a time in LDS, and an
// entry's place is the number of marked rows below it: one pass over the list per segment of rows instead of one
// pass per entry, whatever the atomic fill's order was.  Keeps the transpose linear in the list length when many
// queries pick the same key (constant keys: every row lists blocks 0 .. K-1).
constexpr int kSegRows = 8192, kSegWords = kSegRows / 32;
__global__ void __launch_bounds__(256) csc_sort_long_kernel(CscLevels a) {
    __shared__ uint32_t bm_sh[4][kSegWords];
    __shared__ int32_t pre_sh[4][kSegWords];
    const CscLevel &L = a.lv[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t key0 = ((int64_t)blockIdx.x * 4 + wave) * 64;          // this wave's keys (over all heads)
    if (key0 >= L.nk) return;
    const int64_t mykey = min(key0 + lane, L.nk - 1);
    const int32_t mybeg = L.C[(mykey / L.T) * (L.T + 1) + mykey % L.T];
    const int32_t mylen = L.C[(mykey / L.T) * (L.T + 1) + mykey % L.T + 1] - mybeg;
    uint64_t todo = __ballot(key0 + lane < L.nk && mylen > kLongList);
    uint32_t *bm = bm_sh[wave];
    int32_t *pre = pre_sh[wave];
    while (todo) {
        const int j = (int)__builtin_ctzll(todo);
        todo &= todo - 1;
        const int64_t bh = (key0 + j) / L.T;
        const int32_t beg = __shfl(mybeg, j, 64), len = __shfl(mylen, j, 64);
        const int32_t *src = L.Iq_tmp + bh * L.eph + beg;
        int32_t *dst = L.Iq + bh * L.eph + beg;
        int32_t base = 0;                                   // entries in the segments done so far
        for (int64_t s0 = 0; s0 < L.T; s0 += kSegRows) {
            for (int w = lane; w < kSegWords; w += 64) bm[w] = 0u;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (int32_t e = lane; e < len; e += 64) {
                const int64_t x = src[e] - s0;
                if (x >= 0 && x < kSegRows) atomicOr(&bm[x >> 5], 1u << (x & 31));
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // marked rows below every word: lane holds kSegWords / 64 consecutive words
            constexpr int PL = kSegWords / 64;
            int32_t c[PL], mine = 0;
#pragma unroll
            for (int i = 0; i < PL; ++i) { c[i] = __popc(bm[PL * lane + i]); mine += c[i]; }
            int32_t incl = mine;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int32_t y = __shfl_up(incl, o, 64);
                if (lane >= o) incl += y;
            }
            int32_t run = incl - mine;
#pragma unroll
            for (int i = 0; i < PL; ++i) { pre[PL * lane + i] = run; run += c[i]; }
            const int32_t total = __shfl(incl, 63, 64);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (int32_t e = lane; e < len; e += 64) {
                const int32_t v = src[e];
                const int64_t x = v - s0;
                if (x >= 0 && x < kSegRows) {
                    const int w = (int)(x >> 5);
                    dst[base + pre[w] + __popc(bm[w] & ((1u << (x & 31)) - 1u))] = v;
                }
            }
            base += total;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();                // the bitmap is cleared again only after these reads
        }
    }
}

// The workgroups' work of levels 0 .. top where there are few rows (level 0 has the most): one launch while its O(T^2) reading is cheap
// (measured with the dK/dV kernels it runs beside).
static bool csc_one_launch(const Plan &p) { return p.n[1] <= kSmallRows; }
bool csc_small_args(const Plan &p, int top, const int32_t *indices, void *ws, CscSmall *a) {
    memset(a, 0, sizeof(*a));
    if (!csc_one_launch(p)) return false;
    char *w = static_cast<char *>(ws);
    int64_t wg = 0;
    for (int l = 0; l <= top; ++l) {
        a->lv[l] = {reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(indices) + p.idx_off[l]), (int32_t *)(w + p.C_off[l]),
                    (int32_t *)(w + p.Iq_off[l]), (int32_t)p.n[l + 1], p.Kl[l]};
        wg += p.bh * ((p.n[l + 1] + kRangeKeys - 1) / kRangeKeys);
        a->wg_end[l] = (uint32_t)wg;
    }
    a->levels = top + 1;
    if (dkv_by_tiles(p)) {
        a->tiles = (FineTile *)(w + p.tiles_off);
        a->arrived = (int32_t *)(w + p.arrived_off);
        a->lc = fine_piece_log2(p);
    }
    a->wgs = (uint32_t)((wg + 7) & ~(int64_t)7);            // workgroups behind them stay on their XCDs
    return true;
}

// bytes of scratch memory the transpose of level l needs
size_t csc_scratch_bytes(const Plan &p, int l) {
    const int64_t T = p.n[l + 1];
    if (csc_one_launch(p)) return 0;
    if (p.n[1] <= kSegRowsMax) return (size_t)p.bh * ((T + kGroupRows - 1) / kGroupRows) * ((T + 3) & ~(int64_t)3) * (kSegPerGroup + 4);
    return (size_t)p.bh * T * p.Kl[l] * sizeof(int32_t);
}

// level 0's lists as tiles in a launch of their own, 16 lanes per key
__global__ void __launch_bounds__(256) fine_tiles_kernel(const int32_t *C, TileRows r, int T, int E) {
    const unsigned per_head = ((unsigned)T + 15u) / 16u, bh = blockIdx.x / per_head;
    const int j = (int)((blockIdx.x - bh * per_head) * 16 + (threadIdx.x >> 4));
    if (j < T) tiles_of(r, C + (int64_t)bh * (T + 1), bh, T, E, j, (int)(threadIdx.x & 15));
}
static hipError_t launch_fine_tiles(const Plan &p, char *w, hipStream_t s) {
    if (!dkv_by_tiles(p)) return hipGetLastError();
    fine_tiles_kernel<<<(unsigned)((p.n[1] + 15) / 16 * p.bh), 256, 0, s>>>((const int32_t *)(w + p.C_off[0]), tile_rows(p, w), (int)p.n[1],
                                                                           (int)(p.n[1] * p.Kl[0]));
    return hipGetLastError();
}

// Alg. 2 for levels 0 .. top (the levels whose lists the backward uses)
hipError_t launch_csc(const Plan &p, int top, const int32_t *indices, void *ws, hipStream_t s) {
    CscSmall few;
    if (csc_small_args(p, top, indices, ws, &few)) {
        csc_bitmap_kernel<<<few.wgs, 256, 0, s>>>(few);
        return hipGetLastError();
    }
    char *w = static_cast<char *>(ws);
    CscLevels a;
    int64_t max_nk = 0, max_total = 0;
    for (int l = 0; l <= top; ++l) {
        CscLevel &L = a.lv[l];
        L.T = p.n[l + 1];
        L.Kl = p.Kl[l];
        L.eph = L.T * L.Kl;
        L.total = L.eph * p.bh;
        L.nk = L.T * p.bh;
        L.I = reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(indices) + p.idx_off[l]);
        L.cnt = (int32_t *)(w + p.cnt_off[l]);
        L.C = (int32_t *)(w + p.C_off[l]);
        L.Iq = (int32_t *)(w + p.Iq_off[l]);
        L.Iq_tmp = (int32_t *)(w + p.Iqtmp_off[l]);
        L.Tp = (int)((L.T + 3) & ~(int64_t)3);
        L.ngrp = (int)((L.T + kGroupRows - 1) / kGroupRows);
        L.cnt8 = (uint32_t *)(w + p.Iqtmp_off[l]);          // the segment path's counts, 16-byte aligned both
        L.tot = (int32_t *)(L.cnt8 + (size_t)p.bh * L.ngrp * L.Tp * (kSegPerGroup / 4));
        if (L.nk > max_nk) max_nk = L.nk;
        if (L.total > max_total) max_total = L.total;
    }
    // level 0 has the most rows
    CscRanges r;
    auto ranges = [&](auto wgs) -> unsigned {               // lays the levels' workgroups one after the other
        int64_t wg = 0;
        for (int l = 0; l <= top; ++l) {
            r.lv[l] = a.lv[l];
            wg += p.bh * wgs(a.lv[l].T);
            r.wg_end[l] = (unsigned)wg;
        }
        return (unsigned)wg;
    };
    if (p.n[1] <= kSegRowsMax) {
        auto kr = [](int64_t T) { return (T + kKeyRange - 1) / kKeyRange; };
        unsigned wgs = ranges([&](int64_t T) { return kr(T) * ((T + kGroupRows - 1) / kGroupRows); });
        csc_seg_count_kernel<<<wgs, 256, 0, s>>>(r);
        csc_seg_scan_kernel<<<dim3(p.bh, top + 1), 256, 0, s>>>(a);
        wgs = ranges([&](int64_t T) { return kr(T) * ((T + kSegR - 1) / kSegR); });
        csc_seg_fill_kernel<<<wgs, 256, 0, s>>>(r, tile_rows(p, w));
        return hipGetLastError();
    }
    const unsigned nl = (unsigned)(top + 1);
    csc_zero_kernel<<<dim3((unsigned)((max_nk + 255) / 256), nl), 256, 0, s>>>(a);
    csc_count_kernel<<<dim3((unsigned)((max_total + 255) / 256), nl), 256, 0, s>>>(a);
    csc_scan_kernel<<<dim3(p.bh, nl), kScanThreads, 0, s>>>(a);
    csc_fill_kernel<<<dim3((unsigned)((max_total + 255) / 256), nl), 256, 0, s>>>(a);
    csc_sort_kernel<<<dim3((unsigned)((max_total + 255) / 256), nl), 256, 0, s>>>(a);
    csc_sort_long_kernel<<<dim3((unsigned)((max_nk + 255) / 256), nl), 256, 0, s>>>(a);
    return launch_fine_tiles(p, w, s);
}

// ------------------------------------------------------- key-major lists through a dense block mask (comparator)
// The mask-based baseline of Sec. 5.4 ("Efficient Backward Implementation", Fig. 4): the row-major lists I^(0) are
// turned into a dense binary T x T block mask and the key/value backward scans it, skipping the unmarked blocks.
// Here the mask is kept key-major (mask[key block][query block], one byte each: the layout that makes the scan a
// contiguous read, the baseline's best case), and the scan of a key block's row writes the marked query blocks, in
// ascending order, as that key's list -- the same (C, Iq) pair Alg. 2 produces in O(T K) -- so that the very same
// dK / dV kernel runs behind both.  Work and memory of this path are O(T^2) per head.
__global__ void __launch_bounds__(256) mask_zero_kernel(uint4 *mask16, int64_t n16) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n16) mask16[i] = make_uint4(0u, 0u, 0u, 0u);
}
// one thread per entry of I^(0): marks (key, query block) and counts the key's listers
__global__ void __launch_bounds__(256) mask_mark_kernel(const int32_t *I, uint8_t *mask, int32_t *cnt, int64_t T, int Kl,
                                                        int64_t total) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    const int64_t eph = T * Kl, bh = e / eph, row = (e % eph) / Kl;
    const int32_t key = I[e];
    mask[(bh * T + key) * T + row] = 1;
    atomicAdd(&cnt[bh * T + key], 1);
}
// one wave per key block: scans its T mask bytes, 1024 at a time, and appends the marked query blocks to its list.  A row begins at
// a multiple of T bytes: it is read in vectors of 16 or 4 bytes only if T is a multiple of that.
__global__ void __launch_bounds__(256) mask_scan_kernel(const uint8_t *mask, const int32_t *C, int32_t *Iq, int64_t T,
                                                        int64_t eph, int64_t nk) {
    const int lane = threadIdx.x & 63;
    const int64_t kb = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);           // flat key block over (batch, head)
    if (kb >= nk) return;
    const int64_t bh = kb / T, key = kb % T;
    const uint8_t *row = mask + kb * T;
    int32_t *dst = Iq + bh * eph + C[bh * (T + 1) + key];
    int written = 0;
    for (int64_t base = 0; base < T; base += 1024) {
        const int64_t i0 = base + 16 * lane;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        if (T % 16 == 0) {
            if (i0 < T) {
                const uint4 v = *reinterpret_cast<const uint4 *>(row + i0);
                w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
            }
        } else if (T % 4 == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (i0 + 4 * k < T) w[k] = *reinterpret_cast<const uint32_t *>(row + i0 + 4 * k);
        } else {
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if (i0 + k < T) w[k >> 2] |= (uint32_t)row[i0 + k] << (8 * (k & 3));
        }
        int mine = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) mine += __popc(w[k] & 0x01010101u);
        int incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        int pos = written + incl - mine;
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if ((w[k >> 2] >> (8 * (k & 3))) & 1u) dst[pos++] = (int32_t)(i0 + k);
        written += __shfl(incl, 63, 64);
    }
}

// Level 0's key-major lists through the dense mask: C and Iq of level 0 in the backward workspace, as launch_csc.
hipError_t launch_mask_lists(const Plan &p, const int32_t *indices, void *ws, void *mask, hipStream_t s) {
    char *w = static_cast<char *>(ws);
    const int64_t T = p.n[1], nk = T * p.bh, eph = T * p.Kl[0], total = eph * p.bh;
    CscLevels a;
    CscLevel &L = a.lv[0];
    L.T = T; L.Kl = p.Kl[0]; L.eph = eph; L.total = total; L.nk = nk;
    L.I = reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(indices) + p.idx_off[0]);
    L.cnt = (int32_t *)(w + p.cnt_off[0]);
    L.C = (int32_t *)(w + p.C_off[0]);
    L.Iq = (int32_t *)(w + p.Iq_off[0]);
    L.Iq_tmp = (int32_t *)(w + p.Iqtmp_off[0]);
    const int64_t n16 = (nk * T + 15) / 16;
    if (n16 / 256 >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    mask_zero_kernel<<<dim3((unsigned)((n16 + 255) / 256)), 256, 0, s>>>(static_cast<uint4 *>(mask), n16);
    csc_zero_kernel<<<dim3((unsigned)((nk + 255) / 256), 1), 256, 0, s>>>(a);
    mask_mark_kernel<<<dim3((unsigned)((total + 255) / 256)), 256, 0, s>>>(L.I, static_cast<uint8_t *>(mask), L.cnt, T, L.Kl, total);
    csc_scan_kernel<<<dim3(p.bh, 1), kScanThreads, 0, s>>>(a);
    mask_scan_kernel<<<dim3((unsigned)((nk + 3) / 4)), 256, 0, s>>>(static_cast<const uint8_t *>(mask), L.C, L.Iq, T, eph, nk);
    return launch_fine_tiles(p, w, s);
}

// ---------------------------------------------------------------------------- index reordering (Sec. 5.1)
// Tokens of a W x W pixel grid in nested-patch order: token t is the pixel whose x / y are the even / odd bits
// of t, so every aligned run of 4^i tokens is one aligned 2^i x 2^i patch.  One thread per 16-byte chunk of a
// row; forward: out[t] = in[y W + x], inverse: out[y W + x] = in[t].
__global__ void __launch_bounds__(256) reorder_kernel(const uint4 *in, uint4 *out, int64_t N, int cpr, int bits,
                                                       int inverse, int64_t total) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int64_t row = idx / cpr, bh = row / N, t = row % N;
    const int c = (int)(idx % cpr);
    int64_t x = 0, y = 0;
    for (int b = 0; b < bits; ++b) {
        x |= ((t >> (2 * b)) & 1) << b;
        y |= ((t >> (2 * b + 1)) & 1) << b;
    }
    const int64_t r = (y << bits) + x;
    const int64_t src = inverse ? t : r, dst = inverse ? r : t;
    out[(bh * N + dst) * cpr + c] = in[(bh * N + src) * cpr + c];
}

hipError_t launch_reorder(int64_t bh, int64_t N, int row_bytes, int bits, int inverse, const void *in, void *out,
                          hipStream_t s) {
    const int cpr = row_bytes / 16;
    const int64_t total = bh * N * cpr;
    reorder_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>((const uint4 *)in, (uint4 *)out, N, cpr, bits, inverse,
                                                                   total);
    return hipGetLastError();
}

}  // namespace llsa
