// What the tile kernels share (attention forward, dQ and dK/dV in fp32 arithmetic, any block size, d = 16 .. 128): the walk of a
// query block's gathered list token by token, the exponential, vectors of both I/O types.
#pragma once
#include <type_traits>

#include "mfma_common.h"

namespace llsa {

// E consecutive channels as fp32
template <int E> struct FVec { float v[E]; };
template <int E> __device__ __forceinline__ FVec<E> ld_e(const float *p) {
    FVec<E> r;
    if constexpr (E == 4) { const f32x4 x = *reinterpret_cast<const f32x4 *>(p); for (int i = 0; i < 4; ++i) r.v[i] = x[i]; }
    else if constexpr (E == 2) { const float2 x = *reinterpret_cast<const float2 *>(p); r.v[0] = x.x; r.v[1] = x.y; }
    else r.v[0] = p[0];
    return r;
}
template <int E> __device__ __forceinline__ void st_e(float *p, const FVec<E> &x) {
    if constexpr (E == 4) *reinterpret_cast<f32x4 *>(p) = f32x4{x.v[0], x.v[1], x.v[2], x.v[3]};
    else for (int i = 0; i < E; ++i) p[i] = x.v[i];
}
__device__ __forceinline__ void st_e(uint16_t *p, const FVec<4> &x) {
    *reinterpret_cast<u32x2 *>(p) = u32x2{pack_bf16(x.v[0], x.v[1]), pack_bf16(x.v[2], x.v[3])};
}

// Logits, maxima and logsumexps are in natural units: scale and weight folded into base-2 units for the bare hardware
// exponential (each factor rounded on its own, at the size of the whole exponent) put dQ 1.05 to 1.35 times and the logsumexp
// 1.05 to 1.4 times as far from a 64-bit computation.

// exp(x) to about a unit: x log2(e) in two parts, the hardware's 2^t of the rounded one, the rest to first order.  (Below -104
// the result is 0; a NaN stays one.)  Forward with it and with expf: one head of 256 tokens 8.8 : 9.2 us, 16 x 4096 62.9 : 65.5.
__device__ __forceinline__ float exp_nat(float x) {
    constexpr float kHi = 1.44269504f, kLo = (float)(1.4426950408889634 - (double)kHi);
    x = x < -104.f ? -104.f : x;
    const float t = x * kHi, rest = fmaf(x, kLo, fmaf(x, kHi, -t)), p = __builtin_amdgcn_exp2f(t);
    return fmaf(p, rest * kLn2, p);
}

// m + log(x) for x >= 1 to about the rounding of the result: the hardware's logarithm t, what it leaves of x as a first-order term,
// and the sum's own rounding added back.
__device__ __forceinline__ float add_log(float m, float x) {
    constexpr float kHi = 0.69314718f, kLo = (float)(0.6931471805599453 - (double)kHi);
    const float t = __builtin_amdgcn_logf(x), rest = fmaf(x, __builtin_amdgcn_exp2f(-t), -1.f);
    const float s = fmaf(t, kHi, m);
    return s + (fmaf(t, kHi, m - s) + fmaf(t, kLo, rest));
}

// A level of the list as the kernels read it from their arguments (which begin with a TokArgs).
struct __attribute__((aligned(64))) TokLevel {
    const void *K, *V;
    const int32_t *I;               // null for a dense level
    FastDiv span;                   // query block b reads row span(b) of I
    int32_t n, rows, Kl;
    int32_t first;                  // its first block in the list
    float bias;                     // log of its tokens' weight
};
struct TokArgs {
    TokLevel lev[kMaxL + 1];
    int32_t end[kMaxL + 1];         // blocks of the list up to and with level l (the list's last level and above: all)
    FastDiv B, per_head, tpb;       // tokens per block; query tiles per head; query tiles per block
    int32_t len, total;             // positions of the list; query tiles in all
    float scale;
};
typedef const __attribute__((address_space(4))) TokArgs *tok_args_ptr;
__device__ __forceinline__ tok_args_ptr kernel_tok_args() { return (tok_args_ptr)__builtin_amdgcn_kernarg_segment_ptr(); }

// 64 positions of a query block's gathered list (Alg. 1, enrichment loop), handed round in LDS: addresses of the tokens' key and
// value rows, log of the weight (-inf past the end of the list, whose rows repeat the last one).
struct TokTable {
    uint64_t k[64], v[64];
    float bias[64];
};

// The list of one query block.  Every level of it is whole blocks of B tokens (a dense level, always the last, is cut into blocks
// too, the last of them short), so position p is token p % B of the list's block p / B.  Lane x of the wave holds block
// 64 * chunk + x, fetched for 64 blocks at a time: one pass over the levels and one load per list, mostly, where looking the
// positions up token by token cost a tile of 16 queries as much as its products (1600 of 4500 cycles per 16 x 16 tile).
template <int ROWB> struct TokWalk {
    uint64_t k, v;
    float bias;
    int chunk;
    FastDiv B;
    __device__ __forceinline__ void fetch(tok_args_ptr t, int64_t bh, unsigned blk, int c, int lane) {
        chunk = c;
        const int j = 64 * c + lane;
        int l = 0;
#pragma unroll
        for (int x = 0; x < kMaxL; ++x) l += j >= t->end[x] ? 1 : 0;      // past the end of the list: any level
        const auto *L = &t->lev[l];
        const int32_t *I = L->I;
        const int in = j - L->first;
        const int64_t head = bh * L->n;
        FastDiv span;
        span.d = L->span.d; span.m = L->span.m; span.s = L->span.s;
        int tok = in;
        if (I && j < t->end[kMaxL]) tok = gload<int32_t>(I + (bh * L->rows + span(blk)) * L->Kl + in);
        const uint64_t off = (uint64_t)(head + (int64_t)tok * B.d) * ROWB;
        k = reinterpret_cast<uint64_t>(L->K) + off;
        v = reinterpret_cast<uint64_t>(L->V) + off;
        bias = L->bias;
    }
    __device__ __forceinline__ void begin(tok_args_ptr t, int64_t bh, unsigned blk, int lane) {
        B.d = t->B.d; B.m = t->B.m; B.s = t->B.s;
        fetch(t, bh, blk, 0, lane);
    }
    static __device__ __forceinline__ uint32_t from(uint32_t x, int lane4) { return (uint32_t)__builtin_amdgcn_ds_bpermute(lane4, (int)x); }
    // positions pos0 .. pos0 + 63 (pos0 a multiple of 64, so that they lie in one chunk of 64 blocks)
    __device__ __forceinline__ void put(TokTable &tab, tok_args_ptr t, int64_t bh, unsigned blk, int pos0, int lane) {
        const int c = (int)(B((uint32_t)pos0) >> 6);
        if (c != chunk) fetch(t, bh, blk, c, lane);
        const int len = t->len, pos = min(pos0 + lane, len - 1);
        const unsigned b = B((uint32_t)pos), off = (pos - b * B.d) * ROWB;
        const int src = (int)(b & 63) << 2;
        tab.k[lane] = (((uint64_t)from((uint32_t)(k >> 32), src) << 32) | from((uint32_t)k, src)) + off;
        tab.v[lane] = (((uint64_t)from((uint32_t)(v >> 32), src) << 32) | from((uint32_t)v, src)) + off;
        const float w = __uint_as_float(from(__float_as_uint(bias), src));
        tab.bias[lane] = pos0 + lane < len ? w : -INFINITY;
    }
};

// The query tile of a wave: up to 16 consecutive queries of one block of B.
struct QTile {
    int64_t bh, row;             // head; first query row of the tile, over all heads
    unsigned blk;                // query block inside the head
    int nq;                      // queries in the tile
};
__device__ __forceinline__ QTile query_tile(const TokArgs &a, unsigned tile, int64_t N) {
    QTile q;
    q.bh = a.per_head(tile);
    const unsigned in = tile - (unsigned)q.bh * a.per_head.d;
    q.blk = a.tpb(in);
    const int first = 16 * (int)(in - q.blk * a.tpb.d);
    q.nq = min(16, (int)a.B.d - first);
    q.row = q.bh * N + (int64_t)q.blk * a.B.d + first;
    return q;
}

// attention and dQ of the bf16 tile kernels (tile_bf16.hip)
hipError_t launch_attn_fwd_tile_bf16(const Plan &p, const TokArgs &a, const void *Q, void *O, float *LSE, hipStream_t s);
hipError_t launch_dq_tile_bf16(const Plan &p, const TokArgs &a, const void *Q, const void *O, const void *dO, const float *LSE,
                               float *D, void *dQ, const CscSmall &csc, hipStream_t s);

}  // namespace llsa
