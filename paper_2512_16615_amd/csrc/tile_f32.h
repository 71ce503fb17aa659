// Operands of the fp32 matrix instruction (tile_kernels.hip describes their layout).
#pragma once
#include "tile_common.h"

namespace llsa {

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <int D> struct TShape {
    static constexpr int KS = D / 4;                    // matrix instructions over the channels
    static constexpr int E = D >= 64 ? 4 : D / 16;      // channels per lane and row piece of the second product
    static constexpr int H = D / (16 * E);              // row pieces
    static constexpr int NT = D / 16;                   // 16-channel accumulator tiles: tile E h + e, row i = channel 16 E h + E i + e
};

// a row as an operand of the first product
template <int D> struct RowOp { float x[D / 4]; };
template <int D> __device__ __forceinline__ RowOp<D> row_op(const float *row, int g) {
    RowOp<D> r;
#pragma unroll
    for (int m = 0; m < D / 16; ++m) {
        const FVec<4> v = ld_e<4>(row + 16 * m + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) r.x[4 * m + e] = v.v[e];
    }
    return r;
}
template <int D> __device__ __forceinline__ f32x4 row_product(const RowOp<D> &a, const RowOp<D> &b) {
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D / 4; ++s) c = mfma4(a.x[s], b.x[s], c);
    return c;
}
// the lane's pieces of tile rows 4g + r (r = 0 .. 3) as an operand of the second product
template <int D> struct ColOp { FVec<TShape<D>::E> x[4][TShape<D>::H]; };
template <int D> __device__ __forceinline__ void col_gload(ColOp<D> &c, int r, uint64_t row, int i16) {
    using S = TShape<D>;
    typedef float vec __attribute__((ext_vector_type(S::E)));
#pragma unroll
    for (int h = 0; h < S::H; ++h) {
        const vec x = gload<vec>(row + 4 * (16 * S::E * h + S::E * i16));
#pragma unroll
        for (int e = 0; e < S::E; ++e) c.x[r][h].v[e] = x[e];
    }
}
template <int D> __device__ __forceinline__ void col_product(f32x4 (&acc)[D / 16], const ColOp<D> &c, const f32x4 &p) {
    using S = TShape<D>;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int h = 0; h < S::H; ++h)
#pragma unroll
            for (int e = 0; e < S::E; ++e) acc[S::E * h + e] = mfma4(c.x[r][h].v[e], p[r], acc[S::E * h + e]);
}
// 16 rows in LDS, 16-byte chunk c of row r where the rows that 16 lanes read at one chunk get different bank groups.  Fetched as
// whole rows (64 lanes cover RPR rows a round): the operand layout straight from memory is 16 rows x half a line per instruction,
// which caps gathers at a third of what the L2 delivers.
template <int D> struct RowTile {
    static constexpr int CH = D / 4, RPR = 64 / CH, R = 16 / RPR;    // 16-byte chunks a row, rows a round, rounds
    static constexpr int ROWB = 4 * D, BYTES = 16 * ROWB;
    static __device__ __forceinline__ int at(int r, int c) {
        return r * ROWB + ((c ^ (D >= 64 ? r : D == 32 ? (r >> 1) & 7 : (r >> 2) & 3)) << 4);
    }
    static __device__ __forceinline__ void put(char *b, int lane, const u32x4 (&x)[R]) {
#pragma unroll
        for (int u = 0; u < R; ++u) *reinterpret_cast<u32x4 *>(b + at(lane / CH + RPR * u, lane % CH)) = x[u];
    }
    static __device__ __forceinline__ RowOp<D> row(const char *b, int i16, int g) {
        RowOp<D> r;
#pragma unroll
        for (int m = 0; m < D / 16; ++m) {
            const f32x4 v = *reinterpret_cast<const f32x4 *>(b + at(i16, 4 * m + g));
#pragma unroll
            for (int e = 0; e < 4; ++e) r.x[4 * m + e] = v[e];
        }
        return r;
    }
    static __device__ __forceinline__ ColOp<D> col(const char *b, int i16, int g) {
        using S = TShape<D>;
        ColOp<D> c;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int h = 0; h < S::H; ++h) {
                const int ch = 16 * S::E * h + S::E * i16;
                c.x[r][h] = ld_e<S::E>(reinterpret_cast<const float *>(b + at(4 * g + r, ch >> 2) + (ch & 3) * 4));
            }
        return c;
    }
};

// bf16 tiles, where an input is not finite: acc += x^T p with fp32 operands.  x: 16 channels of 32 rows as two transposing reads leave
// them (lds_tr_pair; slots 4h .. 4h + 3: rows 16h + 4g ..), of which the first `rows` exist; the others count as zeros.
__device__ __forceinline__ f32x4 product_fp32(bf16x8 x, const f32x4 (&p)[2], int rows, int g, f32x4 acc) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool row = 16 * h + 4 * g + r < rows;
            acc = mfma4(row ? (float)x[4 * h + r] : 0.f, row ? p[h][r] : 0.f, acc);
        }
    __builtin_amdgcn_sched_barrier(0);                      // one operand at a time: this is no place to spend registers
    return acc;
}
// is one of these sums a NaN in any lane of the wave (or the sum of infinities of both signs)?
template <int n> __device__ __forceinline__ bool any_nan(const f32x4 (&acc)[n]) {
    f32x4 x = acc[0];
#pragma unroll
    for (int i = 1; i < n; ++i) x += acc[i];
    const float y = (x[0] + x[1]) + (x[2] + x[3]);
    return __builtin_amdgcn_ballot_w64(y != y) != 0;
}

// the lane's results of a second product: channels 16 E h + E (4g + r) .. + E - 1 of column i16, handed out as vectors
template <int D, class Emit> __device__ __forceinline__ void col_emit(const f32x4 (&acc)[D / 16], int g, Emit emit) {
    using S = TShape<D>;
#pragma unroll
    for (int h = 0; h < S::H; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            FVec<S::E> v;
#pragma unroll
            for (int e = 0; e < S::E; ++e) v.v[e] = acc[S::E * h + e][r];
            emit(16 * S::E * h + S::E * (4 * g + r), v);
        }
}

}  // namespace llsa
