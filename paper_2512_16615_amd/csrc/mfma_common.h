// Device helpers shared by the bf16 MFMA kernels (gfx950): vector types, the 16x16x32 bf16 MFMA, the LDS
// transpose read, cross-row reductions and the table of 16-token key blocks of a query block's list.
//
// Register layouts of v_mfma_f32_16x16x32_bf16 (lane = 16*g + i, g = 0..3, i = 0..15):
//   A (16 x 32): lane holds row i,    contraction slots 8g .. 8g+7
//   B (32 x 16): lane holds column i, contraction slots 8g .. 8g+7
//   D (16 x 16): lane holds column i, rows 4g .. 4g+3
// ds_read_b64_tr_b16 (per block of 16 lanes, lane r supplies the address of 4 consecutive 16-bit
// values): output lane i, element e = element (i % 4) of the chunk addressed by lane 4e + i / 4.
// v_permlane16_swap / v_permlane32_swap with both operands equal to x return {x[l], x[l ^ 16]} resp.
// {x[l], x[l ^ 32]} (in some order) in every lane l.
#pragma once
#include "llsa_internal.h"

namespace llsa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

#define LLSA_LDS __attribute__((address_space(3)))

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// A load through an address that came as a number (from LDS, a lane table, a kernel argument's struct): named as global memory.
// The compiler makes a flat load of it otherwise, which also counts as an LDS operation, so that every LDS wait behind it waits
// for memory and nothing is in flight during the math.
template <class T> __device__ __forceinline__ T gload(uint64_t addr) {
    return *reinterpret_cast<const __attribute__((address_space(1))) T *>(addr);
}
template <class T> __device__ __forceinline__ T gload(const void *p) { return gload<T>(reinterpret_cast<uint64_t>(p)); }

__device__ __forceinline__ bf16x8 ld_bf16x8(const void *p) { return *reinterpret_cast<const bf16x8 *>(p); }

// two fp32 -> packed bf16 (round to nearest even; one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    union { bf16x2 v; uint32_t u; } r;
    r.v[0] = (__bf16)lo;
    r.v[1] = (__bf16)hi;
    return r.u;
}

__device__ __forceinline__ bf16x8 pack8(const f32x4 &a, const f32x4 &b) {
    bf16x8 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) { r[i] = (__bf16)a[i]; r[4 + i] = (__bf16)b[i]; }
    return r;
}

// fp32 values as three bf16 parts, x = p[0] + p[1] + p[2] exactly: each part is the upper half of what the ones before it leave,
// and each difference is exact.  A product of a bf16 operand with the three parts, summed in fp32, is the product with x itself.
// (Finite values only: an infinite x has a NaN for its second part, and a part that is 0 times an infinite operand is one; the callers
// look for a NaN.)
struct Parts3 { bf16x8 p[3]; };
__device__ __forceinline__ Parts3 split8(const f32x4 &a, const f32x4 &b) {
    union { uint32_t u[4]; bf16x8 v; } r[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x0 = i < 2 ? a[2 * i] : b[2 * i - 4], x1 = i < 2 ? a[2 * i + 1] : b[2 * i - 3];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const uint32_t u0 = __float_as_uint(x0), u1 = __float_as_uint(x1);
            r[p].u[i] = __builtin_amdgcn_perm(u1, u0, 0x07060302);      // the upper halves, x0's first
            x0 -= __uint_as_float(u0 & 0xffff0000u);
            x1 -= __uint_as_float(u1 & 0xffff0000u);
        }
    }
    return {{r[0].v, r[1].v, r[2].v}};
}

// Two transposing LDS reads glued into one 8-slot MFMA operand.
__device__ __forceinline__ bf16x8 lds_tr_pair(const char *lo, const char *hi) {
    union { s16x4 h[2]; bf16x8 v; } r;
    r.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LLSA_LDS s16x4 *)(lo));
    r.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LLSA_LDS s16x4 *)(hi));
    return r.v;
}

// All-reduce over the four lanes {i, i+16, i+32, i+48} (the four row groups of one MFMA column).
__device__ __forceinline__ float rows_max(float x) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float rows_sum(float x) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Results of a matrix product, transposed, to a row of 16-bit values: lane 16 g + i has channels 16 n + 4 g .. + 3 of row i in `a` and
// 16 n + 16 + 4 g .. + 3 in `b`.  The lanes of an odd g hand their `a` to the ones before them and take those lanes' `b`, so that each has 8 channels in a
// row: 16 bytes a lane, and four lanes write 64 bytes of a row where they wrote 32.  row: channel 0 of row i.
// The L2 takes 64 bytes a request: with 32 a sixth of the forward kernel's requests were its result.  Kernels in a step with 32 and with 64, us: 16 heads
// x 65536 tokens forward 210.7 and 198.6, dQ 271.8 and 260.7, level-0 dK/dV 264.9 and 254.6 (Gaussian 236.6 and 225.2, 301.3 and 292.4, 323.6
// and 305.5), 32 x 16384 97.1 and 90.6, 134.1 and 127.9, 141.5 and 134.5, 8 x 262144, d = 128 1324 and 1279, 1568 and 1539, 1646 and 1636.
__device__ __forceinline__ void store_pair(uint16_t *row, int n, int g, u32x2 a, u32x2 b) {
    u32x4 w;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto r = __builtin_amdgcn_permlane16_swap(a[k], b[k], false, false);
        w[k] = r[0];
        w[2 + k] = r[1];
    }
    *reinterpret_cast<u32x4 *>(row + 16 * (n + (g & 1)) + 8 * (g >> 1)) = w;
}

// arr[idx] for a small kernel-argument array without dynamic indexing (which would spill the table to
// scratch memory): a chain of selects over compile-time positions.
template <class T, int n>
__device__ __forceinline__ T pick(const T (&arr)[n], int idx) {
    T v = arr[0];
#pragma unroll
    for (int j = 1; j < n; ++j) v = (idx == j) ? arr[j] : v;
    return v;
}

// Rows of D bf16 kept unpadded in LDS, the 16-byte chunk c of row r stored at chunk c ^ swz_key(r).  The LDS serves a row-wise
// 16-byte read (lane 16 g + i: row i, chunk g + const) in four passes of 16 lanes over its 64 banks, lanes 0-3, 12-15 and 20-27 first:
// all 16 rows, the middle eight at the next chunk; a transposed 8-byte read in two passes of 32 lanes: 32 bytes each of 8 rows.
// Both are free of conflicts if the key spreads 8 consecutive rows over the 32-byte pieces of the 256 bytes the banks span and
// leaves the lowest bit alone: d = 64 (two rows span the banks) 4 keys, one per row pair, d = 128 8 keys, d = 32 2.  Measured per read
// of a wave: 4.6 cycles row-wise, 2.5 transposed; a key per row instead ((r >> 1) & 7) 4.6 and 4.9, at d = 128 8.6 and 2.5.
template <int D> __device__ __forceinline__ int swz_key(int r) {
    return D == 64 ? ((r >> 1) & 3) << 1 : D == 128 ? (r & 7) << 1 : D == 32 ? ((r >> 2) & 1) << 1 : 0;
}

// Per-lane byte offsets of the MFMA operand reads inside a 16-row slice of such unpadded, swizzled rows (2 D bytes
// each): row[ks] = the 16-byte row-wise read of row lane % 16, contraction step ks (A or B operand with the rows as
// the 16-wide dimension; d = 16: lanes 32 .. 63 repeat the row's two chunks); tr[n] = the address a lane supplies to the
// transposing 64-bit read for the n-th group of 16 channels (rows 4 (lane / 16) + (lane % 16) / 4).  The swizzle key of a
// row depends on the lane only.
template <int D> struct TileOffsets { int row[(D + 31) / 32], tr[D / 16]; };
template <int D> __device__ __forceinline__ TileOffsets<D> tile_offsets(int lane) {
    constexpr int ROWB = 2 * D;
    const int i16 = lane & 15, g = lane >> 4;
    const int key_row = swz_key<D>(i16), key_tr = swz_key<D>(4 * g + (i16 >> 2));
    TileOffsets<D> o;
#pragma unroll
    for (int ks = 0; ks < (D + 31) / 32; ++ks) o.row[ks] = i16 * ROWB + ((((g + 4 * ks) & (D / 8 - 1)) ^ key_row) << 4);
#pragma unroll
    for (int n = 0; n < D / 16; ++n)
        o.tr[n] = (4 * g + (i16 >> 2)) * ROWB + (((2 * n + ((i16 >> 1) & 1)) ^ key_tr) << 4) + ((i16 & 1) << 3);
    return o;
}

// Memory straight into LDS: every lane fetches 16 bytes at base + v, the wave's 1024 bytes land in lane order at `lds`; N times, each time
// 1024 bytes further on both sides, v0 and v1 taken in turn.  A tile brought in this way costs no registers and next to none of the
// LDS's time: a wave that fetches 8 KB and reads them 2 or 4 times, as the tiles do, took 1.4 to 1.6 times as long through registers
// and LDS writes (ds_write_b128: 13.5 cycles of the CU per 1024 bytes, a read 4.6).  Rows are swizzled by choosing each lane's source
// chunk (row_source).  The compiler does not know of these loads (it would wait for all of them at every LDS read): vm_wait before the
// data is read, and nothing may still be reading what they overwrite, which lgkmcnt(0) sees to for the wave's own reads.
// `base` and `lds` are the same in every lane.
// Where the compiler has `base` in vector registers, v_readfirstlane writes it right before the asm, into which the compiler's own
// wait states do not reach: a vector memory instruction must not read an SGPR within five wait states of the vector instruction that
// wrote it, and the hardware does not look.  Scalar instructions may read it at once and what they write may be read at once, so the loads
// take a scalar copy.  It stands between m0 and the first load, which must not follow m0's write at once either (one wait state; an
// s_waitcnt with nothing to wait for may be none).  (s_nop 3 in its place: 0.3 to 0.6 % slower steps at 16 heads x 4096, 32 x 16384 and 16 x 65536 tokens.)
#define LLSA_LOAD_LDS "s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\ts_waitcnt lgkmcnt(0)\n\tglobal_load_lds_dwordx4 %2, %0"
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"         // m0 is on the clobber list so that nothing else is kept in it meanwhile
template <int N> __device__ __forceinline__ void load_lds(uint64_t base, unsigned v0, unsigned v1, unsigned lds) {
    static_assert(N == 1 || N == 2 || N == 4, "");
    base = (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(base >> 32)) << 32 | (unsigned)__builtin_amdgcn_readfirstlane((int)base);
    uint64_t copy;
    if constexpr (N == 1)
        asm volatile(LLSA_LOAD_LDS : "=&s"(copy) : "s"(lds), "v"(v0), "s"(base) : "memory", "m0");
    else if constexpr (N == 2)
        asm volatile(LLSA_LOAD_LDS "\n\tglobal_load_lds_dwordx4 %4, %0 offset:1024"
                     : "=&s"(copy) : "s"(lds), "v"(v0), "s"(base), "v"(v1) : "memory", "m0");
    else
        asm volatile(LLSA_LOAD_LDS "\n\tglobal_load_lds_dwordx4 %4, %0 offset:1024\n\tglobal_load_lds_dwordx4 %2, %0 offset:2048\n\t"
                     "global_load_lds_dwordx4 %4, %0 offset:3072"
                     : "=&s"(copy) : "s"(lds), "v"(v0), "s"(base), "v"(v1) : "memory", "m0");
}
#undef LLSA_LOAD_LDS
// the same with 4 bytes a lane, from an address of its own each, to 256 bytes at `lds` (behind a load_lds, whose wait for the wave's LDS reads
// covers these too)
__device__ __forceinline__ void load_lds_dword(const float *p, unsigned lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds), "v"(p) : "memory", "m0");
}
#pragma clang diagnostic pop
// Rows of D bf16 brought into LDS as swz_key wants them, 1024 bytes (512 / D rows) at a time: what a lane adds to the address of the
// first of them.  Of two 1024 bytes of a 16-row slice in turn (v0, v1): at d = 128 the second four rows have other keys.
template <int D> struct RowSource {
    unsigned v0, v1;
    __device__ __forceinline__ explicit RowSource(int lane) {
        constexpr int PARTS = D / 8, KPU = 64 / PARTS;
        const int r = lane / PARTS, c = lane % PARTS;
        v0 = (unsigned)(r * 2 * D + ((c ^ swz_key<D>(r)) << 4));
        v1 = (unsigned)(r * 2 * D + ((c ^ swz_key<D>(r + KPU)) << 4));
    }
};
// at most N of the wave's loads are still on their way (they complete in order)
template <int N> __device__ __forceinline__ void vm_wait() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// the same, and every wave of the workgroup has come this far and read what it wanted from LDS
template <int N> __device__ __forceinline__ void vm_wait_barrier() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory"); }
__device__ __forceinline__ unsigned lds_address(const void *p) { return (unsigned)(uintptr_t)(const LLSA_LDS char *)p; }

// Workgroup id -> work item so that the workgroups one XCD receives (ids congruent modulo 8) cover a
// contiguous range of work items: neighbouring query blocks gather overlapping keys, which then stay in
// that XCD's L2.
__device__ __forceinline__ int64_t xcd_contiguous(int64_t w, int64_t total) {
    const int64_t per = total >> 3;
    return (w < per * 8) ? (w & 7) * per + (w >> 3) : w;
}

__device__ __forceinline__ unsigned xcd_contiguous32(unsigned w, unsigned total) {
    const unsigned per = total >> 3;
    return w < per * 8 ? (w & 7) * per + (w >> 3) : w;
}

// The 16-token key tiles of one 16-query tile's list (Alg. 1, enrichment loop), 64 at a time: lane j of the wave
// describes tile 64 * chunk + j.  A listed block of B = 16 * 2^ls tokens is 2^ls consecutive tiles; query tile `blk`
// (queries 16 blk ...) reads row 16 blk / B^(l+1) of I^(l).  The main loops fetch a block's fields with
// v_readlane (block numbers are wave-uniform), which keeps the per-tile scalar work small.
struct BlockTable {
    uint64_t kptr, vptr;     // address of the block's first key / value row
    float bias2;             // log2 of the level's token weight
    int cnt;                 // valid rows: 16, fewer in the last block of a ragged coarsest level, 0 past the end

    // lane j describes list block base + 64 * chunk + j; only levels below lev_end are looked at
    __device__ __forceinline__ void fill(const LevelTable &t, int64_t bh, int64_t blk, int base, int chunk, int lane,
                                         int d, int lev_end = kMaxL + 1) {
        const int jb = base + chunk * 64 + lane;
        kptr = vptr = 0;
        bias2 = 0.f;
        cnt = 0;
        const int nl = min(t.nlev, lev_end);
        for (int l = 0; l < nl; ++l) {                           // wave-uniform loop over the levels in the list
            const int b0 = pick(t.bseg, l), b1 = pick(t.bseg, l + 1);
            const int64_t n_l = pick(t.n, l);
            const char *Kb = static_cast<const char *>(pick(t.K, l)), *Vb = static_cast<const char *>(pick(t.V, l));
            if (jb >= b0 && jb < b1) {
                const int k = jb - b0;
                int64_t tok0;
                if (l < t.L) {
                    const int64_t row = blk >> (t.lb * (l + 1) - 4);
                    const int32_t listed = gload<int32_t>(pick(t.I, l) + (bh * pick(t.rows, l) + row) * pick(t.Kl, l) + (k >> t.ls));
                    tok0 = ((int64_t)listed << t.lb) + ((k & ((1 << t.ls) - 1)) << 4);
                    cnt = 16;
                } else {
                    tok0 = (int64_t)k * 16;
                    cnt = min(16, (int)(n_l - tok0));
                }
                const int64_t off = (bh * n_l + tok0) * d * 2;
                kptr = reinterpret_cast<uint64_t>(Kb + off);
                vptr = reinterpret_cast<uint64_t>(Vb + off);
                bias2 = pick(t.bias, l) * kLog2e;
            }
        }
    }
    static __device__ __forceinline__ const char *rl_ptr(uint64_t v, int j) {
        const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, j);
        const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), j);
        return reinterpret_cast<const char *>(((uint64_t)hi << 32) | lo);
    }
    __device__ __forceinline__ const char *K(int j) const { return rl_ptr(kptr, j); }
    __device__ __forceinline__ const char *V(int j) const { return rl_ptr(vptr, j); }
    __device__ __forceinline__ int count(int j) const { return __builtin_amdgcn_readlane(cnt, j); }
    __device__ __forceinline__ float bias(int j) const {
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bias2), j));
    }
};

// The coarse tiles (levels >= 1) of a query tile's list, 64 at a time: lane j describes tile 64 * chunk + j.  Every wave of a
// workgroup builds its own copy: with the levels' fields as scalars straight from the kernel arguments that is about 15
// instructions a level and one load in all, less than handing one wave's copy round through LDS and a barrier.
// In two steps, ask and finish, so that other loads can be asked for in between.  The fields of levels 1 to 4 are fetched without
// conditions, all at once: one wait for scalar memory where fetching each where it is needed waited up to seven times a level, and the
// lists are asked for before anything that comes from further away.  From a wave's start to its first tile on the way, forward,
// 16 heads x 4096 tokens: 7900 -> 6100 cycles of 24500 (kernel 16.0 -> 14.6 us), 65536: 10500 -> 8100 of 47900 (195 us either
// way: the other waves of the SIMD have enough to do).
typedef const __attribute__((address_space(4))) ListArgs *list_args_ptr;
// the kernel's arguments begin with its ListArgs
__device__ __forceinline__ list_args_ptr kernel_list_args() { return (list_args_ptr)__builtin_amdgcn_kernarg_segment_ptr(); }

struct CoarseTable {
    uint64_t kptr, vptr;     // address of the tile's first key / value row
    float bias2;             // log2 of the level's token weight
    int cnt;                 // valid rows: 16, fewer in the last tile of a ragged coarsest level
    int raw, k, n;           // between ask and finish: the listed block; the tile in its level; the level's tokens if it is dense, else -1

    // the asm keeps the compiler from moving a field's load behind the branch that it makes of a select
    template <int D> __device__ __forceinline__ void ask(list_args_ptr t, int64_t bh, unsigned tile, int chunk, int lane) {
        const int ls = t->ls, j = min(t->lev[0].end + 64 * chunk + lane, t->lev[t->nlev - 1].end - 1);   // past the end: the last tile
        uint64_t list = reinterpret_cast<uint64_t>(t->lev[0].I);     // the lane's row of I (any place if its level is dense)
        int first = j;
        n = 0;
        kptr = 0;
        bias2 = 0.f;
        struct Fields { uint64_t K, I; int n, rows, Kl, first, shift; float bias2; };
        auto fields = [&](int l) -> Fields {
            const auto &v = t->lev[l];
            return {reinterpret_cast<uint64_t>(v.K), reinterpret_cast<uint64_t>(v.I), v.n, v.rows, v.Kl, v.first, v.shift, v.bias2};
        };
        auto level = [&](const Fields &v) {                  // (of the levels up to the lane's the last one stays)
            const bool in = j >= v.first;
            const uint64_t K = v.K + (uint64_t)(bh * v.n * (2 * D)), row = v.I + (uint64_t)((bh * v.rows + (tile >> v.shift)) * v.Kl) * 4;
            const int dense = v.I ? -1 : v.n;
            kptr = in ? K : kptr;
            list = in ? (v.I ? row : list) : list;
            first = in ? v.first : first;
            n = in ? dense : n;
            bias2 = in ? v.bias2 : bias2;
        };
        Fields v[4];
#pragma unroll
        for (int l = 0; l < 4; ++l) v[l] = fields(l + 1);    // (a level that the list does not have begins behind everything)
#pragma unroll
        for (int l = 0; l < 4; ++l)
            asm volatile("" : "+s"(v[l].K), "+s"(v[l].I), "+s"(v[l].n), "+s"(v[l].rows), "+s"(v[l].Kl), "+s"(v[l].first), "+s"(v[l].shift), "+s"(v[l].bias2));
#pragma unroll
        for (int l = 0; l < 4; ++l) level(v[l]);
        for (int l = 5; l < t->nlev; ++l) level(fields(l));
        k = j - first;
        raw = gload<int32_t>(list + (n < 0 ? (uint64_t)(unsigned)(k >> ls) * 4 : 0));
    }
    template <int D> __device__ __forceinline__ void finish(list_args_ptr t) {
        const int tok = n < 0 ? (raw << t->lb) + ((k & ((1 << t->ls) - 1)) << 4) : k << 4;
        cnt = n < 0 ? 16 : min(16, n - tok);
        kptr += (uint64_t)((int64_t)tok * (2 * D));
        vptr = kptr + (uint64_t)t->to_v;
    }
    template <int D> __device__ __forceinline__ void fill(list_args_ptr t, int64_t bh, unsigned tile, int chunk, int lane) {
        ask<D>(t, bh, tile, chunk, lane);
        finish<D>(t);
    }
    __device__ __forceinline__ const char *K(int j) const { return BlockTable::rl_ptr(kptr, j); }
    __device__ __forceinline__ const char *V(int j) const { return BlockTable::rl_ptr(vptr, j); }
    __device__ __forceinline__ int count(int j) const { return __builtin_amdgcn_readlane(cnt, j); }
    __device__ __forceinline__ float bias(int j) const {
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bias2), j));
    }
};

}  // namespace llsa
