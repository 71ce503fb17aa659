// Hierarchical Top-K selection, one level (Alg. 1, selection loop), K <= 16: scores on the fp32 matrix instruction, the K best
// by merging sorted lists in registers.  Any block size, channel count and number of candidates, both I/O types.
//
// A score is the fp32 fused-multiply-add chain over channels 0 .. d-1 in order (the contract of the selection: it fixes every
// tie).  v_mfma_f32_16x16x1_4b_f32 performs exactly one such step for 16 queries x 64 candidates: one multiplication per
// result, one rounding, denormals kept, so a chain of d of them is bit for bit the scalar chain (checked against fmaf on random,
// wide-range and denormal inputs).  Lane (b, i) supplies channel c of query i (A) and of candidate 16 b + i of the chunk (B),
// and lane (g, i) receives the scores of queries 4g .. 4g+3 against candidates 16 b + i.
//
// A score and its position become one number of type double, larger = better: the score's 32 bits made monotonic, then 20
// bits of position, complemented so that the lower position wins a tie: the 52 bits of the mantissa, under a constant exponent.
// v_max_f64 / v_min_f64 then compare and exchange in one instruction each.  Every lane keeps the sorted K best (KL = 8 or 16) of
// its own candidates per query; at the end the 16 lanes of a query merge theirs pairwise (maximum of one list and the reversed
// other one, then a bitonic clean-up), and so do the waves of the workgroup.
//
// One workgroup per tile of 16 queries that share their candidates, one wave per 64 candidates (up to 4 waves, which then take
// several chunks).  Candidate rows reach LDS in whole cache lines and leave it as one row per lane.  Bound: matrix pipe (32
// cycles per channel and 64 candidates) and the vector instructions of the merges, about even at K = 8 and 128 candidates.
#include <type_traits>

#include "mfma_common.h"

namespace llsa {

typedef float f32x16 __attribute__((ext_vector_type(16)));

struct SelLevel {
    const void *Q, *K;               // Q^(l), K^(l): [bh, n, D]
    const int32_t *parent;           // I^(l): [bh, n / B, Kp], or null: every token of the level is a candidate
    int32_t *out;                    // I^(l-1): [bh, n, Kout]
    int64_t n;
    int C, Kp, Kout;                 // candidates per query, parent picks, picks
};

template <class T> constexpr int kVn = 16 / (int)sizeof(T);      // channels in 16 bytes
template <class T> __device__ __forceinline__ void unpack16(u32x4 w, float *f) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(w[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
}

constexpr uint32_t kPosMax = 0xfffff;                            // 20 bits of position
__device__ __forceinline__ double make_key(float score, uint32_t pos) {
    const uint32_t u = __float_as_uint(score + 0.f);             // -0 ties with +0
    const uint32_t o = u ^ (uint32_t)(((int32_t)u >> 31) | (int32_t)0x80000000);
    return __hiloint2double((int)(0x3ff00000u | (o >> 12)), (int)((o << 20) | (kPosMax - pos)));
}
__device__ __forceinline__ int key_pos(double k) { return (int)(kPosMax - ((uint32_t)__double2loint(k) & kPosMax)); }

__device__ __forceinline__ void cmp_swap(double &a, double &b) { // larger first
    const double x = fmax(a, b), y = fmin(a, b);
    a = x;
    b = y;
}
// a bitonic list into descending order
template <int KL> __device__ __forceinline__ void bitonic(double *l) {
#pragma unroll
    for (int h = KL / 2; h >= 1; h >>= 1)
#pragma unroll
        for (int i = 0; i < KL; ++i)
            if ((i & h) == 0) cmp_swap(l[i], l[i + h]);
}
template <int CTRL> __device__ __forceinline__ double dpp(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// the KL best of a sorted list of N (in l) and another (o, reversed): all of them while 2 N <= KL
template <int N, int KL> __device__ __forceinline__ void merge_list(double (&l)[KL], const double (&o)[N]) {
    if constexpr (2 * N <= KL) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            l[N + i] = fmin(l[i], o[i]);
            l[i] = fmax(l[i], o[i]);
        }
        bitonic<N>(l);
        bitonic<N>(l + N);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) l[i] = fmax(l[i], o[i]);
        bitonic<N>(l);
    }
}
template <int CTRL, int N, int KL> __device__ __forceinline__ void merge_lanes(double (&l)[KL]) {
    double o[N];
#pragma unroll
    for (int i = 0; i < N; ++i) o[i] = dpp<CTRL>(l[N - 1 - i]);
    merge_list<N, KL>(l, o);
}
// Two lists a, b (of two queries) per lane of a pair: the lane with `second` keeps b and merges its partner's b into it, the
// other one keeps a and merges its partner's a, so that every lane goes on with one list instead of two.
template <int CTRL, int N, int KL> __device__ __forceinline__ void merge_swap(double (&a)[KL], const double (&b)[KL], bool second) {
    double o[N];
#pragma unroll
    for (int i = 0; i < N; ++i) o[i] = dpp<CTRL>(second ? a[N - 1 - i] : b[N - 1 - i]);
#pragma unroll
    for (int i = 0; i < N; ++i) a[i] = second ? b[i] : a[i];
    merge_list<N, KL>(a, o);
}
// The lists (N sorted entries each) of queries 4g .. 4g+3 in the 16 lanes of group g: afterwards l[0] of lane i16 is the merged
// list of query 4g + (i16 & 3).  Pairs and quads (quad_perm) halve the number of lists a lane carries, then the quads
// are merged (row_ror by 4 and by 8 lanes, which keeps the query).
template <int N, int KL> __device__ __forceinline__ void merge_rows(double (&l)[4][KL], int i16) {
    constexpr int N1 = 2 * N < KL ? 2 * N : KL, N2 = 2 * N1 < KL ? 2 * N1 : KL, N3 = 2 * N2 < KL ? 2 * N2 : KL;
    merge_swap<0xb1, N, KL>(l[0], l[1], (i16 & 1) != 0);
    merge_swap<0xb1, N, KL>(l[2], l[3], (i16 & 1) != 0);
    merge_swap<0x4e, N1, KL>(l[0], l[2], (i16 & 2) != 0);
    merge_lanes<0x124, N2, KL>(l[0]);
    merge_lanes<0x128, N3, KL>(l[0]);
}
// one list per lane, all of the same query
template <int N, int KL> __device__ __forceinline__ void merge_row(double (&l)[KL]) {
    constexpr int N1 = 2 * N < KL ? 2 * N : KL, N2 = 2 * N1 < KL ? 2 * N1 : KL, N3 = 2 * N2 < KL ? 2 * N2 : KL;
    merge_lanes<0xb1, N, KL>(l);
    merge_lanes<0x4e, N1, KL>(l);
    merge_lanes<0x124, N2, KL>(l);
    merge_lanes<0x128, N3, KL>(l);
}
__device__ __forceinline__ void sort4(double &a, double &b, double &c, double &d) {
    cmp_swap(a, b); cmp_swap(c, d); cmp_swap(a, c); cmp_swap(b, d); cmp_swap(b, c);
}
// four more keys of a lane
template <int KL> __device__ __forceinline__ void insert4(double (&l)[KL], double a, double b, double c, double d) {
    sort4(a, b, c, d);
    l[KL - 1] = fmax(l[KL - 1], a);
    l[KL - 2] = fmax(l[KL - 2], b);
    l[KL - 3] = fmax(l[KL - 3], c);
    l[KL - 4] = fmax(l[KL - 4], d);
    bitonic<KL>(l);
}

template <class T, int D> struct SelShape {
    static constexpr int ROWB = D * (int)sizeof(T), SB = ROWB < 128 ? ROWB : 128;     // bytes of a row; of a staged slice of it
    static constexpr int NS = ROWB / SB, PC = SB / 16, RPI = 64 / PC, STRIDE = SB + 16;
};

// Scores of 16 query rows (qrow: this lane's row i16) against 64 candidate rows (id: the row of candidate `lane`).
// `lds`: 64 * STRIDE bytes of the wave's own.
template <class T, int D>
__device__ __forceinline__ f32x16 score_chunk(const T *qrow, const T *Kb, char *lds, int lane, int id) {
    using S = SelShape<T, D>;
    u32x4 kreg[S::PC], qreg[S::PC];
    auto load = [&](int slice) {                                 // the candidates' slice, whole cache lines per instruction
#pragma unroll
        for (int u = 0; u < S::PC; ++u) {
            const int64_t row = __shfl(id, S::RPI * u + lane / S::PC, 64);
            kreg[u] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(Kb) + row * S::ROWB + slice * S::SB + (lane % S::PC) * 16);
        }
    };
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    load(0);
#pragma unroll
    for (int s = 0; s < S::NS; ++s) {
#pragma unroll
        for (int u = 0; u < S::PC; ++u)
            qreg[u] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(qrow) + s * S::SB + u * 16);
        __builtin_amdgcn_wave_barrier();                         // one wave's LDS operations stay in order
#pragma unroll
        for (int u = 0; u < S::PC; ++u)
            *reinterpret_cast<u32x4 *>(lds + (S::RPI * u + lane / S::PC) * S::STRIDE + (lane % S::PC) * 16) = kreg[u];
        __builtin_amdgcn_wave_barrier();
        if (s + 1 < S::NS) load(s + 1);                          // flies during this slice's products
#pragma unroll
        for (int u = 0; u < S::PC; ++u) {
            float q[kVn<T>], k[kVn<T>];
            unpack16<T>(qreg[u], q);
            unpack16<T>(*reinterpret_cast<const u32x4 *>(lds + lane * S::STRIDE + u * 16), k);
#pragma unroll
            for (int e = 0; e < kVn<T>; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x1f32(q[e], k[e], acc, 0, 0, 0);
        }
    }
    return acc;
}

// Entries first, first + 4, ... of a list whose first Kout entries are the winners: emit(position, winners below it).
template <int KL, class Emit> __device__ __forceinline__ void winners(const double (&l)[KL], int first, int Kout, Emit emit) {
    int pos[KL];
#pragma unroll
    for (int i = 0; i < KL; ++i) pos[i] = i < Kout ? key_pos(l[i]) : 0x7fffffff;
#pragma unroll
    for (int j = 0; j < KL; j += 4) {
        int mine = pos[j], rank = 0;
#pragma unroll
        for (int x = 1; x < 4; ++x) mine = first == x ? pos[j + x] : mine;
#pragma unroll
        for (int i = 0; i < KL; ++i) rank += pos[i] < mine ? 1 : 0;
        if (j + first < Kout) emit(mine, rank);
    }
}

// NW waves; ONE: at most one chunk of 64 candidates each.  TOP: the launch also does the level above (1) or several (2), up to level L,
// which is dense over at most 64 tokens; the ones between have at most 64 candidates too.  The first wave of every workgroup scores the
// tokens above its queries, level by level from the top, which yields the row of I^(l) it needs; the workgroup with a token's first queries
// also writes the token's row out.  A level less by a launch on a latency-bound path: three levels of one head x 256 tokens, fp32, in
// two launches and in one, a step 33.8 and 32.0 us.
constexpr int kSelAbove = 3;
template <int N> struct SelAbove {
    SelLevel lev[N];                 // from the level next above
    int n;
};
template <> struct SelAbove<0> {};
template <class T, int D, int KL, int NW, bool ONE, int TOP>
__global__ void __launch_bounds__(64 * NW) select_mfma_kernel(SelLevel a, int B, int tpb, unsigned tiles, SelAbove<(TOP < 2 ? TOP : kSelAbove)> up) {
    using S = SelShape<T, D>;
    static_assert(16 * KL * 8 <= 64 * S::STRIDE, "a wave's lists must fit in its staging rows");
    __shared__ __attribute__((aligned(16))) char lds[NW * 64 * S::STRIDE];
    __shared__ int32_t rows[2][64];
    int32_t *prow = rows[0];
    const int tid = threadIdx.x, lane = tid & 63, i16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t bh = blockIdx.x / tiles;
    const unsigned in = blockIdx.x - (unsigned)bh * tiles;
    // the tile: queries first .. first + nq - 1 of block blk (= token blk of the level above); 16 consecutive ones at the top
    const bool dense = !TOP && a.parent == nullptr;
    const unsigned blk = dense ? 0 : in / (unsigned)tpb;
    const int sub = 16 * (int)(in - blk * tpb);
    const int64_t first = dense ? (int64_t)in * 16 : (int64_t)blk * B + sub;
    const int nq = dense ? (int)min((int64_t)16, a.n - first) : min(16, B - sub);
    const T *Kb = static_cast<const T *>(a.K) + bh * a.n * D;
    const T *qrow = static_cast<const T *>(a.Q) + (bh * a.n + first + min(i16, nq - 1)) * D;
    char *my = lds + wave * 64 * S::STRIDE;
    const unsigned magic = 0xffffffffu / (unsigned)B + 1;        // ceil(2^32 / B), also for powers of two

    if constexpr (TOP > 0) {
        if (wave == 0)
            for (int u = TOP > 1 ? up.n - 1 : 0; u >= 0; --u) {
                const SelLevel &v = up.lev[u];
                int q = (int)blk;                                // the token of that level above these queries
                bool begins = sub == 0;                          // ... whose first ones they are
                for (int x = 0; TOP > 1 && x < u; ++x) {
                    const int above = (int)__umulhi((unsigned)q, magic);
                    begins &= above * B == q;
                    q = above;
                }
                const bool all = TOP == 1 || u == up.n - 1;
                const int nt = (int)v.n, C = all ? nt : v.Kp * B, q0 = q & ~15;
                const int32_t *par = rows[(u + 1) & 1];
                int32_t *mine = rows[u & 1];
                auto cand = [&](int p) {
                    const int k = (int)__umulhi((unsigned)p, magic);
                    return all ? p : par[k] * B + (p - k * B);
                };
                const T *tq = static_cast<const T *>(v.Q) + (bh * nt + min(q0 + i16, nt - 1)) * D;
                __builtin_amdgcn_wave_barrier();
                const f32x16 acc = score_chunk<T, D>(tq, static_cast<const T *>(v.K) + bh * nt * D, my, lane, cand(min(lane, C - 1)));
                double l[KL];
#pragma unroll
                for (int b = 0; b < 4; ++b) {                    // the one query's scores (in the lanes of its group)
                    float sc = acc[4 * b];
#pragma unroll
                    for (int r = 1; r < 4; ++r) sc = (q & 3) == r ? acc[4 * b + r] : sc;
                    const int p = 16 * b + i16;
                    l[b] = p < C ? make_key(sc, (uint32_t)p) : 0.0;
                }
                sort4(l[0], l[1], l[2], l[3]);
                merge_row<4, KL>(l);
                if (g == ((q & 15) >> 2) && i16 < 4)
                    winners<KL>(l, i16, v.Kout, [&](int pos, int rank) {
                        const int id = cand(pos);
                        mine[rank] = id;
                        if (begins) v.out[(bh * nt + q) * v.Kout + rank] = id;
                    });
            }
        __syncthreads();
    } else if (!dense) {
        for (int i = tid; i < a.Kp; i += 64 * NW) prow[i] = a.parent[(bh * (a.n / B) + blk) * a.Kp + i];
        __syncthreads();
    }
    auto id_of = [&](int p) -> int {
        if (dense) return p;
        const int k = (int)__umulhi((unsigned)p, magic);         // p / B: exact for p < 2^20, B <= 64
        return prow[k] * B + (p - k * B);
    };

    auto keys = [&](const f32x16 &acc, int c, int r, double (&k)[4]) {
#pragma unroll
        for (int b = 0; b < 4; ++b) k[b] = make_key(acc[4 * b + r], (uint32_t)(64 * c + 16 * b + i16));
        if (64 * c + 64 > a.C)                                   // the last chunk: positions past the candidates
#pragma unroll
            for (int b = 0; b < 4; ++b) k[b] = 64 * c + 16 * b + i16 < a.C ? k[b] : 0.0;
    };
    double l[4][KL];                                             // this lane's lists of queries 4g + r
    if constexpr (ONE) {                                         // at most one chunk per wave
        const f32x16 acc = score_chunk<T, D>(qrow, Kb, my, lane, id_of(min(64 * wave + lane, a.C - 1)));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double k[4];
            keys(acc, wave, r, k);
            sort4(k[0], k[1], k[2], k[3]);
#pragma unroll
            for (int b = 0; b < 4; ++b) l[r][b] = k[b];
        }
        merge_rows<4, KL>(l, i16);
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < KL; ++i) l[r][i] = 0.0;
        for (int c = wave; 64 * c < a.C; c += NW) {
            const f32x16 acc = score_chunk<T, D>(qrow, Kb, my, lane, id_of(min(64 * c + lane, a.C - 1)));
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double k[4];
                keys(acc, c, r, k);
                insert4<KL>(l[r], k[0], k[1], k[2], k[3]);
            }
        }
        merge_rows<KL, KL>(l, i16);
    }
    // lane i16 holds the wave's list of query 4g + i16 % 4; the first wave merges in the other waves' lists, through LDS
    const int qi = 4 * g + (i16 & 3);
    if constexpr (NW > 1) {
        double *ex = reinterpret_cast<double *>(my) + qi * KL;   // (the wave's staged rows are done with)
        __builtin_amdgcn_wave_barrier();
        if (wave > 0 && i16 < 4)
#pragma unroll
            for (int i = 0; i < KL; ++i) ex[i] = l[0][i];
        __syncthreads();
        if (wave > 0) return;
#pragma unroll
        for (int x = 1; x < NW; ++x) {
            const double *src = reinterpret_cast<const double *>(lds + x * 64 * S::STRIDE) + qi * KL;
            double o[KL];
#pragma unroll
            for (int i = 0; i < KL; ++i) o[i] = src[KL - 1 - i];
            merge_list<KL, KL>(l[0], o);
        }
    }
    if (qi < nq)
        winners<KL>(l[0], i16 >> 2, a.Kout, [&](int pos, int rank) { a.out[(bh * a.n + first + qi) * a.Kout + rank] = id_of(pos); });
}

// K <= 16 and positions that fit their 20 bits
bool select_mfma_ok(const Plan &p, int l) {
    const int64_t C = (l == p.L) ? p.n[l] : (int64_t)p.Kl[l] * p.B;
    return p.desc.kernel_path == 0 && p.Kl[l - 1] <= 16 && C <= (int64_t)kPosMax && p.n[l] < ((int64_t)1 << 30);
}

// Lowest level below L that a launch can take along with all levels above it, at least `low`, or 0.  Below level L - 1 for few workgroups, where the
// launch is what a level costs.
int select_top_fused(const Plan &p, int low) {
    if (p.L <= low || !select_mfma_ok(p, p.L) || !select_mfma_ok(p, p.L - 1) || p.n[p.L] > 64) return 0;
    int l = p.L - 1;
    while (l > low && p.L - l < kSelAbove && select_mfma_ok(p, l - 1) && p.Kl[l] * p.B <= 64 && p.bh * p.n[l] * ((p.B + 15) / 16) <= 1024) --l;
    return l;
}

// above: the lists of all levels, of which the launch makes those above `out` too, or null
hipError_t launch_select_mfma(const Plan &p, int l, const void *ws, const int32_t *parent, int32_t *out, hipStream_t s,
                              char *above) {
    const char *w = static_cast<const char *>(ws);
    auto level = [&](int x, const int32_t *par, int32_t *o) {
        SelLevel v;
        v.Q = w + p.pyr_off[0][x];
        v.K = w + p.pyr_off[1][x];
        v.parent = x == p.L ? nullptr : par;
        v.out = o;
        v.n = p.n[x];
        v.C = x == p.L ? (int)p.n[x] : p.Kl[x] * p.B;
        v.Kp = x == p.L ? 0 : p.Kl[x];
        v.Kout = p.Kl[x - 1];
        return v;
    };
    const SelLevel a = level(l, parent, out);
    SelAbove<kSelAbove> up;
    up.n = above ? p.L - l : 0;
    for (int x = 0; x < kSelAbove; ++x) {
        const int y = l + 1 + (x < up.n ? x : 0);
        up.lev[x] = above ? level(y, nullptr, reinterpret_cast<int32_t *>(above + p.idx_off[y - 1])) : a;
    }
    const int tpb = l == p.L ? 1 : (p.B + 15) / 16;
    const int64_t tiles = l == p.L ? (p.n[l] + 15) / 16 : p.n[l + 1] * tpb;
    int kmax = a.Kout;
    for (int x = 0; x < up.n; ++x) kmax = up.lev[x].Kout > kmax ? up.lev[x].Kout : kmax;
    const int chunks = (a.C + 63) / 64;
    const unsigned grid = (unsigned)(p.bh * tiles);
    auto go = [&](auto ty, auto d, auto kl) {
        using T = decltype(ty);
        constexpr int D = decltype(d)::value, KL = decltype(kl)::value;
        auto with = [&](auto nw, auto one) {
            constexpr int NW = decltype(nw)::value;
            constexpr bool ONE = decltype(one)::value;
            auto run = [&](auto top, auto above) {
                select_mfma_kernel<T, D, KL, NW, ONE, decltype(top)::value><<<grid, 64 * NW, 0, s>>>(a, p.B, tpb, (unsigned)tiles, above);
            };
            if (up.n == 0) run(std::integral_constant<int, 0>{}, SelAbove<0>{});
            else if (up.n == 1) run(std::integral_constant<int, 1>{}, SelAbove<1>{{up.lev[0]}, 1});
            else run(std::integral_constant<int, 2>{}, up);
        };
        if (chunks == 1) with(std::integral_constant<int, 1>{}, std::true_type{});
        else if (chunks == 2) with(std::integral_constant<int, 2>{}, std::true_type{});
        else if (chunks <= 4) with(std::integral_constant<int, 4>{}, std::true_type{});
        else with(std::integral_constant<int, 4>{}, std::false_type{});
    };
    auto by_k = [&](auto ty, auto d) {
        if (kmax <= 8) go(ty, d, std::integral_constant<int, 8>{});
        else go(ty, d, std::integral_constant<int, 16>{});
    };
    auto by_d = [&](auto ty) {
        if (p.d == 16) by_k(ty, std::integral_constant<int, 16>{});
        else if (p.d == 32) by_k(ty, std::integral_constant<int, 32>{});
        else if (p.d == 64) by_k(ty, std::integral_constant<int, 64>{});
        else by_k(ty, std::integral_constant<int, 128>{});
    };
    if (p.elt == 4) by_d(float{});
    else by_d(uint16_t{});
    return hipGetLastError();
}

}  // namespace llsa
