// Alg. 2's key-major lists of a problem with few rows, as the work of single workgroups, which need nothing from each other: the
// kernel of their own (generic_kernels.hip) or a few workgroups of the dQ launch, whose result they do not read.
#pragma once
#include "fine_tiles.h"

namespace llsa {

// A workgroup makes the lists of kRangeKeys consecutive keys of one head.  It reads all of the head's entries (from L2: 16 KB at 512 rows
// of 8), marks the rows that list one of its keys in a bitmap of a row per key in LDS and counts the entries of the keys below its
// own (their number is where its lists start); then every group of lanes turns a key's bitmap into its ascending list.  Marking has
// no order, so neither a fill in order nor a sort is needed.  Against count, scan, fill and sort in launches of their own this
// saves four launches, which is most of the time at these sizes.  Reading grows with rows^2, hence the limit; the bitmap of 32
// keys is 2 KB at 512 rows.
constexpr int kRangeKeys = 32, kCscSmallLds = kRangeKeys * kSmallRows / 8 + 4 * kRangeKeys + 64;   // bytes of LDS
template <int NT> __device__ __forceinline__ void csc_small(const CscSmall &a, unsigned wg, uint32_t *lds) {
    if (wg >= a.wg_end[a.levels - 1]) return;
    int l = 0;
    while (wg >= a.wg_end[l]) ++l;
    const CscSmallLevel &L = a.lv[l];
    const unsigned id = wg - (l ? a.wg_end[l - 1] : 0), T = (unsigned)L.T, E = T * (unsigned)L.Kl;
    const unsigned ranges = (T + kRangeKeys - 1) / kRangeKeys, bh = id / ranges, r0 = (id - bh * ranges) * kRangeKeys;
    const unsigned words = ((T + 63) >> 6) * 2;
    uint32_t *bm = lds;                                     // [kRangeKeys][words], words = rows in 64s, times 2
    int32_t *tot = reinterpret_cast<int32_t *>(lds + kRangeKeys * kSmallRows / 32), *below_sh = tot + kRangeKeys;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (unsigned i = tid; i < kRangeKeys * words; i += NT) bm[i] = 0;
    if (tid < kRangeKeys) tot[tid] = 0;
    __syncthreads();
    const int32_t *I = L.I + (int64_t)bh * E;
    int32_t below = 0;
    auto mark = [&](unsigned e, unsigned key) {
        below += key < r0 ? 1 : 0;
        if (key - r0 < (unsigned)kRangeKeys) {
            const unsigned row = e / (unsigned)L.Kl;
            atomicOr(&bm[(key - r0) * words + (row >> 5)], 1u << (row & 31));
            atomicAdd(&tot[key - r0], 1);
        }
    };
    unsigned e = tid;
    for (; e + 7 * NT < E; e += 8 * NT) {                 // eight loads in flight
        int32_t k[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) k[u] = I[e + NT * u];
#pragma unroll
        for (int u = 0; u < 8; ++u) mark(e + NT * u, (unsigned)k[u]);
    }
    for (; e < E; e += NT) mark(e, (unsigned)I[e]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) below += __shfl_xor(below, o, 64);
    if (lane == 0) below_sh[wave] = below;
    __syncthreads();
    // every wave scans the 32 counts for itself
    const int32_t n = lane < kRangeKeys ? tot[lane] : 0;
    int32_t start = n;
#pragma unroll
    for (int o = 1; o < kRangeKeys; o <<= 1) {
        const int32_t y = __shfl_up(start, o, 64);
        if (lane >= o) start += y;
    }
    start -= n;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) start += below_sh[w];
    int32_t *C = L.C + (int64_t)bh * (T + 1);
    if (wave == 0 && lane < kRangeKeys && r0 + lane < T) C[r0 + lane] = start;
    if (tid == 0 && r0 + kRangeKeys >= T) C[T] = (int32_t)E;
    if (l == 0 && a.tiles) {                                // the lists as tiles, a wave per key
        const int64_t places = tile_places(T, E);
        for (int k = wave; k < kRangeKeys && r0 + k < T; k += NT / 64) {
            const int s0 = __shfl(start, k, 64), len = __shfl(n, k, 64);
            write_tiles(a.tiles + bh * places, a.arrived + bh * piece_slots(T, E, a.lc), a.lc, (int)r0 + k, s0, len,
                        r0 + k + 1 == T ? (int)places : tile_place(s0 + len, (int)r0 + k + 1), lane, 64);
        }
    }
    // G lanes per key, each over 64-row words G apart
    int32_t *Iq = L.Iq + (int64_t)bh * E;
    const unsigned w64 = words / 2;
    int G = 1;
    while (G < 64 && (unsigned)G < w64) G <<= 1;
    const int sub = lane & (G - 1), per = 64 / G;           // keys of a wave at a time
    for (int k0 = wave * per; k0 < kRangeKeys; k0 += NT / 64 * per) {
        const int k = k0 + lane / G;                        // 64 / G <= 32 keys or, for one word, two passes' worth of lanes
        const int kk = min(k, kRangeKeys - 1);
        const int32_t cnt = k < kRangeKeys ? __shfl(n, kk, 64) : 0;
        int32_t pos = __shfl(start, kk, 64);
        const int32_t end = pos + cnt;
        if (__ballot(cnt > 0) == 0) continue;
        for (unsigned w0 = 0; w0 < w64; w0 += G) {
            uint64_t bits = 0;
            if (cnt > 0 && w0 + sub < w64) bits = *reinterpret_cast<const uint64_t *>(&bm[kk * words + 2 * (w0 + sub)]);
            int32_t mine = __popcll(bits), incl = mine;
            for (int o = 1; o < G; o <<= 1) {
                const int32_t y = __shfl_up(incl, o, 64);
                if (sub >= o) incl += y;
            }
            int32_t at = pos + incl - mine;
            while (bits) {
                Iq[at++] = (int32_t)(64 * (w0 + sub)) + (int32_t)__builtin_ctzll(bits);
                bits &= bits - 1;
            }
            pos += __shfl(incl, (lane & ~(G - 1)) + G - 1, 64);
        }
        // a key listed twice by one row (no valid selection has that) is marked once: fill its list with the last row
        if (sub == 0)
            for (; pos < end; ++pos) Iq[pos] = (int32_t)T - 1;
    }
}

}  // namespace llsa
