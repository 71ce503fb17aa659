// Level 0's key-major lists (B = 16) as a row of tiles, for the waves of dkv_fine_kernel (dkv_mfma.hip).
//
// A tile is two entries of a list.  The list of key block j, entries start .. start + len of its head's lists, takes the places from
// tile_place(start, j) on: (start + j + 1) / 2 is at least the number of tiles that the lists of the blocks before it have (each rounds up
// once), and leaves at least len / 2, rounded up, for its own.  So every list finds its places by itself, without a scan, at the price of
// some places that stay empty.  Long lists are cut into pieces of 2^lc tiles, the last one of half as many at least and one and a half at most.
#pragma once
#include "llsa_internal.h"

namespace llsa {

constexpr int kGap = -2, kGoesOn = -1, kPiece = 1 << 30;   // FineTile::key: no tile; not the first tile of a list or piece; of a list that is cut
struct FineTile { int32_t key, entry; };                    // the block whose list or piece begins here; the first entry e, or ~e if it is the tile's only one

__host__ __device__ __forceinline__ int tile_place(int start, int j) { return (int)(((unsigned)start + (unsigned)j + 1u) >> 1); }
__host__ __device__ __forceinline__ bool piece_begins(int x, int tiles, int lc) { return x == 0 || ((x & ((1 << lc) - 1)) == 0 && tiles - x >= 1 << (lc - 1)); }
__host__ __device__ __forceinline__ int piece_count(int tiles, int lc) { return tiles < 1 << lc ? 1 : ((tiles - (1 << (lc - 1))) >> lc) + 1; }
// places of a head with T key blocks and E entries; pieces of cut lists begin at least 2^(lc - 1) places apart: slot of the one at place t
__host__ __device__ __forceinline__ int64_t tile_places(int64_t T, int64_t E) { return (T + E + 1) / 2; }
__host__ __device__ __forceinline__ int piece_slot(int t, int lc) { return t >> (lc - 1); }
__host__ __device__ __forceinline__ int64_t piece_slots(int64_t T, int64_t E, int lc) { return (tile_places(T, E) >> (lc - 1)) + 1; }

// lane `lane` of `lanes` that write the places of block j's list (next: where the following block's places begin)
__device__ __forceinline__ void write_tiles(FineTile *tiles, int32_t *arrived, int lc, int j, int start, int len, int next, int lane, int lanes) {
    const int t0 = tile_place(start, j), n = (len + 1) >> 1;
    const bool cut = piece_count(n, lc) > 1;
    for (int x = lane; t0 + x < next; x += lanes) {
        const int e = start + 2 * x;
        tiles[t0 + x] = x >= n ? FineTile{kGap, 0} : FineTile{piece_begins(x, n, lc) ? j | (cut ? kPiece : 0) : kGoesOn, 2 * x + 1 < len ? e : ~e};
    }
    if (cut && lane == 0) arrived[piece_slot(t0, lc)] = 0;
}

}  // namespace llsa
