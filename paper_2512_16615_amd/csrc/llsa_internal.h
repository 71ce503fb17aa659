// Internal declarations shared by the translation units of libllsa (host plan + kernel launchers).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/llsa.h"

namespace llsa {

constexpr int kMaxL = 8;            // coarse levels supported (levels 0..8)
constexpr int kMaxCand = 4096;      // candidates per selection row held in LDS (n_L or K_l * B)

// Host-side description of one problem: level table and buffer layout.
struct Plan {
    llsa_desc desc;
    int L, Le, B, K, d, bh, elt;    // elt = bytes per element of the I/O type
    int64_t N;
    float scale;
    int64_t n[kMaxL + 1];           // tokens per head at level l
    int Kl[kMaxL];                  // K_l = min(K, n_{l+1})
    size_t idx_off[kMaxL];          // byte offset of I^(l) inside `indices`
    size_t idx_bytes;
    size_t pyr_off[3][kMaxL + 1];   // workspace byte offset of pooled level l (1..L) of Q/K/V
    size_t D_off;                   // [bh, N] fp32: rowsum(dO * O)
    size_t C_off[kMaxL], cnt_off[kMaxL], Iq_off[kMaxL], Iqtmp_off[kMaxL];
    size_t tiles_off, arrived_off, piece_off;   // level 0's lists as tiles (fine_tiles.h), pieces of a cut list that are done, their sums
    size_t dKacc_off[kMaxL + 1], dVacc_off[kMaxL + 1]; // fp32 gradients of pooled level l (1..L)
    size_t part_off, part_bytes;    // partial sums of the key-major reductions
    size_t grp_slab_off, grp_red_off[2];   // partials of the query-grouped coarse dK/dV kernel and its reductions
    bool group;                     // coarse levels' dK/dV run grouped by level-1 query block
    size_t ws_fwd, ws_bwd;
    int list_len;                   // tokens one query attends to
    bool fast;                      // bf16 MFMA kernels apply (bf16, B in {16, 32, 64}, d in {64, 128}, N % 64 == 0)
    bool blocks16;                  // the same for any N: what the bf16 selection kernels take
    int lb;                         // log2 B when blocks16
};

// What the attention-type kernels need to walk the gathered list of a query block.
struct LevelTable {
    const void *K[kMaxL + 1];       // level-l keys   [bh, n_l, d]
    const void *V[kMaxL + 1];       // level-l values [bh, n_l, d]
    const int32_t *I[kMaxL + 1];    // I^(l) [bh, rows_l, K_l]; unused for l = L
    int64_t n[kMaxL + 1];
    int64_t rows[kMaxL + 1];
    int Kl[kMaxL + 1];
    int seg[kMaxL + 2];             // list position where level l starts; seg[nlev] = list length
    int bseg[kMaxL + 2];            // same in units of 16-token key blocks (used when B = 16)
    float bias[kMaxL + 1];          // l * ln B (or 0)
    int nlev;                       // levels in the list = Le + 1
    int L, B, d;
    int lb, ls;                     // log2 B and log2(B / 16) when B is 16, 32 or 64 (MFMA kernels), else 0
    float scale;
};

// x / d for x < 2^31 by one 32-bit multiplication (a workgroup's first instructions: the compiler's division of two 64-bit
// numbers is more than a hundred)
struct FastDiv {
    uint32_t d, m, s;
    FastDiv() = default;
    explicit FastDiv(int64_t div) : d((uint32_t)div), m(0), s(0) {
        while (((int64_t)1 << s) < div) ++s;
        m = (uint32_t)((((uint64_t)1 << (31 + s)) + d - 1) / d);
    }
    __host__ __device__ uint32_t operator()(uint32_t x) const { return (uint32_t)(((uint64_t)x * m) >> (31 + s)); }
};

// A level of the list as the workgroups of the shared-level kernels read it: one 64-byte scalar load from the kernel arguments.
struct __attribute__((aligned(64))) ListLevel {
    const void *K, *V;
    const int32_t *I;               // null for a dense level
    int32_t n, rows, Kl;
    int32_t first, end;             // its 16-token tiles in the list
    int32_t shift;                  // query tile q reads row q >> shift of I
    float bias2;                    // log2 of its tokens' weight
    int32_t pad[3];
};
struct ListArgs {
    ListLevel lev[kMaxL + 1];
    int32_t nlev, lb, ls;
    float scale;
    int64_t to_v;                   // from a pooled level's keys to its values: the same for all of them
};
ListArgs make_list_args(const LevelTable &t);

// Alg. 2 for a problem of at most kSmallRows level-0 rows, as workgroups that any launch can take along (csc_small.h).
constexpr int kSmallRows = 512;
struct CscSmallLevel {
    const int32_t *I;               // I^(l) [bh, T, Kl]
    int32_t *C, *Iq;
    int32_t T, Kl;                  // keys per head = rows per head
};
struct FineTile;
struct CscSmall {
    CscSmallLevel lv[kMaxL];
    uint32_t wg_end[kMaxL];         // level l's workgroups end here
    int32_t levels;
    uint32_t wgs;                   // in all, rounded up to a multiple of 8; 0: none
    FineTile *tiles;                // level 0's tiles and counters (fine_tiles.h), or null
    int32_t *arrived;
    int32_t lc;                     // log2 of the tiles of a piece
};

LevelTable make_level_table(const Plan &p, const void *K0, const void *V0, const int32_t *indices,
                            const void *workspace);

// ---- any supported shape ----
hipError_t launch_pool(const Plan &p, const void *Q, const void *K, const void *V, void *ws, bool q_too,
                       hipStream_t s);
// QK-Norm + RoPE of Q and K fused with level-1 pooling, then the remaining pooled levels (fills Qout, Kout and ws)
hipError_t launch_qknorm_rope_pool(const Plan &p, const void *Qpre, const void *Kpre, const void *V,
                                   const float *gamma_q, const float *gamma_k, const float *cos_t, const float *sin_t,
                                   float eps, void *Qout, void *Kout, void *ws, hipStream_t s);
hipError_t launch_select(const Plan &p, int l, const void *ws, const int32_t *parent, int32_t *out, hipStream_t s);
hipError_t launch_csc(const Plan &p, int top_level, const int32_t *I, void *ws, hipStream_t s);  // levels 0..top_level
bool csc_small_args(const Plan &p, int top_level, const int32_t *I, void *ws, CscSmall *a);   // false (and none): too many rows
size_t csc_scratch_bytes(const Plan &p, int l);   // scratch memory at Iqtmp_off[l]
// level 0's key-major lists through a dense T x T block mask (`mask`: bh * T * T bytes, rounded up to 16) instead of Alg. 2
hipError_t launch_mask_lists(const Plan &p, const int32_t *indices, void *ws, void *mask, hipStream_t s);
// nested-patch token order of a 2^bits x 2^bits grid (or back); rows of row_bytes (a multiple of 16) bytes
hipError_t launch_reorder(int64_t bh, int64_t N, int row_bytes, int bits, int inverse, const void *in, void *out,
                          hipStream_t s);

// ---- attention, dQ (and D = rowsum(dO * O)) and dK / dV of every level in fp32 arithmetic (tile_kernels.hip) ----
hipError_t launch_attn_fwd_tile(const Plan &p, const LevelTable &t, const void *Q, void *O, float *LSE, hipStream_t s);
hipError_t launch_dq_tile(const Plan &p, const LevelTable &t, const void *Q, const void *O, const void *dO, const float *LSE,
                          float *D, void *dQ, const CscSmall &csc, hipStream_t s);   // csc: the key-major lists too, in the same launch
hipError_t launch_dkv_tile(const Plan &p, const LevelTable &t, const void *Q, const void *dO, const float *LSE, const float *D,
                           void *ws, void *dK, void *dV, hipStream_t s);
bool dkv_tile_folds(const Plan &p);      // is there anything to fold behind it?
hipError_t launch_dkv_tile_fold(const Plan &p, const LevelTable &t, void *ws, void *dK, void *dV, hipStream_t s);
size_t dkv_tile_bytes(const Plan &p);    // workspace of its partial sums

// ---- selection: K <= 16 (any shape), bf16 with B = 16 / 32 / 64 and K <= 64 ----
bool select_mfma_ok(const Plan &p, int l);
bool select_dense_ok(const Plan &p, int l);
bool select_dense_top_ok(const Plan &p);
// top_out: l = L - 1 and the launch also does level L, writing I^(L-1) to top_out (allowed if select_dense_top_ok)
hipError_t launch_select_dense(const Plan &p, int l, const void *ws, const int32_t *parent, int32_t *out, hipStream_t s,
                               int32_t *top_out = nullptr);
// above: the lists of all levels; the launch also does the levels above l, up to L (allowed at select_top_fused's l)
hipError_t launch_select_mfma(const Plan &p, int l, const void *ws, const int32_t *parent, int32_t *out, hipStream_t s,
                              char *above = nullptr);
int select_top_fused(const Plan &p, int low);

// ---- bf16 MFMA kernels (B = 16 / 32 / 64, d = 64 or 128, N % 64 == 0) ----
// select (or null): the launch selects the lists of level 0 itself (attn_selects(p) = 1: those of level 1 are there), or those of both levels (2)
struct AttnSelect { const void *workspace; int32_t *I0, *I1; };
int attn_selects(const Plan &p);         // 0: it cannot, or a launch of the selection's own is faster
hipError_t launch_attn_fwd_mfma(const Plan &p, const LevelTable &t, const void *Q, void *O, float *LSE, const AttnSelect *select, hipStream_t s);
// variant that shares the coarse levels among the 8 or 16 sibling query blocks of a workgroup
hipError_t launch_attn_fwd_shared(const Plan &p, const LevelTable &t, const void *Q, void *O, float *LSE, const AttnSelect *select, hipStream_t s);
struct GroupAlong;                       // dkv_group.h
// also writes D = rowsum(dO * O) for the key-major kernels that follow
hipError_t launch_dq_mfma(const Plan &p, const LevelTable &t, const void *Q, const void *O, const void *dO,
                          const float *LSE, float *D, void *dQ, const CscSmall &csc, const GroupAlong *group, hipStream_t s);
bool dq_takes_lists(const Plan &p);      // does launch_dq_mfma take the key-major lists along?
hipError_t launch_dq_shared(const Plan &p, const LevelTable &t, const void *Q, const void *O, const void *dO,
                            const float *LSE, float *D, void *dQ, const CscSmall &csc, const GroupAlong *group, hipStream_t s);
bool dq_takes_group(const Plan &p);      // does it take the grouped dK / dV kernel's work along (dkv_group.h; with the lists)?
// key-major dK/dV of level l; levels >= 1 also fold their split slabs and the level above into the
// level's fp32 gradient buffer, so they must be launched from the coarsest level down
hipError_t launch_dkv_mfma(const Plan &p, const LevelTable &t, int l, const void *Q, const void *dO, const float *LSE,
                           const float *D, void *ws, void *dK, void *dV, hipStream_t s, bool level0_alone = false);
bool dkv_by_tiles(const Plan &p);         // does level 0 take its lists as tiles (fine_tiles.h)?
int fine_piece_log2(const Plan &p);       // in pieces of how many tiles
int dkv_splits(const Plan &p, int l);    // workgroups sharing one key block's query list at level l
int dkv_block_tiles(const Plan &p, int l), dkv_block_splits(const Plan &p, int l);   // the same for dkv_block.hip's levels
// all coarse levels (dkv_group_top .. 1) at once, grouped by level-1 query block; fills the levels' fp32
// gradients.  `lists` (or null): event after which the key-major lists are complete, recorded on another stream;
// `s` waits for it behind the kernels that need no list, before the gathers.  `side`, `upper_done` (or null): the
// stream the lists are made on and a spare event; the reductions and gathers of levels >= 2 then run on `side` behind
// the lists, beside the level-1 kernel, and `lists` is recorded once more behind them (so it still marks the end of `side`).
hipError_t launch_dkv_group(const Plan &p, const LevelTable &t, const void *Q, const void *dO, const float *LSE,
                            const float *D, void *ws, bool taken, hipStream_t s, hipEvent_t lists, hipStream_t side = nullptr,
                            hipEvent_t upper_done = nullptr);
void dkv_group_sizes(const Plan &p, size_t *slab_bytes, size_t *red_bytes);
int dkv_group_top(const Plan &p);         // highest level the grouped kernel takes (the rest: split kernel)

// ---- measured peaks for the benchmark (calibrate.hip) ----
hipError_t launch_peak_mfma(float *out, int iters, int workgroups, hipStream_t s);
hipError_t launch_peak_copy(const void *src, void *dst, int64_t bytes, hipStream_t s);

}  // namespace llsa
