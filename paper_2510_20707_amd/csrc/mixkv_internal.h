// Internal declarations shared by the libmixkv translation units (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "mixkv.h"

namespace mixkv {

constexpr int kWave = 64;
constexpr int kTileKeys = 32;          // keys per MFMA tile
constexpr int kLayersPerLaunch = 32;   // pointer-table entries that fit in one kernel-argument block
constexpr int kSelectThreads = 1024;
constexpr int kMaxCandPerHead = 1024;   // head-adaptive budgets: list length of the selection-only workspace layout
constexpr int kMaxSegs = 32;            // segments a long row is cut into at most
constexpr int kMaxStreamGrid = 1024;    // upper bound on the workgroups of a streaming kernel launch

// Loads of cache rows carry the non-temporal bit where a launch streams more than the Infinity Cache would keep of it for the next
// reader.  A plain read of 0.5 to 4 GB then runs at 7.0 to 7.4 TB/s, without the bit at 6.2.  Whole calls, without -> with, by the bytes of K
// and V: 67 MB 60.8 -> 63.8 us, 134 MB 80.9 -> 83.1, 168 MB 101 -> 104, 197 MB (f32) 79.4 -> 77.2, 235 MB 130 -> 126, 336 MB 166 ->
// 157, 2.1 GB 730 -> 686; block sums of 117 MB of keys 28.3 -> 29.7, of 235 MB 58.7 -> 54.2.  Time without over time with, one to twelve query
// tiles, caches in turn: 182 MB 0.99-1.08, 260 MB 1.00-1.12, 400 MB 0.98-1.12; the same cache again and again (a cache is compressed
// once): 182 MB 0.87-0.99, 260 MB 0.84-1.00, 400 MB 0.97-1.03.
// A template parameter, not a branch: the branch in the tile loops cost 2 to 5 %.
constexpr int64_t kInfinityCache = 256 * 1000 * 1000;
constexpr int64_t kCachedBytes = 180 * 1000 * 1000;
inline bool read_once(int64_t bytes) { return bytes >= kCachedBytes; }

// Per-layer device pointers handed to the kernels by value.
struct LayerIn {
  const void *K, *V, *Q;
  int64_t sb, sh, sn;                  // K/V strides in elements
  const float *r_given;                // caller's head weights (mix mode GIVEN_R), else null
};
struct LayerInTable { LayerIn l[kLayersPerLaunch]; };

// The window rows' log-sum-exp per layer, when the caller has it (else all null).
struct LseTable { const float *l[kLayersPerLaunch]; };

struct LayerOut {
  float *scores;                       // may point into the workspace
  float *redundancy;                   // may be null
  int32_t *indices, *counts, *offsets; // offsets may be null (fixed mode)
  void *K_out, *V_out;
};
struct LayerOutTable { LayerOut l[kLayersPerLaunch]; };

// Problem shape, identical for every layer of a call.
struct Shape {
  int32_t batch, hq, hkv, G, D, N, W, Nc, B, Bp;   // Bp = B - W
  int32_t GW;            // G * W query rows per KV head
  int32_t QT;            // ceil(GW / 32) query tiles
  int32_t chunk;         // keys per workgroup in the two streaming kernels
  int32_t nchunks;       // ceil(N / chunk)
  int32_t Npad;          // nchunks * chunk, row length of the per-unit float arrays
  int32_t units_per_layer;
  int32_t nb_rows;       // row length of the per-unit exponent offsets: QT*32 rounded up to 256
  int32_t pool, pool_k, causal, intrinsic, mix, adaptive, per_head, floor_;
  int32_t kstats;        // 1 / |K_i|, the mean normalised key and r are needed (else nothing reads them: the
                         // importance-only mix without the key-norm intrinsic score and without a redundancy output)
  float scale_log2e;     // softmax_scale * log2(e)
  float eps;
};

// read_once for the two passes over `nunits` heads.
inline bool pass_once(const Shape &s, int dtype, int nunits) {
  return read_once((int64_t)nunits * s.N * s.D * (dtype == MIXKV_BF16 ? 2 : 4) * (s.intrinsic == MIXKV_INTRINSIC_VNORM ? 2 : 1));
}

// Workspace carve-up (byte offsets from a 256-byte aligned base).  Sizes are per call (all units).
struct Workspace {
  size_t budgets;        // int32  [layers][hkv]             per-head budget mode: the caller's table (first, so
                         //                                  that selection alone can run on a workspace this small)
  size_t part_ml;        // float2 [slots][QT*32]            per-run (max, sum) of each softmax row, log2 domain
  size_t part_ksum;      // float  [slots][D]                per-run partial sums of normalised keys
  size_t rbar;           // float  [units]
  size_t nb;             // float  [units][nb_rows]          -b_r per window-query row (-inf past G*W)
  size_t kbarp;          // uint4  [units][64]               mean normalised key as MFMA operand pieces
  size_t invnorm;        // float  [units][Npad]             1 / |K_i|
  size_t vnorm;          // float  [units][Npad]             |V_i|
  size_t araw;           // float  [units][Npad]             window/group mean attention before pooling
  size_t sdiv;           // float  [units][Npad]             K_i . Kbar (the mix kernel applies -1/|K_i|)
  size_t cand_idx;       // int32  [units][kMaxCandPerHead]  adaptive mode, selection alone: every head's best
  size_t cand_key;       // uint32 [units][kMaxCandPerHead]  candidates, ascending, and their order keys (unused in the full layout)
  size_t scores;         // float  [units][N]                used when the caller passes no scores buffer
  size_t total;
};

// Where the heads' candidate lists for the head-adaptive split live: positions and order keys of unit u at
// idx / key (byte offsets into the workspace) + u * stride entries.
struct CandLists {
  size_t idx, key;
  int64_t stride;
};

// Bit 31 of a candidate-list entry: the candidate is one of its head's `floor` best.
constexpr uint32_t kFloorFlag = 0x80000000u;

// How a long row is cut over several workgroups: nseg segments of seg candidates, whose lists have `merge` entries
// together (seg 0: the row cannot be cut); with `rounds` > 0 lists are merged in groups that many times first, and the
// last merge has up to `merge` entries.
struct SegPlan { int seg, nseg, merge, rounds; };

mixkv_status make_shape(const mixkv_params *p, Shape *s);
void carve_workspace(const Shape &s, int64_t units, Workspace *w, bool select_only = false);

// Kernel launchers (one per pipeline stage).  `unit0` is the first unit of this launch group,
// `nunits` the number of units it covers (whole layers).
// `grid` (from stream_grid) is the number of workgroups of the two streaming kernels; `slot0` is the
// first partial slot of this launch group (each group owns kMaxStreamGrid + its units).
int stream_grid(const Shape &s, int nunits, int num_cus);
// `given_lse`: the caller supplies the softmax normalisers, so the first pass takes key and value
// statistics only; `lse` then holds them per layer (all null otherwise).
hipError_t launch_stats(const Shape &s, int dtype, const LayerInTable &in, char *ws, const Workspace &w, int64_t unit0,
                        int nunits, int grid, int64_t slot0, bool given_lse, hipStream_t st);
// A launch's rows of the budget table (per-head mode), which fold_kernel writes to the workspace: its other arguments leave room for 256
// entries in 4 KB (28 layers of 4 heads, 32 of 8).  More of them, and calls without the scoring passes, go through upload_ints, a
// launch of its own.  Calls with that launch -> without: one layer of 4096 tokens 40.8 -> 38.1 us, 28 of 512 48.8 -> 47.4, 8 of 2000
// tokens and 8 heads 54.0 -> 52.8.
constexpr int kFoldBudgets = 256;
struct BudgetRows { int32_t *dst; int32_t n; int32_t v[kFoldBudgets]; };
// Folds the first pass's per-run partials per unit (exponent offsets, mean key, redundancy).  `grid`
// and `items_per_unit` describe the work split of the first-pass kernel that wrote them.
hipError_t launch_fold(const Shape &s, int dtype, const LayerOutTable &out, const LseTable &lse, char *ws, const Workspace &w,
                       int64_t unit0, int nunits, int grid, int items_per_unit, int64_t slot0, const BudgetRows *budgets, hipStream_t st);
hipError_t launch_attn(const Shape &s, int dtype, const LayerInTable &in, const LayerOutTable &out, const LseTable &lse,
                       char *ws, const Workspace &w, int64_t unit0, int nunits, int grid, int64_t slot0, hipStream_t st);
// The two passes for few query rows (mixkv_keysplit.hip); `grid` from keysplit_grid.
bool keysplit_supported(const Shape &s, int dtype);
int keysplit_grid(const Shape &s, int dtype, int nunits, int num_cus);
hipError_t launch_ks_stats(const Shape &s, int dtype, const LayerInTable &in, char *ws, const Workspace &w, int64_t unit0, int nunits,
                           int grid, int64_t slot0, hipStream_t st);
hipError_t launch_ks_attn(const Shape &s, int dtype, const LayerInTable &in, char *ws, const Workspace &w, int64_t unit0, int nunits,
                          int grid, hipStream_t st);
// The first pass of long bf16 launches (mixkv_qstats.hip); `max_stride_n`: largest row stride of the launch, in elements.
bool qstats_supported(const Shape &s, int dtype, int nunits, int num_cus, int64_t max_stride_n);
int qstats_grid(const Shape &s, int nunits, int num_cus);
hipError_t launch_qstats(const Shape &s, const LayerInTable &in, char *ws, const Workspace &w, int64_t unit0, int nunits, int grid,
                         int64_t slot0, hipStream_t st);
// The second pass of long bf16 launches (mixkv_keystat.hip).
bool keystat_supported(const Shape &s, int dtype, int nunits, int num_cus);
hipError_t launch_kst_attn(const Shape &s, const LayerInTable &in, char *ws, const Workspace &w, int64_t unit0, int nunits, int num_cus,
                           hipStream_t st);
hipError_t launch_mix(const Shape &s, const LayerInTable &in, const LayerOutTable &out, char *ws, const Workspace &w,
                      int64_t unit0, int nunits, hipStream_t st);
// Weights of s_imp and of the scaled diversity in s_comp (Sec. 3.3, Eq. 5; Table 4's variants);
// r is the head's redundancy, rg the caller's weight.
__device__ __forceinline__ void mix_weights(int mix, float r, float rg, float &wi, float &wd) {
  switch (mix) {
    case MIXKV_MIX_SUM: wi = 1.f; wd = 1.f; break;
    case MIXKV_MIX_DIV_ONLY: wi = 0.f; wd = 1.f; break;
    case MIXKV_MIX_IMP_ONLY: wi = 1.f; wd = 0.f; break;
    case MIXKV_MIX_GIVEN_R: wi = 1.f - rg; wd = rg; break;
    default: wi = 1.f - r; wd = r; break;
  }
}
// |K_i| from its stored reciprocal (0 for a key that normalises to the zero vector).
__device__ __forceinline__ float neg_key_norm(float inv_norm) { return inv_norm > 0.f ? -1.f / inv_norm : 0.f; }
// `budgets` (per-head budget mode, else null): device table [layers of this launch][hkv].
hipError_t launch_select(const Shape &s, const LayerOutTable &out, int nlayers, const int32_t *budgets, hipStream_t st);
// Copies `n` ints from host memory to device memory through kernel arguments (no memcpy, so the
// call neither synchronises nor depends on how the host memory was allocated).
hipError_t upload_ints(const int32_t *host, int n, int32_t *dev, hipStream_t st);
// Head-adaptive budget split from the per-head candidate lists (cand_m entries each) in the workspace.
int adaptive_candidates(const Shape &s);   // cand_m, 0 if no head keeps anything but its window
hipError_t launch_select_candidates(const Shape &s, const LayerOutTable &out, char *ws, const CandLists &cl, int64_t unit0,
                                    int nlayers, int cand_m, hipStream_t st);
hipError_t launch_split_stream(const Shape &s, const LayerOutTable &out, char *ws, const CandLists &cl, int64_t unit0, int nlayers,
                               int cand_m, hipStream_t st);
// Long rows (mixkv_longrow.hip): the cut for up to `keep` kept candidates per head, the mix (and with `select` the
// segments' lists), the lists from scores in memory, and their merge.
SegPlan plan_segments(const Shape &s, int keep);
CandLists merged_lists(const SegPlan &pl, const Shape &s, const Workspace &w);   // where the heads' lists are after the merge
hipError_t launch_segmix(const Shape &s, const SegPlan &pl, bool select, const LayerInTable &in, const LayerOutTable &out, char *ws,
                         const Workspace &w, int64_t unit0, int nunits, int cand_m, const int32_t *budgets, hipStream_t st);
hipError_t launch_segtop(const Shape &s, const SegPlan &pl, const LayerOutTable &out, char *ws, const Workspace &w, int64_t unit0,
                         int nunits, int cand_m, const int32_t *budgets, hipStream_t st);
hipError_t launch_mergetop(const Shape &s, const SegPlan &pl, int keep, const LayerOutTable &out, char *ws, const Workspace &w,
                           const CandLists &cl, int64_t unit0, int nunits, int cand_m, const int32_t *budgets, hipStream_t st);
hipError_t launch_gather(const Shape &s, int dtype, const LayerInTable &in, const LayerOutTable &out, int nlayers,
                         hipStream_t st);

}  // namespace mixkv
