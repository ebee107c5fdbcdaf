// Mixing and selection of long rows: several workgroups per head.
//
// A head's candidates are cut into segments of THREADS * EPT, one workgroup each.
//   segstat_kernel   pools the segment's attention and takes its share of the head's statistics;
//   segmix_kernel    folds the shares, forms the segment's mixed scores and, if a selection follows, hands the
//                    segment's best `keep` candidates on as a list (ascending positions, with their order keys);
//   segtop_kernel    the same lists from scores that are already in memory (mixkv_select);
//   mergetop_kernel  one workgroup per head selects from the head's lists laid end to end; lists too long for one
//                    workgroup are merged in groups first, each group's best `keep` being the next round's list.
// A head that keeps `keep` candidates keeps none that is not among the `keep` best of its own segment, and the
// lists hold equal scores in ascending position, so the result is the one a ranking of the whole row gives.
//
// Bound: HBM (four rows of floats per key, read by the statistics and again by the mix; the diversity and the
// intrinsic score stay in registers from then on).  One 130 688-token prompt of 28 layers and 4 KV heads (234 MB of
// rows, budget 128, head-adaptive): statistics 37 us (6.3 TB/s), mix and lists 65, merge 20, split 5.9 (44, 82, 31 and 8.8 before
// the loads of a thread were in flight together and the search took six barriers).  One workgroup
// per head for the mix and one per layer for the selection left most of the chip idle: 784 + 2 583 us.
// At 32 768 tokens (448 heads) mixsel_kernel, which holds a whole head, takes 97 us, and the three kernels took no less than it.
//
// Paper: Sec. 3.2 Eq. 2, Sec. 3.3 Eq. 5, Sec. 3.1 / Algorithm 1 (TopB), as in mixsel_kernel.
#include <cfloat>
#include <type_traits>
#include <utility>

#include "mixkv_topsel.h"

namespace mixkv {

constexpr int kHalo = 32;                // candidates on either side of a segment that the pooling window may reach
constexpr int kMaxMerge = 1024 * 32;     // list entries mergetop_kernel can hold (registers and LDS)

// Shares of a head's statistics, one per segment (in the rows that held the softmax offsets: the second pass was
// their last reader).  Sums of intrinsic score and diversity are taken above the share's own minimum: every term is
// non-negative, here and where two shares meet, so no outlier costs the sums of the others their low bits.
struct SegStat {
  float sum_a, sum_v, sum_d, min_v, min_d, max_v, max_d;
  float n;                               // candidates in the share
};

// Two shares as one.  Products and sums are written out (the compiler may not contract them one way here and another
// there), and a share of no candidates leaves the other one as it is.
__device__ __forceinline__ SegStat join(const SegStat &x, const SegStat &y) {
  auto above = [](const SegStat &s, float sum, float lo, float lo_all) { return s.n > 0.f ? fmaf(s.n, lo - lo_all, sum) : 0.f; };
  SegStat r;
  r.n = x.n + y.n;
  r.sum_a = x.sum_a + y.sum_a;
  r.min_v = fminf(x.min_v, y.min_v); r.max_v = fmaxf(x.max_v, y.max_v);
  r.min_d = fminf(x.min_d, y.min_d); r.max_d = fmaxf(x.max_d, y.max_d);
  r.sum_v = above(x, x.sum_v, x.min_v, r.min_v) + above(y, y.sum_v, y.min_v, r.min_v);
  r.sum_d = above(x, x.sum_d, x.min_d, r.min_d) + above(y, y.sum_d, y.min_d, r.min_d);
  return r;
}

// The share that the neighbouring group of 2^LEVEL lanes holds, where all lanes of an aligned group hold the same one.
template <int LEVEL>
__device__ __forceinline__ float of_neighbour(float x) {
  if constexpr (LEVEL == 4) return __shfl_xor(x, 16);
  constexpr int ctrl = LEVEL == 0 ? 0xB1 : (LEVEL == 1 ? 0x4E : (LEVEL == 2 ? 0x141 : 0x140));   // quad_perm, quad_perm, half mirror, mirror
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xf, 0xf, true));
}
template <int LEVEL>
__device__ __forceinline__ SegStat join_neighbour(const SegStat &x) {
  return join(x, SegStat{of_neighbour<LEVEL>(x.sum_a), of_neighbour<LEVEL>(x.sum_v), of_neighbour<LEVEL>(x.sum_d),
                         of_neighbour<LEVEL>(x.min_v), of_neighbour<LEVEL>(x.min_d), of_neighbour<LEVEL>(x.max_v),
                         of_neighbour<LEVEL>(x.max_d), of_neighbour<LEVEL>(x.n)});
}
__device__ __forceinline__ SegStat *seg_stats(const Shape &s, char *ws, const Workspace &w, int64_t unit) {
  static_assert(sizeof(SegStat) * kMaxSegs <= 256 * sizeof(float), "a head's shares fit its row of softmax offsets");
  return reinterpret_cast<SegStat *>(reinterpret_cast<float *>(ws + w.nb) + unit * s.nb_rows);
}

// Intrinsic score and diversity of the thread's groups of four, all loads in flight together.
template <int EPT, class GroupOf>
__device__ __forceinline__ void load_rows(const UnitRows &rows, int s0, float (&v)[EPT], float (&d)[EPT], GroupOf group_of) {
  constexpr int G = EPT / 4;
  int at[G];
  float4 vr[G], dr[G];
#pragma unroll
  for (int g = 0; g < G; ++g) at[g] = rows.inside(s0 + group_of(g) * 4);
  rows.load_vd<G>(at, vr, dr);
#pragma unroll
  for (int g = 0; g < G; ++g) {
    v[4 * g] = vr[g].x; v[4 * g + 1] = vr[g].y; v[4 * g + 2] = vr[g].z; v[4 * g + 3] = vr[g].w;
    d[4 * g] = dr[g].x; d[4 * g + 1] = dr[g].y; d[4 * g + 2] = dr[g].z; d[4 * g + 3] = dr[g].w;
  }
}

// Loads the raw attention of the segment [s0, s0 + THREADS * EPT) and its halo into LDS (out-of-range
// candidates hold the pooling's neutral element) and leaves the pooled values of the thread's candidates in
// a[]: group_of(0), group_of(1), ... are the thread's groups of four, consecutive threads holding consecutive groups
// so that all loads are coalesced.  Ends past its reads of LDS only after the caller's next barrier.
template <int THREADS, int EPT, class GroupOf>
__device__ __forceinline__ void load_pooled(const Shape &s, const UnitRows &rows, int s0, float (&a)[EPT], float *a_s, GroupOf group_of) {
  const float *araw = rows.araw;
  const int tid = threadIdx.x, Nc = s.Nc;
  const bool pooled = s.pool != MIXKV_POOL_NONE && s.pool_k > 1, is_max = s.pool == MIXKV_POOL_MAX;
  const float fill = is_max ? -INFINITY : 0.f;          // out-of-range taps: ignored by max, zero for avg
  float4 raw[EPT / 4];                                  // the rows are padded past the last group
#pragma unroll
  for (int g = 0; g < EPT / 4; ++g) raw[g] = *reinterpret_cast<const float4 *>(araw + rows.inside(s0 + group_of(g) * 4));
  if (tid < 2 * kHalo) {
    const int i = tid < kHalo ? s0 - kHalo + tid : s0 + THREADS * EPT + tid - kHalo;
    const int li = tid < kHalo ? tid : THREADS * EPT + tid;
    a_s[slot4(li)] = (pooled && i >= 0 && i < Nc) ? araw[i] : fill;
  }
#pragma unroll
  for (int g = 0; g < EPT / 4; ++g) {
    const int li = group_of(g) * 4, i = s0 + li;
    float4 r = raw[g];
    if (i >= Nc) r.x = fill;
    if (i + 1 >= Nc) r.y = fill;
    if (i + 2 >= Nc) r.z = fill;
    if (i + 3 >= Nc) r.w = fill;
    a[4 * g] = r.x; a[4 * g + 1] = r.y; a[4 * g + 2] = r.z; a[4 * g + 3] = r.w;
    *reinterpret_cast<float4 *>(&a_s[slot4(kHalo + li)]) = r;
  }
  __syncthreads();
  if (!pooled) return;
  const int hk = s.pool_k >> 1;
  if (hk <= 3) {
    // sliding window in registers over each group: its own values and the aligned groups on either side
#pragma unroll
    for (int g = 0; g < EPT / 4; ++g) {
      const int li = kHalo + group_of(g) * 4;
      const float4 lo = *reinterpret_cast<const float4 *>(&a_s[slot4(li - 4)]);
      const float4 hi = *reinterpret_cast<const float4 *>(&a_s[slot4(li + 4)]);
      const float win[10] = {lo.y, lo.z, lo.w, a[4 * g], a[4 * g + 1], a[4 * g + 2], a[4 * g + 3], hi.x, hi.y, hi.z};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float acc;
        if (is_max) {
          acc = win[3 + e];
          if (hk >= 1) acc = fmaxf(acc, fmaxf(win[2 + e], win[4 + e]));
          if (hk >= 2) acc = fmaxf(acc, fmaxf(win[1 + e], win[5 + e]));
          if (hk >= 3) acc = fmaxf(acc, fmaxf(win[e], win[6 + e]));
        } else {                                        // taps from left to right
          acc = 0.f;
          if (hk >= 3) acc += win[e];
          if (hk >= 2) acc += win[1 + e];
          if (hk >= 1) acc += win[2 + e];
          acc += win[3 + e];
          if (hk >= 1) acc += win[4 + e];
          if (hk >= 2) acc += win[5 + e];
          if (hk >= 3) acc += win[6 + e];
          acc = acc / (float)s.pool_k;
        }
        a[4 * g + e] = acc;
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int li = kHalo + group_of(e >> 2) * 4 + (e & 3);
      float acc = a_s[slot4(li - hk)];
      for (int j = li - hk + 1; j <= li + hk; ++j) acc = is_max ? fmaxf(acc, a_s[slot4(j)]) : acc + a_s[slot4(j)];
      a[e] = is_max ? acc : acc / (float)s.pool_k;
    }
  }
}

// The statistics are shares of a wave's 512 candidates, joined along one tree over the row: the eight waves of a block of
// 4096, neighbouring blocks here if a segment has several, the segments in segmix_kernel.  The tree is the same
// for every cut, so the bits of the statistics, and with them the scores', depend neither on the budget nor on
// whether a selection follows.  A block is the work of 512 threads, eight candidates each; a workgroup has one or
// two such halves, and at four blocks a half takes two.  Against one reduction over whatever the workgroup holds:
// statistics and mix 125 -> 126 us (one block, 112 heads of 130 688), 137 -> 139 (two, 140 001), 173 -> 182 (four, 131 000).
constexpr int kStatThreads = 512, kStatEpt = 8, kStatBlock = kStatThreads * kStatEpt, kStatWaves = kStatThreads / 64;

template <int BLOCKS>
__global__ __launch_bounds__(kStatThreads * (BLOCKS > 1 ? 2 : 1)) void segstat_kernel(Shape s, char *ws, Workspace w, int64_t unit0, int nseg) {
  static_assert((BLOCKS == 1 || BLOCKS == 2 || BLOCKS == 4) && kStatWaves == 8, "a tree of neighbours, up to five levels");
  constexpr int HALVES = BLOCKS > 1 ? 2 : 1, THREADS = HALVES * kStatThreads, TURNS = BLOCKS / HALVES, EPT = TURNS * kStatEpt;
  __shared__ __align__(16) float a_s[slots4(BLOCKS * kStatBlock + 2 * kHalo)];
  __shared__ SegStat share_s[BLOCKS * kStatWaves];
  const int ul = blockIdx.x / nseg, seg = blockIdx.x - ul * nseg, s0 = seg * BLOCKS * kStatBlock, tid = threadIdx.x, lane = tid & 63;
  const int half = tid / kStatThreads, ht = tid % kStatThreads, hw = ht / 64;
  const int64_t unit = unit0 + ul;
  const UnitRows rows(s, ws, w, unit);
  // group g of the thread: turn g / 2 is block HALVES * (g / 2) + half
  auto group_of = [&](int g) { return ((HALVES * (g >> 1) + half) * 2 + (g & 1)) * kStatThreads + ht; };
  float v[EPT], d[EPT], a[EPT];
  load_rows<EPT>(rows, s0, v, d, group_of);
  load_pooled<THREADS, EPT>(s, rows, s0, a, a_s, group_of);
#pragma unroll
  for (int t = 0; t < TURNS; ++t) {
    auto on = [&](int e) { return s0 + group_of(e >> 2) * 4 + (e & 3) < s.Nc; };
    float min_v = INFINITY, min_d = INFINITY, max_v = -INFINITY, max_d = -INFINITY, sum_a = 0.f, sum_v = 0.f, sum_d = 0.f;
#pragma unroll
    for (int e = t * kStatEpt; e < (t + 1) * kStatEpt; ++e)
      if (on(e)) {
        min_v = fminf(min_v, v[e]); min_d = fminf(min_d, d[e]);
        max_v = fmaxf(max_v, v[e]); max_d = fmaxf(max_d, d[e]);
      }
    min_v = wave_reduce<WMin>(min_v, INFINITY); min_d = wave_reduce<WMin>(min_d, INFINITY);
    max_v = wave_reduce<WMax>(max_v, -INFINITY); max_d = wave_reduce<WMax>(max_d, -INFINITY);
#pragma unroll
    for (int e = t * kStatEpt; e < (t + 1) * kStatEpt; ++e)
      if (on(e)) { sum_a += a[e]; sum_v += v[e] - min_v; sum_d += d[e] - min_d; }
    sum_a = wave_reduce<WSum>(sum_a, 0.f); sum_v = wave_reduce<WSum>(sum_v, 0.f); sum_d = wave_reduce<WSum>(sum_d, 0.f);
    const int block = HALVES * t + half, left = s.Nc - s0 - block * kStatBlock - hw * 256;   // the wave's first and second 64 groups
    const int n = min(max(left, 0), 256) + min(max(left - kStatBlock / 2, 0), 256);
    if (lane == 0) share_s[block * kStatWaves + hw] = SegStat{sum_a, sum_v, sum_d, min_v, min_d, max_v, max_d, (float)n};
  }
  __syncthreads();
  if (tid >= 64) return;
  SegStat x{0.f, 0.f, 0.f, INFINITY, INFINITY, -INFINITY, -INFINITY, 0.f};
  if (lane < BLOCKS * kStatWaves) x = share_s[lane];
  x = join_neighbour<0>(x); x = join_neighbour<1>(x); x = join_neighbour<2>(x);
  if constexpr (BLOCKS > 1) x = join_neighbour<3>(x);
  if constexpr (BLOCKS > 2) x = join_neighbour<4>(x);
  if (lane == 0) seg_stats(s, ws, w, unit)[seg] = x;
}

// 1 / den for quotient().  An eps too small for a float reciprocal leaves a head of equal values (range 0) such a
// denominator: the quotients are 0 then, not 0 times infinity.
__device__ __forceinline__ float reciprocal(float den) { return fminf(1.f / den, FLT_MAX); }
// num / den to within half a unit in the last place, given rden = 1 / den
__device__ __forceinline__ float quotient(float num, float den, float rden) {
  const float q = num * rden;
  return fmaf(fmaf(-q, den, num), rden, q);
}

// Candidates a head hands on from every segment: the rows it keeps besides the window (fixed and per-head
// mode), or its candidates for the head-adaptive split.
__device__ __forceinline__ int head_keep(const Shape &s, const int32_t *budgets, int layer, int h, int cand_m) {
  return cand_m > 0 ? cand_m : (budgets ? budgets[layer * s.hkv + h] : s.B) - s.W;
}

// The segment's best min(keep, len) candidates, out of the order keys in k_s (slot4(0) is candidate s0).
template <int THREADS, int EPT>
__device__ __forceinline__ void segment_list(const uint32_t *k_s, int s0, int len, int keep, int32_t *idx, uint32_t *ckey, MsScratch &sc) {
  const int base = threadIdx.x * EPT;
  uint32_t key[EPT];
  read_keys<EPT>(k_s, base, len, key);
  top_select_keys<THREADS, EPT>(key, min(keep, len), idx, ckey, 0, sc, [&](int e) { return s0 + base + e; });
}

template <int THREADS, int EPT, bool SELECT>
__global__ __launch_bounds__(THREADS) void segmix_kernel(Shape s, LayerInTable in, LayerOutTable out, char *ws, Workspace w,
                                                         int64_t unit0, int nseg, int cand_m, const int32_t *budgets) {
  constexpr int SEG = THREADS * EPT;
  __shared__ __align__(16) float a_s[slots4(SEG + 2 * kHalo)];
  __shared__ MsScratch sc;
  const int ul = blockIdx.x / nseg, seg = blockIdx.x - ul * nseg, s0 = seg * SEG, tid = threadIdx.x, lane = tid & 63;
  const int64_t unit = unit0 + ul;
  const int layer = ul / s.units_per_layer, bh = ul - layer * s.units_per_layer, Nc = s.Nc;
  const LayerOut O = out.l[layer];
  const UnitRows rows(s, ws, w, unit);

  float v[EPT], d[EPT], a[EPT];
  auto group_of = [&](int g) { return g * THREADS + tid; };
  load_rows<EPT>(rows, s0, v, d, group_of);
  load_pooled<THREADS, EPT>(s, rows, s0, a, a_s, group_of);

  // ---- the head's statistics: lane l holds segment l's share, every wave folds neighbours, then pairs of them, ...
  // From here on products and sums that the compiler could contract in two ways are written out: all instantiations
  // give the same bits.
  static_assert(kMaxSegs == 32, "five levels");
  const SegStat *shares = seg_stats(s, ws, w, unit);
  SegStat x{0.f, 0.f, 0.f, INFINITY, INFINITY, -INFINITY, -INFINITY, 0.f};
  if (lane < nseg) x = shares[lane];
  x = join_neighbour<0>(x); x = join_neighbour<1>(x); x = join_neighbour<2>(x); x = join_neighbour<3>(x); x = join_neighbour<4>(x);
  const float vmin = read_lane(x.min_v, 0), dmin = read_lane(x.min_d, 0), vmax = read_lane(x.max_v, 0), dmax = read_lane(x.max_d, 0);
  const float inv_n = 1.f / (float)Nc;
  const float r = reinterpret_cast<const float *>(ws + w.rbar)[unit];
  float wi, wd;
  mix_weights(s.mix, r, s.mix == MIXKV_MIX_GIVEN_R ? in.l[layer].r_given[bh] : 0.f, wi, wd);
  const float mean_ex = read_lane(x.sum_a, 0) * inv_n;
  const float vden = vmax - vmin + s.eps, dden = dmax - dmin + s.eps, rvden = reciprocal(vden), rdden = reciprocal(dden);
  const float mean_in = read_lane(x.sum_v, 0) * inv_n / vden;           // mean((x - min) / den)
  const float mean_dn = read_lane(x.sum_d, 0) * inv_n / dden;
  const float f_in = rows.use_v ? mean_ex / (mean_in + s.eps) : 0.f;    // Sec. 3.2: scale VNorm to mean(s_ex)
  const float mean_imp = rows.use_v ? fmaf(f_in, mean_in, mean_ex) : mean_ex;
  const float f_div = mean_imp / (mean_dn + s.eps);                      // Sec. 3.3: scale diversity to mean(s_imp)
  const int len = min(SEG, Nc - s0);
  float *scores = O.scores ? O.scores + (int64_t)bh * s.N + s0 : nullptr;
  uint32_t *k_s = reinterpret_cast<uint32_t *>(a_s);
  KeyRange range;
  if constexpr (SELECT) __syncthreads();                // the pooling is done with the raw attention: the order keys replace it
#pragma unroll
  for (int g = 0; g < EPT / 4; ++g) {
    const int li = group_of(g) * 4;
    uint32_t k4[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = 4 * g + j;
      const float imp = rows.use_v ? fmaf(quotient(v[e] - vmin, vden, rvden), f_in, a[e]) : a[e];   // Eq. 2
      const float c = fmaf(wi, imp, wd * (quotient(d[e] - dmin, dden, rdden) * f_div));              // Eq. 5
      if (scores && li + j < len) scores[li + j] = c;
      k4[j] = li + j < len ? order_key_u(c) : 0u;
      range.add_or_none(k4[j], li + j < len);
    }
    if constexpr (SELECT) *reinterpret_cast<uint4 *>(&k_s[slot4(li)]) = make_uint4(k4[0], k4[1], k4[2], k4[3]);
  }
  if (scores && seg == nseg - 1)
    for (int i = len + tid; i < s.N - s0; i += THREADS) scores[i] = INFINITY;
  if constexpr (SELECT) thresholds_begin<THREADS>(range, sc);
  if constexpr (SELECT) __syncthreads();
  if constexpr (SELECT) {
    // the list takes the place of the segment's own share of two rows that have been read
    const int keep = head_keep(s, budgets, layer, bh % s.hkv, cand_m);
    int32_t *idx = reinterpret_cast<int32_t *>(ws + w.sdiv) + unit * s.Npad + s0;
    uint32_t *ckey = reinterpret_cast<uint32_t *>(ws + w.invnorm) + unit * s.Npad + s0;
    if (keep > 0) segment_list<THREADS, EPT>(k_s, s0, len, keep, idx, ckey, sc);
  }
}

template <int THREADS, int EPT>
__global__ __launch_bounds__(THREADS) void segtop_kernel(Shape s, LayerOutTable out, char *ws, Workspace w, int64_t unit0,
                                                         int nseg, int cand_m, const int32_t *budgets) {
  constexpr int SEG = THREADS * EPT;
  __shared__ __align__(16) uint32_t k_s[slots4(SEG)];
  __shared__ MsScratch sc;
  const int ul = blockIdx.x / nseg, seg = blockIdx.x - ul * nseg, s0 = seg * SEG, tid = threadIdx.x;
  const int64_t unit = unit0 + ul;
  const int layer = ul / s.units_per_layer, bh = ul - layer * s.units_per_layer, len = min(SEG, s.Nc - s0);
  const float *scores = out.l[layer].scores + (int64_t)bh * s.N + s0;
  float a[EPT];
#pragma unroll
  for (int k = 0; k < EPT; ++k) a[k] = scores[min(k * THREADS + tid, len - 1)];     // all in flight together
  KeyRange range;
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const uint32_t key = order_key_u(a[k]);
    range.add(key);                                     // past the segment its last score again
    k_s[slot4(k * THREADS + tid)] = key;
  }
  thresholds_begin<THREADS>(range, sc);
  __syncthreads();
  const int keep = head_keep(s, budgets, layer, bh % s.hkv, cand_m);
  int32_t *idx = reinterpret_cast<int32_t *>(ws + w.sdiv) + unit * s.Npad + s0;
  uint32_t *ckey = reinterpret_cast<uint32_t *>(ws + w.invnorm) + unit * s.Npad + s0;
  if (keep > 0) segment_list<THREADS, EPT>(k_s, s0, len, keep, idx, ckey, sc);
}

// One workgroup per head: its rows (fixed and per-head mode) or its candidates for the head-adaptive split, out
// of its lists: nseg of them in `from`, each with the best of `seg` candidates.  PART: one workgroup per `group`
// lists, which leaves the best of them as one list in `to`, at the group's first candidate.
template <int THREADS, int EPT, bool PART>
__global__ __launch_bounds__(THREADS) void mergetop_kernel(Shape s, LayerOutTable out, char *ws, CandLists from, CandLists to,
                                                           int64_t unit0, int seg, int nseg, int group, int cand_m, const int32_t *budgets) {
  extern __shared__ __align__(16) uint32_t k_s[];
  __shared__ MsScratch sc;
  const int ngroups = PART ? (nseg + group - 1) / group : 1;
  const int ul = PART ? blockIdx.x / ngroups : blockIdx.x, first = PART ? (blockIdx.x - ul * ngroups) * group : 0, tid = threadIdx.x;
  const int64_t unit = unit0 + ul;
  const int layer = ul / s.units_per_layer, bh = ul - layer * s.units_per_layer, h = bh % s.hkv, b = bh / s.hkv;
  const LayerOut O = out.l[layer];
  const int32_t *lidx = reinterpret_cast<const int32_t *>(ws + from.idx) + unit * from.stride + first * seg;
  const uint32_t *lkey = reinterpret_cast<const uint32_t *>(ws + from.key) + unit * from.stride + first * seg;
  const int keep = head_keep(s, budgets, layer, h, cand_m), per = min(keep, seg);   // entries per list, the row's last one may have fewer
  const int lists = PART ? min(group, nseg - first) : nseg;
  const int n = per > 0 ? (lists - 1) * per + min(per, s.Nc - (first + lists - 1) * seg) : 0;
  auto at = [&](int e) { const int g = e / per; return g * seg + (e - g * per); };
  const int base = tid * EPT;
  uint32_t key[EPT];
  KeyRange range;
  if (n > 0) {
#pragma unroll
    for (int k = 0; k < EPT; ++k) key[k] = lkey[at(min(k * THREADS + tid, n - 1))];  // all in flight together
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      range.add(key[k]);                                // past the lists the last entry again
      if (k * THREADS + tid < n) k_s[slot4(k * THREADS + tid)] = key[k];
    }
  }
  thresholds_begin<THREADS>(range, sc);
  __syncthreads();
  read_keys<EPT>(k_s, base, n, key);
  auto pos = [&](int e) { return lidx[at(base + e)]; };
  if (PART || cand_m > 0) {
    int32_t *idx = reinterpret_cast<int32_t *>(ws + to.idx) + unit * to.stride + first * seg;
    uint32_t *ckey = reinterpret_cast<uint32_t *>(ws + to.key) + unit * to.stride + first * seg;
    if (!PART) top_select_keys<THREADS, EPT>(key, cand_m, idx, ckey, s.floor_, sc, pos);
    else if (n > 0) top_select_keys<THREADS, EPT>(key, min(keep, n), idx, ckey, 0, sc, pos);
    return;
  }
  int Bh, row0;
  head_rows(s, budgets, layer, h, Bh, row0);
  int32_t *idx = O.indices + (int64_t)b * s.hkv * s.B + row0;
  if (keep > 0) top_select_keys<THREADS, EPT>(key, keep, idx, nullptr, 0, sc, pos);
  finish_head(s, O, b, h, Bh, row0, idx, THREADS);
}

// ------------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------------
// Entries of the lists of up to `keep` candidates that nseg segments of `seg` candidates leave of a row.
static int64_t list_entries(const Shape &s, int keep, int64_t seg, int nseg) {
  const int64_t per = keep < seg ? keep : seg, last = s.Nc - (nseg - 1) * seg;
  return (nseg - 1) * per + (per < last ? per : last);
}

// Lists per workgroup of a round that leaves fewer lists, as even as they come: `keep` <= kMaxMerge / 2 entries each.
static int round_group(int keep, int nseg) {
  const int most = kMaxMerge / keep, groups = (nseg + most - 1) / most;
  return (nseg + groups - 1) / groups;
}

// The cut of a row of Nc candidates of which up to `keep` survive per head (0: no selection): the smallest
// segments that give at most kMaxSegs of them, as long as the merge has no more than 16 384 entries to look at
// (beyond that its one workgroup per head is the longer half); failing that the largest that fit it.  Longer lists, of up
// to half of what a workgroup holds, are merged in rounds.  Beyond that one workgroup ranks whole rows
// (select_adaptive_kernel: all heads' rows of a batch item), which took these, too: selection alone, head-adaptive, us before ->
// after: 130 688 tokens, 4 heads, budget 1200 1856 -> 84, 28 layers of them 2399 -> 142, budget 960 (one merge of 29 696 entries) 2396 -> 54;
// 8 heads, budget 600 3671 -> 110; 14 layers of 131 072 tokens, 8 heads, budget 2048 4603 -> 873; 60 000 tokens, 8 heads, budget 2048
// 1691 -> 372.
SegPlan plan_segments(const Shape &s, int keep) {
  SegPlan best{0, 0, 0, 0};
  for (int seg : {4096, 8192, 16384}) {
    const int nseg = (s.Nc + seg - 1) / seg;
    if (nseg < 2 || nseg > kMaxSegs) continue;
    const int64_t n = list_entries(s, keep, seg, nseg);
    if (n > kMaxMerge) continue;
    best = SegPlan{seg, nseg, (int)n, 0};
    if (n <= 16384) break;
  }
  const int seg = 16384, nseg = (s.Nc + seg - 1) / seg;
  if (best.seg == 0 && keep <= seg && nseg >= 2 && nseg <= kMaxSegs) {
    best = SegPlan{seg, nseg, kMaxMerge, 0};
    for (int64_t len = seg, left = nseg; list_entries(s, keep, len, (int)left) > kMaxMerge; ++best.rounds) {
      const int group = round_group(keep, (int)left);
      left = (left + group - 1) / group;
      len *= group;
    }
  }
  return best;
}

CandLists merged_lists(const SegPlan &pl, const Shape &s, const Workspace &w) {
  return pl.rounds % 2 ? CandLists{w.sdiv, w.invnorm, s.Npad} : CandLists{w.araw, w.vnorm, s.Npad};
}

template <int THREADS, int EPT>
static hipError_t launch_segmix_e(const Shape &s, const SegPlan &pl, bool select, const LayerInTable &in, const LayerOutTable &out,
                                  char *ws, const Workspace &w, int64_t unit0, int nunits, int cand_m, const int32_t *budgets,
                                  hipStream_t st) {
  const dim3 grid((unsigned)(nunits * pl.nseg)), block(THREADS);
  hipLaunchKernelGGL((segstat_kernel<THREADS * EPT / kStatBlock>), grid, block, 0, st, s, ws, w, unit0, pl.nseg);
  if (select) hipLaunchKernelGGL((segmix_kernel<THREADS, EPT, true>), grid, block, 0, st, s, in, out, ws, w, unit0, pl.nseg, cand_m, budgets);
  else hipLaunchKernelGGL((segmix_kernel<THREADS, EPT, false>), grid, block, 0, st, s, in, out, ws, w, unit0, pl.nseg, 0, nullptr);
  return hipGetLastError();
}

hipError_t launch_segmix(const Shape &s, const SegPlan &pl, bool select, const LayerInTable &in, const LayerOutTable &out, char *ws,
                         const Workspace &w, int64_t unit0, int nunits, int cand_m, const int32_t *budgets, hipStream_t st) {
  if (pl.seg == 4096) return launch_segmix_e<512, 8>(s, pl, select, in, out, ws, w, unit0, nunits, cand_m, budgets, st);
  if (pl.seg == 8192) return launch_segmix_e<1024, 8>(s, pl, select, in, out, ws, w, unit0, nunits, cand_m, budgets, st);
  return launch_segmix_e<1024, 16>(s, pl, select, in, out, ws, w, unit0, nunits, cand_m, budgets, st);
}

hipError_t launch_segtop(const Shape &s, const SegPlan &pl, const LayerOutTable &out, char *ws, const Workspace &w, int64_t unit0,
                         int nunits, int cand_m, const int32_t *budgets, hipStream_t st) {
  const dim3 grid((unsigned)(nunits * pl.nseg));
  if (pl.seg == 4096) hipLaunchKernelGGL((segtop_kernel<512, 8>), grid, dim3(512), 0, st, s, out, ws, w, unit0, pl.nseg, cand_m, budgets);
  else if (pl.seg == 8192) hipLaunchKernelGGL((segtop_kernel<1024, 8>), grid, dim3(1024), 0, st, s, out, ws, w, unit0, pl.nseg, cand_m, budgets);
  else hipLaunchKernelGGL((segtop_kernel<1024, 16>), grid, dim3(1024), 0, st, s, out, ws, w, unit0, pl.nseg, cand_m, budgets);
  return hipGetLastError();
}

// Rounds of merges, the lists going to and fro between the two pairs of rows, and the last merge.
template <int THREADS, int EPT, bool PART>
static hipError_t launch_mergetop_e(const Shape &s, int entries, const LayerOutTable &out, char *ws, const CandLists &from, const CandLists &to,
                                    int64_t unit0, int nunits, int seg, int nseg, int group, int cand_m, const int32_t *budgets, hipStream_t st) {
  auto kern = mergetop_kernel<THREADS, EPT, PART>;
  static LdsLimitOnce once;
  const hipError_t attr = once.raise(reinterpret_cast<const void *>(kern));
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kern, dim3(nunits * (PART ? (nseg + group - 1) / group : 1)), dim3(THREADS), (size_t)slots4(entries) * 4, st, s, out, ws,
                     from, to, unit0, seg, nseg, group, cand_m, budgets);
  return hipGetLastError();
}

hipError_t launch_mergetop(const Shape &s, const SegPlan &pl, int keep, const LayerOutTable &out, char *ws, const Workspace &w,
                           const CandLists &cl, int64_t unit0, int nunits, int cand_m, const int32_t *budgets, hipStream_t st) {
  CandLists from{w.sdiv, w.invnorm, s.Npad}, to{w.araw, w.vnorm, s.Npad};
  int seg = pl.seg, nseg = pl.nseg;
  for (int r = 0; r < pl.rounds; ++r) {
    const int group = round_group(keep, nseg);
    const hipError_t e = launch_mergetop_e<1024, 32, true>(s, group * keep, out, ws, from, to, unit0, nunits, seg, nseg, group, cand_m, budgets, st);
    if (e != hipSuccess) return e;
    nseg = (nseg + group - 1) / group;
    seg *= group;
    std::swap(from, to);
  }
  auto merge = [&](auto threads, auto ept) {
    return launch_mergetop_e<decltype(threads)::value, decltype(ept)::value, false>(s, pl.merge, out, ws, from, cl, unit0, nunits, seg, nseg, nseg,
                                                                                    cand_m, budgets, st);
  };
  using std::integral_constant;
  if (pl.merge <= 512 * 8) return merge(integral_constant<int, 512>{}, integral_constant<int, 8>{});
  if (pl.merge <= 1024 * 8) return merge(integral_constant<int, 1024>{}, integral_constant<int, 8>{});
  if (pl.merge <= 1024 * 16) return merge(integral_constant<int, 1024>{}, integral_constant<int, 16>{});
  return merge(integral_constant<int, 1024>{}, integral_constant<int, 32>{});
}

}  // namespace mixkv
