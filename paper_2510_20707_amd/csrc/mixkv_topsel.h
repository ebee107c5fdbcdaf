// Workgroup-level selection code shared by the kernels that rank one head's candidates: block reductions and
// scans, the most-significant-digit radix select on order-preserving keys held in registers, and the
// ordered emission of the kept positions.
#pragma once
#include <mutex>

#include "mixkv_internal.h"
#include "mixkv_wave.h"

namespace mixkv {

constexpr int kMsMaxThreads = 1024, kMsMaxWaves = kMsMaxThreads / 64;
constexpr int kDigit = 11, kBins = 1 << kDigit;     // a histogram of the threshold search
constexpr int kSurvivors = 128;                      // keys of a boundary bin that are ranked by counting

struct MsScratch {
  float f[kMsMaxWaves][8];
  uint2 wrange[kMsMaxWaves];             // every wave's KeyRange
  uint2 bin_range[2][kMsMaxWaves];       // per threshold: every wave's greatest and least distance inside its bin
  int i[kMsMaxWaves], i2[kMsMaxWaves];
  int hist[kBins];
  struct { int bin, k, count; } cut[2];  // per threshold: its bin, the keys still needed of that bin, the keys in it
  int nsurv[2], krem[2];
  uint32_t tau[2], surv[2][kSurvivors];
};

// LDS slot of a word: four pad words per 32 keep every aligned group of four together and spread the groups of
// owners a power of two apart over the banks.
__device__ __forceinline__ int slot4(int i) { return i + ((i >> 5) << 2); }
__host__ __device__ constexpr int slots4(int n) { return n + n / 32 * 4 + 4; }

// Block-wide reduction of NS sums, NMIN minima and NMAX maxima at once; every thread gets the
// results back in place.  Fixed order: lanes in lane order inside a wave, then waves in wave order.
template <int NW, int NS, int NMIN, int NMAX>
__device__ __forceinline__ void block_reduce_mixed(float (&v)[NS + NMIN + NMAX], MsScratch &sc) {
  constexpr int NV = NS + NMIN + NMAX;
  static_assert(NV <= 8 && NW <= 16, "scratch holds eight values for sixteen waves");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k)
    v[k] = k < NS ? wave_reduce<WSum>(v[k], 0.f)
                  : (k < NS + NMIN ? wave_reduce<WMin>(v[k], INFINITY) : wave_reduce<WMax>(v[k], -INFINITY));
  __syncthreads();                       // scratch may still be read from a previous call
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < NV; ++k) sc.f[wave][k] = v[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    // every wave folds the NW partials itself (one row of lanes), so no third barrier is needed
    const float id = k < NS ? 0.f : (k < NS + NMIN ? INFINITY : -INFINITY);
    float x = (lane & 15) < NW ? sc.f[lane & 15][k] : id;
    x = k < NS ? row_scan_incl<WSum>(x, id) : (k < NS + NMIN ? row_scan_incl<WMin>(x, id) : row_scan_incl<WMax>(x, id));
    v[k] = read_lane(x, 15);
  }
}

__device__ __forceinline__ int read_lane_dyn(int x, int lane_uniform) {
  return __builtin_amdgcn_readlane(x, __builtin_amdgcn_readfirstlane(lane_uniform));
}

// Exclusive prefix sums of one int per wave's thread, given every wave's total in tot[]; *total receives the block sum.
template <int NW>
__device__ __forceinline__ int waves_before(const int *tot, int *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int x = (lane & 15) < NW ? tot[lane & 15] : 0;
  const int y = row_scan_incl<WSum>(x, 0);              // inclusive over the waves, in every row of lanes
  *total = read_lane(y, 15);
  return wave == 0 ? 0 : read_lane_dyn(y, wave - 1);
}

// Exclusive prefix sum of one int per thread (thread order) behind one barrier; *total receives the block sum.  A barrier
// must lie between this and the last reads of sc.i.
template <int NW>
__device__ __forceinline__ int block_scan_excl(int v, MsScratch &sc, int *total) {
  int wtot;
  const int inc = wave_scan_incl_add(v, &wtot);
  if ((threadIdx.x & 63) == 0) sc.i[threadIdx.x >> 6] = wtot;
  __syncthreads();
  return waves_before<NW>(sc.i, total) + inc - v;
}

// The same for two ints; *total receives the block sum of the first.  A barrier must lie between this and the last reads of sc.i and sc.i2.
template <int NW>
__device__ __forceinline__ void block_scan_excl(int &v, int &v2, MsScratch &sc, int *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int wtot, wtot2, total2;
  const int inc = wave_scan_incl_add(v, &wtot), inc2 = wave_scan_incl_add(v2, &wtot2);
  if (lane == 0) { sc.i[wave] = wtot; sc.i2[wave] = wtot2; }
  __syncthreads();
  v = waves_before<NW>(sc.i, total) + inc - v;
  v2 = waves_before<NW>(sc.i2, &total2) + inc2 - v2;
}

// Order-preserving map float -> uint32 >= 1 (larger float <=> larger key); 0 is left for "no candidate".
__device__ __forceinline__ uint32_t order_key_u(float x) {
  uint32_t u = __float_as_uint(x);
  if (u == 0x80000000u) u = 0;                          // -0 and +0 are the same score
  return max(u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u), 1u);
}

// One count into a shared histogram bin per lane (all lanes take part), with the lanes that share lane 0's bin merged into
// a single atomic: scores of one head often agree in their leading bits, and 64 atomics on one LDS word would run one
// after the other.
__device__ __forceinline__ void hist_add(int *hist, int bin) {
  const int b0 = __builtin_amdgcn_readfirstlane(bin);
  const bool same = bin == b0, lead = (threadIdx.x & 63) == 0;
  const int n = __popcll(__ballot(same));
  if (!same || lead) atomicAdd(&hist[bin], lead ? n : 1);
}

// The same for the lanes with `in` set, merged on the bin of the first of them.
__device__ __forceinline__ void hist_add(int *hist, int bin, bool in) {
  const int first = max(__ffsll((long long)__ballot(in)) - 1, 0);         // wave-uniform
  const bool same = in && bin == __builtin_amdgcn_readlane(bin, first), lead = (int)(threadIdx.x & 63) == first;
  const int n = __popcll(__ballot(same));
  if (in && (!same || lead)) atomicAdd(&hist[bin], lead ? n : 1);
}

// Whether an eighth of the wave's keys with `in` set equal the first of them (or none is set: not known).
__device__ __forceinline__ bool wave_tied(uint32_t key, bool in) {
  const unsigned long long on = __ballot(in);
  const uint32_t k0 = (uint32_t)__builtin_amdgcn_readlane((int)key, max(__ffsll((long long)on) - 1, 0));
  const int n = __popcll(__ballot(in && key == k0));
  return on == 0 || (n > 1 && 8 * n >= __popcll(on));
}

// The bins of sc.hist in which the first k[q] counts end (q < NK; none for k[q] < 1), to sc.cut[Q0 + q].  Ends behind a
// barrier.
template <int THREADS, int NK, int Q0 = 0>
__device__ __forceinline__ void find_bins(const int (&k)[NK], MsScratch &sc) {
  constexpr int NW = THREADS / 64, BPT = kBins / THREADS;
  const int tid = threadIdx.x;
  int c[BPT], cnt = 0;
#pragma unroll
  for (int j = 0; j < BPT; ++j) { c[j] = sc.hist[tid * BPT + j]; cnt += c[j]; }
  int wtot, total;
  const int inc = wave_scan_incl_add(cnt, &wtot);
  if ((tid & 63) == 0) sc.i[tid >> 6] = wtot;
  __syncthreads();
  const int excl = waves_before<NW>(sc.i, &total) + inc - cnt;
#pragma unroll
  for (int q = 0; q < NK; ++q)
    if (excl < k[q] && k[q] <= excl + cnt) {
      int run = excl;
#pragma unroll
      for (int j = 0; j < BPT; ++j) {
        if (run < k[q] && k[q] <= run + c[j]) sc.cut[Q0 + q] = {tid * BPT + j, k[q] - run, c[j]};
        run += c[j];
      }
    }
  __syncthreads();
}

// Sum over aligned groups of L = 1, 2, 4 or 8 lanes, in every lane.
template <int L>
__device__ __forceinline__ int group_sum(int x) {
  if (L >= 2) x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, true);      // quad_perm [1,0,3,2]
  if (L >= 4) x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, true);      // quad_perm [2,3,0,1]
  if (L >= 8) x += __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, true);     // row_half_mirror
  return x;
}

// A thread's largest and smallest key.
struct KeyRange {
  uint32_t largest = 0, smallest = 0xffffffffu;
  __device__ __forceinline__ void add(uint32_t key) { largest = max(largest, key); smallest = min(smallest, key); }
  // key 0 where there is none
  __device__ __forceinline__ void add_or_none(uint32_t key, bool there) { largest = max(largest, key); smallest = min(smallest, there ? key : 0xffffffffu); }
};
// What the threshold search needs from before a barrier: every wave's range of keys and an empty histogram.
template <int THREADS>
__device__ __forceinline__ void thresholds_begin(const KeyRange &r, MsScratch &sc) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int i = 0; i < kBins / THREADS; ++i) sc.hist[i * THREADS + tid] = 0;
  if (tid < 2) sc.nsurv[tid] = 0;
  const uint32_t m = wave_reduce<WMax>(r.largest, 0u), n = wave_reduce<WMin>(r.smallest, 0xffffffffu);
  if ((tid & 63) == 0) sc.wrange[tid >> 6] = make_uint2(m, n);
}

// Thresholds of the want[q] largest of a workgroup's keys (q < NK; want[q] < 1: not asked for, else at most the number of
// keys): every thread holds EPT keys, 0 where there is none.  The want[q] largest are the keys above tau[q] and, if
// krem[q] > 0, the first krem[q] (by position) of those equal to it.  thresholds_begin and a barrier come before.
// The first histogram takes the distance of a key to the largest one in steps of 2^17 (a float's upper six mantissa bits), up
// to 32 powers of two below it, or in smaller steps if they reach the smallest; the keys of a threshold's bin, if they are no more than
// kSurvivors and not all needed, are listed and ranked by counting, a few lanes to a key; fuller bins and what lies further below are
// divided by more histograms.
// Equal keys: one atomic per key would send all lanes to one word, so the waves merge such counts.  A head of equal keys needs no
// search; a bin with an eighth of all keys or more is first cut to the range that its keys really have (which ends the search where they
// are equal), by the waves whose first keys look tied, and those merge their lanes' counts.  Keys that are not tied pay for the look at one
// key per thread only.
// Bound: instruction issue (16 waves on one compute unit) and, with few waves, the length of the chain.  A search from the
// first bit in which the keys differ (a histogram per eleven bits and threshold, masks of valid keys) took 3 to 6 us more.  us a
// selection of 28 layers, that search -> one with an atomic per key and no look at the range -> this: 4 heads of 8160, normal scores 11.7 ->
// 8.3 -> 8.5, all equal 6.3 -> 22 -> 5.6, 1 % twice the others 14.0 -> 22 -> 7.2, four neighbouring values 9.9 -> 17.6 -> 8.5; head-adaptive, 4 heads of
// 32 000, normal 56 -> 30 -> 29, all equal 29 -> 145 -> 19, 1 % twice the others 69 -> 94 -> 29, all equal but one far above 64 -> 200 -> 25, four
// neighbouring values 42 -> 110 -> 28.
constexpr int kFirstShift = 17;
template <int THREADS, int EPT, int NK>
__device__ __forceinline__ void radix_thresholds(const uint32_t (&key)[EPT], const int (&want)[NK], MsScratch &sc, uint32_t (&tau)[NK],
                                                 int (&krem)[NK]) {
  constexpr int NW = THREADS / 64, L = THREADS / kSurvivors;        // L lanes to a listed key
  static_assert(kBins % THREADS == 0 && THREADS % kSurvivors == 0, "whole bins and lanes per thread");
  const int tid = threadIdx.x, lane = tid & 63;
  const uint2 wr = (lane & 15) < NW ? sc.wrange[lane & 15] : make_uint2(0u, 0xffffffffu);
  const uint32_t kmax = read_lane(row_scan_incl<WMax>(wr.x, 0u), 15), kmin = read_lane(row_scan_incl<WMin>(wr.y, 0xffffffffu), 15);
  if (kmax == kmin) {                                    // equal keys: the first ones
#pragma unroll
    for (int q = 0; q < NK; ++q) {
      tau[q] = want[q] < 1 ? 0xffffffffu : kmax;
      krem[q] = max(want[q], 0);
    }
    return;
  }
  const int shift1 = min(kFirstShift, max(0, 32 - __clz((int)(kmax - kmin)) - kDigit));
#pragma unroll
  for (int e = 0; e < EPT; ++e) hist_add(sc.hist, (int)min((kmax - key[e]) >> shift1, (uint32_t)kBins - 1));
  __syncthreads();
  find_bins<THREADS, NK>(want, sc);
  uint32_t hi[NK], width[NK];                            // a threshold's bin: the keys from hi - width to hi
  int count[NK];
  bool ranked[NK], any = false;
#pragma unroll
  for (int q = 0; q < NK; ++q) {
    ranked[q] = false;
    tau[q] = 0xffffffffu;
    krem[q] = 0;
    if (want[q] < 1) continue;
    const int bin = sc.cut[q].bin;
    hi[q] = kmax - ((uint32_t)bin << shift1);
    width[q] = min(hi[q] - kmin, bin == kBins - 1 ? 0xffffffffu : (1u << shift1) - 1);
    krem[q] = sc.cut[q].k;
    count[q] = sc.cut[q].count;
    bool wide = bin == kBins - 1;                        // as wide as it gets, and "no key" is counted here: look again
    while (width[q] > 0 && (wide || (count[q] > kSurvivors && count[q] != krem[q]))) {        // uniform over the workgroup
      const bool crowd = count[q] > THREADS * EPT / 8;
      wide = false;
#pragma unroll
      for (int i = 0; i < kBins / THREADS; ++i) sc.hist[i * THREADS + tid] = 0;
      auto inside = [&](int e) { return hi[q] - key[e] <= width[q]; };
      const bool tied = crowd && wave_tied(key[0], inside(0));
      if (crowd) {
        // the range that the bin's keys really have, if every wave looks for it: equal keys are told apart no further
        uint32_t near = 0, far = width[q];
        if (tied) {
          near = 0xffffffffu;
          far = 0;
#pragma unroll
          for (int e = 0; e < EPT; ++e) {
            const uint32_t d = hi[q] - key[e];
            near = min(near, d);                         // (a key outside the bin is further than `width`)
            far = max(far, d <= width[q] ? d : 0u);
          }
          near = wave_reduce<WMin>(near, 0xffffffffu);
          far = wave_reduce<WMax>(far, 0u);
        }
        if (lane == 0) sc.bin_range[q][tid >> 6] = make_uint2(far, near);
        __syncthreads();
        const uint2 br = (lane & 15) < NW ? sc.bin_range[q][lane & 15] : make_uint2(0u, 0xffffffffu);
        far = read_lane(row_scan_incl<WMax>(br.x, 0u), 15);
        near = read_lane(row_scan_incl<WMin>(br.y, 0xffffffffu), 15);
        hi[q] -= near;
        width[q] = far - near;
        if (width[q] == 0) break;
      } else {
        __syncthreads();
      }
      const int shift = max(0, 32 - __clz((int)width[q]) - kDigit);
      auto bin_of = [&](int e) { return (int)((hi[q] - key[e]) >> shift); };
      if (tied) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) hist_add(sc.hist, bin_of(e), inside(e));
      } else {
#pragma unroll
        for (int e = 0; e < EPT; ++e)
          if (inside(e)) atomicAdd(&sc.hist[bin_of(e)], 1);
      }
      __syncthreads();
      const int k1[1] = {krem[q]};
      if (q == 0) find_bins<THREADS, 1, 0>(k1, sc); else find_bins<THREADS, 1, NK - 1>(k1, sc);
      const uint32_t step = (uint32_t)sc.cut[q].bin << shift;
      hi[q] -= step;
      width[q] = min(width[q] - step, (1u << shift) - 1);
      krem[q] = sc.cut[q].k;
      count[q] = sc.cut[q].count;
    }
    if (count[q] == krem[q]) {                           // the whole bin is needed
      tau[q] = hi[q] - width[q] - 1;
      krem[q] = 0;
      continue;
    }
    tau[q] = hi[q];
    if (width[q] == 0) continue;                         // the bin is one key
    ranked[q] = any = true;
#pragma unroll
    for (int e = 0; e < EPT; ++e)
      if (hi[q] - key[e] <= width[q]) {
        const int at = atomicAdd(&sc.nsurv[q], 1);
        if (at < kSurvivors) sc.surv[q][at] = key[e];
      }
  }
  if (!any) return;
  __syncthreads();
  const int mine = tid / L, part = tid % L;
#pragma unroll
  for (int q = 0; q < NK; ++q)
    if (ranked[q] && mine < sc.nsurv[q]) {
      const int n = sc.nsurv[q];
      const uint32_t x = sc.surv[q][mine];
      int above = 0, equal = 0;
      for (int j = part; j < n; j += L) {
        const uint32_t y = sc.surv[q][j];
        above += y > x ? 1 : 0;
        equal += y == x ? 1 : 0;
      }
      above = group_sum<L>(above);
      equal = group_sum<L>(equal);
      if (above < krem[q] && krem[q] <= above + equal) {                          // equal keys write the same
        const bool all = krem[q] == above + equal;
        sc.tau[q] = all ? x - 1 : x;
        sc.krem[q] = all ? 0 : krem[q] - above;
      }
    }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NK; ++q)
    if (ranked[q]) { tau[q] = sc.tau[q]; krem[q] = sc.krem[q]; }
}

// The Bp >= 1 largest of a workgroup's keys, ties to the smaller position: every thread holds EPT consecutive
// keys, 0 where there is none, in ascending order of position over the threads (Sec. 3.1 /
// Algorithm 1, TopB).  pos(e) is the position of the thread's key e; it is asked for kept keys only.  The
// kept positions go to idx[0, Bp) in ascending order.  With ckey not null the list is a head's candidates for
// the head-adaptive split: the order keys go beside the positions, and the head's `floor` <= Bp best carry
// kFloorFlag in their position word.  `kept`, if not null, is an LDS array that receives the positions too; it may be where
// the keys came from.  thresholds_begin and a barrier come before.
template <int THREADS, int EPT, class Pos>
__device__ __forceinline__ void top_select_keys(const uint32_t (&key)[EPT], int Bp, int32_t *idx, uint32_t *ckey, int floor, MsScratch &sc,
                                                Pos pos_of, int32_t *kept = nullptr) {
  const bool flags = ckey != nullptr && floor > 0;
  const int want[2] = {Bp, flags ? floor : 0};
  uint32_t tau[2];
  int k[2];
  radix_thresholds<THREADS, EPT, 2>(key, want, sc, tau, k);
  auto put = [&](int e, int pos, bool in_floor) {
    if (pos >= Bp) return;
    const int32_t word = (int32_t)((uint32_t)pos_of(e) | (in_floor ? kFloorFlag : 0u));
    idx[pos] = word;
    if (ckey) ckey[pos] = key[e];
    if (kept) kept[pos] = word;
  };
  int total;
  if (k[0] == 0 && k[1] == 0) {                         // no key equal to a threshold is left out
    int pos = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) pos += key[e] > tau[0] ? 1 : 0;
    pos = block_scan_excl<THREADS / 64>(pos, sc, &total);
#pragma unroll
    for (int e = 0; e < EPT; ++e)
      if (key[e] > tau[0]) put(e, pos++, key[e] > tau[1]);
    return;
  }
  // keys above tau (low half) and keys equal to tau (high half) share a word
  int packed = 0, seenf = 0;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    packed += (key[e] > tau[0] ? 1 : 0) + (key[e] == tau[0] ? 1 << 16 : 0);
    seenf += key[e] == tau[1] ? 1 : 0;
  }
  block_scan_excl<THREADS / 64>(packed, seenf, sc, &total);
  int seen = packed >> 16;                          // equal keys at smaller indices
  int pos = (packed & 0xffff) + min(seen, k[0]);    // kept entries at smaller indices
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    bool sel = key[e] > tau[0], inf = key[e] > tau[1];
    if (key[e] == tau[0]) sel = seen++ < k[0];
    if (key[e] == tau[1]) inf = seenf++ < k[1];
    if (sel) put(e, pos++, inf);
  }
}

// The EPT consecutive order keys from `base` on out of the LDS row k_s of n keys (whole groups of four were written), 0 past it.
template <int EPT>
__device__ __forceinline__ void read_keys(const uint32_t *k_s, int base, int n, uint32_t (&key)[EPT]) {
#pragma unroll
  for (int e = 0; e < EPT; e += 4) {
    const uint4 v = base + e < n ? *reinterpret_cast<const uint4 *>(&k_s[slot4(base + e)]) : make_uint4(0u, 0u, 0u, 0u);
    key[e] = v.x; key[e + 1] = v.y; key[e + 2] = v.z; key[e + 3] = v.w;
#pragma unroll
    for (int j = 1; j < 4; ++j) key[e + j] = base + e + j < n ? key[e + j] : 0u;
  }
}

// Rows head h of a layer keeps and its first row inside the batch item: B each, or the layer's
// row of the budget table (per-head mode), the heads packed back to back.
__device__ __forceinline__ void head_rows(const Shape &s, const int32_t *budgets, int layer, int h, int &Bh, int &row0) {
  Bh = s.B;
  row0 = h * s.B;
  if (budgets) {
    const int32_t *bl = budgets + layer * s.hkv;
    row0 = 0;
    for (int j = 0; j < h; ++j) row0 += bl[j];
    Bh = bl[h];
  }
}

// After the candidates of a head: the W window positions, the head's count and its offsets.
__device__ __forceinline__ void finish_head(const Shape &s, const LayerOut &O, int b, int h, int Bh, int row0,
                                            int32_t *idx, int threads) {
  const int tid = threadIdx.x, Bp = Bh - s.W;
  for (int wv = tid; wv < s.W; wv += threads) idx[Bp + wv] = s.Nc + wv;
  if (tid == 0) {
    O.counts[b * s.hkv + h] = Bh;
    if (O.offsets) {
      O.offsets[b * (s.hkv + 1) + h] = row0;
      if (h == s.hkv - 1) O.offsets[b * (s.hkv + 1) + s.hkv] = row0 + Bh;
    }
  }
}

// The per-key rows the streaming passes left for a unit, and the two scores formed from them.
struct UnitRows {
  const float *araw, *vnorm, *kdot, *invn;
  int Nc;
  bool kstats, use_v, knorm;             // use_v: an intrinsic score takes part
  __device__ UnitRows(const Shape &s, const char *ws, const Workspace &w, int64_t unit)
      : araw(reinterpret_cast<const float *>(ws + w.araw) + unit * s.Npad),
        vnorm(reinterpret_cast<const float *>(ws + w.vnorm) + unit * s.Npad),
        kdot(reinterpret_cast<const float *>(ws + w.sdiv) + unit * s.Npad),
        invn(reinterpret_cast<const float *>(ws + w.invnorm) + unit * s.Npad), Nc(s.Nc), kstats(s.kstats != 0),
        use_v(s.intrinsic != MIXKV_INTRINSIC_NONE), knorm(s.intrinsic == MIXKV_INTRINSIC_KNORM) {}
  // A group of four candidates to read for the group from i on: a group past the row re-reads the row's last one (its
  // values are not used), so that no load waits behind a branch on the one before.
  __device__ __forceinline__ int inside(int i) const { return min(i, (Nc - 1) & ~3); }
  // Intrinsic score and diversity of G groups of four candidates, group g from i[g] on (a multiple of four, inside()
  // the row): all loads are in flight together.
  template <int G>
  __device__ __forceinline__ void load_vd(const int (&i)[G], float4 (&vr)[G], float4 (&dr)[G]) const {
    float4 nr[G];
#pragma unroll
    for (int g = 0; g < G; ++g) vr[g] = dr[g] = nr[g] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (kstats) {                            // else nobody wrote them: the diversity is 0 and carries weight 0
#pragma unroll
      for (int g = 0; g < G; ++g) dr[g] = *reinterpret_cast<const float4 *>(kdot + i[g]);
#pragma unroll
      for (int g = 0; g < G; ++g) nr[g] = *reinterpret_cast<const float4 *>(invn + i[g]);
    }
    if (use_v && !knorm) {
#pragma unroll
      for (int g = 0; g < G; ++g) vr[g] = *reinterpret_cast<const float4 *>(vnorm + i[g]);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (knorm) vr[g] = make_float4(neg_key_norm(nr[g].x), neg_key_norm(nr[g].y), neg_key_norm(nr[g].z), neg_key_norm(nr[g].w));
      // s_div: a product rounded on its own.  The minimum is taken from the first reading and must
      // cancel exactly against the second, so the compiler may not fuse the product into the
      // subtraction that follows there (it may by default); the empty statements hide where it came from.
      dr[g] = make_float4(-dr[g].x * nr[g].x, -dr[g].y * nr[g].y, -dr[g].z * nr[g].z, -dr[g].w * nr[g].w);
      asm("" : "+v"(dr[g].x), "+v"(dr[g].y), "+v"(dr[g].z), "+v"(dr[g].w));
    }
  }
};

// Most dynamic LDS any of these kernels asks for, next to their scratch.
constexpr int kMsMaxLds = 146 * 1024;

// Raises a kernel's dynamic-LDS limit to kMsMaxLds the first time it is launched on a device.
struct LdsLimitOnce {
  static constexpr int kMaxDevices = 64;
  std::mutex mu;
  bool done[kMaxDevices] = {};
  hipError_t raise(const void *kern) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!done[dev]) {
      e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, kMsMaxLds);
      if (e != hipSuccess) return e;
      done[dev] = true;
    }
    return hipSuccess;
  }
};

}  // namespace mixkv
