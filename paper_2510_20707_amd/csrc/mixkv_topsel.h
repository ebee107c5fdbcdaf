// Workgroup-level selection code shared by the kernels that rank one head's candidates: block reductions and
// scans, the most-significant-digit radix select on order-preserving keys held in registers, and the
// ordered emission of the kept positions.
#pragma once
#include <mutex>

#include "mixkv_internal.h"
#include "mixkv_wave.h"

namespace mixkv {

constexpr int kMsMaxThreads = 1024, kMsMaxWaves = kMsMaxThreads / 64;
constexpr int kDigit = 11, kBins = 1 << kDigit;     // radix-select digit

struct MsScratch {
  float f[kMsMaxWaves][8];
  float fr[8];
  uint32_t ur[2];
  int i[kMsMaxWaves + 1];
  int hist[kBins];
  int hist0[kBins];                      // the first round's histogram of a head, for a second threshold on the same keys
  int bin, krem, cut;
};

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

// Block-wide minimum and maximum of unsigned keys through two LDS atomics per wave (integer
// min / max do not depend on the order).  sc.ur must hold {0xffffffff, 0} from before an earlier
// barrier of the kernel.
__device__ __forceinline__ void block_minmax_u32(uint32_t &lo, uint32_t &hi, MsScratch &sc) {
  const int lane = threadIdx.x & 63;
  lo = wave_reduce<WMin>(lo, 0xffffffffu);
  hi = wave_reduce<WMax>(hi, 0u);
  if (lane == 0) { atomicMin(&sc.ur[0], lo); atomicMax(&sc.ur[1], hi); }
  __syncthreads();
  lo = sc.ur[0];
  hi = sc.ur[1];
}

// Exclusive prefix sum of one int per thread (thread order); *total receives the block sum.
__device__ __forceinline__ int read_lane_dyn(int x, int lane_uniform) {
  return __builtin_amdgcn_readlane(x, __builtin_amdgcn_readfirstlane(lane_uniform));
}

template <int NW>
__device__ __forceinline__ int block_scan_excl(int v, MsScratch &sc, int *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int wtot;
  const int inc = wave_scan_incl_add(v, &wtot);
  __syncthreads();
  if (lane == 0) sc.i[wave] = wtot;
  __syncthreads();
  const int x = (lane & 15) < NW ? sc.i[lane & 15] : 0;
  const int y = row_scan_incl<WSum>(x, 0);              // inclusive over the waves, in every row of lanes
  *total = read_lane(y, 15);
  const int before = wave == 0 ? 0 : read_lane_dyn(y, wave - 1);
  return before + inc - v;
}

__device__ __forceinline__ uint32_t order_key_u(float x) {
  uint32_t u = __float_as_uint(x);
  if (u == 0x80000000u) u = 0;                          // -0 and +0 are the same score
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// One count into a shared histogram bin per lane, with the lanes that share the wave's most common
// bin (as seen from its first active lane) merged into a single atomic.
__device__ __forceinline__ void hist_add(int *hist, int bin, bool on) {
  const unsigned long long act = __ballot(on);
  if (act == 0) return;
  const int first = __ffsll((long long)act) - 1;                  // wave-uniform
  const int b0 = __builtin_amdgcn_readlane(bin, first);
  const unsigned long long same = __ballot(on && bin == b0);
  const int lane = threadIdx.x & 63;
  if (lane == first) atomicAdd(&hist[b0], __popcll(same));
  if (on && bin != b0) atomicAdd(&hist[bin], 1);
}

// Threshold of the k largest of a workgroup's keys (1 <= k <= number of valid keys): every thread holds
// EPT keys, those with their bit set in `vmask` valid, and [kmin, kmax] is the range of all valid keys.  Most-significant-digit radix select from the first
// bit in which the keys differ.  Returns tau, the k-th largest key, and in krem how many of the
// keys equal to tau still belong to the k (0: all of them).  Ends behind a barrier: may be called again.
// The first round counts every valid key and does not depend on k: FIRST = 1 keeps its histogram
// aside, FIRST = 2 takes it from there (a second threshold on the same keys), 0 does neither.
template <int THREADS, int EPT, int FIRST = 0>
__device__ __forceinline__ uint32_t radix_threshold(const uint32_t (&key)[EPT], uint32_t vmask, uint32_t kmin, uint32_t kmax,
                                                    int k, MsScratch &sc, int &krem) {
  constexpr int NW = THREADS / 64;
  const int tid = threadIdx.x;
  // bits at and above `undecided` are common to all keys; digits of up to kDigit bits from there down
  int undecided = kmin == kmax ? 0 : 32 - __clz((int)(kmin ^ kmax));
  uint32_t prefix = undecided >= 32 ? 0u : (kmax >> undecided) << undecided;
  bool all_equal = false, first = true;
  while (undecided > 0) {
    const int wbits = min(kDigit, undecided), shift = undecided - wbits;
    const uint32_t himask = undecided >= 32 ? 0u : ~0u << undecided;
    const bool saved = FIRST == 2 && first;             // this round's histogram is already in hist0
    int *hist = saved ? sc.hist0 : sc.hist;
    if (!saved) {
      for (int i = tid; i < kBins; i += THREADS) sc.hist[i] = 0;
      __syncthreads();
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const bool on = ((vmask >> e) & 1u) != 0 && (key[e] & himask) == (prefix & himask);
        hist_add(sc.hist, (int)((key[e] >> shift) & ((1u << wbits) - 1u)), on);
      }
      __syncthreads();
    }
    // walk the bins from the top: thread t sums bins [kBins - (t+1)*BPT, kBins - t*BPT)
    constexpr int BPT = (kBins + THREADS - 1) / THREADS;
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      const int bi = kBins - 1 - (tid * BPT + j);
      const int c = bi >= 0 ? hist[bi] : 0;
      if (FIRST == 1 && first && bi >= 0) sc.hist0[bi] = c;
      cnt += c;
    }
    first = false;
    int total;
    const int excl = block_scan_excl<NW>(cnt, sc, &total);
    if (excl < k && k <= excl + cnt) {
      int run = excl;
#pragma unroll
      for (int j = 0; j < BPT; ++j) {
        const int bi = kBins - 1 - (tid * BPT + j);
        const int c = bi >= 0 ? hist[bi] : 0;
        if (run < k && k <= run + c) { sc.bin = bi; sc.krem = k - run; sc.cut = c; }
        run += c;
      }
    }
    __syncthreads();
    prefix |= (uint32_t)sc.bin << shift;
    k = sc.krem;
    undecided = shift;
    const bool whole_bin = sc.cut == k && shift > 0 && prefix != 0;
    __syncthreads();
    // Every key of the bin is needed: the kept set is "all keys at or above the bin", whatever
    // the lower digits are, so the remaining rounds can be skipped.
    if (whole_bin) { prefix -= 1; all_equal = true; break; }
  }
  krem = all_equal ? 0 : k;
  return prefix;
}

// The Bp >= 1 largest of a workgroup's keys, ties to the smaller position: every thread holds EPT consecutive
// keys of which the first `nvalid` exist, in ascending order of position over the threads (Sec. 3.1 /
// Algorithm 1, TopB).  pos(e) is the position of the thread's key e; it is asked for kept keys only.  The
// kept positions go to idx[0, Bp) in ascending order.  With ckey not null the list is a head's candidates for
// the head-adaptive split: the order keys go beside the positions, and the head's `floor` <= Bp best carry
// kFloorFlag in their position word.  sc.ur must hold {0xffffffff, 0} from before an earlier barrier.
template <int THREADS, int EPT, class Pos>
__device__ __forceinline__ void top_select_keys(const uint32_t (&key)[EPT], int nvalid, int Bp, int32_t *idx, uint32_t *ckey,
                                                int floor, MsScratch &sc, Pos pos_of) {
  constexpr int NW = THREADS / 64;
  uint32_t kmin = 0xffffffffu, kmax = 0;
#pragma unroll
  for (int e = 0; e < EPT; ++e)
    if (e < nvalid) { kmin = min(kmin, key[e]); kmax = max(kmax, key[e]); }
  block_minmax_u32(kmin, kmax, sc);
  const uint32_t vmask = nvalid >= EPT ? (EPT >= 32 ? 0xffffffffu : (1u << (EPT & 31)) - 1u)
                                       : (nvalid <= 0 ? 0u : (1u << nvalid) - 1u);
  int k;                             // of the keys equal to tau, the first k (by position) are kept
  const bool flags = ckey != nullptr && floor > 0;
  int kf = 0;
  uint32_t tau, tauf = 0xffffffffu;
  if (flags) {
    tau = radix_threshold<THREADS, EPT, 1>(key, vmask, kmin, kmax, Bp, sc, k);
    tauf = radix_threshold<THREADS, EPT, 2>(key, vmask, kmin, kmax, floor, sc, kf);
  } else {
    tau = radix_threshold<THREADS, EPT>(key, vmask, kmin, kmax, Bp, sc, k);
  }
  // one scan carries both counts: keys above tau (low half) and keys equal to tau (high half)
  int ngt = 0, neq = 0, neqf = 0;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const bool in = e < nvalid;
    ngt += (in && key[e] > tau) ? 1 : 0;
    neq += (in && key[e] == tau) ? 1 : 0;
    neqf += (in && key[e] == tauf) ? 1 : 0;
  }
  int total;
  const int packed = block_scan_excl<NW>(ngt | (neq << 16), sc, &total);
  int seen = packed >> 16;                          // equal keys at smaller indices
  int pos = (packed & 0xffff) + min(seen, k);       // kept entries at smaller indices
  int seenf = flags ? block_scan_excl<NW>(neqf, sc, &total) : 0;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    if (e < nvalid) {
      bool sel = key[e] > tau;
      if (key[e] == tau) sel = seen++ < k;
      bool inf = flags && key[e] > tauf;
      if (flags && key[e] == tauf) inf = seenf++ < kf;
      if (sel) {
        if (pos < Bp) {
          idx[pos] = (int32_t)((uint32_t)pos_of(e) | (inf ? kFloorFlag : 0u));
          if (ckey) ckey[pos] = key[e];
        }
        ++pos;
      }
    }
  }
}

// top_select_keys on the scores a[] of the EPT consecutive candidates base .. base + nvalid - 1.
template <int THREADS, int EPT>
__device__ __forceinline__ void top_select(const float (&a)[EPT], int nvalid, int base, int Bp, int32_t *idx,
                                           uint32_t *ckey, int floor, MsScratch &sc) {
  uint32_t key[EPT];
#pragma unroll
  for (int e = 0; e < EPT; ++e) key[e] = order_key_u(a[e]);
  top_select_keys<THREADS, EPT>(key, nvalid, Bp, idx, ckey, floor, sc, [&](int e) { return base + e; });
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
  // intrinsic score and diversity of the four candidates from i on (i a multiple of four; zeros past the row)
  __device__ __forceinline__ void load_vd(int i, float4 &vr, float4 &dr) const {
    float4 kr = make_float4(0.f, 0.f, 0.f, 0.f), nr = kr;
    vr = kr;
    if (i < Nc) {
      if (kstats) {                          // else nobody wrote them: the diversity is 0 and carries weight 0
        kr = *reinterpret_cast<const float4 *>(kdot + i);
        nr = *reinterpret_cast<const float4 *>(invn + i);
      }
      if (knorm) vr = make_float4(neg_key_norm(nr.x), neg_key_norm(nr.y), neg_key_norm(nr.z), neg_key_norm(nr.w));
      else if (use_v) vr = *reinterpret_cast<const float4 *>(vnorm + i);
    }
    // s_div: a product rounded on its own.  The minimum is taken from the first reading and must
    // cancel exactly against the second, so the compiler may not fuse the product into the
    // subtraction that follows there (it may by default); the empty statements hide where it came from.
    dr = make_float4(-kr.x * nr.x, -kr.y * nr.y, -kr.z * nr.z, -kr.w * nr.w);
    asm("" : "+v"(dr.x), "+v"(dr.y), "+v"(dr.z), "+v"(dr.w));
  }
};

// Most dynamic LDS any of these kernels asks for, next to their scratch.
constexpr int kMsMaxLds = 140 * 1024;

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
