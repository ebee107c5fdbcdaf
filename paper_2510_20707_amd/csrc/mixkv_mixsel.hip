// mixsel_kernel: score mixing and (optionally) the fixed-budget top-B' selection of one unit in a
// single workgroup, with every per-key quantity held in registers.
//
// Loading, pooling, statistics and mixing deal the candidates to the threads in groups of four,
// round-robin, so that every load is coalesced; the pooled attention needs neighbours, so the raw
// attention row is staged once in LDS.  For the selection thread t owns the EPT consecutive
// candidates [t*EPT, (t+1)*EPT) (the order keys of the mixed scores change hands through the same LDS row), so the
// kept indices come out in ascending order from a plain prefix sum.  The selection is a threshold search by histograms
// on order-preserving integer keys kept in registers (radix_thresholds).
//
// Bound: the instructions of a workgroup's 4 to 16 waves and the length of their chain (112 workgroups use less than half of the
// chip); past 16 384 candidates the loads of four rows too.  All of a thread's loads in flight together, keys formed as
// they are dealt, whole groups through LDS, one search of six barriers for both thresholds, us a launch before and now:
// 2 heads of 504 11.6 -> 7.6, 4 of 4064 13.4 -> 10.9, 112 of 8160 18.5 -> 15.9, 256 of 16 128 49.7 -> 40.6, 448 of 32 736
// 137 -> 97 (head-adaptive lists).
//
// Paper: Sec. 3.2 Eq. 2 (importance = attention + scaled value norm), Sec. 3.3 (min-max and mean
// matching of the diversity, Eq. 5 mix), Sec. 3.1 / Algorithm 1 (TopB with B' = B - W); Sec. 4.3 /
// Table 4 for the variants (key-norm intrinsic score, un-weighted and one-sided mixes, given weights).
#include "mixkv_topsel.h"

namespace mixkv {

// 16 bytes of a cache row (arrays of HIP's own uint4 end up in scratch memory in the gather below)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int THREADS, int EPT, bool SELECT>
__global__ __launch_bounds__(THREADS) void mixsel_kernel(Shape s, LayerOutTable out, char *ws, Workspace w,
                                                           int64_t unit0, LayerInTable in, int gather_eb, int cand_m,
                                                           CandLists cl, const int32_t *budgets) {
  constexpr int NW = THREADS / 64;
  extern __shared__ __align__(16) float a_s[];          // raw window attention of this head, later its order keys
  __shared__ MsScratch sc;
  const int ul = blockIdx.x;
  int tid = threadIdx.x;
  const int64_t unit = unit0 + ul;
  const int layer = ul / s.units_per_layer, bh = ul - layer * s.units_per_layer;
  const LayerOut O = out.l[layer];
  const UnitRows rows(s, ws, w, unit);
  const float r = reinterpret_cast<const float *>(ws + w.rbar)[unit];
  const int Nc = s.Nc, N = s.N, base = threadIdx.x * EPT;
  const bool use_v = rows.use_v;
  const float inv_n = 1.f / (float)Nc;
  float wi, wd;
  mix_weights(s.mix, r, s.mix == MIXKV_MIX_GIVEN_R ? in.l[layer].r_given[bh] : 0.f, wi, wd);

  // ---- load.  The first phases deal the candidates to the threads in groups of four, group
  // g * THREADS + tid to thread tid: consecutive lanes read consecutive 16 bytes (the per-unit rows
  // are padded past Nc).  The sums and extrema of the intrinsic score and the diversity are taken as
  // they pass.  Up to 16 candidates per thread all three rows stay in registers until the mix; at 32 they would not
  // fit the 128 registers a 1024-thread workgroup leaves each lane, so only the attention does and the mix reads
  // the two a second time (that reading cost 0.7 us at 8 per thread on 4 heads of 4096, 3 us at 16 on 256 heads of 16 384).
  // Runs of EPT consecutive candidates per thread would touch one cache line per lane and load, but the selection needs
  // consecutive runs (ascending output from one prefix sum): s_comp reaches their owners through LDS.
  auto cidx = [&](int e) { return (((e >> 2) * THREADS + tid) << 2) + (e & 3); };
  // up to 16 candidates per thread the other two fit beside it
  constexpr bool KEEP = EPT <= 16;
  float a[EPT], vk[KEEP ? EPT : 1], dk[KEEP ? EPT : 1];
  float st[7] = {0.f, 0.f, 0.f, INFINITY, INFINITY, -INFINITY, -INFINITY};   // sums a, v, d | min v, d | max v, d
  constexpr int GB = EPT <= 16 ? EPT / 4 : 2;           // groups whose loads are in flight together
  // The raw attention row goes to LDS four words up, between the pooling's neutral element on either side.
  const bool pooled = s.pool != MIXKV_POOL_NONE && s.pool_k > 1, is_max = s.pool == MIXKV_POOL_MAX;
  const float fill = is_max ? -INFINITY : 0.f;          // out-of-range taps: ignored by max, zero for avg
  if (threadIdx.x < 2) {
    const int at = threadIdx.x == 0 ? 0 : 4 + ((Nc + 3) & ~3);
    *reinterpret_cast<float4 *>(&a_s[slot4(at)]) = make_float4(fill, fill, fill, fill);
  }
#pragma unroll
  for (int g0 = 0; g0 < EPT / 4; g0 += GB) {
    if constexpr (!KEEP) __builtin_amdgcn_sched_barrier(0);      // the next batch's loads would not fit the registers
    int at[GB];
    float4 ar[GB], vr[GB], dr[GB];
#pragma unroll
    for (int g = 0; g < GB; ++g) {
      at[g] = rows.inside(cidx(4 * (g0 + g)));
      ar[g] = *reinterpret_cast<const float4 *>(rows.araw + at[g]);
    }
    rows.load_vd<GB>(at, vr, dr);
#pragma unroll
    for (int g = 0; g < GB; ++g) {
      const int e4 = 4 * (g0 + g), i = cidx(e4);
      const float a4[4] = {ar[g].x, ar[g].y, ar[g].z, ar[g].w};
      const float v4[4] = {vr[g].x, vr[g].y, vr[g].z, vr[g].w}, d4[4] = {dr[g].x, dr[g].y, dr[g].z, dr[g].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        a[e4 + j] = a4[j];
        if constexpr (KEEP) { vk[e4 + j] = v4[j]; dk[e4 + j] = d4[j]; }
        if (i + j < Nc) {
          st[1] += v4[j]; st[2] += d4[j];
          st[3] = fminf(st[3], v4[j]); st[4] = fminf(st[4], d4[j]);
          st[5] = fmaxf(st[5], v4[j]); st[6] = fmaxf(st[6], d4[j]);
        }
      }
      if (i < Nc)
        *reinterpret_cast<float4 *>(&a_s[slot4(4 + i)]) =
            make_float4(a4[0], i + 1 < Nc ? a4[1] : fill, i + 2 < Nc ? a4[2] : fill, i + 3 < Nc ? a4[3] : fill);
    }
  }
  __syncthreads();
  if constexpr (!KEEP) asm("" : "+v"(tid));             // positions and LDS slots are formed again, not held in registers

  // ---- pooled attention (candidates only) and the first round of statistics
  if (pooled) {
    const int hk = s.pool_k >> 1;
    if (hk <= 3) {
      // sliding window in registers over each group of four: its own values and the groups on either side
#pragma unroll
      for (int e0 = 0; e0 < EPT; e0 += 4) {
        const int at = 4 + rows.inside(cidx(e0));
        const float4 lo = *reinterpret_cast<const float4 *>(&a_s[slot4(at - 4)]);
        const float4 own = *reinterpret_cast<const float4 *>(&a_s[slot4(at)]);
        const float4 hi = *reinterpret_cast<const float4 *>(&a_s[slot4(at + 4)]);
        const float win[10] = {lo.y, lo.z, lo.w, own.x, own.y, own.z, own.w, hi.x, hi.y, hi.z};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float acc = win[3 + e];
          if (is_max) {
            if (hk >= 1) acc = fmaxf(acc, fmaxf(win[2 + e], win[4 + e]));
            if (hk >= 2) acc = fmaxf(acc, fmaxf(win[1 + e], win[5 + e]));
            if (hk >= 3) acc = fmaxf(acc, fmaxf(win[e], win[6 + e]));
          } else {
            // same left-to-right order as a plain loop over the taps
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
          a[e0 + e] = acc;
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int i = cidx(e);
        if (i < Nc) {
          const int lo = max(0, i - hk), hi = min(Nc - 1, i + hk);
          float acc = a_s[slot4(4 + lo)];
          if (is_max) {
            for (int j = lo + 1; j <= hi; ++j) acc = fmaxf(acc, a_s[slot4(4 + j)]);
          } else {
            for (int j = lo + 1; j <= hi; ++j) acc += a_s[slot4(4 + j)];
            acc = acc / (float)s.pool_k;
          }
          a[e] = acc;
        }
      }
    }
  }
  // One round of statistics over the candidates.  The means of the min-max normalised intrinsic score
  // and diversity follow from the plain sums: sum((x - min) * c) = (sum(x) - Nc * min) * c, and
  // mean(s_imp) = mean(s_ex) + f_in * mean(s_in_norm).
#pragma unroll
  for (int e = 0; e < EPT; ++e)
    if (cidx(e) < Nc) st[0] += a[e];
  block_reduce_mixed<NW, 3, 2, 2>(st, sc);
  const float mean_ex = st[0] * inv_n;
  const float vmin = st[3], dmin = st[4];
  const float rvden = 1.f / (st[5] - vmin + s.eps), rdden = 1.f / (st[6] - dmin + s.eps);
  const float mean_in = (st[1] - (float)Nc * vmin) * rvden * inv_n;     // mean of the normalised value norm
  const float mean_dn = (st[2] - (float)Nc * dmin) * rdden * inv_n;     // mean of the normalised diversity
  const float f_in = use_v ? mean_ex / (mean_in + s.eps) : 0.f;         // Sec. 3.2: scale VNorm to mean(s_ex)
  const float mean_imp = use_v ? mean_ex + f_in * mean_in : mean_ex;
  const float f_div = mean_imp / (mean_dn + s.eps);                      // Sec. 3.3: scale diversity to mean(s_imp)
  auto s_comp = [&](float ai, float vi, float di) {
    const float imp = use_v ? ai + (vi - vmin) * rvden * f_in : ai;       // Eq. 2
    return wi * imp + wd * ((di - dmin) * rdden * f_div);                 // Eq. 5
  };
  // Every thread is past the reduction's barriers, so the pooling has read all it needs of the raw row: the order keys
  // of s_comp replace it in LDS and come back dealt in consecutive runs of EPT.
  uint32_t *k_s = reinterpret_cast<uint32_t *>(a_s);
  float *scores = O.scores ? O.scores + (int64_t)bh * N : nullptr;
  KeyRange range;
#pragma unroll
  for (int g0 = 0; g0 < EPT / 4; g0 += GB) {
    float4 vr[GB], dr[GB];
    if constexpr (!KEEP) {
      __builtin_amdgcn_sched_barrier(0);
      int at[GB];
#pragma unroll
      for (int g = 0; g < GB; ++g) at[g] = rows.inside(cidx(4 * (g0 + g)));
      rows.load_vd<GB>(at, vr, dr);
    }
#pragma unroll
    for (int g = 0; g < GB; ++g) {
      const int e4 = 4 * (g0 + g), i = cidx(e4);
      float v4[4], d4[4];
      if constexpr (KEEP) {
#pragma unroll
        for (int j = 0; j < 4; ++j) { v4[j] = vk[e4 + j]; d4[j] = dk[e4 + j]; }
      } else {
        v4[0] = vr[g].x; v4[1] = vr[g].y; v4[2] = vr[g].z; v4[3] = vr[g].w;
        d4[0] = dr[g].x; d4[1] = dr[g].y; d4[2] = dr[g].z; d4[3] = dr[g].w;
      }
      uint32_t k4[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float c = s_comp(a[e4 + j], v4[j], d4[j]);
        if (scores && i + j < Nc) scores[i + j] = c;
        k4[j] = i + j < Nc ? order_key_u(c) : 0u;
        range.add_or_none(k4[j], i + j < Nc);
      }
      if constexpr (SELECT)
        if (i < Nc) *reinterpret_cast<uint4 *>(&k_s[slot4(i)]) = make_uint4(k4[0], k4[1], k4[2], k4[3]);
    }
  }
  if (scores)
    for (int i = Nc + tid; i < N; i += THREADS) scores[i] = INFINITY;
  if constexpr (!SELECT) return;
  thresholds_begin<THREADS>(range, sc);
  __syncthreads();
  uint32_t key[EPT];
  read_keys<EPT>(k_s, base, Nc, key);

  // ---- TopB': the B' candidates with the largest s_comp, ties to the smaller index.  In fixed
  // budget mode B' = B - W and the indices are the head's final ones; with a budget table (per-head
  // mode) B is the head's own entry and the heads of a batch item are packed back to back.  With cand_m > 0 (head-adaptive
  // mode) the head's best cand_m candidates go to the workspace with their keys instead: no head
  // can end up keeping more than that, so the budget split only has to look at those.
  const bool cand = cand_m > 0;
  const int h = bh % s.hkv, b = bh / s.hkv;
  int Bh, row0;                                        // rows this head keeps, and its first row in the batch item
  head_rows(s, budgets, layer, h, Bh, row0);
  const int64_t out_row0 = (int64_t)b * s.hkv * s.B + row0;
  int32_t *idx = cand ? reinterpret_cast<int32_t *>(ws + cl.idx) + unit * cl.stride : O.indices + out_row0;
  uint32_t *ckey = reinterpret_cast<uint32_t *>(ws + cl.key) + unit * cl.stride;
  const int Bp = cand ? cand_m : Bh - s.W;
  int32_t *kept = gather_eb > 0 ? reinterpret_cast<int32_t *>(a_s) : nullptr;      // in place of the keys: the gather's rows
  if (Bp > 0) top_select_keys<THREADS, EPT>(key, Bp, idx, cand ? ckey : nullptr, s.floor_, sc, [&](int e) { return base + e; }, kept);
  if (cand) return;
  finish_head(s, O, b, h, Bh, row0, idx, THREADS);
  // ---- gather of the kept rows (Sec. 3.1, the compacted cache), if asked for: gather_eb is the
  // element size in bytes, 0 to skip.  16 bytes per thread and step, four rows in flight per thread, their positions
  // out of LDS: a step is one memory round trip (one row in flight, positions read back from memory: 256 heads of 1024 rows of
  // 4096 72 -> 56 us, 512 of 225 fp32 rows 62 -> 47).
  if (gather_eb > 0) {
    __syncthreads();
    const LayerIn L = in.l[layer];
    const int lppr = 31 - __clz(s.D * gather_eb / 16), pieces = Bh << lppr;         // pieces per row: 8, 16 or 32
    const char *Kh = reinterpret_cast<const char *>(L.K) + ((int64_t)b * L.sb + (int64_t)h * L.sh) * gather_eb;
    const char *Vh = reinterpret_cast<const char *>(L.V) + ((int64_t)b * L.sb + (int64_t)h * L.sh) * gather_eb;
    char *Ko = reinterpret_cast<char *>(O.K_out) + out_row0 * s.D * gather_eb;
    char *Vo = reinterpret_cast<char *>(O.V_out) + out_row0 * s.D * gather_eb;
    constexpr int U = 4;
    for (int p0 = threadIdx.x; p0 < pieces; p0 += U * THREADS) {
      u32x4 kv[U], vv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = min(p0 + u * THREADS, pieces - 1), row = p >> lppr, piece = p & ((1 << lppr) - 1);
        const int at = row < Bp ? kept[row] : Nc + row - Bp;
        const int src = min(max(at, 0), N - 1);        // positions come from the selection above; the clamp only guards the load
        const int64_t so = (int64_t)src * L.sn * gather_eb + piece * 16;
        kv[u] = *reinterpret_cast<const u32x4 *>(Kh + so);
        vv[u] = *reinterpret_cast<const u32x4 *>(Vh + so);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = p0 + u * THREADS;
        if (p < pieces) {
          *reinterpret_cast<u32x4 *>(Ko + (int64_t)p * 16) = kv[u];
          *reinterpret_cast<u32x4 *>(Vo + (int64_t)p * 16) = vv[u];
        }
      }
    }
  }
}

// topsel_kernel: the selection half alone, on scores that are already in memory (the caller's, for
// mixkv_select).  One workgroup per unit reads the Nc candidate scores of its head once (coalesced,
// their order keys through the padded LDS row to their consecutive-range owners) and selects from registers as
// above: the head's final rows in fixed and per-head mode, or with cand_m > 0 its best cand_m
// candidates with their keys for the head-adaptive split (Sec. 3.1 / Algorithm 1, TopB).  112 heads of 8160, 1536 candidates
// and a floor each: 14.9 -> 9.2 us with the search of mixkv_topsel.h as it is now.
template <int THREADS, int EPT>
__global__ __launch_bounds__(THREADS) void topsel_kernel(Shape s, LayerOutTable out, char *ws, CandLists cl, int64_t unit0,
                                                           int cand_m, const int32_t *budgets) {
  extern __shared__ __align__(16) float a_s[];          // the head's order keys
  __shared__ MsScratch sc;
  const int tid = threadIdx.x, ul = blockIdx.x;
  const int64_t unit = unit0 + ul;
  const int layer = ul / s.units_per_layer, bh = ul - layer * s.units_per_layer;
  const LayerOut O = out.l[layer];
  const float *scores = O.scores + (int64_t)bh * s.N;
  const int Nc = s.Nc, base = tid * EPT;
  uint32_t *k_s = reinterpret_cast<uint32_t *>(a_s);
  float c[EPT];
#pragma unroll
  for (int e = 0; e < EPT; ++e) c[e] = scores[min(e * THREADS + tid, Nc - 1)];      // all in flight together
  uint32_t key[EPT];
  KeyRange range;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    key[e] = order_key_u(c[e]);
    range.add(key[e]);                                  // past the row the last score again
    if (e * THREADS + tid < Nc) k_s[slot4(e * THREADS + tid)] = key[e];
  }
  thresholds_begin<THREADS>(range, sc);
  __syncthreads();
  read_keys<EPT>(k_s, base, Nc, key);
  const bool cand = cand_m > 0;
  const int h = bh % s.hkv, b = bh / s.hkv;
  int Bh, row0;
  head_rows(s, budgets, layer, h, Bh, row0);
  int32_t *idx = cand ? reinterpret_cast<int32_t *>(ws + cl.idx) + unit * cl.stride
                      : O.indices + (int64_t)b * s.hkv * s.B + row0;
  uint32_t *ckey = cand ? reinterpret_cast<uint32_t *>(ws + cl.key) + unit * cl.stride : nullptr;
  const int Bp = cand ? cand_m : Bh - s.W;
  if (Bp > 0) top_select_keys<THREADS, EPT>(key, Bp, idx, ckey, s.floor_, sc, [&](int e) { return base + e; });
  if (!cand) finish_head(s, O, b, h, Bh, row0, idx, THREADS);
}

// candsplit_kernel: head-adaptive budgets from candidate lists, one workgroup per (layer, batch
// item).  Every head brings its best M candidates (ascending positions, with keys, its f best
// marked); a head keeps its floor, i.e. its f best, and the rest of the layer's pool goes to the
// best remaining candidates of all heads together, ties to the smaller head, then the smaller
// position.  A head can keep at most f + H * (B' - f) <= M candidates, so the lists hold every
// candidate that can be kept and the result is the same as ranking all scores.  Thread t owns EPT
// consecutive entries of the H lists laid end to end, each rounded up to whole threads: that order is the tie order,
// the kept entries of a head come out in ascending position from one prefix sum, and a thread's entries are one
// aligned run of one list.  Up to 32 entries per thread stay in registers with their positions; of 64 the keys alone, the
// positions of kept entries being read again.
template <int THREADS, int EPT>
__global__ __launch_bounds__(THREADS) void candsplit_kernel(Shape s, LayerOutTable out, char *ws, CandLists cl, int64_t unit0,
                                                              int M) {
  constexpr int NW = THREADS / 64;
  __shared__ MsScratch sc;
  __shared__ int hstart[65];                           // kept entries before each head's list; [H]: all
  const int tid = threadIdx.x, lb = blockIdx.x, layer = lb / s.batch, b = lb - layer * s.batch;
  const LayerOut O = out.l[layer];
  const int Nc = s.Nc, H = s.hkv, rest = H * (s.Bp - s.floor_);
  const int64_t unit = unit0 + (int64_t)lb * H;        // first head of this (layer, batch item)
  int32_t *idx = O.indices + (int64_t)b * H * s.B;
  const int tph = (M + EPT - 1) / EPT;                 // threads to a list
  const int h = tid / tph, i0 = (tid - h * tph) * EPT, left = h < H ? M - i0 : 0;    // entries from the thread's first one on
  // Whole runs: what lies behind a list's last entry (inside its row of the workspace) is not looked at.
  const int64_t at = (unit + min(h, H - 1)) * cl.stride + i0;
  const uint4 *krun = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint32_t *>(ws + cl.key) + at);
  const uint4 *prun = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint32_t *>(ws + cl.idx) + at);
  constexpr bool HOLD = EPT <= 32;
  constexpr int STEP = HOLD ? EPT : 16;                 // entries loaded together
  uint32_t key[EPT], pw[HOLD ? EPT : 1];
  // the search sees the entries outside the floors (key 0: not this one)
  KeyRange range;
  uint32_t floors[EPT / STEP];             // entries that are kept as they are
#pragma unroll
  for (int j0 = 0; j0 < EPT; j0 += STEP) {
    uint32_t p[STEP];
#pragma unroll
    for (int g = 0; g < STEP / 4; ++g) {
      // behind a list that ends earlier its last group of four again, which is inside the workspace
      const int gi = HOLD ? g : min(j0 / 4 + g, max(left - 1, 0) / 4);
      const uint4 kq = krun[gi], pq = prun[gi];
      key[j0 + 4 * g] = kq.x; key[j0 + 4 * g + 1] = kq.y; key[j0 + 4 * g + 2] = kq.z; key[j0 + 4 * g + 3] = kq.w;
      p[4 * g] = pq.x; p[4 * g + 1] = pq.y; p[4 * g + 2] = pq.z; p[4 * g + 3] = pq.w;
    }
    floors[j0 / STEP] = 0;
#pragma unroll
    for (int j = 0; j < STEP; ++j) {
      const bool flag = (p[j] & kFloorFlag) != 0;
      floors[j0 / STEP] |= j0 + j < left && flag ? 1u << j : 0u;
      const bool there = j0 + j < left && !flag && rest > 0;
      key[j0 + j] = there ? key[j0 + j] : 0u;
      if constexpr (HOLD) range.add_or_none(key[j0 + j], there);
      else range.largest = max(range.largest, key[j0 + j]);
      if constexpr (HOLD) pw[j] = p[j];
    }
    if constexpr (!HOLD) __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (!HOLD) range.smallest = 1;              // keys are at least that; the smallest of 64 per thread took 1.9 us of 54 to find
  thresholds_begin<THREADS>(range, sc);
  __syncthreads();
  const int want[1] = {rest};
  uint32_t tau[1] = {0xffffffffu};
  int k[1] = {0};
  if (rest > 0) radix_thresholds<THREADS, EPT, 1>(key, want, sc, tau, k);
  // kept for sure (low half) and equal to the threshold (high half) share a word
  int packed = 0, total;
#pragma unroll
  for (int j = 0; j < EPT / STEP; ++j) packed += __popc(floors[j]);
#pragma unroll
  for (int j = 0; j < EPT; ++j) packed += key[j] > tau[0] ? 1 : 0;
  if (k[0] > 0) {
#pragma unroll
    for (int j = 0; j < EPT; ++j) packed += key[j] == tau[0] ? 1 << 16 : 0;
  }
  packed = block_scan_excl<NW>(packed, sc, &total);
  int seen = (int)((uint32_t)packed >> 16);
  int pos = (packed & 0xffff) + min(seen, k[0]);       // kept entries before this thread's
  const int kept = (total & 0xffff) + min((int)((uint32_t)total >> 16), k[0]);
  if (i0 == 0 && h < H) hstart[h] = pos;
  pos += h * s.W;
#pragma unroll
  for (int j = 0; j < EPT; ++j) {
    bool keep = ((floors[j / STEP] >> (j % STEP)) & 1u) != 0 || key[j] > tau[0];
    if (k[0] > 0 && key[j] == tau[0]) keep = seen++ < k[0];
    if (keep) idx[pos++] = (int32_t)((HOLD ? pw[HOLD ? j : 0] : reinterpret_cast<const uint32_t *>(prun)[j]) & ~kFloorFlag);
  }
  if (tid == 0) hstart[H] = kept;
  __syncthreads();
  // per head: count, offset, and the window behind the kept candidates
  for (int hh = tid >> 6; hh < H; hh += NW) {
    const int lane = tid & 63, first = hstart[hh] + hh * s.W, cnt = hstart[hh + 1] - hstart[hh];
    for (int wv = lane; wv < s.W; wv += 64) idx[first + cnt + wv] = Nc + wv;
    if (lane == 0) {
      O.counts[b * H + hh] = cnt + s.W;
      O.offsets[b * (H + 1) + hh] = first;
      if (hh == H - 1) O.offsets[b * (H + 1) + H] = first + cnt + s.W;
    }
  }
}

// Largest sequence the fused kernel handles: 32 candidates per thread, and the raw attention row
// must fit in LDS next to the scratch.
static size_t mixsel_lds(const Shape &s) { return (size_t)slots4(s.Nc + 12) * 4; }      // the row, four words up, with fill on either side
bool mixsel_supported(const Shape &s) { return s.Nc <= kMsMaxThreads * 32 && mixsel_lds(s) <= (size_t)kMsMaxLds; }

template <int THREADS, int EPT>
static hipError_t launch_mixsel_e(const Shape &s, bool select, const LayerOutTable &out, char *ws, const Workspace &w,
                                  int64_t unit0, int nunits, const LayerInTable &in, int gather_eb, int cand_m,
                                  const CandLists &cl, const int32_t *budgets, hipStream_t st) {
  const size_t lds = mixsel_lds(s);
  // The kernels may use more dynamic LDS than the default limit.  The limit is a property of the
  // kernel, shared by every stream and thread, so it is raised once, to the most mixsel_supported
  // admits, once per device, and never touched again (a per-launch value could be lowered by another
  // thread between this thread's call and its launch).
  if (select) {
    auto kern = mixsel_kernel<THREADS, EPT, true>;
    static LdsLimitOnce once;
    const hipError_t attr = once.raise(reinterpret_cast<const void *>(kern));
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kern, dim3(nunits), dim3(THREADS), lds, st, s, out, ws, w, unit0, in, gather_eb, cand_m, cl, budgets);
  } else {
    auto kern = mixsel_kernel<THREADS, EPT, false>;
    static LdsLimitOnce once;
    const hipError_t attr = once.raise(reinterpret_cast<const void *>(kern));
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kern, dim3(nunits), dim3(THREADS), lds, st, s, out, ws, w, unit0, in, 0, 0, cl, nullptr);
  }
  return hipGetLastError();
}

// Mix (and, with `select`, selection: the final fixed-budget one, or with cand_m > 0 every head's
// best cand_m candidates for the head-adaptive split; with `gather_eb` > 0 also the gather of the
// kept rows, gather_eb being the element size) for `nunits` units starting at unit0.  Threads and candidates per thread by
// what takes the time, a wave's instructions (504 candidates: 256 threads of 4 8.9 us, of 8 10.5; 4064: 512 of 8 and 1024 of 4
// the same 11.1, 256 of 16 13.9; 8160 on 112 heads: 1024 of 8 16.3, 512 of 16 17.9; 16 352 on 256 heads: 1024 of 16 44, 512 of 32 52).
hipError_t launch_mixsel(const Shape &s, bool select, const LayerOutTable &out, char *ws, const Workspace &w,
                         int64_t unit0, int nunits, const LayerInTable &in, int gather_eb, int cand_m,
                         const CandLists &cl, const int32_t *budgets, hipStream_t st) {
  const int nc = s.Nc;
  if (nc <= 256 * 4) return launch_mixsel_e<256, 4>(s, select, out, ws, w, unit0, nunits, in, gather_eb, cand_m, cl, budgets, st);
  if (nc <= 512 * 4) return launch_mixsel_e<512, 4>(s, select, out, ws, w, unit0, nunits, in, gather_eb, cand_m, cl, budgets, st);
  if (nc <= 512 * 8) return launch_mixsel_e<512, 8>(s, select, out, ws, w, unit0, nunits, in, gather_eb, cand_m, cl, budgets, st);
  if (nc <= 1024 * 8) return launch_mixsel_e<1024, 8>(s, select, out, ws, w, unit0, nunits, in, gather_eb, cand_m, cl, budgets, st);
  if (nc <= 1024 * 16) return launch_mixsel_e<1024, 16>(s, select, out, ws, w, unit0, nunits, in, gather_eb, cand_m, cl, budgets, st);
  return launch_mixsel_e<1024, 32>(s, select, out, ws, w, unit0, nunits, in, gather_eb, cand_m, cl, budgets, st);
}

template <int THREADS, int EPT>
static hipError_t launch_topsel_e(const Shape &s, const LayerOutTable &out, char *ws, const CandLists &cl, int64_t unit0,
                                  int nunits, int cand_m, const int32_t *budgets, hipStream_t st) {
  const size_t lds = mixsel_lds(s);
  auto kern = topsel_kernel<THREADS, EPT>;
  static LdsLimitOnce once;
  const hipError_t attr = once.raise(reinterpret_cast<const void *>(kern));
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kern, dim3(nunits), dim3(THREADS), lds, st, s, out, ws, cl, unit0, cand_m, budgets);
  return hipGetLastError();
}

// Selection on scores in memory for `nunits` units starting at unit0 (requires mixsel_supported):
// final rows, or with cand_m > 0 every head's best cand_m candidates for the head-adaptive split.
hipError_t launch_topsel(const Shape &s, const LayerOutTable &out, char *ws, const CandLists &cl, int64_t unit0, int nunits,
                         int cand_m, const int32_t *budgets, hipStream_t st) {
  const int nc = s.Nc;
  if (nc <= 256 * 4) return launch_topsel_e<256, 4>(s, out, ws, cl, unit0, nunits, cand_m, budgets, st);
  if (nc <= 512 * 4) return launch_topsel_e<512, 4>(s, out, ws, cl, unit0, nunits, cand_m, budgets, st);
  if (nc <= 512 * 8) return launch_topsel_e<512, 8>(s, out, ws, cl, unit0, nunits, cand_m, budgets, st);
  if (nc <= 1024 * 8) return launch_topsel_e<1024, 8>(s, out, ws, cl, unit0, nunits, cand_m, budgets, st);
  if (nc <= 1024 * 16) return launch_topsel_e<1024, 16>(s, out, ws, cl, unit0, nunits, cand_m, budgets, st);
  return launch_topsel_e<1024, 32>(s, out, ws, cl, unit0, nunits, cand_m, budgets, st);
}

// The head-adaptive split of `nlayers` layers' candidate lists of M entries per head: one workgroup per (layer, batch
// item) with all entries in registers, or, past 64 of them per thread, streamed from memory.  As many threads as there
// are groups of four entries, up to 1024: a wave's instructions are what takes the time (4 lists of 1536 entries: 1024 threads
// of 8 7.4 us, 512 of 16 8.6; with lists that shared a thread and branches on every entry 13.2).  64 of them against the stream, the
// selection's whole call: 8 lists of 5344 entries 126 -> 58 us, of 7744 161 -> 67, 28 layers of those 176 -> 85.
template <int THREADS, int EPT>
static hipError_t launch_candsplit_e(const Shape &s, const LayerOutTable &out, char *ws, const CandLists &cl, int64_t unit0,
                                     int grid, int cand_m, hipStream_t st) {
  hipLaunchKernelGGL((candsplit_kernel<THREADS, EPT>), dim3(grid), dim3(THREADS), 0, st, s, out, ws, cl, unit0, cand_m);
  return hipGetLastError();
}
hipError_t launch_select_candidates(const Shape &s, const LayerOutTable &out, char *ws, const CandLists &cl, int64_t unit0,
                                    int nlayers, int cand_m, hipStream_t st) {
  const int grid = nlayers * s.batch;
  auto fits = [&](int threads, int ept) { return (int64_t)((cand_m + ept - 1) / ept) * s.hkv <= threads; };
  if (fits(256, 4)) return launch_candsplit_e<256, 4>(s, out, ws, cl, unit0, grid, cand_m, st);
  if (fits(512, 4)) return launch_candsplit_e<512, 4>(s, out, ws, cl, unit0, grid, cand_m, st);
  if (fits(1024, 4)) return launch_candsplit_e<1024, 4>(s, out, ws, cl, unit0, grid, cand_m, st);
  if (fits(1024, 8)) return launch_candsplit_e<1024, 8>(s, out, ws, cl, unit0, grid, cand_m, st);
  if (fits(1024, 16)) return launch_candsplit_e<1024, 16>(s, out, ws, cl, unit0, grid, cand_m, st);
  if (fits(1024, 32)) return launch_candsplit_e<1024, 32>(s, out, ws, cl, unit0, grid, cand_m, st);
  // (kept entries and entries equal to the threshold are counted in 16 bits each)
  if (fits(1024, 64) && (int64_t)cand_m * s.hkv < 1 << 16) return launch_candsplit_e<1024, 64>(s, out, ws, cl, unit0, grid, cand_m, st);
  return launch_split_stream(s, out, ws, cl, unit0, nlayers, cand_m, st);
}

}  // namespace mixkv
