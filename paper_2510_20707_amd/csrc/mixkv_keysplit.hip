// The two streaming passes for few query rows: every wave takes key tiles of its own.
//
// stats_kernel and attn_kernel deal the query tiles of a head to the waves of a workgroup, which walk the key
// tiles together.  With one or two query tiles that leaves most waves without matrix work: one wave's chain of
// matrix instructions is the length of every tile step, and every step ends in a barrier.  Here a wave holds all TQ
// query tiles in registers and takes every kKsWaves-th key tile of the workgroup's run by itself:
//   * the tile travels global -> registers (whole rows, coalesced, the next tile's rows requested before the
//     matrix work of the present one), so the row norms, the normalised-key sum and K_i . Kbar are taken
//     from registers;
//   * the keys then cross a private 32-row LDS image into MFMA fragments; no barrier, no other wave;
//   * column sums are complete inside the wave, and one store per tile and output carries 32 keys.
// Waves meet once per run, where their softmax partials and key sums are folded in wave order.
//
// Bound: HBM, once no wave waits for another's matrix instructions (f32 with two tiles: the matrix cores).  First
// pass / second pass with the fold, us, 14 layers x 8 KV heads, 8192 keys (f32: 4096), by query tiles, before -> now
// (before: the kernels of mixkv_stream.hip):
//   f32  D = 128   one 179 -> 110 (4.3 TB/s) / 146 -> 72    two 188 -> 144 / 152 -> 104
//   f32  D = 64    one  68 ->  47 (5.0 TB/s) /  87 -> 36    two  93 ->  66 /  89 ->  62
//   bf16 D = 64    one  58 ->  43 (5.5 TB/s) /  45 -> 30    two  65 ->  47 /  46 ->  33
//   bf16 D = 128   one 102 ->  99 (4.7 TB/s) /  62 -> 56    two 105 -> 108 /  64 -> 64: not taken
// Three and four tiles spill (their fragments, 32 or 64 registers a tile, are what fills the file): not taken.
#include "mixkv_stream.h"

namespace mixkv {

constexpr int kKsWaves = 4, kKsThreads = kKsWaves * 64;

// Workgroups per compute unit: tiles of 16 KB take the full register file; three for the smallest tiles (the
// registers allow it) were slower than two (46 -> 50 us on 117 MB).
__host__ __device__ constexpr int ks_wgs(int dtype, int D) {
  return D * (dtype == MIXKV_BF16 ? 2 : 4) > 256 ? 1 : 2;
}

// The 32-row tile that starts at `tile` (wave-uniform) in row layout: load j holds rows j * RPL + lane / PPR, piece
// lane % PPR.  A whole tile is a uniform address per load plus one lane offset; rows past the last one (row
// `rows` - 1) repeat it.
// (The plain load stands here and not in load_piece: behind a call the compiler lays the first pass out 8 % longer, 29.8 -> 30.3 us a call
// of 2 heads of 512 keys.)
template <int DT, int D, bool ONCE, int NL>
__device__ __forceinline__ void load_rows(uint4 (&r)[NL], const char *tile, int64_t row_bytes, int rows, int lane) {
  constexpr int PPR = D * Tr<DT>::EB / 16, RPL = 64 / PPR;
  const int lrow = lane / PPR, lq = lane % PPR;
  if (rows >= 32) {
    const uint32_t off = (uint32_t)lrow * (uint32_t)row_bytes + (uint32_t)lq * 16;
#pragma unroll
    for (int j = 0; j < NL; ++j)
      if constexpr (ONCE) r[j] = load_piece<true>(tile + (int64_t)(j * RPL) * row_bytes + off);
      else r[j] = *reinterpret_cast<const uint4 *>(tile + (int64_t)(j * RPL) * row_bytes + off);
  } else {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int row = min(j * RPL + lrow, rows - 1);
      if constexpr (ONCE) r[j] = load_piece<true>(tile + row * row_bytes + lq * 16);
      else r[j] = *reinterpret_cast<const uint4 *>(tile + row * row_bytes + lq * 16);
    }
  }
}

// Row-layout registers into the wave's tile image (the rotation of read_key_frag).
template <int DT, int D, int NL>
__device__ __forceinline__ void image_of_rows(uint4 *img, const uint4 (&r)[NL], int lane) {
  constexpr int PPR = D * Tr<DT>::EB / 16, RPL = 64 / PPR;
  const int lrow = lane / PPR, lq = lane % PPR;
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int row = j * RPL + lrow;
    img[row * PPR + (lq ^ tile_swz<DT, D>(row))] = r[j];
  }
}

// ------------------------------------------------------------------------------------------------
// First pass (see stats_kernel for what it computes): softmax partials, key norms, the sum of normalised keys, value norms.
// ------------------------------------------------------------------------------------------------
template <int DT, int D, int TQ, bool ONCE>
__global__ __launch_bounds__(kKsThreads, ks_wgs(DT, D)) void ks_stats_kernel(Shape s, LayerInTable in, char *ws, Workspace w, int64_t unit0,
                                                                int nunits, int64_t slot0) {
  constexpr int EB = Tr<DT>::EB, EPC = Tr<DT>::EPC, NCHK = D / (2 * EPC), PPR = D * EB / 16, RPL = 64 / PPR, TILE = 32 * PPR;
  constexpr int NL = TILE / 64, KT = chunk_tiles(DT, D), W = kKsWaves;
  __shared__ uint4 img_s[W * TILE];
  __shared__ float ks_s[W * D];
  __shared__ float2 ml_s[W * TQ * 32];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5, lrow = lane / PPR, lq = lane % PPR;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint4 *img = img_s + wave * TILE;
  const int N = s.N, Nc = s.Nc, QTR = s.QT * 32;
  const float c2 = s.scale_log2e;
  const int free_limit = s.causal ? Nc : N - 1;      // keys <= this are visible to every row
  const bool use_v = s.intrinsic == MIXKV_INTRINSIC_VNORM;
  const int64_t T = (int64_t)nunits * s.nchunks;
  int64_t item = wg_first_item(blockIdx.x, gridDim.x, T);
  const int64_t item_end = wg_first_item(blockIdx.x + 1, gridDim.x, T);

  while (item < item_end) {
    const int ul = (int)(item / s.nchunks), c0 = (int)(item - (int64_t)ul * s.nchunks);
    const int nit = (int)min((int64_t)(s.nchunks - c0), item_end - item);
    const int64_t unit = unit0 + ul;
    const UnitCoord uc = unit_coord(s, ul);
    const LayerIn L = in.l[uc.layer];
    const int64_t head_off = ((int64_t)uc.b * L.sb + (int64_t)uc.h * L.sh) * EB;
    const int64_t row_bytes = L.sn * EB;
    const int key0 = c0 * KT * 32;                                   // first key of the run
    const int nt = min(nit * KT, (N - key0 + 31) / 32);              // tiles of the run that hold keys
    const char *Kr = reinterpret_cast<const char *>(L.K) + head_off + key0 * row_bytes;
    const char *Vr = reinterpret_cast<const char *>(L.V) + head_off + key0 * row_bytes;
    const char *Qb = reinterpret_cast<const char *>(L.Q) + ((int64_t)(uc.b * s.hq + uc.h * s.G) * s.W * D) * EB;
    float *invnorm = reinterpret_cast<float *>(ws + w.invnorm) + unit * s.Npad + key0;
    float *vnorm = reinterpret_cast<float *>(ws + w.vnorm) + unit * s.Npad + key0;

    uint4 kr[NL], vr[NL];
    auto request = [&](int t) {
      load_rows<DT, D, ONCE, NL>(kr, Kr + (int64_t)t * 32 * row_bytes, row_bytes, N - key0 - t * 32, lane);
      if (use_v) load_rows<DT, D, ONCE, NL>(vr, Vr + (int64_t)t * 32 * row_bytes, row_bytes, N - key0 - t * 32, lane);
    };
    if (wave < nt) request(wave);
    Frag qf[TQ][NCHK];
    int lim[TQ];
    float m[TQ], l[TQ];
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
      const int row = q * 32 + l32;
      const bool live = row < s.GW;
      const char *qrow = Qb + ((int64_t)(live ? row : 0) * D) * EB + half * 16;
#pragma unroll
      for (int c = 0; c < NCHK; ++c) {
        const uint4 v = *reinterpret_cast<const uint4 *>(qrow + c * 32);
        qf[q][c].q = live ? v : make_uint4(0, 0, 0, 0);
      }
      lim[q] = s.causal ? Nc + row % s.W : N - 1;     // last key this row attends to
      m[q] = -INFINITY;
      l[q] = 0.f;
    }
    float ksacc[EPC];                                 // lane (lrow, lq): piece lq of the normalised rows it has seen
#pragma unroll
    for (int e = 0; e < EPC; ++e) ksacc[e] = 0.f;

    for (int t = wave; t < nt; t += W) {
      const int tb = key0 + t * 32;
      // ---- norms from the rows in registers; lane lq of a row group keeps the value of load lq for the store
      if (use_v) {
        float keep = 0.f;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
          Frag f;
          f.q = vr[j];
          const float ss = seg_sum<PPR>(piece_sumsq<DT>(f));
          keep = lq == j ? ss : keep;
        }
        const int row = lq * RPL + lrow;
        if (lq < NL && tb + row < Nc) vnorm[t * 32 + row] = __builtin_amdgcn_sqrtf(keep);
      }
      if (s.kstats) {
        float keep = 0.f;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
          Frag f;
          f.q = kr[j];
          const float ss = seg_sum<PPR>(piece_sumsq<DT>(f));
          const float inv = tb + j * RPL + lrow < N ? inv_norm<DT>(ss) : 0.f;
          keep = lq == j ? inv : keep;
#pragma unroll
          for (int e = 0; e < EPC; ++e) ksacc[e] = fmaf(inv, frag_elem<DT>(f, e), ksacc[e]);
        }
        const int row = lq * RPL + lrow;
        if (lq < NL && tb + row < N) invnorm[t * 32 + row] = keep;
      }
      wave_lds_fence();
      image_of_rows<DT, D, NL>(img, kr, lane);
      wave_lds_fence();
      if (t + W < nt) request(t + W);

      // ---- per query tile: scores (keys on the MFMA output rows, query rows on the columns), then the running
      // softmax with an offset that moves only on overflow (as in stats_kernel)
      __builtin_amdgcn_sched_barrier(0);
      Frag kf[NCHK];
#pragma unroll
      for (int c = 0; c < NCHK; ++c) kf[c].q = read_key_frag<DT, D>(img, 0, c, l32, half);
#pragma unroll
      for (int q = 0; q < TQ; ++q) {
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
        for (int c = 0; c < NCHK; ++c) acc = mma<DT>(kf[c], qf[q][c], acc);
        if (tb + 31 > free_limit) {                    // tile reaches into the window or past N: mask
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[i] = (tb + 8 * (i >> 2) + 4 * half + (i & 3) > lim[q]) ? -INFINITY : acc[i];
        }
        float sum[4];
        const float nmu = -m[q];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float term = fast_exp2(fmaf(acc[i], c2, nmu));
          sum[i & 3] = i < 4 ? term : sum[i & 3] + term;
        }
        float lnew = l[q] + ((sum[0] + sum[1]) + (sum[2] + sum[3]));
        if (__builtin_amdgcn_ballot_w64(!(lnew < kSumLimit)) != 0) {
          float tmax = fmaxf(acc[0], acc[1]);
#pragma unroll
          for (int i = 2; i < 16; i += 2) tmax = fmaxf(fmaxf(tmax, acc[i]), acc[i + 1]);
          const float mn = fmaxf(m[q], ceilf(tmax * c2));   // whole offsets: every rescaling, here and in the merges, is exact
          const float mu = (mn == -INFINITY) ? 0.f : mn;
          float s2[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < 16; ++i) s2[i & 3] += fast_exp2(fmaf(acc[i], c2, -mu));
          lnew = l[q] * fast_exp2(m[q] - mu) + ((s2[0] + s2[1]) + (s2[2] + s2[3]));
          m[q] = mn;
        }
        l[q] = lnew;
      }
    }

    // ---- run partials: the waves' shares meet in LDS and are folded in wave order
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
      int e;
      l[q] = frexpf(l[q], &e);                         // the sum may be far from 1: see stats_kernel
      m[q] += (float)e;
      ml_merge(m[q], l[q], __shfl_xor(m[q], 32), __shfl_xor(l[q], 32));
      if (half == 0) ml_s[(wave * TQ + q) * 32 + l32] = make_float2(m[q], l[q]);
    }
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
      float x = ksacc[e];
#pragma unroll
      for (int off = PPR; off < 64; off <<= 1) x += __shfl_xor(x, off);
      if (lane < PPR) ks_s[wave * D + lane * EPC + e] = x;
    }
    __syncthreads();
    const int64_t slot = slot0 + blockIdx.x + ul;
    for (int r = tid; r < TQ * 32; r += kKsThreads) {
      float mm = ml_s[r].x, ll = ml_s[r].y;
#pragma unroll
      for (int v = 1; v < W; ++v) ml_merge(mm, ll, ml_s[v * TQ * 32 + r].x, ml_s[v * TQ * 32 + r].y);
      reinterpret_cast<float2 *>(ws + w.part_ml)[slot * QTR + r] = make_float2(mm, ll);
    }
    for (int d = tid; d < D; d += kKsThreads) {
      float a = 0.f;
#pragma unroll
      for (int v = 0; v < W; ++v) a += ks_s[v * D + d];
      reinterpret_cast<float *>(ws + w.part_ksum)[slot * D + d] = a;
    }
    __syncthreads();                                   // before the next run's partials
    item += nit;
  }
}

// ------------------------------------------------------------------------------------------------
// Second pass (see attn_kernel): mean attention weight per key and K_i . Kbar.
// ------------------------------------------------------------------------------------------------
template <int DT, int D, int TQ, bool ONCE>
__global__ __launch_bounds__(kKsThreads, ks_wgs(DT, D)) void ks_attn_kernel(Shape s, LayerInTable in, char *ws, Workspace w, int64_t unit0,
                                                               int nunits) {
  constexpr int EB = Tr<DT>::EB, EPC = Tr<DT>::EPC, NCHK = D / (2 * EPC), PPR = D * EB / 16, RPL = 64 / PPR, TILE = 32 * PPR;
  constexpr int NL = TILE / 64, KT = chunk_tiles(DT, D), W = kKsWaves;
  __shared__ uint4 img_s[W * TILE];
  __shared__ int lim_s[TQ * 32];                         // last key each query row attends to
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5, lrow = lane / PPR, lq = lane % PPR;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint4 *img = img_s + wave * TILE;
  const int N = s.N, Nc = s.Nc;
  const float c2 = s.scale_log2e;
  const int free_limit = s.causal ? Nc : N - 1;
  for (int r = tid; r < TQ * 32; r += kKsThreads) lim_s[r] = s.causal ? Nc + r % s.W : N - 1;
  __syncthreads();
  const int64_t T = (int64_t)nunits * s.nchunks;
  int64_t item = wg_first_item(blockIdx.x, gridDim.x, T);
  const int64_t item_end = wg_first_item(blockIdx.x + 1, gridDim.x, T);

  while (item < item_end) {
    const int ul = (int)(item / s.nchunks), c0 = (int)(item - (int64_t)ul * s.nchunks);
    const int nit = (int)min((int64_t)(s.nchunks - c0), item_end - item);
    const int64_t unit = unit0 + ul;
    const UnitCoord uc = unit_coord(s, ul);
    const LayerIn L = in.l[uc.layer];
    const int64_t row_bytes = L.sn * EB;
    const int key0 = c0 * KT * 32;
    const int nt = min(nit * KT, (N - key0 + 31) / 32);
    const char *Kr = reinterpret_cast<const char *>(L.K) + ((int64_t)uc.b * L.sb + (int64_t)uc.h * L.sh) * EB + key0 * row_bytes;
    const char *Qb = reinterpret_cast<const char *>(L.Q) + ((int64_t)(uc.b * s.hq + uc.h * s.G) * s.W * D) * EB;
    float *araw = reinterpret_cast<float *>(ws + w.araw) + unit * s.Npad + key0;
    float *kdot = reinterpret_cast<float *>(ws + w.sdiv) + unit * s.Npad + key0;   // K_i . Kbar, not yet normalised
    const float *nb = reinterpret_cast<const float *>(ws + w.nb) + unit * s.nb_rows;
    const uint4 *kbarp = reinterpret_cast<const uint4 *>(ws + w.kbarp) + unit * (NCHK * 4);

    uint4 kr[NL];
    auto request = [&](int t) { load_rows<DT, D, ONCE, NL>(kr, Kr + (int64_t)t * 32 * row_bytes, row_bytes, N - key0 - t * 32, lane); };
    if (wave < nt) request(wave);
    // piece lq of the mean key (bf16: head and remainder rows)
    float kbar[EPC];
    {
      Frag hi, lo;
      hi.q = kbarp[lq * 2];
      lo.q = kbarp[lq * 2 + 1];
#pragma unroll
      for (int e = 0; e < EPC; ++e) kbar[e] = DT == MIXKV_BF16 ? frag_elem<DT>(hi, e) + frag_elem<DT>(lo, e) : frag_elem<DT>(hi, e);
    }
    Frag qf[TQ][NCHK];
    float nbv[TQ][16];                                 // exponent offsets of the lane's rows
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
      const int row = q * 32 + l32;
      const bool live = row < s.GW;
      const char *qrow = Qb + ((int64_t)(live ? row : 0) * D) * EB + half * 16;
#pragma unroll
      for (int c = 0; c < NCHK; ++c) {
        const uint4 v = *reinterpret_cast<const uint4 *>(qrow + c * 32);
        qf[q][c].q = live ? v : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int k4 = 0; k4 < 4; ++k4) {
        const float4 v = *reinterpret_cast<const float4 *>(nb + q * 32 + 8 * k4 + 4 * half);
        nbv[q][4 * k4 + 0] = v.x; nbv[q][4 * k4 + 1] = v.y; nbv[q][4 * k4 + 2] = v.z; nbv[q][4 * k4 + 3] = v.w;
      }
    }

    for (int t = wave; t < nt; t += W) {
      const int tb = key0 + t * 32, key = tb + l32;
      if (s.kstats) {                                  // K_i . Kbar from the rows in registers
        float keep = 0.f;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
          Frag f;
          f.q = kr[j];
          float x = 0.f;
#pragma unroll
          for (int e = 0; e < EPC; ++e) x = fmaf(frag_elem<DT>(f, e), kbar[e], x);
          x = seg_sum<PPR>(x);
          keep = lq == j ? x : keep;
        }
        const int row = lq * RPL + lrow;
        if (lq < NL && tb + row < Nc) kdot[t * 32 + row] = keep;
      }
      wave_lds_fence();
      image_of_rows<DT, D, NL>(img, kr, lane);
      wave_lds_fence();
      if (t + W < nt) request(t + W);

      // ---- per query tile: scores (query rows on the MFMA output rows, keys on the columns), then the weights
      __builtin_amdgcn_sched_barrier(0);
      Frag kf[NCHK];
#pragma unroll
      for (int c = 0; c < NCHK; ++c) kf[c].q = read_key_frag<DT, D>(img, 0, c, l32, half);
      float cs4[4];
      int rot = 4 * half;                              // hidden from the compiler: it would keep every row's limit in a register
      asm volatile("" : "+v"(rot));
#pragma unroll
      for (int q = 0; q < TQ; ++q) {
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
        for (int c = 0; c < NCHK; ++c) acc = mma<DT>(qf[q][c], kf[c], acc);
        if (tb + 31 > free_limit) {
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[i] = key <= lim_s[rot + q * 32 + 8 * (i >> 2) + (i & 3)] ? acc[i] : -INFINITY;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float wgt = fast_exp2(fmaf(acc[i], c2, nbv[q][i]));
          cs4[i & 3] = (q == 0 && i < 4) ? wgt : cs4[i & 3] + wgt;
        }
      }
      float colsum = (cs4[0] + cs4[1]) + (cs4[2] + cs4[3]);
      colsum += __shfl_xor(colsum, 32);
      if (half == 0 && key < Nc) araw[t * 32 + l32] = colsum;
    }
    item += nit;
  }
}

// ------------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------------
// Up to two query tiles, one for bf16 rows of 128 elements (the table above has both sides of each).
bool keysplit_supported(const Shape &s, int dtype) {
  return s.QT <= (dtype == MIXKV_BF16 && s.D == 128 ? 1 : 2);
}

int keysplit_grid(const Shape &s, int dtype, int nunits, int num_cus) {
  const int64_t T = (int64_t)nunits * s.nchunks;
  int64_t cap = (int64_t)num_cus * ks_wgs(dtype, s.D);
  if (cap > kMaxStreamGrid) cap = kMaxStreamGrid;
  return (int)(T < cap ? T : cap);
}

template <class F>
static void with_types(int dtype, int D, int QT, bool once, F f) {
  auto tq = [&](auto dt, auto d) {
    auto go = [&](auto t) { once ? f(dt, d, t, std::true_type{}) : f(dt, d, t, std::false_type{}); };
    if constexpr (dt() == MIXKV_BF16 && d() == 128) go(std::integral_constant<int, 1>{});
    else if (QT <= 1) go(std::integral_constant<int, 1>{});
    else go(std::integral_constant<int, 2>{});
  };
  auto dd = [&](auto dt) {
    if (D == 128) tq(dt, std::integral_constant<int, 128>{});
    else tq(dt, std::integral_constant<int, 64>{});
  };
  if (dtype == MIXKV_BF16) dd(std::integral_constant<int, MIXKV_BF16>{});
  else dd(std::integral_constant<int, MIXKV_F32>{});
}

// pass_once, except that a launch which reads keys alone keeps them cacheable up to the Infinity Cache's size: its second pass reads all that
// the first has read.  Time with plain loads over that with non-temporal ones, caches in turn, heads of 400 to 7013 keys: 64 elements bf16
// 182-240 MB 0.95-1.02, 260 MB 0.99-1.03, 300 MB 1.04-1.06; f32 0.98-1.01, 1.00-1.02, 1.00-1.04.  128 elements bf16 gain more by
// the faster first read: 182-250 MB, heads of 400 keys 0.96-0.97, of 1500 and 7013 1.03-1.05.
bool keysplit_once(const Shape &s, int dtype, int nunits) {
  const bool keys_alone = s.intrinsic != MIXKV_INTRINSIC_VNORM, wide = dtype == MIXKV_BF16 && s.D == 128 && s.N >= 1000;
  const int64_t key_bytes = (int64_t)nunits * s.N * s.D * (dtype == MIXKV_BF16 ? 2 : 4);
  return pass_once(s, dtype, nunits) && (!keys_alone || wide || key_bytes >= kInfinityCache);
}

hipError_t launch_ks_stats(const Shape &s, int dtype, const LayerInTable &in, char *ws, const Workspace &w, int64_t unit0, int nunits,
                           int grid, int64_t slot0, hipStream_t st) {
  with_types(dtype, s.D, s.QT, keysplit_once(s, dtype, nunits), [&](auto dt, auto d, auto tq, auto once) {
    hipLaunchKernelGGL((ks_stats_kernel<dt(), d(), tq(), once()>), dim3(grid), dim3(kKsThreads), 0, st, s, in, ws, w, unit0, nunits, slot0);
  });
  return hipGetLastError();
}

hipError_t launch_ks_attn(const Shape &s, int dtype, const LayerInTable &in, char *ws, const Workspace &w, int64_t unit0, int nunits,
                          int grid, hipStream_t st) {
  with_types(dtype, s.D, s.QT, keysplit_once(s, dtype, nunits), [&](auto dt, auto d, auto tq, auto once) {
    hipLaunchKernelGGL((ks_attn_kernel<dt(), d(), tq(), once()>), dim3(grid), dim3(kKsThreads), 0, st, s, in, ws, w, unit0, nunits);
  });
  return hipGetLastError();
}

}  // namespace mixkv
