// Redundancy analysis of cached keys or values: the mean off-diagonal cosine similarity of one
// head's rows and the block-mean heat-map of its cosine matrix (paper: Sec. 1, the figures on
// key / value similarity inside a head and across heads; Sec. 3.3, Eq. 3-4 for the matrix and
// its off-diagonal mean).
//
// The N x N matrix is never formed.  With Xh the L2-normalised rows and S_a the sum of the rows
// of block a, the mean of the matrix over block a x block b is S_a . S_b / (n_a n_b), and the sum
// of all entries is |sum_a S_a|^2.  So one streaming pass over X produces the block sums
// (blocksum_kernel, bound by HBM); blockgram_kernel forms their Gram matrix and folds them into the
// off-diagonal mean.
#include "mixkv_stream.h"

namespace mixkv {

struct RowsIn {
  const void *X;
  int64_t sb, sh, sn;   // strides in elements
};
struct RowsInTable { RowsIn l[kLayersPerLaunch]; };
struct SimOut {
  float *redundancy, *block_map;
};
struct SimOutTable { SimOut l[kLayersPerLaunch]; };

struct AShape {
  int32_t batch, heads, N, D, block, nb, units_per_layer;
};

// 1 / max(|x|, 1e-30) from the sum of squares, 0 for a zero row (same convention as the scoring
// path: tiny sums are scaled by 2^64 before the hardware reciprocal square root).
template <int DT>
__device__ __forceinline__ float inv_norm_a(float ss) {
  const bool tiny = ss < 1e-30f;
  const float x = tiny ? ss * 18446744073709551616.f : ss;
  float y = __builtin_amdgcn_rsqf(x);
  y = y * fmaf(-0.5f * x, y * y, 1.5f);
  y = tiny ? y * 4294967296.f : y;
  return ss > 0.f ? fminf(y, 1e30f) : 0.f;
}

// One wave per block of rows.  A row is PPR consecutive lanes of 16 bytes; a wave load covers
// 64 / PPR rows.  Each lane keeps the running sum of its piece of the normalised rows; at the end
// the lanes holding the same piece are folded and the first PPR lanes store S_a.  diag[a] gets
// sum_i |Xh_i|^2 (the number of non-zero rows up to rounding), the trace part of the matrix.
template <int DT, int D, bool ONCE>
__global__ __launch_bounds__(256) void blocksum_kernel(AShape a, RowsInTable in, float *S, float *diag, int nunits) {
  constexpr int EB = DT == MIXKV_BF16 ? 2 : 4, E = 16 / EB, PPR = D * EB / 16, RPL = 64 / PPR, U = 8;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wgs_per_unit = (a.nb + 3) / 4;
  const int ul = blockIdx.x / wgs_per_unit, blk = (blockIdx.x - ul * wgs_per_unit) * 4 + wave;
  if (ul >= nunits || blk >= a.nb) return;             // whole waves leave; no barrier below
  const int layer = ul / a.units_per_layer, bh = ul - layer * a.units_per_layer;
  const int b = bh / a.heads, h = bh - b * a.heads;
  const RowsIn L = in.l[layer];
  const char *base = reinterpret_cast<const char *>(L.X) + ((int64_t)b * L.sb + (int64_t)h * L.sh) * EB;
  const int r0 = blk * a.block, rend = min(a.N, r0 + a.block);
  const int lr = lane / PPR, piece = lane - lr * PPR;
  float acc[E];
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.f;
  float dsum = 0.f;
  for (int r = r0; r < rend; r += RPL * U) {
    uint4 q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int row = r + u * RPL + lr;
      q[u] = make_uint4(0u, 0u, 0u, 0u);
      const char *p = base + (int64_t)row * L.sn * EB + piece * 16;
      if (row < rend) q[u] = load_piece<ONCE>(p);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float x[E];
      if constexpr (DT == MIXKV_BF16) {
        const uint32_t w[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          x[2 * j] = __uint_as_float(w[j] << 16);
          x[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
        }
      } else {
        x[0] = __uint_as_float(q[u].x); x[1] = __uint_as_float(q[u].y);
        x[2] = __uint_as_float(q[u].z); x[3] = __uint_as_float(q[u].w);
      }
      float ss = 0.f;
#pragma unroll
      for (int e = 0; e < E; ++e) ss = fmaf(x[e], x[e], ss);
      ss = seg_sum<PPR>(ss);
      const float inv = inv_norm_a<DT>(ss);              // rows past the block are all zero: inv = 0
#pragma unroll
      for (int e = 0; e < E; ++e) acc[e] = fmaf(inv, x[e], acc[e]);
      if (piece == 0) dsum = fmaf(inv * inv, ss, dsum);
    }
  }
#pragma unroll
  for (int o = PPR; o < 64; o <<= 1) {
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] += __shfl_xor(acc[e], o);
    dsum += __shfl_xor(dsum, o);
  }
  if (lane < PPR) {
    float *dst = S + ((int64_t)ul * a.nb + blk) * D + piece * E;
#pragma unroll
    for (int e = 0; e < E; e += 4) *reinterpret_cast<float4 *>(dst + e) = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
  }
  if (lane == 0) diag[(int64_t)ul * a.nb + blk] = dsum;
}

// Off-diagonal mean of one unit: the sum of all entries of the cosine matrix is |sum_a S_a|^2 and its trace sum_a
// diag[a].  Partial sums are taken over interleaved blocks and folded in a fixed order, in double.
constexpr int kMapThreads = 256;
template <int D>
__device__ void redundancy_of(const AShape &a, const SimOutTable &out, const float *S, const float *diag, int ul) {
  constexpr int PARTS = kMapThreads / D, U = 32;        // loads in flight
  __shared__ double part[kMapThreads];
  const int layer = ul / a.units_per_layer, bh = ul - layer * a.units_per_layer;
  float *red = out.l[layer].redundancy;
  if (!red) return;                                     // uniform over the workgroup
  const float *Su = S + (int64_t)ul * a.nb * D;
  const int tid = threadIdx.x, d = tid % D, pt = tid / D;
  double t4[4] = {0.0, 0.0, 0.0, 0.0};
  for (int bb = pt; bb < a.nb; bb += U * PARTS) {
    float x[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int at = bb + q * PARTS;
      x[q] = Su[(int64_t)min(at, a.nb - 1) * D + d];
      if (at >= a.nb) x[q] = 0.f;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < U; ++q) t4[q & 3] += (double)x[q];
  }
  part[tid] = (t4[0] + t4[1]) + (t4[2] + t4[3]);
  __syncthreads();
  double share = 0.0;                                   // every thread's share of (all entries - trace)
  if (tid < D) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < PARTS; ++q) v += part[q * D + tid];
    share = v * v;
  }
  for (int bb = tid; bb < a.nb; bb += kMapThreads) share -= (double)diag[(int64_t)ul * a.nb + bb];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) share += __shfl_xor(share, o);
  __syncthreads();
  if ((tid & 63) == 0) part[tid >> 6] = share;
  __syncthreads();
  if (tid == 0) {
    double off = 0.0;
#pragma unroll
    for (int i = 0; i < kMapThreads / 64; ++i) off += part[i];
    const double n = (double)a.N;
    red[bh] = (float)(off / (n * (n - 1.0)));
  }
}

// What follows from the block sums, in one launch: workgroups 0 .. nunits - 1 take a unit's off-diagonal mean each, the
// others one 64 x 64 tile of a unit's heat-map, M[a][b] = S_a . S_b / (n_a n_b).  The two sets of 64 block sums
// cross LDS as images of 32 rows and feed the fp32 matrix instructions, a 32 x 32 quadrant per wave.  Bound:
// latency (loads, D / 2 matrix instructions, stores).  112 units of 128 blocks, D = 128: 13.5 us, against 15.2 (the
// same tiles on the vector ALU) + 7.4 (a launch of its own for the means); fragments straight from memory, 32
// rows of 32 bytes per load: 15 to 20.
constexpr int kMapTile = 64;
template <int D>
__global__ __launch_bounds__(kMapThreads) void blockgram_kernel(AShape a, SimOutTable out, const float *S, const float *diag, int nunits) {
  if ((int)blockIdx.x < nunits) {
    redundancy_of<D>(a, out, S, diag, blockIdx.x);
    return;
  }
  constexpr int DT = MIXKV_F32, NCHK = D / 8, PPR = D / 4, TILE = 32 * PPR, LOADS = TILE / kMapThreads;
  __shared__ uint4 img[4 * TILE];                       // rows a0, a0 + 32, b0, b0 + 32
  // workgroups go to the eight XCDs in turn: each XCD takes a contiguous eighth of the tiles, so that a unit's tiles
  // share one L2
  const int tiles = (a.nb + kMapTile - 1) / kMapTile, wg = blockIdx.x - nunits, per_xcd = (gridDim.x - nunits) / 8;
  const int t = (wg & 7) * per_xcd + (wg >> 3);
  if (t >= nunits * tiles * tiles) return;              // uniform over the workgroup
  const int ul = t / (tiles * tiles), tt = t - ul * tiles * tiles, a0 = (tt / tiles) * kMapTile, b0 = (tt % tiles) * kMapTile;
  const int layer = ul / a.units_per_layer, bh = ul - layer * a.units_per_layer;
  float *map = out.l[layer].block_map;
  if (!map) return;                                     // uniform over the workgroup
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const uint4 *Su = reinterpret_cast<const uint4 *>(S + (int64_t)ul * a.nb * D);
  // rows past the last block repeat it: their entries are not stored
  uint4 v[4 * LOADS];
#pragma unroll
  for (int k = 0; k < 4 * LOADS; ++k) {
    const int r = (k % LOADS * kMapThreads + tid) / PPR, piece = tid % PPR, g = k / LOADS;
    v[k] = Su[(int64_t)min((g < 2 ? a0 : b0) + (g & 1) * 32 + r, a.nb - 1) * PPR + piece];
  }
#pragma unroll
  for (int k = 0; k < 4 * LOADS; ++k) {
    const int r = (k % LOADS * kMapThreads + tid) / PPR, piece = tid % PPR;
    img[k / LOADS * TILE + r * PPR + (piece ^ tile_swz<DT, D>(r))] = v[k];
  }
  __syncthreads();
  const uint4 *xa = img + (wave >> 1) * TILE, *yb = img + (2 + (wave & 1)) * TILE;
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
  for (int c = 0; c < NCHK; ++c) {
    Frag x, y;
    x.q = read_key_frag<DT, D>(xa, 0, c, l32, half);
    y.q = read_key_frag<DT, D>(yb, 0, c, l32, half);
    acc = mma<DT>(x, y, acc);
  }
  auto rows_of = [&](int blk) { return (float)(min(a.N, (blk + 1) * a.block) - blk * a.block); };
  const int bb = b0 + (wave & 1) * 32 + l32;
  if (bb >= a.nb) return;
  const float nb_b = rows_of(bb);
  float *col = map + (int64_t)bh * a.nb * a.nb + bb;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int ba = a0 + (wave >> 1) * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
    if (ba < a.nb) col[(int64_t)ba * a.nb] = acc[i] * (1.f / rows_of(ba)) / nb_b;
  }
}

static size_t align256(size_t x) { return (x + 255) / 256 * 256; }

static mixkv_status analysis_shape(const mixkv_params *p, int32_t block, AShape *a) {
  Shape s;
  mixkv_status st = make_shape(p, &s);
  if (st != MIXKV_OK) return st;
  if (block < 1 || block > s.N) return MIXKV_ERR_INVALID_ARG;
  a->batch = s.batch; a->heads = s.hkv; a->N = s.N; a->D = s.D; a->block = block;
  a->nb = (s.N + block - 1) / block;
  a->units_per_layer = s.units_per_layer;
  const int64_t tiles = (a->nb + kMapTile - 1) / kMapTile, per_launch = (int64_t)kLayersPerLaunch * a->units_per_layer;
  if (a->nb * per_launch > INT32_MAX || tiles * tiles * per_launch > INT32_MAX) return MIXKV_ERR_UNSUPPORTED;   // grid sizes
  return MIXKV_OK;
}

}  // namespace mixkv

extern "C" {

mixkv_status mixkv_similarity_workspace_size(const mixkv_params *params, int32_t n_layers, int32_t block, size_t *bytes) {
  mixkv::AShape a;
  mixkv_status st = mixkv::analysis_shape(params, block, &a);
  if (st != MIXKV_OK) return st;
  if (!bytes || n_layers < 1 || n_layers > MIXKV_MAX_LAYERS) return MIXKV_ERR_INVALID_ARG;
  const size_t units = (size_t)n_layers * a.units_per_layer;
  *bytes = mixkv::align256(units * a.nb * a.D * 4) + mixkv::align256(units * a.nb * 4);
  return MIXKV_OK;
}

mixkv_status mixkv_similarity(const mixkv_params *params, const mixkv_rows_in *in, const mixkv_similarity_out *out,
                              int32_t n_layers, int32_t block, void *workspace, size_t workspace_bytes,
                              void *hip_stream) {
  using namespace mixkv;
  AShape a;
  mixkv_status st = analysis_shape(params, block, &a);
  if (st != MIXKV_OK) return st;
  if (!in || !out || n_layers < 1 || n_layers > MIXKV_MAX_LAYERS) return MIXKV_ERR_INVALID_ARG;
  size_t need = 0;
  st = mixkv_similarity_workspace_size(params, n_layers, block, &need);
  if (st != MIXKV_OK) return st;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return MIXKV_ERR_INVALID_ARG;
  if (workspace_bytes < need) return MIXKV_ERR_WORKSPACE_TOO_SMALL;
  const int eb = params->dtype == MIXKV_BF16 ? 2 : 4;
  for (int l = 0; l < n_layers; ++l) {
    const mixkv_rows_in &li = in[l];
    if (!li.X || (reinterpret_cast<uintptr_t>(li.X) & 15u)) return MIXKV_ERR_INVALID_ARG;
    if (li.stride_n < a.D || li.stride_h < 0 || li.stride_b < 0) return MIXKV_ERR_INVALID_ARG;
    if ((li.stride_n * eb) % 16 || (li.stride_h * eb) % 16 || (li.stride_b * eb) % 16) return MIXKV_ERR_INVALID_ARG;
    if (!out[l].redundancy && !out[l].block_map) return MIXKV_ERR_INVALID_ARG;
  }
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
  const size_t units = (size_t)n_layers * a.units_per_layer;
  float *S = reinterpret_cast<float *>(workspace);
  float *diag = reinterpret_cast<float *>(reinterpret_cast<char *>(workspace) + align256(units * a.nb * a.D * 4));
  for (int l0 = 0; l0 < n_layers; l0 += kLayersPerLaunch) {
    const int nl = (n_layers - l0 < kLayersPerLaunch) ? n_layers - l0 : kLayersPerLaunch;
    RowsInTable ti;
    SimOutTable to;
    for (int l = 0; l < kLayersPerLaunch; ++l) {
      ti.l[l] = RowsIn{nullptr, 0, 0, 0};
      to.l[l] = SimOut{nullptr, nullptr};
    }
    for (int l = 0; l < nl; ++l) {
      ti.l[l] = RowsIn{in[l0 + l].X, in[l0 + l].stride_b, in[l0 + l].stride_h, in[l0 + l].stride_n};
      to.l[l] = SimOut{out[l0 + l].redundancy, out[l0 + l].block_map};
    }
    const int nunits = nl * a.units_per_layer;
    const size_t unit0 = (size_t)l0 * a.units_per_layer;
    float *Sg = S + unit0 * a.nb * a.D, *dg = diag + unit0 * a.nb;
    bool any_map = false;
    for (int l = 0; l < nl; ++l) any_map = any_map || to.l[l].block_map;
    const int64_t tiles = any_map ? (a.nb + kMapTile - 1) / kMapTile : 0;
    const dim3 grid_a((unsigned)(nunits * ((a.nb + 3) / 4))), grid_b((unsigned)(nunits + (nunits * tiles * tiles + 7) / 8 * 8));
    const bool bf = params->dtype == MIXKV_BF16;
    const bool once = read_once((int64_t)nunits * a.N * a.D * eb);
    auto sums = [&](auto kern) { hipLaunchKernelGGL(kern, grid_a, dim3(256), 0, stream, a, ti, Sg, dg, nunits); };
    if (a.D == 128) {
      if (bf) once ? sums(blocksum_kernel<MIXKV_BF16, 128, true>) : sums(blocksum_kernel<MIXKV_BF16, 128, false>);
      else once ? sums(blocksum_kernel<MIXKV_F32, 128, true>) : sums(blocksum_kernel<MIXKV_F32, 128, false>);
      hipLaunchKernelGGL(blockgram_kernel<128>, grid_b, dim3(kMapThreads), 0, stream, a, to, Sg, dg, nunits);
    } else {
      if (bf) once ? sums(blocksum_kernel<MIXKV_BF16, 64, true>) : sums(blocksum_kernel<MIXKV_BF16, 64, false>);
      else once ? sums(blocksum_kernel<MIXKV_F32, 64, true>) : sums(blocksum_kernel<MIXKV_F32, 64, false>);
      hipLaunchKernelGGL(blockgram_kernel<64>, grid_b, dim3(kMapThreads), 0, stream, a, to, Sg, dg, nunits);
    }
    if (hipGetLastError() != hipSuccess) return MIXKV_ERR_HIP;
  }
  return MIXKV_OK;
}

}  // extern "C"
