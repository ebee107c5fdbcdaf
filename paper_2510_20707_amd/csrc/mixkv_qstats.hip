// The first pass over long bf16 caches with five to eight query tiles: two waves hold all window queries in registers.
//
// stats_kernel gives each of eight waves one query tile, so every wave reads the whole key tile from LDS: 64 of the 96 KB of LDS traffic per tile,
// and the card runs both passes below its clock (1.6 to 1.8 of 2.4 GHz here).  Here a wave
// holds three or four tiles (96 to 128 registers), a fragment read serves as many matrix instructions, and the norms come from registers:
//   * 1 / |K_i| from the score fragments (a lane has half a row), on the wave with fewer query tiles or on both in turn;
//   * the sum of normalised keys on the matrix cores: 1 / |K_i| as three bf16 addends (exact: 24 bits) times the keys, read transposed
//     from the tile image (ds_read_b64_tr_b16), eight small instructions and no vector work where stats_kernel takes 16 per 16 bytes;
//   * value rows through a private image per wave, four lanes to a row.
// A tile step: the key tile was asked for two steps ahead, the value rows one; requests, waits and LDS accesses are written out (see lds_read8).
// Bound: 448 heads of 32768 keys, 7 tiles: 1.81 GHz; the matrix units busy in 31 % of the SIMDs' clocks, the vector units in 52 %, one or the
// other in 75 %; 7.6 GB at 4.9 TB/s; bank conflicts in 30 % of the LDS cycles.
// 244 registers, 34 KB of LDS: four workgroups per compute unit.  First pass of 224 heads of 32768 keys, 7 tiles: 820 -> 740 us (stats_kernel
// with non-temporal loads 794 to 828); without its requests 506 to 590, without its arithmetic 757 with plain loads.
#include "mixkv_stream.h"

namespace mixkv {

constexpr int kQsWaves = 2, kQsThreads = kQsWaves * 64;

typedef float f32x4 __attribute__((ext_vector_type(4)));

// The value, unknown to the compiler: what is computed from it inside a loop stays there instead of holding a register
// for each of its results through the loop.
__device__ __forceinline__ int opaque(int x) { asm volatile("" : "+v"(x)); return x; }

// Sum of a value over the two halves of the wave, and over the two rows of 16 lanes of each half, in every lane.
__device__ __forceinline__ float add_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_rows(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// LDS accesses of the tile loop.  The compiler makes every LDS access that it sees wait for all direct-to-LDS loads in flight, which
// would end the requests' lead, so these are written out, each group of reads with its wait.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void lds_read8(u32x4 (&t)[8], uint32_t p0, uint32_t p1, uint32_t p2, uint32_t p3, uint32_t p4, uint32_t p5,
                                          uint32_t p6, uint32_t p7) {
  asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
               "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]), "=&v"(t[6]), "=&v"(t[7])
               : "v"(p0), "v"(p1), "v"(p2), "v"(p3), "v"(p4), "v"(p5), "v"(p6), "v"(p7) : "memory");
}
__device__ __forceinline__ void lds_read4(u32x4 (&t)[4], uint32_t p0, uint32_t p1, uint32_t p2, uint32_t p3) {
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]) : "v"(p0), "v"(p1), "v"(p2), "v"(p3) : "memory");
}
// Two 16-byte pieces and eight transposed 8-byte reads: of four blocks the contraction's first half at x, the second 1024 bytes past y.
__device__ __forceinline__ void lds_read_tr(u32x4 (&a)[2], u32x2 (&f)[8], uint32_t pa, uint32_t pb, uint32_t x0, uint32_t y0, uint32_t x1,
                                            uint32_t y1, uint32_t x2, uint32_t y2, uint32_t x3, uint32_t y3) {
  asm volatile("ds_read_b128 %0, %10\n\tds_read_b64_tr_b16 %2, %12\n\tds_read_b64_tr_b16 %3, %13 offset:1024\n\t"
               "ds_read_b64_tr_b16 %4, %14\n\tds_read_b64_tr_b16 %5, %15 offset:1024\n\tds_read_b128 %1, %11\n\t"
               "ds_read_b64_tr_b16 %6, %16\n\tds_read_b64_tr_b16 %7, %17 offset:1024\n\t"
               "ds_read_b64_tr_b16 %8, %18\n\tds_read_b64_tr_b16 %9, %19 offset:1024\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(a[0]), "=&v"(a[1]), "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7])
               : "v"(pa), "v"(pb), "v"(x0), "v"(y0), "v"(x1), "v"(y1), "v"(x2), "v"(y2), "v"(x3), "v"(y3) : "memory");
}
// Sum of squares over pieces, four chains.
template <int DT, int NP>
__device__ __forceinline__ float pieces_sumsq(const u32x4 (&t)[NP]) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < NP; ++c)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t u = t[c][j];
      const bf16x2 v = __builtin_bit_cast(bf16x2, u);
      s[j] = __builtin_amdgcn_fdot2_f32_bf16(v, v, s[j], false);
    }
  return (s[0] + s[1]) + (s[2] + s[3]);
}
__device__ __forceinline__ void lds_write16(uint32_t p, uint32_t x, uint32_t y) {   // 16 bits at p and at p + 64
  asm volatile("ds_write_b16 %0, %1\n\tds_write_b16 %0, %2 offset:64" :: "v"(p), "v"(x), "v"(y) : "memory");
}

template <int TQ, bool ONCE>
__global__ __launch_bounds__(kQsThreads, 2) void qs_stats_kernel(Shape s, LayerInTable in, char *ws, Workspace w, int64_t unit0,
                                                                 int nunits, int64_t slot0) {
  constexpr int D = 128, WV = kQsWaves, DT = MIXKV_BF16, EB = 2, NCHK = D / 16, PPR = D / 8, TILE = 32 * PPR, KT = chunk_tiles(DT, D);
  constexpr int RING = 3, NB = D / 16;
  constexpr int RPL = 64 / PPR, KL = TILE / 64 / WV;      // rows per load; key loads per wave and tile
  constexpr int VR = 32 / WV, VL = VR * PPR / 64;         // value rows and loads per wave and tile
  __shared__ __align__(1024) uint4 kring[RING * TILE];
  __shared__ __align__(1024) uint4 vimg_s[WV * VR * PPR];               // each wave's value rows of one tile
  __shared__ float ks_s[WV * D];
  __shared__ __align__(256) uint16_t parts_s[WV][4 * 32]; // 1 / |K_i| of a tile as three bf16 addends, and a row of zeros

  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = s.N, Nc = s.Nc, QTR = s.QT * 32;
  const float c2 = s.scale_log2e;
  const int free_limit = s.causal ? Nc : N - 1;
  const int nq = max(0, min(TQ, s.QT - wv * TQ));
  const bool use_v = s.intrinsic == MIXKV_INTRINSIC_VNORM, use_k = s.kstats != 0;
  const uint32_t ring_a = lds_base_of(kring);
  const uint32_t vimg_a = lds_base_of(vimg_s) + (uint32_t)wv * (VR * PPR * 16);
  const uint32_t parts_a = lds_base_of(parts_s) + (uint32_t)wv * 256;
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
    const int key0 = c0 * KT * 32;
    const int nt = min(nit * KT, (N - key0 + 31) / 32);              // tiles of the run
    const char *Kb = reinterpret_cast<const char *>(L.K) + head_off;
    const char *Vb = reinterpret_cast<const char *>(L.V) + head_off;
    const char *Qb = reinterpret_cast<const char *>(L.Q) + ((int64_t)(uc.b * s.hq + uc.h * s.G) * s.W * D) * EB;
    float *invnorm = reinterpret_cast<float *>(ws + w.invnorm) + unit * s.Npad;
    float *vnorm = reinterpret_cast<float *>(ws + w.vnorm) + unit * s.Npad;
    auto tile_row = [&](int i) { return key0 + min(i, nt - 1) * 32; };   // past its last tile the run asks for that one again

    // This wave's share of the group's key tile i into ring image `slot`, and its value rows of tile i.  A whole tile is a uniform
    // address per load plus a lane offset; the last tile of a head repeats its last row.
    const uint32_t rb = (uint32_t)row_bytes, lrow = lane / PPR, lq = lane % PPR;
    auto request = [&](int i, int slot) {
      const int tb = tile_row(i), last = N - 1 - tb;
      const char *tile = Kb + tb * row_bytes;
      const uint32_t dst = ring_a + slot * (TILE * 16);
      const uint32_t ln = (uint32_t)opaque(tid) & 63, row0 = ln / PPR, pc = ln % PPR;
      if (last >= 31) {
#pragma unroll
        for (int jj = 0; jj < KL; ++jj) {
          const int j = jj * WV + wv;
          const uint32_t off = row0 * rb + (pc ^ (uint32_t)tile_swz<DT, D>(j * RPL + row0)) * 16;
          load_to_lds<ONCE>(tile + (int64_t)(j * RPL) * row_bytes + off, dst + j * 1024);
        }
      } else {
#pragma unroll
        for (int jj = 0; jj < KL; ++jj) {
          const int j = jj * WV + wv;
          const uint32_t off = (uint32_t)min((int)(j * RPL + row0), last) * rb + (pc ^ (uint32_t)tile_swz<DT, D>(j * RPL + row0)) * 16;
          load_to_lds<ONCE>(tile + off, dst + j * 1024);
        }
      }
    };
    auto request_v = [&](int i) {
      const int tb = tile_row(i) + wv * VR, last = N - 1 - tb;
      if (last >= VR - 1) {
        const char *tile = Vb + tb * row_bytes;
#pragma unroll
        for (int j = 0; j < VL; ++j)
          load_to_lds<ONCE>(tile + (int64_t)(j * RPL) * row_bytes + (lrow * rb + lq * 16), vimg_a + j * 1024);
      } else {
        const char *tile = Vb + (tb + min(last, 0)) * row_bytes;      // (a wave whose rows all lie past the last one repeats that one)
#pragma unroll
        for (int j = 0; j < VL; ++j)
          load_to_lds<ONCE>(tile + ((uint32_t)min((int)(j * RPL + lrow), max(last, 0)) * rb + lq * 16), vimg_a + j * 1024);
      }
    };
    lds_barrier();                                     // the previous run is done with LDS
    request(0, 0);
    request(1, 1);
    Frag qf[TQ][NCHK];
    float m[TQ], l[TQ];
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
      const int row = (wv * TQ + q) * 32 + l32;
      const bool live = row < s.GW;
      const char *qrow = Qb + ((int64_t)(live ? row : 0) * D) * EB + half * 16;
#pragma unroll
      for (int c = 0; c < NCHK; ++c) {
        const uint4 v = *reinterpret_cast<const uint4 *>(qrow + c * 32);
        qf[q][c].q = live ? v : make_uint4(0, 0, 0, 0);
      }
      m[q] = -INFINITY;
      l[q] = 0.f;
    }
    wait_vm<0>();
    if (use_v) request_v(0);
    f32x4 ks[NB / 4], ks_total[NB / 4];                                  // sum of normalised keys: element b * 16 + lane % 16 on lane group b % 4
#pragma unroll
    for (int b = 0; b < NB / 4; ++b) ks[b] = ks_total[b] = f32x4{0.f, 0.f, 0.f, 0.f};

    int slot = 0;
    for (int i = 0; i < nt; ++i) {
      const int tb = key0 + i * 32;
      const uint32_t img_a = ring_a + slot * (TILE * 16);
      lds_barrier();                                   // tile i has landed for both waves, tile i - 1 is read
      request(i + 2, slot == 0 ? 2 : slot - 1);
      const int ol = opaque(tid) & 63;
      Frag kf[NCHK];
      u32x4 kt[NCHK];
      {
        // piece 2c + half of row r sits at piece (2c + half) ^ swz(r) of its 256-byte row: one exclusive-or per chunk
        const uint32_t r = ol & 31, p = img_a + r * 256 + (((uint32_t)ol >> 5) ^ (uint32_t)tile_swz<DT, D>(r)) * 16;
        lds_read8(kt, p, p ^ 32, p ^ 64, p ^ 96, p ^ 128, p ^ 160, p ^ 192, p ^ 224);
#pragma unroll
        for (int c = 0; c < NCHK; ++c) kf[c].h = __builtin_bit_cast(bf16x8, kt[c]);
      }

      // ---- key norms and the sum of normalised keys
      float inv_mine = -1.f;                           // stored behind the wait for the value rows
      const bool norms = use_k && ((s.QT & 1) ? wv == WV - 1 : (i & 1) == wv);   // the wave with fewer query tiles, else in turn
      if (norms) {
        float ss = pieces_sumsq<DT, NCHK>(kt);
        ss = add_halves(ss);
        const bool valid = tb + l32 < N;
        const float inv = valid ? inv_norm<DT>(ss) : 0.f;
        inv_mine = valid && half == 0 ? inv : -1.f;
        const uint32_t hi = __float_as_uint(inv) & 0xffff0000u;
        const float r1 = inv - __uint_as_float(hi);
        const uint32_t mid = __float_as_uint(r1) & 0xffff0000u;
        const uint32_t lo = __float_as_uint(r1 - __uint_as_float(mid));
        lds_write16(parts_a + (half * 64 + l32) * 2, (half ? lo : hi) >> 16, half ? 0 : mid >> 16);
      }
      // The sum: addends times keys on the matrix cores, the keys read transposed from the image.  Blocks of 16 elements, four to a set
      // of accumulators: block b's addends go to the output rows of lane group b % 4.
      auto key_sum = [&] {
        static_assert(NB == 8, "two blocks per set of addends");
        const int mm = ol & 15, kg = ol >> 4;
        // lane mm of group kg reads row kg * 8 + mm / 4 (and 4 rows further), elements (mm % 4) * 4 of a block
        const uint32_t r0 = kg * 8 + (mm >> 2);
        const uint32_t t0 = img_a + r0 * 256 + ((((uint32_t)mm & 3) >> 1) ^ (uint32_t)tile_swz<DT, D>(r0)) * 16 + (mm & 1) * 8;
        auto pa = [&](int b4) { return parts_a + ((mm >> 2) == b4 ? mm & 3 : 3) * 64 + kg * 16; };
        auto x = [&](int b) { return t0 ^ (uint32_t)(b * 32); };
        auto y = [&](int b) { return t0 ^ (uint32_t)(b * 32) ^ 64u; };   // rows r0 + 4: the rotation's third bit is set
#pragma unroll
        for (int b = 0; b < 4; b += 2) {
          u32x4 a[2];
          u32x2 f[8];
          lds_read_tr(a, f, pa(b), pa(b + 1), x(b), y(b), x(b + 4), y(b + 4), x(b + 1), y(b + 1), x(b + 5), y(b + 5));
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const u32x4 fb = {f[4 * j + 2 * h].x, f[4 * j + 2 * h].y, f[4 * j + 2 * h + 1].x, f[4 * j + 2 * h + 1].y};
              ks[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[j]), __builtin_bit_cast(bf16x8, fb), ks[h], 0, 0, 0);
            }
        }
      };

      // ---- softmax statistics (see stats_kernel): keys on the output rows, the lane follows its query rows
#pragma unroll
      for (int q = 0; q < TQ; ++q) {
        if (q >= nq) break;
        f32x16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
        for (int c = 0; c < NCHK; ++c) acc = mma<DT>(kf[c], qf[q][c], acc);
        if (tb + 31 > free_limit) {                    // tile reaches into the window or past N: mask
          const int lim = s.causal ? Nc + ((wv * TQ + q) * 32 + (ol & 31)) % s.W : N - 1;   // last key the row attends to
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[e] = (tb + 8 * (e >> 2) + 4 * (ol >> 5) + (e & 3) > lim) ? -INFINITY : acc[e];
        }
        const float nmu = -m[q];
        float sum[4];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float term = fast_exp2(fmaf(acc[e], c2, nmu));
          sum[e & 3] = e < 4 ? term : sum[e & 3] + term;
        }
        float lnew = l[q] + ((sum[0] + sum[1]) + (sum[2] + sum[3]));
        if (__builtin_amdgcn_ballot_w64(!(lnew < kSumLimit)) != 0) {
          float tmax = fmaxf(acc[0], acc[1]);
#pragma unroll
          for (int e = 2; e < 16; e += 2) tmax = fmaxf(fmaxf(tmax, acc[e]), acc[e + 1]);
          const float mn = fmaxf(m[q], tmax * c2);
          const float mu = (mn == -INFINITY) ? 0.f : mn;
          float s2[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int e = 0; e < 16; ++e) s2[e & 3] += fast_exp2(fmaf(acc[e], c2, -mu));
          lnew = l[q] * fast_exp2(m[q] - mu) + ((s2[0] + s2[1]) + (s2[2] + s2[3]));
          m[q] = mn;
        }
        l[q] = lnew;
      }
      if (norms) key_sum();
      if ((i & 15) == 15) {                            // in two levels: a single chain over the run rounds more than stats_kernel's many
#pragma unroll
        for (int b = 0; b < NB / 4; ++b) {
          ks_total[b] += ks[b];
          ks[b] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }

      // ---- value norms: lanes r, r + 16, r + 32 and r + 48 hold row r of a set of 16 (which piece a lane gets does not matter)
      float keep = 0.f;
      if (use_v) {
        wait_vm<KL>();                                 // since the value rows only a key tile has been asked for
        const uint32_t r = ol & 15, p = vimg_a + r * 256 + ((((uint32_t)ol >> 4) * 4) ^ r) * 16;
#pragma unroll
        for (int v = 0; v < VR / 16; ++v) {
          u32x4 t[4];
          lds_read4(t, p + v * 4096, (p ^ 16) + v * 4096, (p ^ 32) + v * 4096, (p ^ 48) + v * 4096);
          const float ss = add_halves(add_rows(pieces_sumsq<DT, 4>(t)));
          keep = (ol >> 4) == v ? ss : keep;
        }
        const int key = tb + wv * VR + (ol & 15) + (ol >> 4) * 16;
        if ((ol >> 4) < VR / 16 && key < Nc) vnorm[key] = __builtin_amdgcn_sqrtf(keep);
      } else {
        wait_vm<KL>();                                 // this wave's share of tile i + 1
      }
      if (inv_mine >= 0.f) invnorm[tb + l32] = inv_mine;
      if (use_v) request_v(i + 1);
      slot = slot + 1 == RING ? 0 : slot + 1;
    }
    wait_vm<0>();                                      // requests past the last tile are unused, but must not land later

    // ---- run partials
    const int64_t pslot = slot0 + blockIdx.x + ul;
    float2 *part_ml = reinterpret_cast<float2 *>(ws + w.part_ml) + pslot * QTR;
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
      int e;
      l[q] = frexpf(l[q], &e);                         // the sum may be far from 1: see stats_kernel
      m[q] += (float)e;
      ml_merge(m[q], l[q], __shfl_xor(m[q], 32), __shfl_xor(l[q], 32));
      if (q < nq && half == 0) part_ml[(wv * TQ + q) * 32 + l32] = make_float2(m[q], l[q]);
    }
#pragma unroll
    for (int b = 0; b < NB / 4; ++b) ks_s[wv * D + b * 64 + lane] = ((ks_total[b][0] + ks[b][0]) + (ks_total[b][1] + ks[b][1])) + (ks_total[b][2] + ks[b][2]);
    lds_barrier();
    float *part_ks = reinterpret_cast<float *>(ws + w.part_ksum) + pslot * D;
    for (int d = tid; d < D; d += kQsThreads) {
      float a = 0.f;
#pragma unroll
      for (int v = 0; v < WV; ++v) a += ks_s[v * D + d];   // fixed order
      part_ks[d] = a;
    }
    item += nit;
  }
}

// bf16 rows of 128 elements, 5 to 8 query tiles, from 32 chunks of 128 keys per compute unit on, row strides whose 32-row offsets fit 32
// bits.  stats_kernel -> this, whole calls: 448 heads of 32768 keys (7 tiles, 448 chunks per unit) 2705 -> 2612 us, 112 heads of
// 130688 2674 -> 2585; this pass alone, 224 heads of 8192 keys (5 tiles, 56 chunks) 215 to 230 -> 185 to 188; 112 and 128 heads of 8192 (7
// tiles, 28 and 32 chunks) the same call time, 14 chunks 62 to 72 -> 75 (a workgroup's queries go to registers once per run).
// Short heads, which end a run each, do not move the line: stats_kernel loads its queries as often.  Time of a call with stats_kernel over that
// with this, 32, 48 and 96 chunks per unit:
//   keys per head  256        384        512        768        1024       2048       4096       8192
//     5 tiles      1.04-1.08  1.04-1.05  1.05-1.09  1.02-1.05  0.99-1.03  0.99-1.00  1.00-1.05  0.98-1.02
//     6            1.04-1.09  1.02-1.04  1.06-1.07  1.05-1.08  1.04-1.09  1.01-1.04  1.01-1.03  1.00-1.03
//     7            1.04-1.07  1.01-1.06  1.05-1.06  1.02-1.06  1.04-1.07  1.02-1.04  1.03-1.04  1.01-1.03
//     8            1.05-1.07  1.01-1.05  1.06-1.07  1.02-1.05  1.04       1.02-1.04  1.02-1.03  1.00-1.04
// With up to four tiles one wave would hold all of them: 256 heads of 16384 keys 662 -> 669 us a call.
bool qstats_supported(const Shape &s, int dtype, int nunits, int num_cus, int64_t max_stride_n) {
  return dtype == MIXKV_BF16 && s.D == 128 && s.QT >= 5 && s.QT <= 8 && (int64_t)nunits * s.nchunks >= 32 * (int64_t)num_cus &&
         max_stride_n < (int64_t)1 << 25;
}

// Four workgroups of two waves per compute unit.
int qstats_grid(const Shape &s, int nunits, int num_cus) {
  const int64_t T = (int64_t)nunits * s.nchunks;
  int64_t cap = (int64_t)num_cus * 4;
  if (cap > kMaxStreamGrid) cap = kMaxStreamGrid;
  return (int)(T < cap ? T : cap);
}

hipError_t launch_qstats(const Shape &s, const LayerInTable &in, char *ws, const Workspace &w, int64_t unit0, int nunits, int grid,
                         int64_t slot0, hipStream_t st) {
  const bool once = pass_once(s, MIXKV_BF16, nunits);
  auto kern = s.QT > 6 ? (once ? qs_stats_kernel<4, true> : qs_stats_kernel<4, false>) : (once ? qs_stats_kernel<3, true> : qs_stats_kernel<3, false>);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kQsThreads), 0, st, s, in, ws, w, unit0, nunits, slot0);
  return hipGetLastError();
}

}  // namespace mixkv
