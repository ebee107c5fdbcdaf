// The second pass over long bf16 caches with the keys in registers and the window queries in LDS.
//
// attn_kernel keeps the queries in registers and walks a key tile with all waves of a workgroup, a barrier per tile and two matrix
// instructions per fragment read from LDS.  Here a wave takes 64 keys of its own into registers, and every fragment of a query tile that
// it reads from LDS serves both of its key tiles; column sums are complete inside the wave, and nothing crosses waves until the run ends.
// Any number of query tiles, a loop, shares one kernel.
//   * The keys come through a private 32-row LDS image per wave (direct-to-LDS loads, whole rows): one of the block's two tiles waits in
//     registers, the other is asked for as soon as its predecessor has been read, half a block ahead.  Straight from memory in fragment form
//     (32-byte pieces) the pass reads 4.3 TB/s, through the image 4.9.
//   * Blocks are walked from a run's last to its first: the first pass read those last, and the caches may still hold them (1 % of a call).
//   * K_i . Kbar: 16x16x32 matrix instructions on the same key fragments (half the cost of a 32-row tile): a fragment's lanes 0-15 and
//     16-31 are two groups of keys, told apart by the contraction group, so the mean key's rows are zero for the other group's.
//   * Keys on the output rows: a lane follows one query row, whose offset is one register (with queries on the rows it took four LDS reads per
//     query tile, a third of all), and adds up its 32 keys over the tiles; 32 registers of 32 lanes meet once per block.
//   * The matrix instructions run half a tile ahead of the weights, an eighth (D = 64: a quarter) of them beside each: fma, exp2 and add of a
//     half tile are issued while the next half's scores are formed.
//   * Query rows lie a piece apart in LDS, so that a tile's fragments are one address and immediates.
// Bound: issue, at the clock that the card's power leaves.  448 heads of 32768 keys, 7 query tiles: 1.61 GHz (a copy runs at 2.37); of the
// SIMDs' clocks the matrix units are busy in 54 %, the vector units in 70 %, one or the other in 90 %; 3.8 GB from memory at 3.9 TB/s.
// The same launch, us: queries on the rows, matrix and vector work taking turns 993; keys on the rows 973;
// half a tile ahead 909 (2649 -> 2595 the call: the card holds its power, and the first pass then runs 1 % slower).  28 chunks of
// 128 keys per compute unit: 8 tiles 88.8 -> 79.4, 7 82.0 -> 78.1, 4 58.7 -> 55.9, 3 54.9 -> 55.2; 64-element heads, 16 tiles 97.5 -> 89.0, 4
// 40.2 -> 37.9.
// attn_kernel -> the first of these, us, alone on the chip, 7 query tiles and 224 heads of 32768 keys 535 -> 505, 4 tiles and 256 heads of
// 16384 keys 248 -> 214, 2 tiles and 224 heads of 8192 keys 120 -> 90.
// Not better: three waves per SIMD, blocks dealt by a counter (the younger wave of a SIMD ends later, but the time is the same), four key
// tiles a wave (no registers left for the next).
#include "mixkv_stream.h"

namespace mixkv {

constexpr int kKstWaves = 8, kKstThreads = kKstWaves * 64;

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Wait for everything this wave has in flight towards its image; nothing that reads the image moves up past it.
__device__ __forceinline__ void image_landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// The image's reads have reached registers: it may be requested anew.
__device__ __forceinline__ void image_read() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Sum over 32 lanes of each of 32 registers: lane l (of each half of the wave) gets register l's.  Every step adds the two lanes of a pair
// and keeps half of the registers in either lane.
__device__ __forceinline__ float sum_over_lanes(float (&v)[32], int lane) {
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[j]), __float_as_uint(v[j + 16]), false, false);
    v[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  auto step = [&](auto ctrl_c, auto half_c) {
    constexpr int CTRL = decltype(ctrl_c)::value, H = decltype(half_c)::value;
    const bool upper = (lane & H) != 0;
#pragma unroll
    for (int j = 0; j < H; ++j) {
      const float a = v[j] + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[j]), CTRL, 0xf, 0xf, true));
      const float b = v[j + H] + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[j + H]), CTRL, 0xf, 0xf, true));
      v[j] = upper ? b : a;
    }
  };
  step(std::integral_constant<int, 0x140>{}, std::integral_constant<int, 8>{});   // row_mirror
  step(std::integral_constant<int, 0x141>{}, std::integral_constant<int, 4>{});   // row_half_mirror
  step(std::integral_constant<int, 0x4E>{}, std::integral_constant<int, 2>{});    // quad_perm [2,3,0,1]
  step(std::integral_constant<int, 0xB1>{}, std::integral_constant<int, 1>{});    // quad_perm [1,0,3,2]
  return v[0];
}

template <int D, int QTMAX, bool ONCE>
__global__ __launch_bounds__(kKstThreads, 2) void kst_attn_kernel(Shape s, LayerInTable in, char *ws, Workspace w, int64_t unit0,
                                                                  int nunits, int nblk) {
  constexpr int DT = MIXKV_BF16, EB = 2, NCHK = D / 16, PPR = D / 8, TILE = 32 * PPR, BK = 64;
  constexpr int PITCH = PPR + 1;                       // query rows in LDS, in 16-byte pieces: a piece apart, so that rows meet in no bank
  __shared__ uint4 q_s[QTMAX * 32 * PITCH];            // window queries
  __shared__ uint4 img_s[kKstWaves * TILE];            // one key tile per wave on its way to registers
  __shared__ float nb_s[QTMAX * 32];                   // exponent offsets -b_r
  __shared__ int lim_s[QTMAX * 32];                    // last key each query row attends to
  __shared__ uint4 kb_s[NCHK * 8];                     // mean key: bf16 head and remainder; then zeros
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = s.N, Nc = s.Nc, Npad = s.Npad, QT = s.QT;
  const float c2 = s.scale_log2e;
  const int free_limit = s.causal ? Nc : N - 1;
  const uint4 *img = img_s + wave * TILE;
  const uint32_t img_a = lds_base_of(img_s) + (uint32_t)wave * (TILE * 16);
  for (int r = tid; r < QTMAX * 32; r += kKstThreads) lim_s[r] = s.causal ? Nc + r % s.W : N - 1;
  for (int p = tid; p < NCHK * 4; p += kKstThreads) kb_s[NCHK * 4 + p] = make_uint4(0, 0, 0, 0);
  const int64_t T = (int64_t)nunits * nblk;
  int64_t item = wg_first_item(blockIdx.x, gridDim.x, T);
  const int64_t item_end = wg_first_item(blockIdx.x + 1, gridDim.x, T);
  // K_i . Kbar: row and contraction group of the 16x16x32 operand; lanes of another row or group read the zeros
  const int km = lane & 15, kg = lane >> 4;
  const bool kb_mine = (km >> 2) == (kg & 1) && (km & 2) == 0 && km < 8;
  const uint4 *kb_row = kb_s + (kb_mine ? (kg >> 1) * 2 + (km & 1) : NCHK * 4);
  const uint4 *q_row = q_s + l32 * PITCH + half;
  const int koff = (l32 >> 4) * 32 + 8 * ((l32 >> 2) & 3) + 4 * half + (l32 & 3);   // key of the block whose sum this lane ends with

  while (item < item_end) {
    const int ul = (int)(item / nblk), b0 = (int)(item - (int64_t)ul * nblk);
    const int nb = (int)min((int64_t)(nblk - b0), item_end - item);   // blocks of the run
    const int64_t unit = unit0 + ul;
    const UnitCoord uc = unit_coord(s, ul);
    const LayerIn L = in.l[uc.layer];
    const int64_t row_bytes = L.sn * EB;
    const char *Kb = reinterpret_cast<const char *>(L.K) + ((int64_t)uc.b * L.sb + (int64_t)uc.h * L.sh) * EB;
    const char *Qb = reinterpret_cast<const char *>(L.Q) + ((int64_t)(uc.b * s.hq + uc.h * s.G) * s.W * D) * EB;
    float *araw = reinterpret_cast<float *>(ws + w.araw) + unit * s.Npad;
    float *kdot = reinterpret_cast<float *>(ws + w.sdiv) + unit * s.Npad;
    const float *nbg = reinterpret_cast<const float *>(ws + w.nb) + unit * s.nb_rows;
    const uint4 *kbarp = reinterpret_cast<const uint4 *>(ws + w.kbarp) + unit * (NCHK * 4);

    // Request the key tile of rows [row0, row0 + 32) into the wave's image (rows past the last one repeat it).
    auto request = [&](int row0) {
      const int r0 = min(row0, N - 1);
      fetch_tile<DT, D, 1, ONCE>(Kb + r0 * row_bytes, row_bytes, r0, N, img_a, 0, lane);
    };
    auto take = [&](Frag (&k)[NCHK]) {
#pragma unroll
      for (int c = 0; c < NCHK; ++c) k[c].q = read_key_frag<DT, D>(img, 0, c, l32, half);
    };
    const int b9 = b0 + nb - 1;
    const int row_first = (b9 - min(wave, nb - 1)) * BK;
    lds_barrier();                                     // the previous run is done with LDS
    // the queries (rows past the last one repeat it: their offsets make their weights 0)
    constexpr int QL = QTMAX * TILE / kKstThreads;
    u32x4 qv[QL];
    int qtid = tid;
    asm volatile("" : "+v"(qtid));                     // the pieces' addresses are formed here, once per run, and hold no registers elsewhere
#pragma unroll
    for (int j = 0; j < QL; ++j) {
      const int p = j * kKstThreads + qtid;
      qv[j] = load_vec<false>(Qb + (int64_t)min(p / PPR, s.GW - 1) * (D * EB) + (p % PPR) * 16);
    }
#pragma unroll
    for (int j = 0; j < QL; ++j) {
      const int p = j * kKstThreads + qtid;
      *reinterpret_cast<u32x4 *>(q_s + (p / PPR) * PITCH + p % PPR) = qv[j];
    }
    for (int r = tid; r < QT * 32; r += kKstThreads) nb_s[r] = nbg[r];
    for (int p = tid; p < NCHK * 4; p += kKstThreads) kb_s[p] = kbarp[p];
    request(row_first);
    image_landed();
    lds_barrier();
    // The results of a block are stored at the start of the wave's next one, in front of its requests: the waits for the
    // image then find them long finished.
    int tbp = Npad;                                    // first key of the block whose results are held (none yet)
    float csp = 0.f, kdp[2];
    auto store = [&] {
      if (tbp + koff < Nc) araw[tbp + koff] = csp;
      if (half == 0 && tbp + l32 < Nc) kdot[tbp + l32] = kdp[0];
      if (half == 0 && tbp + 32 + l32 < Nc) kdot[tbp + 32 + l32] = kdp[1];
    };
    Frag kn[NCHK], kf[2][NCHK], qf[NCHK];
    take(kn);
    image_read();
    request(row_first + 32);
    const int qm = QT / 2;
    constexpr int EPS = 16 / NCHK;                     // weights beside one matrix instruction
    f32x16 acc[2];
    auto q_frag = [&](int q, int c) { return q_row[q * (32 * PITCH) + c * 2]; };
    // The chain of matrix instructions runs one half tile (32 keys x 32 queries) ahead of the weights.
#pragma unroll
    for (int c = 0; c < NCHK; ++c) qf[c].q = q_frag(0, c);
    float nbq = nb_s[l32], nbn = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[0][i] = 0.f;
#pragma unroll
    for (int c = 0; c < NCHK; ++c) acc[0] = mma<DT>(kn[c], qf[c], acc[0]);

    for (int blk = wave; blk < nb; blk += kKstWaves) {
      const int tb = (b9 - blk) * BK;
      const int nxt = (b9 - min(blk + kKstWaves, nb - 1)) * BK;
#pragma unroll
      for (int c = 0; c < NCHK; ++c) kf[0][c] = kn[c];
      image_landed();
      take(kf[1]);
      image_read();
      store();
      request(nxt);
      const bool masked = tb + BK - 1 > free_limit;

      // ---- K_i . Kbar: rows 0, 1 (head, remainder) belong to keys 0-15 of a tile, rows 4, 5 to keys 16-31
      {
        f32x4 kacc[2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) kacc[t][i] = 0.f;
#pragma unroll
        for (int c = 0; c < NCHK; ++c) {
          Frag a;
          a.q = kb_row[c * 4];
#pragma unroll
          for (int t = 0; t < 2; ++t) kacc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, kf[t][c].h, kacc[t], 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) kdp[t] = kacc[t][0] + kacc[t][1];
      }

      float cs[32];
#pragma unroll
      for (int i = 0; i < 32; ++i) cs[i] = 0.f;
      // Keys on the output rows: a lane follows one query row and adds up each of its 32 keys over the query tiles.  Weights of the tile on
      // the first 32 keys, one slice beside each matrix instruction of the second 32; tile qn's fragments follow the old ones.
      auto first = [&](int qn) {
        __builtin_amdgcn_sched_barrier(0);
        nbn = nb_s[qn * 32 + l32];
#pragma unroll
        for (int c = 0; c < NCHK; ++c) {
          if (c == 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[1][i] = 0.f;
          }
          acc[1] = mma<DT>(kf[1][c], qf[c], acc[1]);
          qf[c].q = q_frag(qn, c);
#pragma unroll
          for (int i = c * EPS; i < (c + 1) * EPS; ++i) cs[i] += fast_exp2(fmaf(acc[0][i], c2, nbq));
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      // Weights of the second 32 keys beside the next tile's first (of these keys, or the wave's next block).
      auto second = [&](const Frag (&k)[NCHK]) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < NCHK; ++c) {
          if (c == 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[0][i] = 0.f;
          }
          acc[0] = mma<DT>(k[c], qf[c], acc[0]);
#pragma unroll
          for (int i = c * EPS; i < (c + 1) * EPS; ++i) cs[16 + i] += fast_exp2(fmaf(acc[1][i], c2, nbq));
          __builtin_amdgcn_sched_barrier(0);
        }
        nbq = nbn;
      };
      if (!masked) {
        for (int q = 0; q < qm; ++q) { first(q + 1); second(kf[0]); }
        image_landed();
        take(kn);
        image_read();
        request(nxt + 32);
        for (int q = qm; q < QT - 1; ++q) { first(q + 1); second(kf[0]); }
        first(0);
        second(kn);
      } else {
        // a block that reaches into the window or past the last key: no overlap, the next block's first scores at the end
        image_landed();
        take(kn);
        image_read();
        request(nxt + 32);
        for (int q = 0; q < QT; ++q) {
          const float nbm = nb_s[q * 32 + l32];
          const int lim = lim_s[q * 32 + l32] - tb - 4 * half;
#pragma unroll
          for (int c = 0; c < NCHK; ++c) qf[c].q = q_frag(q, c);
#pragma unroll
          for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[0][i] = 0.f;
#pragma unroll
            for (int c = 0; c < NCHK; ++c) acc[0] = mma<DT>(kf[t][c], qf[c], acc[0]);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const float x = (t * 32 + 8 * (i >> 2) + (i & 3) <= lim) ? acc[0][i] : -INFINITY;
              cs[t * 16 + i] += fast_exp2(fmaf(x, c2, nbm));
            }
          }
        }
#pragma unroll
        for (int c = 0; c < NCHK; ++c) qf[c].q = q_frag(0, c);
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[0][i] = 0.f;
#pragma unroll
        for (int c = 0; c < NCHK; ++c) acc[0] = mma<DT>(kn[c], qf[c], acc[0]);
      }
      csp = sum_over_lanes(cs, lane);
      tbp = tb;
    }
    store();
    image_landed();                                    // requests past the run's last block are unused, but must not land later
    item += nb;
  }
}

// The lines below were drawn for an earlier form of this kernel (queries on the output rows); the figures are of the kernel as it is, each of a
// call for the scores.  Where it is taken it is at most 6 % behind attn_kernel (the shortest heads of a line, 16 to 24 chunks per compute unit); the
// lines leave up to 9 % at short heads (64 elements, 9 tiles, 384 keys), more only under the limit for the last round.
// From sixteen 128-key chunks per compute unit on (64 KB of queries are staged per workgroup and run): 7 query tiles, 8192 keys per
// head, attn_kernel -> this, us: 3.5 chunks per unit 54 -> 55, 8 chunks 71 -> 73, 14 chunks 121 -> 117, 40 chunks 261 -> 257; 4 query tiles: 3.5
// chunks 47 -> 48, 8 chunks 62 -> 62, 14 chunks 101 -> 98, 40 chunks 224 -> 214.
// A wave takes whole 64-key blocks: not where the last round of them would leave more than a tenth of the time idle (112 heads of 7013 keys,
// 7 tiles, 6.02 blocks a wave: 175 us with either; 18 chunks per compute unit, 4.5 blocks a wave, heads of 2048 keys and more: 8 tiles 1.06 times
// as fast as attn_kernel, 2 to 7 tiles 0.99 to 1.05; 64 elements, 9 to 16 tiles 1.10 to 1.22, 3 to 8 tiles 1.02 to 1.09).
// A run ends with its head, so that short heads pay the staging and a last round of the eight waves again and again: time of a call with
// attn_kernel over that with this, 16 to 56 chunks per compute unit in whole rounds, by keys per head:
//   128 elements   512          1024         1536         2048         4096         8192
//     8 tiles      0.97-0.98    0.97-1.01    0.99-1.05    1.04-1.05    1.06         1.06-1.08
//     7            0.88-0.92    0.92-0.95    0.93-1.00    0.99-1.01    1.01-1.02    1.02-1.04
//     4 to 6       0.88-0.96    0.91-1.00    0.94-1.03    1.00-1.06    0.99-1.07    1.01-1.08
//     2, 3         0.90-0.96    0.90-1.01    0.95-1.01    0.97-1.03    0.97-1.03    0.97-1.03 (below 24 chunks 0.97-0.98)
//   64 elements
//     9 to 16      1.07-1.17    1.07-1.18    1.07-1.23    1.09-1.24    1.10-1.23    1.11-1.24 (384 keys 0.95-1.09)
//     3 to 8       0.89-0.96    0.95-1.01    0.94-1.04    1.01-1.07    1.01-1.06    1.02-1.07
// Between those lengths the last round counts (blocks of 64 keys a head; 20, 28, 40, 56 chunks per compute unit):
//   64 elements, 16 tiles: 9 blocks 1.02 0.99 1.01 1.01; 10 1.03 1.02 1.03 1.03; 11 1.05 1.02 1.06 1.06; 17 1.07 1.06 1.08 1.08
//     13 tiles: 9 blocks 1.04 1.01 1.03 1.04; 10 1.05 1.04 1.05 1.05; 12 tiles: 9 blocks 1.06 1.03 1.05 1.05; 9 tiles: 9 blocks 1.13 1.08 1.11 1.12
//   128 elements, 6 tiles: 25 blocks 1.00 0.99 0.99 1.00; 28 0.98 1.00 1.01 1.01; 30 0.97 0.98 0.99 1.01; 31 0.98 0.99 1.01 1.01
//     4 and 5 tiles: 25 and 28 blocks 0.98-1.04
// (attn_kernel computes whole slots of 4, 8 or 16 query tiles, and the mean key costs it extra where none is spare: 4, 8, 16.)
bool keystat_supported(const Shape &s, int dtype, int nunits, int num_cus) {
  if (dtype != MIXKV_BF16 || s.QT > (s.D == 128 ? 8 : 16)) return false;
  const int head = (s.N + 63) / 64;                    // blocks of a head
  const bool few = s.D == 128 && s.QT <= 3;
  const int least = s.D == 64 ? (s.QT > 8 ? 8 : 24) : (few || s.QT == 7) ? 64 : s.QT == 8 ? 16 : 24;
  const bool idle_round = s.D == 64 && ((head == 9 && s.QT > 12) || (head == 10 && s.QT > 14));
  const int chunks = few ? 24 : (s.D == 128 && s.QT == 6 && head < 31) ? 32 : 16;    // per compute unit
  if (head < least || idle_round || (int64_t)nunits * s.nchunks < chunks * (int64_t)num_cus) return false;
  const int64_t blocks = (int64_t)nunits * head, waves = (int64_t)num_cus * kKstWaves, rounds = (blocks + waves - 1) / waves;
  return 10 * rounds * waves <= 11 * blocks;
}

hipError_t launch_kst_attn(const Shape &s, const LayerInTable &in, char *ws, const Workspace &w, int64_t unit0, int nunits, int num_cus,
                           hipStream_t st) {
  const int nblk = (s.N + 63) / 64;
  const int64_t T = (int64_t)nunits * nblk, cap = (int64_t)num_cus;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)(T < cap ? T : cap)), dim3(kKstThreads), 0, st, s, in, ws, w, unit0, nunits, nblk);
    return hipGetLastError();
  };
  const bool once = pass_once(s, MIXKV_BF16, nunits);
  if (s.D == 128) return once ? go(kst_attn_kernel<128, 8, true>) : go(kst_attn_kernel<128, 8, false>);
  return once ? go(kst_attn_kernel<64, 16, true>) : go(kst_attn_kernel<64, 16, false>);
}

}  // namespace mixkv
