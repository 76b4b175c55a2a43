// Compression-side assignment step (paper section 4.2, steps 1 and 3 of the post-training
// procedure): every edge's grid of G = 10 coefficients is normalised - its mean becomes the
// bias, the norm of the centred grid the gain - and assigned to the nearest of the K
// codebook shapes.  (Learning the shapes, step 2, is not part of this library.)
//
// Nearest centroid = largest score s(e, k) = n_e . C_k - |C_k|^2 / 2, a dense
// [K x 10] x [10 x E] contraction: it runs on the matrix cores.  To keep the decision at
// fp32 quality with fp16 operands, both operands are split into a high and a low fp16 part
// and the contraction runs over 32 slots (two v_mfma_f32_32x32x16_f16 per 32 x 32 tile):
//     shape  [ hi(C) (10) | hi(-|C|^2/2) | lo(C) 0..4 ]   [ lo(C) 5..9 | hi(C) (10) | lo(-|C|^2/2) ]
//     edge   [ hi(n) (10) |      1       | hi(n) 0..4 ]   [ hi(n) 5..9 | lo(n) (10) |      1       ]
// (the dropped lo x lo term is ~1e-7 of the score).  Centroids are the MFMA rows and edges
// the columns, so a lane owns one edge and 16 of the 32 centroids of a tile: the running
// maximum over centroids never crosses lanes until the very end.
//
// The arg-max costs vector instructions per score, which is what would bound the kernel, so the
// common case is kept to half an instruction per score: the maximum of a lane's 16 scores of a
// tile is 8 three-input maxima, and only when it beats the lane's running best - the t-th tile
// does so with probability ~1/t - is the row looked up.  Exactly equal scores (duplicate shapes)
// resolve to the lower index within a half-wave's rows; which of two half-waves' equal scores
// wins is decided by index at the end.

// That is the whole search (kan_assign_whole_kernel, kan_assign_own_kernel).  Large codebooks take the bounded search further down, which
// finds the same shapes from a small part of the scores.

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "kan_device.hpp"
#include "kan_internal.hpp"
#include "kan_mfma_common.hpp"

namespace kan {
namespace {

constexpr int kAssignThreads = 256;
constexpr int kEdgeTilesPerWave = 4;                                   // 4 x 32 edges per wave
constexpr int kEdgesPerWg = (kAssignThreads / kWave) * kEdgeTilesPerWave * 32;   // 512

__device__ __forceinline__ void split_h(float v, _Float16& hi, _Float16& lo) {
  hi = (_Float16)v;
  lo = (_Float16)(v - (float)hi);
}

// Slots s0 .. s0+7 of a shape's operand.  Without a shape (its row is zeros then) (rows past the last one) the norm term is minus infinity,
// so that the row never wins, whatever the norms of the shapes.  Both searches take these, and the products in this
// order: a score has the same bits in either.
__device__ __forceinline__ uint4 shape_slots(const float (&row)[kG], bool there, int s0) {
  h16x8 v;
  float nrm = 0.f;
#pragma unroll
  for (int m = 0; m < kG; ++m) nrm = fmaf(row[m], row[m], nrm);
  const float half_norm = there ? -0.5f * nrm : -INFINITY;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int s = s0 + t;
    float src = half_norm;
    bool low = s == 31;
#pragma unroll
    for (int m = 0; m < kG; ++m)
      if (s == m || s == 11 + m || s == 21 + m) {
        src = row[m];
        low = s >= 11 && s < 21;
      }
    _Float16 hi, lo;
    split_h(src, hi, lo);
    v[t] = low ? (there ? lo : (_Float16)0.0f) : hi;
  }
  return __builtin_bit_cast(uint4, v);
}

// Centroid-side operands in MFMA A-fragment order: record [(tile * 2 + kstep) * 64 + lane]
// holds slots kstep*16 + (lane/32)*8 .. +8 of centroid tile*32 + (lane & 31).
__global__ __launch_bounds__(256) void kan_assign_prep_kernel(const float* __restrict__ cb, int K, int n_tiles,
                                                              uint4* __restrict__ out) {
  const long long rec = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (rec >= (long long)n_tiles * 2 * 64) return;
  const int lane = (int)(rec & 63), ks = (int)((rec >> 6) & 1);
  const int c = (int)(rec >> 7) * 32 + (lane & 31);
  float row[kG];
#pragma unroll
  for (int m = 0; m < kG; ++m) row[m] = c < K ? cb[(long long)c * kG + m] : 0.f;
  out[rec] = shape_slots(row, c < K, ks * 16 + (lane >> 5) * 8);
}

// Step 1 of an edge: bias = mean, gain = norm of the centred grid, direction = centred / gain.
__device__ __forceinline__ void normalise(const float* __restrict__ coef, float (&c)[kG], float& mean, float& g) {
#pragma unroll
  for (int m = 0; m < kG / 2; ++m) {
    const float2 v = ((const float2*)coef)[m];
    c[2 * m] = v.x;
    c[2 * m + 1] = v.y;
  }
  mean = 0.f;
#pragma unroll
  for (int m = 0; m < kG; ++m) mean += c[m];
  mean /= (float)kG;       // a true division: the mean of ten equal values is that value
  float ss = 0.f;
#pragma unroll
  for (int m = 0; m < kG; ++m) {
    c[m] -= mean;
    ss = fmaf(c[m], c[m], ss);
  }
  g = sqrtf(ss);
  const float inv = g > 0.f ? 1.0f / g : 0.f;
#pragma unroll
  for (int m = 0; m < kG; ++m) c[m] *= inv;
}

__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// Maximum of a lane's 16 scores: 8 three-input maxima.
__device__ __forceinline__ float max_of(const f32x16& v) {
  const float m0 = max3(v[0], v[1], v[2]), m1 = max3(v[3], v[4], v[5]);
  const float m2 = max3(v[6], v[7], v[8]), m3 = max3(v[9], v[10], v[11]);
  const float m4 = max3(v[12], v[13], v[14]);
  return max3(max3(m0, m1, m2), m3, max3(m4, v[15], -3.0e38f));
}
// The first register that holds it: of the first three whose maximum it is (25 instructions; one register after the
// other 45, half of them waits for the condition of the one before).
__device__ __forceinline__ int row_of(const f32x16& v, float m) {
  float x = v[15], y = v[15];
  int base = 15;
#pragma unroll
  for (int q = 4; q >= 0; --q) {
    const bool here = max3(v[3 * q], v[3 * q + 1], v[3 * q + 2]) == m;
    x = here ? v[3 * q] : x;
    y = here ? v[3 * q + 1] : y;
    base = here ? 3 * q : base;
  }
  return base + (x == m ? 0 : (y == m ? 1 : (base < 15 ? 2 : 0)));
}

// The bounded search's tiles are four groups of eight shapes: a lane's registers 4 g .. 4 g + 3 are its rows of group g,
// rows 4 (lane / 32) .. of its eight, and these lie by id.  found(g, row among the four, score) for every group whose best
// score is at least `best`, which it may raise: equal scores of several groups are all reported.
constexpr int kGroupShapes = 8;
constexpr int kGroupRecords = kGroupShapes * 4;            // [instruction][half of a wave][shape] records of 16 bytes
template <typename Found>
__device__ __forceinline__ void for_groups_with(const f32x16& v, const float& best, Found found) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const float a = v[4 * g], b = v[4 * g + 1], c = v[4 * g + 2], d = v[4 * g + 3], m = fmaxf(max3(a, b, c), d);
    if (m >= best) found(g, a == m ? 0 : (b == m ? 1 : (c == m ? 2 : 3)), m);
  }
}

// An edge's operand, in pieces of eight slots.
__device__ __forceinline__ void edge_pieces(const float (&c)[kG], uint4 (&piece)[4]) {
  _Float16 hi[kG], lo[kG];
#pragma unroll
  for (int m = 0; m < kG; ++m) split_h(c[m], hi[m], lo[m]);
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    h16x8 v;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int s = n * 8 + t;
      v[t] = s < 10 ? hi[s] : (s == 10 || s == 31 ? (_Float16)1.0f : (s < 21 ? hi[s - 11] : lo[s - 21]));
    }
    piece[n] = __builtin_bit_cast(uint4, v);
  }
}
// An edge's operand in LDS, four pieces of eight slots; edges four apart keep them in another order, so that the sixteen
// lanes that store or read a piece together meet different banks.
__device__ __forceinline__ int piece_at(int q, int piece) { return q * 4 + (piece ^ ((q >> 2) & 3)); }
__device__ __forceinline__ void store_edge(uint4* sB, int q, const float (&c)[kG]) {
  uint4 piece[4];
  edge_pieces(c, piece);
#pragma unroll
  for (int n = 0; n < 4; ++n) sB[piece_at(q, n)] = piece[n];
}

// What the second product can add to the score of a shape at distance d or less of an edge (|n| = 1): its norm is at
// most 1 + d, the low parts are at most 2^-11 of what they complete, on either side of n . C and in |C|^2 / 2.
constexpr float kFar = 100.0f;                    // distances above are not bounded in fp16
__device__ __forceinline__ float first_product_slack(float d) {
  const float r = 1.001f + d;
  return d <= kFar ? fmaf(r, fmaf(r, 2.45e-4f, 9.8e-4f), 1e-5f) : INFINITY;
}

// ---- whole search ---------------------------------------------------------------------------------
// Eight waves share 128 edges and take the tiles of shapes in turn; with few edges several workgroups share them as well,
// each on a part of the codebook, and a second launch takes the best of the parts.  (One workgroup per 128 edges left most of
// the chip idle: 2^13 edges x 65,536 shapes 171 us, 44 in eight parts; 10,388 x 5,377 24.0 / 16.0, 4,096 x 4,096 19.7 / 11.4.)
// The waves tell each other through LDS what an edge's best shape reaches at least: a wave's own best starts anew with it, and
// the row of a new best is a third of the work of a tile (131,072 edges x 4,096 shapes 55 -> 43 us).
// FILTER: the second product, half of the matrix work, only for tiles whose first one comes near that (first_product_slack):
// after the first hundreds of tiles that is rare.  65,536 edges x 65,536 shapes 281 -> 217 us, 98,304 x 16,384 113 -> 97; with
// 169 or 128 tiles a part it loses (10,388 x 5,377 15.4 -> 16.9, 131,072 x 4,096 48 -> 51).
// Bound: matrix and vector instructions, at clocks that the matrix instructions lower; the loads are one tile of 2 KB for four of edges.
constexpr int kWholeWaves = 8, kWholeEdges = kEdgeTilesPerWave * 32;

// The two half-waves hold different rows of the same edge, the waves different tiles: the better score, of equal ones the
// lower id.
__device__ __forceinline__ void keep_better(float sc, int id, int q, float* s_best, int* s_id) {
  const float sc_o = __shfl_xor(sc, 32, kWave);
  const int id_o = __shfl_xor(id, 32, kWave);
  if (sc_o > sc || (sc_o == sc && id_o < id)) {
    id = id_o;
    sc = sc_o;
  }
  if ((threadIdx.x & 63) < 32) {
    s_best[q] = sc;
    s_id[q] = id;
  }
}
__device__ __forceinline__ uint2 best_of_waves(const float (&s_best)[kWholeWaves][kWholeEdges], const int (&s_id)[kWholeWaves][kWholeEdges], int q) {
  float sc = s_best[0][q];
  int id = s_id[0][q];
#pragma unroll
  for (int w = 1; w < kWholeWaves; ++w) {
    const float o = s_best[w][q];
    const int io = s_id[w][q];
    if (o > sc || (o == sc && io < id)) {
      sc = o;
      id = io;
    }
  }
  return make_uint2(__float_as_uint(sc), (uint32_t)id);
}
// Row r of a lane's sixteen is row 8 (r / 4) + 4 (lane / 32) + r % 4 of its tile.
__device__ __forceinline__ int shape_of(int tile, int r, int half) { return tile * 32 + 8 * (r >> 2) + 4 * half + (r & 3); }

struct WholeArgs {
  const float* coef;        // [E][10]
  const uint4* cent;        // prepared centroid operands
  long long E;
  int n_tiles, parts, part_tiles;
  uint2* found;             // [parts][E] score and shape of every part; parts = 1: not used
  void* idx;
  float *gain, *bias;
};

// The slack for every shape that scores m or more, in steps: d = sqrt(1 - 2 m) at most.
__device__ __forceinline__ float slack_from(float m) {
  return m >= 0.f ? 2.97e-3f : (m >= -4.f ? 7.9e-3f : (m >= -420.f ? 0.25f : INFINITY));       // (of d = 1, 3, 29)
}

template <typename IdxT, bool FILTER>
__global__ __launch_bounds__(kWholeWaves * kWave, 4) void kan_assign_whole_kernel(const WholeArgs a) {
  __shared__ uint4 sB[kWholeEdges * 4];
  // A score that an edge's best shape reaches with the first product alone ([edge of the tile][tile]), and whether that is known to hold
  __shared__ __attribute__((aligned(16))) float s_near[32][kEdgeTilesPerWave];
  __shared__ uint8_t s_unit[kWholeEdges];
  __shared__ float s_best[kWholeWaves][kWholeEdges];
  __shared__ int s_id[kWholeWaves][kWholeEdges];
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, half = lane >> 5;
  const int part = (int)(blockIdx.x % (unsigned)a.parts);
  const long long e_wg = (long long)(blockIdx.x / (unsigned)a.parts) * kWholeEdges;
  const int t_end = min(a.n_tiles, (part + 1) * a.part_tiles);

  const uint4* cp = a.cent + lane;
  auto load_tile = [&](int t, uint4 (&fa)[2]) {
    const int tc = min(t, t_end - 1);            // past the end: a harmless re-read
    fa[0] = cp[(long long)(tc * 2) * 64];
    fa[1] = cp[(long long)(tc * 2) * 64 + 64];
  };
  uint4 fa0[2], fa1[2];
  const int t0 = part * a.part_tiles + wave;
  load_tile(t0, fa0);
  load_tile(t0 + kWholeWaves, fa1);

  if (tid < kWholeEdges) {
    const long long at = e_wg + tid;
    float c[kG], mean, g, nn = 0.f;
    normalise(a.coef + min(at, a.E - 1) * kG, c, mean, g);
    if (part == 0 && at < a.E) {
      a.gain[at] = g;
      a.bias[at] = mean;
    }
#pragma unroll
    for (int m = 0; m < kG; ++m) nn = fmaf(c[m], c[m], nn);
    s_unit[tid] = nn <= 1.000003f;               // (longer: squares in the subnormal range lose bits; what is no number)
    store_edge(sB, tid, c);
    s_near[tid & 31][tid >> 5] = -INFINITY;
  }
  __syncthreads();

  h16x8 fb[kEdgeTilesPerWave][2];
  float best[kEdgeTilesPerWave];
  int best_tile[kEdgeTilesPerWave], best_row[kEdgeTilesPerWave];
#pragma unroll
  for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) fb[nb][ks] = __builtin_bit_cast(h16x8, sB[piece_at(nb * 32 + col, ks * 2 + half)]);
    best[nb] = -3.0e38f;
    best_tile[nb] = 0;
    best_row[nb] = 0;
  }
  int unit = 0;
#pragma unroll
  for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) unit |= s_unit[nb * 32 + col] << nb;
  f32x16 zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
  auto score_tile = [&](int t, const uint4 (&fa)[2]) {
    const h16x8 a0 = __builtin_bit_cast(h16x8, fa[0]), a1 = __builtin_bit_cast(h16x8, fa[1]);
    const f32x4 near = *(const volatile f32x4*)&s_near[col][0];        // (raised meanwhile: more is looked at than need be)
#pragma unroll
    for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
      f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, fb[nb][0], zero, 0, 0, 0);
      bool may = true;
      if constexpr (FILTER) {
        may = max_of(acc) >= near[nb];
        if (__ballot(may) == 0) continue;        // (for the whole wave: matrix instructions heed no lane mask)
      }
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, fb[nb][1], acc, 0, 0, 0);
      const float m = max_of(acc);
      if constexpr (!FILTER) may = m >= near[nb];
      // Strictly greater: the earliest tile, and in it the lowest register, keeps a tie.
      if (may && m > best[nb]) {
        best[nb] = m;
        best_tile[nb] = t;
        best_row[nb] = row_of(acc, m);
        const float slack = FILTER ? ((unit >> nb) & 1 ? slack_from(m) : INFINITY) : 0.f;
        __hip_atomic_fetch_max(&s_near[col][nb], m - slack, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  };
  for (int t = t0; t < t_end; t += 2 * kWholeWaves) {
    score_tile(t, fa0);
    load_tile(t + 2 * kWholeWaves, fa0);
    if (t + kWholeWaves < t_end) score_tile(t + kWholeWaves, fa1);
    load_tile(t + 3 * kWholeWaves, fa1);
  }

#pragma unroll
  for (int nb = 0; nb < kEdgeTilesPerWave; ++nb)
    keep_better(best[nb], shape_of(best_tile[nb], best_row[nb], half), nb * 32 + col, s_best[wave], s_id[wave]);
  __syncthreads();
  const long long at = e_wg + tid;
  if (tid < kWholeEdges && at < a.E) {
    const uint2 top = best_of_waves(s_best, s_id, tid);
    if (a.parts > 1) a.found[part * a.E + at] = top;
    else ((IdxT*)a.idx)[at] = (IdxT)top.y;
  }
}

// Small codebooks, and more edges than the shared form has use for: every wave has TILES * 32 edges of its own.  A lane
// normalises an edge; the two halves of the wave then exchange pieces of the operands, which puts every piece where the matrix
// instruction wants it, without LDS.  LOCAL: the workgroup builds the shapes' operands in its LDS and goes through the edges:
// one launch, and only edges are read in its loop.  256 shapes and 28,672 / 182,784 / 394,240 edges 9.6 / 13.5 / 19.3 us with
// operands of both kinds stored in pieces of two bytes and fetched from memory, 7.9 / 9.8 / 15.3 so; 2^20 x 4,096 (not LOCAL)
// 293 -> 271.  Bound: reads and writes of the edges (16 MB in 6 us) beside a new best in almost every tile.
template <typename IdxT, int TILES, bool LOCAL>
__global__ __launch_bounds__(kAssignThreads, 4) void kan_assign_own_kernel(const WholeArgs a, const float* __restrict__ cb, int K) {
  static_assert(TILES % 2 == 0, "a lane per edge of two tiles");
  extern __shared__ uint4 s_cent[];
  constexpr int kOwn = TILES * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
  if constexpr (LOCAL) {
    for (int c = tid; c < a.n_tiles * 32; c += kAssignThreads) {
      float row[kG];
#pragma unroll
      for (int m = 0; m < kG; ++m) row[m] = c < K ? cb[(long long)c * kG + m] : 0.f;
#pragma unroll
      for (int piece = 0; piece < 4; ++piece)
        s_cent[((c >> 5) * 2 + (piece >> 1)) * 64 + (piece & 1) * 32 + (c & 31)] = shape_slots(row, c < K, piece * 8);
    }
    __syncthreads();
  }
  const uint4* cp = (LOCAL ? (const uint4*)s_cent : a.cent) + lane;
  auto load_tile = [&](int t, uint4 (&fa)[2]) {
    const int tc = min(t, a.n_tiles - 1);        // past the end: a harmless re-read
    fa[0] = cp[(long long)(tc * 2) * 64];
    fa[1] = cp[(long long)(tc * 2) * 64 + 64];
  };
  f32x16 zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
  for (long long e0 = ((long long)blockIdx.x * 4 + wave) * kOwn; e0 < a.E; e0 += (long long)gridDim.x * 4 * kOwn) {
    h16x8 fb[TILES][2];
    float best[TILES];
    int best_tile[TILES], best_row[TILES];
#pragma unroll
    for (int h = 0; h < TILES / 2; ++h) {
      const long long at = e0 + h * 64 + lane;
      float c[kG], mean, g;
      normalise(a.coef + min(at, a.E - 1) * kG, c, mean, g);
      if (at < a.E) {
        a.gain[at] = g;
        a.bias[at] = mean;
      }
      uint4 piece[4];
      edge_pieces(c, piece);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        uint32_t lo[4], hi[4];
        const uint4 x = piece[2 * ks], y = piece[2 * ks + 1];
        const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
        for (int w = 0; w < 4; ++w) {            // (upper half of the first, lower half of the second)
          const auto sw = __builtin_amdgcn_permlane32_swap(xs[w], ys[w], false, false);
          lo[w] = sw[0];
          hi[w] = sw[1];
        }
        fb[2 * h][ks] = __builtin_bit_cast(h16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
        fb[2 * h + 1][ks] = __builtin_bit_cast(h16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
      }
    }
#pragma unroll
    for (int nb = 0; nb < TILES; ++nb) {
      best[nb] = -3.0e38f;
      best_tile[nb] = 0;
      best_row[nb] = 0;
    }
    auto score_tile = [&](int t, const uint4 (&fa)[2]) {
      const h16x8 a0 = __builtin_bit_cast(h16x8, fa[0]), a1 = __builtin_bit_cast(h16x8, fa[1]);
#pragma unroll
      for (int nb = 0; nb < TILES; ++nb) {
        f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, fb[nb][0], zero, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, fb[nb][1], acc, 0, 0, 0);
        const float m = max_of(acc);
        // A new best is rare (the t-th tile improves a lane's running maximum with probability
        // ~1/t), so the row is looked for only then.  Strictly greater: the earliest tile, and in
        // it the lowest register, keeps a tie.
        if (m > best[nb]) {
          best[nb] = m;
          best_tile[nb] = t;
          best_row[nb] = row_of(acc, m);
        }
      }
    };
    uint4 fa0[2], fa1[2];
    load_tile(0, fa0);
    load_tile(1, fa1);
    for (int t = 0; t < a.n_tiles; t += 2) {
      score_tile(t, fa0);
      load_tile(t + 2, fa0);
      if (t + 1 < a.n_tiles) score_tile(t + 1, fa1);
      load_tile(t + 3, fa1);
    }
    // the two halves hold different rows of the same edges: the better one, the lower id.  (In registers: an array that a
    // lane indexes by its half goes to LDS or scratch, and the address in LDS comes from the launch's packet in host memory,
    // which cost a launch 9 to 12 us: 2^20 edges x 64 / 1,000 / 4,096 shapes in four tiles a wave 28 / 97 / 282 us so, 17 / 84 /
    // 271 in registers.)
    auto better = [&](int nb) {
      const int id = shape_of(best_tile[nb], best_row[nb], half);
      const float sc_o = __shfl_xor(best[nb], 32, kWave);
      const int id_o = __shfl_xor(id, 32, kWave);
      return sc_o > best[nb] || (sc_o == best[nb] && id_o < id) ? id_o : id;
    };
#pragma unroll
    for (int h = 0; h < TILES / 2; ++h) {
      const long long at = e0 + h * 64 + lane;
      const int first = better(2 * h), second = better(2 * h + 1);
      if (at < a.E) ((IdxT*)a.idx)[at] = (IdxT)(half ? second : first);
    }
  }
}

// The edges that the bounded search leaves, against its groups of eight shapes, four to a tile: the same scores, and of
// equal ones the lowest id, whatever tile it lies in.  Eight waves share 128 edges of its order.
struct RestArgs {
  const float* coef;
  const uint4* cent;        // operands of the groups
  long long E;
  const uint32_t* list;     // the edges in the bounded search's order ...
  const uint8_t* left;      // ... and of every 32 whether they are left (their gains and biases are there already)
  const uint32_t *groups, *ids;      // the number of groups and the shape of every row
  void* idx;
};

template <typename IdxT>
__global__ __launch_bounds__(kWholeWaves * kWave, 4) void kan_assign_rest_kernel(const RestArgs a) {
  __shared__ uint4 sB[kWholeEdges * 4];
  __shared__ float s_best[kWholeWaves][kWholeEdges];
  __shared__ int s_id[kWholeWaves][kWholeEdges];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, half = lane >> 5;
  const int n_tiles = ((int)*a.groups + 3) / 4;
  const uint4* cp = a.cent + (col >> 3) * kGroupRecords + half * kGroupShapes + (lane & 7);
  auto load_tile = [&](int t, uint4 (&fa)[2]) {
    const int tc = min(t, n_tiles - 1);          // past the end: a harmless re-read
    fa[0] = cp[(long long)(tc * 2) * 64];
    fa[1] = cp[(long long)(tc * 2) * 64 + kGroupRecords / 2];
  };
  f32x16 zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
  // The edges from e_wg on, of these the tiles with their byte set in `tiles`.
  auto serve = [&](long long e_wg, uint32_t tiles) {
    if (tid < kWholeEdges) {
      float c[kG], mean, g;
      normalise(a.coef + (long long)a.list[min(e_wg + tid, a.E - 1)] * kG, c, mean, g);
      store_edge(sB, tid, c);
    }
    __syncthreads();
    h16x8 fb[kEdgeTilesPerWave][2];
    float best[kEdgeTilesPerWave];
    int best_id[kEdgeTilesPerWave];
#pragma unroll
    for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) fb[nb][ks] = __builtin_bit_cast(h16x8, sB[piece_at(nb * 32 + col, ks * 2 + half)]);
      best[nb] = -3.0e38f;
      best_id[nb] = 0;
    }
    auto score_tile = [&](int t, const uint4 (&fa)[2]) {
      const h16x8 a0 = __builtin_bit_cast(h16x8, fa[0]), a1 = __builtin_bit_cast(h16x8, fa[1]);
#pragma unroll
      for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
        if (!((tiles >> (8 * nb)) & 1u)) continue;
        f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, fb[nb][0], zero, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, fb[nb][1], acc, 0, 0, 0);
        if (max_of(acc) >= best[nb])
          for_groups_with(acc, best[nb], [&](int g, int r, float mg) {
            const int id = (int)a.ids[t * 32 + g * kGroupShapes + 4 * half + r];
            if (mg > best[nb] || (uint32_t)id < (uint32_t)best_id[nb]) best_id[nb] = id;
            best[nb] = mg;
          });
      }
    };
    uint4 fa0[2], fa1[2];
    load_tile(wave, fa0);
    load_tile(wave + kWholeWaves, fa1);
    for (int t = wave; t < n_tiles; t += 2 * kWholeWaves) {
      score_tile(t, fa0);
      load_tile(t + 2 * kWholeWaves, fa0);
      if (t + kWholeWaves < n_tiles) score_tile(t + kWholeWaves, fa1);
      load_tile(t + 3 * kWholeWaves, fa1);
    }
#pragma unroll
    for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) keep_better(best[nb], best_id[nb], nb * 32 + col, s_best[wave], s_id[wave]);
    __syncthreads();
    const long long at = e_wg + tid;
    if (tid < kWholeEdges && at < a.E && ((tiles >> (8 * (tid >> 5))) & 1u))
      ((IdxT*)a.idx)[a.list[at]] = (IdxT)best_of_waves(s_best, s_id, tid).y;
  };
  const long long groups = (a.E + kWholeEdges - 1) / kWholeEdges;
  for (long long g0 = blockIdx.x; g0 < groups; g0 += (long long)kWave * gridDim.x) {
    const long long mine = g0 + (long long)lane * gridDim.x;
    const uint32_t flags = mine < groups ? ((const uint32_t*)a.left)[mine] : 0u;
    for (unsigned long long m = __ballot(flags != 0); m; m &= m - 1) {
      const int l = __ffsll(m) - 1;
      serve((g0 + (long long)l * gridDim.x) * kWholeEdges, (uint32_t)__builtin_amdgcn_readlane((int)flags, l));
      __syncthreads();
    }
  }
}

// The best of the parts' shapes; they are in the order of the ids, but for an edge without any (id 0 everywhere).
template <typename IdxT>
__global__ __launch_bounds__(256) void kan_assign_join_kernel(const uint2* __restrict__ found, int parts, long long E, IdxT* __restrict__ idx) {
  const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= E) return;
  uint2 top = found[e];
#pragma unroll 4
  for (int p = 1; p < parts; ++p) {
    const uint2 o = found[p * E + e];
    if (__uint_as_float(o.x) > __uint_as_float(top.x)) top = o;
  }
  idx[e] = (IdxT)top.y;
}

// ---- bounded search -------------------------------------------------------------------------------
// The codebook is cut into cells (the shapes nearest to one of M = K / 64 sampled shapes, the cell's centre) and a cell
// into groups of eight shapes that lie close together.  Shapes that all lie within R of a point c can be left out for an
// edge n that knows a shape at distance d already when |n - c| > R + d; in scores (|n| = 1)
//     n . c - |c|^2 / 2 + R^2 / 2 + R d  <  (1 - d^2) / 2 .
// The left side is a product of an edge's vector (n, 1, d) with the ball's vector (c, (R^2 - |c|^2) / 2, R), so one
// v_mfma_f32_32x32x16_f16 tests 32 edges against 32 balls, the right side included; what the fp16 operands
// round away is covered by a margin.  The cells are tested first, then the groups of those that any edge of the wave asks
// for; four groups that any edge asks for make up a tile of the search, wherever they lie.  The edges are sorted by their
// nearest centre and the side of it that they lie on, so that the 32 of a wave ask for about the same groups:
//     (1) the groups of the edges' own cells: seven of ten edges with 5 % noise find their shape here;
//     (2) those within R + min(d, what a typical edge of the wave has): finds nearly all of the others, whose d of
//         step 1 alone would ask for a large part of the codebook;
//     (3) where an edge is left with a larger d than it asked at: what that one still asks for.
// The scores are those of the whole search, bit for bit, no group that can hold the best one is left out and equal
// scores go to the lowest id: the result is the whole search's, whichever edges share a wave (the sort places them in
// no particular order) and whichever of them are handed over: a wave that would visit more than kRestShare of the groups
// in (2) or in (3) leaves its edges to the whole search.  A visit costs about what a tile costs there, so that is worth
// it only for edges that ask for nearly everything (vectors that the bounds do not hold for, codebooks of one shape):
// grids that fit their codebook poorly ask for less, and stay.
//
// What bounds it: instruction issue (vector instructions for 60 % of the time) and operands (the address units 66 % busy).
// A wave makes about 47 tests of 32 cells, 38 of 32 groups, and visits 68 tiles of four groups, each with one matrix, one
// 1 KB load and some 15 vector instructions (65,536 shapes, 5 % noise).  Groups of eight in place of tiles of 32 shapes around the
// cell's centre took 258 visits down to 92 at 101 tests in place of 80; the sides of the centre to the figures above;
// resources of the loads that were not known to be the same for the wave had cost a loop around every load.
// 2048 x 512 edges against 65,536 shapes, the whole call: 737 -> 480 us (the kernel 650 -> 400); 2 % / 15 % noise / unrelated
// grids 545 / 1290 / 1332 -> 332 / 885 / 908.  The whole search takes 3.7 ms.

constexpr int kCellShapes = 64;                   // shapes per cell on average
constexpr int kCellMaxGroups = 49152;             // (listed in 16 bits)
constexpr float kRestShare = 0.9f;                // (0.6 / 0.7: K = 8,192, unrelated grids 1153 / 873 us)
// Step (2): edges within kFound of the mean of those below the wave's mean have found their shape where that is well below
// the mean of all; the others ask at kAsk of it.  Where edges are not apart like that, all ask at kPoor of the mean at most:
// nearly none is left for (3), which would test the cells again and visit most groups once more.
constexpr float kFound = 1.8f, kAsk = 1.5f, kApart = 1.3f, kPoor = 1.2f;

constexpr int kRestWorkgroups = 1024;             // of the whole search behind it: twice what is resident
constexpr int kAhead = 2;                         // tiles in flight per wave
// Lists of a wave in LDS: cells that may hold a best shape (of 32 words of cells), a window of their groups, groups to visit
constexpr int kListCells = 1024, kListGroups = 640, kListVisits = 1024;
constexpr int kPadGroups = 8;                     // groups without shapes behind the last one (a tile may reach past it)
constexpr int kSortThreads = 1024, kSortGroups = 128;
// Edges of a cell are sorted by the side of its centre they lie on along kMaxSub directions as well, so that a wave's 32 lie
// closer together: 49 + 71 in place of 57 + 94 tiles tested and visited a wave (65,536 shapes, 5 % noise).
constexpr int kMaxSub = 3, kMaxBins = 8192;       // (bins are counted in LDS)
constexpr int kBuildThreads = 512;
constexpr int kBuildChunk = 512;                  // members of a cell that are grouped together, a power of two

// Where the pieces of the search lie in the workspace.
struct CellLayout {
  int M;                   // cells, a multiple of 32
  int sub;                 // log2 of the parts of a cell that the edges are sorted by
  int bins[2];             // of the sort, one for edges without direction included
  int groups_max;
  int groups[2];           // workgroups of the sort: over the shapes, over the edges
  long long chunk[2];      // items per workgroup
  size_t centres, frag, ids, cell_bound, bound, member, perm, key[2], hist[2], total[2], first[2], first_group, wg_least, least, left, bytes;
};

size_t centroid_bytes(int K) { return (size_t)((K + 31) / 32) * 2 * 64 * sizeof(uint4); }

CellLayout cell_layout(long long E, int K) {
  CellLayout g;
  g.M = (K / kCellShapes + 31) / 32 * 32;
  g.sub = 0;
  while (g.sub < kMaxSub && (g.M << (g.sub + 1)) <= kMaxBins) ++g.sub;
  g.bins[0] = g.M + 1;
  g.bins[1] = (g.M << g.sub) + 1;
  g.groups_max = (K + kGroupShapes - 1) / kGroupShapes + g.M;
  size_t at = 0;
  auto take = [&](size_t bytes) {
    const size_t here = at;
    at += (bytes + 255) / 256 * 256;
    return here;
  };
  g.centres = take((size_t)g.M * 2 * sizeof(uint4));
  g.frag = take((size_t)(g.groups_max + kPadGroups) * kGroupRecords * sizeof(uint4));
  g.ids = take((size_t)(g.groups_max + kPadGroups) * kGroupShapes * 4);
  g.cell_bound = take((size_t)g.M * 2 * sizeof(uint4));
  g.bound = take((size_t)g.groups_max * 2 * sizeof(uint4));
  g.member = take((size_t)K * 4);
  g.perm = take((size_t)E * 4);
  for (int p = 0; p < 2; ++p) {
    const long long n = p ? E : K;
    const long long groups = (n + kSortThreads - 1) / kSortThreads;
    g.groups[p] = (int)(groups < kSortGroups ? groups : kSortGroups);
    g.chunk[p] = (n + g.groups[p] - 1) / g.groups[p];
    g.key[p] = take((size_t)n * 2);
    g.hist[p] = take((size_t)g.groups[p] * g.bins[p] * 4);
    g.total[p] = take((size_t)g.bins[p] * 4);
    g.first[p] = take((size_t)g.bins[p] * 4);
  }
  g.first_group = take((size_t)(g.M + 1) * 4);
  g.wg_least = take((size_t)((K + kEdgesPerWg - 1) / kEdgesPerWg) * 8);
  g.least = take(4);
  g.left = take((size_t)((E + 127) / 128) * 4);
  g.bytes = at;
  return g;
}

struct CellArgs {
  const float* coef;
  const float* cb;
  long long E;
  int K, M, sub;
  int bins[2];
  int shape_wgs;                 // kan_cells_kernel: workgroups over the shapes, in front of those over the edges
  int groups[2];
  long long chunk[2];
  uint4* centres;                // operands of the centres
  uint4* frag;                   // operands of the groups, kGroupRecords each
  uint32_t* ids;                 // shape of every group row
  uint4* cell_bound;             // bound operands of the cells, 32 to a matrix operand
  uint4* bound;                  // bound operands of the groups, two records each
  uint32_t* sorted[2];           // shapes, edges in the order of their cells
  uint16_t* key[2];              // bin of every shape (its cell), edge (its cell's part; the last one: an edge without direction)
  uint32_t *hist[2], *total[2], *first[2];
  uint32_t* first_group;         // [M + 1]
  unsigned long long* wg_least;
  uint8_t* left;                 // [4 * ceil(E / 128)] waves whose edges are left to the whole search
  uint32_t* least;               // shape of the smallest norm: the nearest to an edge of gain 0
  void* idx;
  float *gain, *bias;
};

// Over the 64 lanes, for all of them: moves within rows of 16, then of the rows' results (an LDS permute for each step is a
// round trip).
template <typename Op>
__device__ __forceinline__ float wave_fold(float v, float none, Op op) {
  auto moved = [&](auto ctrl, auto rows) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(none), __float_as_int(v), ctrl.value, rows.value, 0xf, false));
  };
  using std::integral_constant;
  v = op(v, moved(integral_constant<int, 0x111>(), integral_constant<int, 0xf>()));
  v = op(v, moved(integral_constant<int, 0x112>(), integral_constant<int, 0xf>()));
  v = op(v, moved(integral_constant<int, 0x114>(), integral_constant<int, 0xf>()));
  v = op(v, moved(integral_constant<int, 0x118>(), integral_constant<int, 0xf>()));
  v = op(v, moved(integral_constant<int, 0x142>(), integral_constant<int, 0xa>()));
  v = op(v, moved(integral_constant<int, 0x143>(), integral_constant<int, 0xc>()));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_total(float v) {
  return wave_fold(v, 0.f, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_most(float v) {       // v >= -1
  return wave_fold(v, -1.f, [](float a, float b) { return fmaxf(a, b); });
}

__device__ __forceinline__ int sums_up_to(int v) {          // of the lanes up to this one
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return v;
}

// A row's sixteen slots as the two halves of a wave hold them.
__device__ __forceinline__ uint4 pack_slots(const float (&v)[8]) {
  h16x8 p;
#pragma unroll
  for (int t = 0; t < 8; ++t) p[t] = (_Float16)v[t];
  return __builtin_bit_cast(uint4, p);
}
__device__ __forceinline__ float fp16_of(float v) { return (float)(_Float16)v; }
__device__ __forceinline__ float fp16_up(float v) {           // v >= 0: an fp16 number of at least v
  return fp16_of(fmaf(v, 1.0f + 1.0f / 1024.0f, 1e-7f));
}

__device__ __forceinline__ const float* centre_row(const CellArgs& a, int m) {
  return a.cb + (long long)m * a.K / a.M * kG;
}

// Centres as matrix operands [c (10) | hi, lo of -|c|^2/2 | 0 (4)]: fp16 is enough to choose a cell.
__global__ __launch_bounds__(256) void kan_cell_centres_kernel(const CellArgs a) {
  const int rec = blockIdx.x * 256 + threadIdx.x;
  if (rec >= a.M * 2) return;
  const float* row = centre_row(a, (rec >> 6) * 32 + (rec & 31));
  float c[kG], nrm = 0.f;
#pragma unroll
  for (int k = 0; k < kG; ++k) {
    c[k] = row[k];
    nrm = fmaf(c[k], c[k], nrm);
  }
  // (beyond fp16, or no number: a centre that nothing is near)
  const bool fits = nrm < 1.19e5f;
#pragma unroll
  for (int k = 0; k < kG; ++k) c[k] = fits ? c[k] : 0.f;
  const float hn = fits ? -0.5f * nrm : -6e4f, hi = fp16_of(hn);
  const float v0[8] = {c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7]};
  const float v1[8] = {c[8], c[9], hi, hn - hi, 0.f, 0.f, 0.f, 0.f};
  a.centres[rec] = (rec & 32) ? pack_slots(v1) : pack_slots(v0);
}

// Nearest centre of every shape and every edge, and on which side of it an edge lies; gains and biases of the edges.  Any
// cell is a valid one, so the choice is cheap: the maxima of four rows each, the group's number in the low two bits of the
// mantissa, one running maximum - sixteen vector instructions per 32 x 32 scores - and the four rows of the winning
// group are told apart at the end.  Four is added to the scores, so that those that matter are positive and compare as
// integers (floating-point maxima of two operands cost an instruction each to quiet what may be no number).
__global__ __launch_bounds__(kAssignThreads, 4) void kan_cells_kernel(const CellArgs a) {
  __shared__ uint4 sB[kEdgesPerWg * 2];
  __shared__ uint8_t s_flat[kEdgesPerWg];
  __shared__ unsigned long long s_least;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool shapes = (int)blockIdx.x < a.shape_wgs;
  const long long n = shapes ? a.K : a.E;
  const long long first = (long long)(shapes ? blockIdx.x : blockIdx.x - a.shape_wgs) * kEdgesPerWg;
  uint16_t* key = a.key[shapes ? 0 : 1];
  if (tid == 0) s_least = ~0ull;
  __syncthreads();
  for (int q = tid; q < kEdgesPerWg; q += kAssignThreads) {
    const long long e = first + q, ec = e < n ? e : n - 1;
    float c[kG];
    bool flat = false;
    if (shapes) {
      float nrm = 0.f;
#pragma unroll
      for (int m = 0; m < kG; ++m) {
        c[m] = a.cb[ec * kG + m];
        nrm = fmaf(c[m], c[m], nrm);
      }
      // (by the norm term as the operands hold it, so that equal ones are equal here as well)
      _Float16 hi, lo;
      split_h(-0.5f * nrm, hi, lo);
      atomicMin(&s_least, ((unsigned long long)__float_as_uint(fabsf((float)hi + (float)lo)) << 32) | (uint32_t)ec);
    } else {
      float mean, g;
      normalise(a.coef + ec * kG, c, mean, g);
      flat = !(g > 0.f);
      if (e < n) {
        a.gain[e] = g;
        a.bias[e] = mean;
      }
    }
    const float v0[8] = {c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7]};
    const float v1[8] = {c[8], c[9], 1.f, 1.f, 0.f, 0.f, 0.f, 0.f};
    sB[q * 2] = pack_slots(v0);
    sB[q * 2 + 1] = pack_slots(v1);
    s_flat[q] = flat;
  }
  __syncthreads();
  if (shapes && tid == 0) a.wg_least[blockIdx.x] = s_least;

  h16x8 fb[kEdgeTilesPerWave];
  int best[kEdgeTilesPerWave], best_tile[kEdgeTilesPerWave];
#pragma unroll
  for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
    const int q = (wave * kEdgeTilesPerWave + nb) * 32 + (lane & 31);
    fb[nb] = __builtin_bit_cast(h16x8, sB[q * 2 + (lane >> 5)]);
    best[nb] = 0;
    best_tile[nb] = 0;
  }
  f32x16 four;
#pragma unroll
  for (int r = 0; r < 16; ++r) four[r] = 4.f;
  const uint4* cp = a.centres + lane;
  const int n_tiles = a.M / 32;
  uint4 next = cp[0];
  for (int t = 0; t < n_tiles; ++t) {
    const h16x8 fa = __builtin_bit_cast(h16x8, next);
    next = cp[min(t + 1, n_tiles - 1) * 64];
#pragma unroll
    for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
      const f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa, fb[nb], four, 0, 0, 0);
      int m = best[nb];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        auto bits = [&](int r) { return __float_as_int(acc[r]); };
        const int v = max(max(max(bits(q), bits(q + 4)), bits(q + 8)), bits(q + 12));
        m = max(m, (v & ~3) | q);
      }
      best_tile[nb] = m > best[nb] ? t : best_tile[nb];
      best[nb] = m;
    }
  }
  typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));
  auto dot = [](const h16x8& u, const h16x8& v) {
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < 8; k += 2) sum = __builtin_amdgcn_fdot2(h16x2{u[k], u[k + 1]}, h16x2{v[k], v[k + 1]}, sum, false);
    return sum;
  };
  const int half = lane >> 5;
  // the directions of the parts: orthogonal, of sum 0 as the shapes are
  h16x8 way[kMaxSub];
  {
    constexpr signed char kWay[kMaxSub][kG] = {{1, 1, 1, 1, 1, -1, -1, -1, -1, -1}, {1, -1, 1, -1, 0, 1, -1, 1, -1, 0}, {1, 1, -1, -1, 0, 0, 1, 1, -1, -1}};
#pragma unroll
    for (int b = 0; b < kMaxSub; ++b)
#pragma unroll
      for (int k = 0; k < 8; ++k) way[b][k] = (_Float16)(float)(half ? (k < 2 ? kWay[b][8 + k] : 0) : kWay[b][k]);
  }
#pragma unroll
  for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
    const int best_o = __shfl_xor(best[nb], 32, kWave), tile_o = __shfl_xor(best_tile[nb], 32, kWave);
    const bool other = best_o > best[nb] || (best_o == best[nb] && half);
    const int grp = (other ? best_o : best[nb]) & 3, tile = other ? tile_o : best_tile[nb];
    const int row0 = 4 * (half ^ (int)other) + grp;                // of the tile: rows row0 + 8 k
    const int q = (wave * kEdgeTilesPerWave + nb) * 32 + (lane & 31);
    // this half's eight slots of the four
    const uint4* rec = a.centres + tile * 64 + half * 32 + row0;
    h16x8 row[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) row[k] = __builtin_bit_cast(h16x8, rec[8 * k]);
    h16x8 near = row[0];
    int id = row0;
    float top = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float sc = dot(fb[nb], row[k]);
      sc += __shfl_xor(sc, 32, kWave);
      if (k == 0 || sc > top) {
        top = sc;
        near = row[k];
        id = row0 + 8 * k;
      }
    }
    int bin = tile * 32 + id;
    if (!shapes) {
      const h16x8 off = fb[nb] - near;
#pragma unroll
      for (int b = 0; b < kMaxSub; ++b) {
        float side = dot(off, way[b]);
        side += __shfl_xor(side, 32, kWave);
        if (b < a.sub) bin = 2 * bin + (side > 0.f);
      }
      if (s_flat[q]) bin = a.M << a.sub;
    }
    if (lane < 32 && first + q < n) key[first + q] = (uint16_t)bin;
  }
}

// Counting sort of shapes (blockIdx.y = 0) and edges (1) by bin, in chunks: bins counted per chunk, added up over the
// chunks, over the bins, items put in their places.  No order is kept within a bin of a chunk.
__global__ __launch_bounds__(kSortThreads) void kan_cell_count_kernel(const CellArgs a) {
  extern __shared__ uint32_t h[];
  const int p = blockIdx.y, g = blockIdx.x;
  if (g >= a.groups[p]) return;
  const int bins = a.bins[p];
  for (int m = threadIdx.x; m < bins; m += kSortThreads) h[m] = 0;
  __syncthreads();
  const long long n = p ? a.E : a.K, begin = g * a.chunk[p], end = min(n, begin + a.chunk[p]);
  for (long long i = begin + threadIdx.x; i < end; i += kSortThreads) atomicAdd(&h[a.key[p][i]], 1u);
  __syncthreads();
  for (int m = threadIdx.x; m < bins; m += kSortThreads) a.hist[p][(long long)g * bins + m] = h[m];
}

// A bin's counts of the chunks become running sums: a thread per bin and quarter of the chunks.
__global__ __launch_bounds__(256) void kan_cell_chunks_kernel(const CellArgs a) {
  constexpr int kQuarter = kSortGroups / 4;
  __shared__ uint32_t of_quarter[4][64];
  const int p = blockIdx.y, col = threadIdx.x & 63, quarter = threadIdx.x >> 6, m = blockIdx.x * 64 + col;
  const int bins = a.bins[p], groups = a.groups[p];
  const bool there = m < bins;
  uint32_t* h = a.hist[p] + min(m, bins - 1);
  uint32_t v[kQuarter], sum = 0;
#pragma unroll
  for (int k = 0; k < kQuarter; ++k) {
    const int g = quarter * kQuarter + k;
    v[k] = there && g < groups ? h[(long long)g * bins] : 0u;
  }
#pragma unroll
  for (int k = 0; k < kQuarter; ++k) sum += v[k];
  of_quarter[quarter][col] = sum;
  __syncthreads();
  uint32_t run = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) run += q < quarter ? of_quarter[q][col] : 0u;
#pragma unroll
  for (int k = 0; k < kQuarter; ++k) {
    const int g = quarter * kQuarter + k;
    if (there && g < groups) h[(long long)g * bins] = run;
    run += v[k];
  }
  if (there && quarter == 3) a.total[p][m] = run;
}

// One workgroup: running sums over the bins (shapes, groups, edges) and the shape of the smallest norm.
__global__ __launch_bounds__(kSortThreads) void kan_cell_scan_kernel(const CellArgs a) {
  constexpr int kPer = kMaxBins / kSortThreads + 1;         // bins of a thread
  __shared__ int of_wave[3][kSortThreads / kWave];
  __shared__ unsigned long long least;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) least = ~0ull;
  uint32_t n[2][kPer];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int m = tid * kPer + k;
      n[p][k] = m < a.bins[p] ? a.total[p][m] : 0u;
    }
  auto groups_of = [](uint32_t shapes) { return (shapes + kGroupShapes - 1) / kGroupShapes; };
  uint32_t own[3] = {0, 0, 0};
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    own[0] += n[0][k];
    own[1] += groups_of(n[0][k]);
    own[2] += n[1][k];
  }
  uint32_t run[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int upto = sums_up_to((int)own[q]);
    if (lane == kWave - 1) of_wave[q][wave] = upto;
    run[q] = (uint32_t)upto - own[q];
  }
  __syncthreads();
  unsigned long long l = ~0ull;
  for (int k = tid; k < a.shape_wgs; k += kSortThreads) l = min(l, a.wg_least[k]);
  if (l != ~0ull) atomicMin(&least, l);
#pragma unroll
  for (int q = 0; q < 3; ++q)
    for (int w = 0; w < wave; ++w) run[q] += (uint32_t)of_wave[q][w];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int m = tid * kPer + k;
    if (m < a.bins[0]) {
      a.first[0][m] = run[0];
      a.first_group[m] = run[1];
    }
    if (m < a.bins[1]) a.first[1][m] = run[2];
    run[0] += n[0][k];
    run[1] += groups_of(n[0][k]);
    run[2] += n[1][k];
  }
  __syncthreads();
  if (tid == 0) *a.least = (uint32_t)least;
}

__global__ __launch_bounds__(kSortThreads) void kan_cell_place_kernel(const CellArgs a) {
  extern __shared__ uint32_t at[];
  const int p = blockIdx.y, g = blockIdx.x;
  if (g >= a.groups[p]) return;
  const int bins = a.bins[p];
  for (int m = threadIdx.x; m < bins; m += kSortThreads) at[m] = a.first[p][m] + a.hist[p][(long long)g * bins + m];
  __syncthreads();
  const long long n = p ? a.E : a.K, begin = g * a.chunk[p], end = min(n, begin + a.chunk[p]);
  for (long long i = begin + threadIdx.x; i < end; i += kSortThreads)
    a.sorted[p][atomicAdd(&at[a.key[p][i]], 1u)] = (uint32_t)i;
}

// Bound operands of a ball of radius R (squared: far) around c: an edge asks for it, or not (see the head of this search).
__device__ __forceinline__ void ball_operands(const float (&c)[kG], float far, bool empty, uint4& lower, uint4& upper) {
  float cn = 0.f;
#pragma unroll
  for (int k = 0; k < kG; ++k) cn = fmaf(c[k], c[k], cn);
  const float R = fp16_up(sqrtf(far) * 1.00001f);
  // (fp16 operands: n and c are off by 2^-11 of themselves each, or flushed below 6e-5)
  float cst = 0.5f * (R * R - cn) + 1.5e-3f * sqrtf(cn) + 1e-4f;
  const bool fits = cn < 1e5f && R < 300.f && fabsf(cst) < 6e4f;
  if (!fits) cst = 6e4f;                          // beyond fp16, or no number: always asked for
  if (empty) cst = -6e4f;                         // never
  const float hi = fp16_of(cst), Rf = empty ? 0.f : (fits ? R : 300.f);
  const bool zero = empty || !fits;
  const float v0[8] = {zero ? 0.f : c[0], zero ? 0.f : c[1], zero ? 0.f : c[2], zero ? 0.f : c[3],
                       zero ? 0.f : c[4], zero ? 0.f : c[5], zero ? 0.f : c[6], zero ? 0.f : c[7]};
  const float v1[8] = {zero ? 0.f : c[8], zero ? 0.f : c[9], hi, cst - hi, Rf, 1.f, 1.f, 0.f};
  lower = pack_slots(v0);
  upper = pack_slots(v1);
}

// Part `at` of a chunk of n members after `level` halvings: [lo, hi), halved between whole groups while it is more than one.
__device__ __forceinline__ void part_of(int n, int level, int at, int& lo, int& hi) {
  lo = 0;
  hi = n;
  for (int l = level - 1; l >= 0; --l) {
    const int groups = (hi - lo + kGroupShapes - 1) / kGroupShapes, cut = lo + groups / 2 * kGroupShapes;
    if (groups < 2) {
      if ((at >> l) & 1) lo = hi;                  // (one group stays whole, in the first of the two)
    } else if ((at >> l) & 1) {
      lo = cut;
    } else {
      hi = cut;
    }
  }
}
// The same for the part that holds position i.
__device__ __forceinline__ void part_around(int n, int level, int i, int& lo, int& hi) {
  lo = 0;
  hi = n;
  for (int l = 0; l < level; ++l) {
    const int groups = (hi - lo + kGroupShapes - 1) / kGroupShapes, cut = lo + groups / 2 * kGroupShapes;
    if (groups < 2) return;
    if (i >= cut) lo = cut;
    else hi = cut;
  }
}

// Groups of one cell: its members are halved along the direction in which they spread most until eight are left (two
// steps of the power iteration from the member farthest from the mean; exact directions: 59 in place of 63 tiles a wave, the
// longest axis: 77), the operands of the search and the bounds of groups and cell are written.
// The first M workgroups take the first kBuildChunk members of a cell each.  Shapes that coincide (the unused rows of a
// trained codebook) all fall into one cell: the workgroups behind start at every kBuildChunk-th shape in the order of
// the cells and take the further chunk of its cell that begins there or next (one workgroup for the whole cell: with
// 30 % of 65,536 rows unused 658 us, now 35).
__global__ __launch_bounds__(kBuildThreads) void kan_cell_build_kernel(const CellArgs a) {
  __shared__ float x[kG][kBuildChunk];                     // the members' shapes
  __shared__ uint32_t id[kBuildChunk];
  __shared__ uint16_t order[2][kBuildChunk];               // members in the order of the parts
  __shared__ __attribute__((aligned(16))) uint32_t spot[kBuildChunk + 4];       // where along its part's direction the member at a position lies
  __shared__ uint32_t farthest;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int m = blockIdx.x, n0 = 0;
  if (m >= a.M) {
    const uint32_t at = (uint32_t)(m - a.M) * kBuildChunk;
    m = 0;
    for (int up = a.M; up - m > 1;) {            // the last cell that begins at `at` or before
      const int mid = (m + up) >> 1;
      if (a.first[0][mid] <= at) m = mid;
      else up = mid;
    }
    n0 = (int)((at - a.first[0][m] + kBuildChunk - 1) / kBuildChunk) * kBuildChunk;
    if (n0 == 0) return;
  }
  const int n = (int)a.total[0][m];
  const uint32_t* member = a.sorted[0] + a.first[0][m];
  const int nc = min(kBuildChunk, n - n0), groups = (nc + kGroupShapes - 1) / kGroupShapes;
  if (nc > 0) {
    for (int i = tid; i < nc; i += kBuildThreads) {
      const uint32_t k = member[n0 + i];
      id[i] = k;
      order[0][i] = (uint16_t)i;
#pragma unroll
      for (int q = 0; q < kG; ++q) x[q][i] = a.cb[(long long)k * kG + q];
    }
    __syncthreads();
    if (tid < 4) spot[nc + tid] = ~0u;
    int now = 0, levels = 0;
    while ((1 << levels) < groups) ++levels;
    for (int level = 0; level < levels; ++level) {
      // every member's place along its part's direction, a wave per part
      for (int p = wave; p < (1 << level); p += kBuildThreads / kWave) {
        int lo, hi;
        part_of(nc, level, p, lo, hi);
        if (hi - lo <= kGroupShapes) continue;             // (the same for the whole wave)
        float mean[kG], v[kG];
#pragma unroll
        for (int q = 0; q < kG; ++q) mean[q] = 0.f;
        for (int i = lo + lane; i < hi; i += 64) {
          const int t = order[now][i];
#pragma unroll
          for (int q = 0; q < kG; ++q) mean[q] += x[q][t];
        }
        const float inv = 1.0f / (float)(hi - lo);
#pragma unroll
        for (int q = 0; q < kG; ++q) mean[q] = wave_total(mean[q]) * inv;
        float top = -1.f;
        int who = lo;
        for (int i = lo + lane; i < hi; i += 64) {
          const int t = order[now][i];
          float d2 = 0.f;
#pragma unroll
          for (int q = 0; q < kG; ++q) d2 = fmaf(x[q][t] - mean[q], x[q][t] - mean[q], d2);
          if (d2 > top) {
            top = d2;
            who = i;
          }
        }
        const unsigned long long most = __ballot(top == wave_most(top));       // (0 for a part of no numbers)
        const int t0 = order[now][__builtin_amdgcn_readlane(who, most ? __ffsll(most) - 1 : 0)];
#pragma unroll
        for (int q = 0; q < kG; ++q) v[q] = x[q][t0] - mean[q];
        for (int step = 0; step < 2; ++step) {
          float w[kG], big = 0.f;
#pragma unroll
          for (int q = 0; q < kG; ++q) w[q] = 0.f;
          for (int i = lo + lane; i < hi; i += 64) {
            const int t = order[now][i];
            float dot = 0.f;
#pragma unroll
            for (int q = 0; q < kG; ++q) dot = fmaf(x[q][t] - mean[q], v[q], dot);
#pragma unroll
            for (int q = 0; q < kG; ++q) w[q] = fmaf(x[q][t] - mean[q], dot, w[q]);
          }
#pragma unroll
          for (int q = 0; q < kG; ++q) {
            v[q] = wave_total(w[q]);
            big = fmaxf(big, fabsf(v[q]));
          }
          const float by = big > 0.f ? 1.0f / big : 0.f;
#pragma unroll
          for (int q = 0; q < kG; ++q) v[q] *= by;
        }
        for (int i = lo + lane; i < hi; i += 64) {
          const int t = order[now][i];
          float dot = 0.f;
#pragma unroll
          for (int q = 0; q < kG; ++q) dot = fmaf(x[q][t] - mean[q], v[q], dot);
          const uint32_t bits = __float_as_uint(dot);      // in the order of the numbers; what is none has a place as well
          spot[i] = ((bits >> 31 ? ~bits : bits | 0x80000000u) & ~(kBuildChunk - 1u)) | (uint32_t)i;      // (no two alike)
        }
      }
      __syncthreads();
      for (int i = tid; i < nc; i += kBuildThreads) {
        int lo, hi, at;
        part_around(nc, level, i, lo, hi);
        at = i;
        if (hi - lo > kGroupShapes) {
          const uint32_t mine = spot[i];
          at = lo;
          for (int j = lo; j < hi; j += 4) {               // (parts begin and, but the last, end at whole groups)
            const uint4 o = *(const uint4*)&spot[j];
            at += (int)(o.x < mine) + (int)(o.y < mine) + (int)(o.z < mine) + (int)(o.w < mine);
          }
        }
        order[now ^ 1][at] = order[now][i];
      }
      now ^= 1;
      __syncthreads();
    }
    // Within a group by id: of equal scores a lane keeps the first row, which is then the lowest id, as in the whole search.
    // A thread per row (spot: the member there).
    for (int i = tid; i < nc; i += kBuildThreads) {
      const int t = order[now][i], g = i & ~(kGroupShapes - 1);
      const uint32_t k = id[t];
      int at = g;
      for (int j = g; j < min(g + kGroupShapes, nc); ++j) at += id[order[now][j]] < k;
      spot[at] = (uint32_t)t;
    }
    __syncthreads();
    const int group0 = (int)a.first_group[m] + n0 / kGroupShapes;
    for (int rec = tid; rec < groups * kGroupRecords; rec += kBuildThreads) {      // [group][shape][instruction, half]
      const int row = rec >> 2, part = rec & 3, r = row & (kGroupShapes - 1), g = group0 + row / kGroupShapes;
      const bool there = row < nc;
      const int t = there ? (int)spot[row] : 0;
      float shape[kG];
#pragma unroll
      for (int q = 0; q < kG; ++q) shape[q] = there ? x[q][t] : 0.f;
      a.frag[(long long)g * kGroupRecords + part * kGroupShapes + r] = shape_slots(shape, there, (part >> 1) * 16 + (part & 1) * 8);
      if (part == 0) a.ids[g * kGroupShapes + r] = there ? id[t] : 0xffffffffu;
    }
    for (int row = tid; row < (groups * kGroupShapes + 63) / 64 * 64; row += kBuildThreads) {       // (whole waves: eight lanes a group)
      const bool there = row < nc;
      const int t = there ? (int)spot[row] : 0;
      const float share = 1.0f / (float)max(1, min(kGroupShapes, nc - (row & ~(kGroupShapes - 1))));
      float c[kG], d2 = 0.f;
#pragma unroll
      for (int q = 0; q < kG; ++q) {
        c[q] = there ? x[q][t] : 0.f;
#pragma unroll
        for (int o = 1; o < kGroupShapes; o <<= 1) c[q] += __shfl_xor(c[q], o, kWave);
        c[q] *= share;
        const float d = there ? x[q][t] - c[q] : 0.f;
        d2 = fmaf(d, d, d2);
      }
      if (!(d2 >= 0.f)) d2 = 3.0e38f;             // (a row that is no number: its group is never left out)
#pragma unroll
      for (int o = 1; o < kGroupShapes; o <<= 1) d2 = fmaxf(d2, __shfl_xor(d2, o, kWave));
      uint4 rec[2];
      ball_operands(c, d2, false, rec[0], rec[1]);
      if ((row & (kGroupShapes - 1)) == 0 && there) {
        a.bound[(long long)(group0 + row / kGroupShapes) * 2] = rec[0];
        a.bound[(long long)(group0 + row / kGroupShapes) * 2 + 1] = rec[1];
      }
    }
  }
  if (n0 == 0) {                                  // the cell: the ball around its centre
    if (tid == 0) farthest = 0u;
    __syncthreads();
    const float* cr = centre_row(a, m);
    float c[kG];
#pragma unroll
    for (int k = 0; k < kG; ++k) c[k] = cr[k];
    float far = 0.f;
    for (int i = tid; i < n; i += kBuildThreads) {
      const float* s = a.cb + (long long)member[i] * kG;
      float d2 = 0.f;
#pragma unroll
      for (int q = 0; q < kG; ++q) {
        const float d = (i < nc ? x[q][i] : s[q]) - c[q];
        d2 = fmaf(d, d, d2);
      }
      if (!(d2 >= 0.f)) d2 = 3.0e38f;
      far = fmaxf(far, d2);
    }
    atomicMax(&farthest, __float_as_uint(far));
    __syncthreads();
    if (tid == 0) {
      uint4* rec = a.cell_bound + (long long)(m >> 5) * 64 + (m & 31);
      ball_operands(c, __uint_as_float(farthest), n == 0, rec[0], rec[32]);
    }
  }
  if (blockIdx.x == 0) {                          // groups without shapes behind the last one
    const int T = (int)a.first_group[a.M];
    for (int rec = tid; rec < kPadGroups * kGroupRecords; rec += kBuildThreads) {
      const int part = (rec / kGroupShapes) & 3;
      const float none[kG] = {};
      a.frag[(long long)T * kGroupRecords + rec] = shape_slots(none, false, (part >> 1) * 16 + (part & 1) * 8);
      if (rec < kPadGroups * kGroupShapes) a.ids[T * kGroupShapes + rec] = 0xffffffffu;
    }
  }
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}

template <typename IdxT>
__global__ __launch_bounds__(256, 6) void kan_assign_bounded_kernel(const CellArgs a) {
  // A wave's lists.  Only the wave itself reads them: LDS serves its accesses in order, and order() keeps the compiler to it.
  __shared__ uint16_t s_cells[4][kListCells], s_window[4][kListGroups + 64 * kAhead], s_visits[4][kListVisits + 16 * kAhead];
  auto order = [] { asm volatile("" ::: "memory"); };
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  // runs of consecutive workgroups on one XCD (workgroups go to the eight in turn): neighbours ask for the same groups
  const unsigned W = gridDim.x, xcd = blockIdx.x & 7u, q8 = W >> 3, r8 = W & 7u;
  const long long wg = xcd * q8 + min(xcd, r8) + (blockIdx.x >> 3);
  const long long pos = (wg * 4 + wave) * 32 + (lane & 31);
  if ((wg * 4 + wave) * 32 >= a.E) {                       // (no barrier in this kernel)
    if (lane == 0) a.left[wg * 4 + wave] = 0;
    return;
  }
  uint16_t* const cells = s_cells[wave];
  uint16_t* const window = s_window[wave];
  uint16_t* const visits = s_visits[wave];
  auto first_group = [&](int cell) { return __builtin_amdgcn_readfirstlane((int)a.first_group[cell]); };     // (for the whole wave)
  const int T = first_group(a.M), words = a.M / 32, most = (int)(kRestShare * T);

  const uint32_t e = a.sorted[1][min(pos, a.E - 1)];
  const int key = a.key[1][e] >> a.sub;           // its cell
  const bool there = pos < a.E, live = there && key < a.M;

  // edge operands of the search (see the head of the file) and of the bound
  h16x8 fb[2], fe;
  bool unit;
  {
    float n[kG], mean, gain;
    normalise(a.coef + (long long)e * kG, n, mean, gain);
    float nn = 0.f;
#pragma unroll
    for (int m = 0; m < kG; ++m) nn = fmaf(n[m], n[m], nn);
    unit = nn <= 1.000003f;      // (longer: squares in the subnormal range, below 1e-38, lose bits; the bounds do not hold)
    _Float16 hi[kG], lo[kG];
#pragma unroll
    for (int m = 0; m < kG; ++m) split_h(n[m], hi[m], lo[m]);
    auto slot = [&](int s) {
      return s < 10 ? hi[s] : (s == 10 || s == 31 ? (_Float16)1.0f : (s < 21 ? hi[s - 11] : lo[s - 21]));
    };
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      fb[0][t] = half ? slot(8 + t) : slot(t);
      fb[1][t] = half ? slot(24 + t) : slot(16 + t);
      fe[t] = half ? (t < 2 ? hi[8 + t] : (_Float16)(t < 4 ? 1.0f : 0.0f)) : hi[t];
    }
  }
  f32x16 zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;

  float best = -3.0e38f;
  int best_row = -1;             // where in the groups' rows the best shape lies
  // The first product of a shape that can win reaches `near` = best - slack (see first_product_slack).
  float slack = 0.f, near = 0.f;
  auto take = [&](float sc, int row) {           // (equal scores: the lower id)
    if (sc > best || (sc == best && a.ids[row] < a.ids[max(best_row, 0)])) best_row = row;
    best = fmaxf(best, sc);
    near = best - slack;
  };
  auto leave = [&] {                             // to the whole search
    if (lane == 0) a.left[wg * 4 + wave] = 1;
  };
  const __amdgpu_buffer_rsrc_t cell_rsrc = buffer_of(a.cell_bound, (size_t)a.M * 32);
  const __amdgpu_buffer_rsrc_t bound_rsrc = buffer_of(a.bound, (size_t)T * 32);
  const __amdgpu_buffer_rsrc_t frag_rsrc = buffer_of(a.frag, (size_t)(T + kPadGroups) * kGroupRecords * 16);
  auto load = [&](const __amdgpu_buffer_rsrc_t& rsrc, int lane_at, int at) {
    return __builtin_bit_cast(h16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_at, at, 0));
  };
  // A tile of the search: four groups, a lane's rows are those of group g (its own argument)
  const int row_at = (half * kGroupShapes + (lane & (kGroupShapes - 1))) * 16;
  auto load_rows = [&](int g, int instruction) {
    return load(frag_rsrc, g * (kGroupRecords * 16) + row_at, instruction * (kGroupRecords * 8));
  };
  // (g: the tile's four groups, the same for the whole wave.  Read from lanes inside the branch, the registers of the lanes
  // that are switched off there would not need to hold them.)
  auto take_tile = [&](const f32x16& acc, const int (&g)[4]) {
    for_groups_with(acc, best, [&](int q, int r, float m) { take(m, g[q] * kGroupShapes + 4 * half + r); });
  };

  // (1) own cells, both instructions of every tile
  int visited = 0;
  unsigned long long firsts = 0;                 // a lane of every own cell
  for (unsigned long long w = __ballot(live); w != 0;) {
    const int first = __ffsll(w) - 1, cell = __builtin_amdgcn_readlane(key, first);
    firsts |= 1ull << first;
    w &= ~__ballot(key == cell);
    const int g0 = first_group(cell), g1 = first_group(cell + 1);
    visited += g1 - g0;
    if (visited > most) {
      leave();
      return;
    }
    for (int t = g0; t < g1; t += 4) {           // (past the cell's last group: the next cell's, or one without shapes)
      const int g = t + ((lane & 31) >> 3);
      const h16x8 f0 = load_rows(g, 0), f1 = load_rows(g, 1);
      f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(f0, fb[0], zero, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(f1, fb[1], acc, 0, 0, 0);
      const int four[4] = {t, t + 1, t + 2, t + 3};
      take_tile(acc, four);
    }
  }

  // Distance to the best shape so far (scores are good to 1e-6).  The two lanes of an edge hold different rows:
  // they agree on the better shape first.
  auto distance = [&] {
    const float sc_o = __shfl_xor(best, 32, kWave);
    const int row_o = __shfl_xor(best_row, 32, kWave);
    if (row_o >= 0) take(sc_o, row_o);
    float dist = live ? sqrtf(fmaxf(0.f, 1.0f - 2.0f * best) + 4e-6f) : 0.f;
    if (live && !unit) dist = 2.0f * kFar;       // (every tile: the wave goes to the whole search)
    slack = live ? first_product_slack(dist) : -INFINITY;      // (an edge without direction asks for nothing)
    near = best - slack;
    return dist;
  };
  // The groups listed so far.  A tile whose first product comes near the best score gets the second instruction.
  int n_visits = 0;
  auto visit = [&] {
    // (to whole tiles and pairs of them: the last group again; what is loaded ahead of that is not used)
    order();
    const uint16_t last = visits[n_visits - 1];
    if (lane < 4 * kAhead) visits[n_visits + lane] = last;
    order();
    const uint16_t* at = visits + ((lane & 31) >> 3);
    auto examine = [&](int g, const f32x16& first) {
      int four[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) four[q] = __builtin_amdgcn_readlane(g, q * kGroupShapes);
      take_tile(__builtin_amdgcn_mfma_f32_32x32x16_f16(load_rows(g, 1), fb[1], first, 0, 0, 0), four);
    };
    int g[kAhead];
    h16x8 f[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      g[k] = at[4 * k];
      f[k] = load_rows(g[k], 0);
    }
    for (int i = 0; i < n_visits; i += 4 * kAhead) {
      at += 4 * kAhead;
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        const f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[k], fb[0], zero, 0, 0, 0);
        const int u = g[k];
        g[k] = at[4 * k];
        f[k] = load_rows(g[k], 0);
        if (__ballot(max_of(acc) >= near)) examine(u, acc);
      }
    }
    order();
    n_visits = 0;
  };
  // Every group that an edge with its bit in `who` asks for at distance d: of the cells that it asks for but the own ones,
  // a lane a cell, then of their groups.  False: too many.
  auto search = [&](bool who, float d) -> bool {
    int asked = 0;
    const bool far = d > kFar;                   // (no shape known yet, or beyond fp16: every tile)
    const float thr = who ? (far ? -6e4f : 0.5f * (1.0f - d * d) - 1e-5f) : 6e4f;
    const float thr_hi = fp16_of(thr);
    if (half) {
      fe[4] = (_Float16)(far ? 0.f : fp16_up(d));
      fe[5] = (_Float16)-thr_hi;
      fe[6] = (_Float16)(thr_hi - thr);
    }
    // bit c: an edge (the rows) asks for the ball of column c
    auto asks = [&](const h16x8& ball) {
      const unsigned long long any = __ballot(!(max_of(__builtin_amdgcn_mfma_f32_32x32x16_f16(fe, ball, zero, 0, 0, 0)) <= 0.f));
      return (uint32_t)any | (uint32_t)(any >> 32);
    };
    for (int w0 = 0; w0 < words; w0 += kListCells / 32) {
      const int w1 = min(words - w0, kListCells / 32);
      int mine = 0;                              // lane w: the cells of word w0 + w
      h16x8 f[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) f[k] = load(cell_rsrc, lane * 16, (w0 + min(k, w1 - 1)) * 1024);
      for (int w = 0; w < w1; w += kAhead) {     // (past the last word: that one again, struck out below)
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
          const int any = (int)asks(f[k]);
          f[k] = load(cell_rsrc, lane * 16, (w0 + min(w + k + kAhead, w1 - 1)) * 1024);
          mine = lane == w + k ? any : mine;
        }
      }
      if (lane >= w1) mine = 0;
      for (unsigned long long w = firsts; w != 0; w &= w - 1) {
        const int cell = __builtin_amdgcn_readlane(key, __ffsll(w) - 1);
        if (lane == (cell >> 5) - w0) mine &= ~(1 << (cell & 31));
      }
      const int own = __popc(mine), cells_to = sums_up_to(own), n_cells = __builtin_amdgcn_readlane(cells_to, 63);
      order();
      for (int at = cells_to - own; mine; ++at) {
        cells[at] = (uint16_t)((w0 + lane) * 32 + __ffs(mine) - 1);
        mine &= mine - 1;
      }
      order();
      for (int c0 = 0; c0 < n_cells; c0 += 64) {
        const bool one = c0 + lane < n_cells;
        const int cell = one ? cells[c0 + lane] : 0, g0 = (int)a.first_group[cell];
        const int ng = one ? (int)a.first_group[cell + 1] - g0 : 0, to = sums_up_to(ng), from = to - ng;
        const int total = __builtin_amdgcn_readlane(to, 63);
        for (int v0 = 0; v0 < total; v0 += kListGroups) {
          const int n = min(total - v0, kListGroups);
          order();
          for (int j = max(0, v0 - from); j < min(ng, v0 + kListGroups - from); ++j) window[from + j - v0] = (uint16_t)(g0 + j);
          order();
          int g[kAhead];
          const uint16_t* at = window + (lane & 31);
          auto load_ball = [&](int i) { return load(bound_rsrc, i * 32 + half * 16, 0); };
          // (past the last one: whatever stands there, struck out below)
#pragma unroll
          for (int k = 0; k < kAhead; ++k) {
            g[k] = at[32 * k];
            f[k] = load_ball(g[k]);
          }
          for (int i = 0; i < n; i += 32 * kAhead) {
            at += 32 * kAhead;
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
              const int group = g[k], rest = n - i - 32 * k;
              const uint32_t ones = asks(f[k]) & (rest >= 32 ? ~0u : (rest > 0 ? (1u << rest) - 1u : 0u));
              g[k] = at[32 * k];
              f[k] = load_ball(g[k]);
              if (lane < 32 && ((ones >> lane) & 1u)) visits[__builtin_amdgcn_mbcnt_lo(ones, n_visits)] = (uint16_t)group;
              n_visits += __popc(ones);
              asked += __popc(ones);
            }
          }
          if (asked > most) return false;
          const bool last = v0 + kListGroups >= total && c0 + 64 >= n_cells;       // (no empty cell is asked for)
          if (n_visits > (last ? 0 : kListVisits - kListGroups)) visit();
        }
      }
    }
    return true;
  };

  float d = distance(), asked_at;
  {
    auto mean_of = [&](bool which) {
      const int n = __popcll(__ballot(which));
      return n > 0 ? wave_total(which ? d : 0.f) / (float)n : 2.0f * kFar;
    };
    const float mean = mean_of(live && d <= kFar), low = mean_of(live && d <= mean);
    // the edges that have found their shape: their own distance, and the others what those would ask for
    const bool apart = kFound * low < kApart * mean;
    asked_at = !apart ? fminf(d, kPoor * mean) : (d <= kFound * low ? d : fminf(d, kAsk * low));
  }
  bool who = live;
  for (int step = 2; step <= 3 && __ballot(who); ++step) {
    if (!search(who, step == 2 ? asked_at : d)) {
      leave();
      return;
    }
    d = distance();
    who = live && d > asked_at;
  }
  if (lane == 0) a.left[wg * 4 + wave] = 0;
  // (an edge without direction: the shape of the smallest norm; one that is no number has no scores and gets row 0)
  if (lane < 32 && there) {
    const uint32_t id = live ? (best_row >= 0 ? a.ids[best_row] : 0u) : (a.gain[e] == a.gain[e] ? *a.least : 0u);
    ((IdxT*)a.idx)[e] = (IdxT)id;
  }
}

// ---- reconstruction quality ---------------------------------------------------------------------
// Sums for R^2 between the dense grids and their reconstruction gain * C[idx] + bias:
// per workgroup {sum of squared residuals, sum of c, sum of c^2} in fp64, then one
// fixed-order pass over the workgroups.
template <typename IdxT>
__global__ __launch_bounds__(256) void kan_recon_partial_kernel(const float* __restrict__ coef,
                                                                const float* __restrict__ cb,
                                                                const IdxT* __restrict__ idx,
                                                                const float* __restrict__ gain,
                                                                const float* __restrict__ bias, long long E,
                                                                double* __restrict__ part) {
  __shared__ double red[3][256];
  double sr = 0.0, s1 = 0.0, s2 = 0.0;
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < E; e += (long long)gridDim.x * blockDim.x) {
    const float* c = coef + e * kG;
    const float* r = cb + (long long)idx[e] * kG;
    const double g = gain[e], b = bias[e];
#pragma unroll
    for (int m = 0; m < kG; ++m) {
      const double v = c[m], d = v - (g * (double)r[m] + b);
      sr += d * d;
      s1 += v;
      s2 += v * v;
    }
  }
  red[0][threadIdx.x] = sr;
  red[1][threadIdx.x] = s1;
  red[2][threadIdx.x] = s2;
  __syncthreads();
  if (threadIdx.x < 3) {
    double t = 0.0;
    for (int q = 0; q < 256; ++q) t += red[threadIdx.x][q];
    part[(long long)blockIdx.x * 3 + threadIdx.x] = t;
  }
}

// sums[0..2] = the three totals; sums[3] = R^2 = 1 - SS_res / SS_tot with SS_tot taken about the
// overall mean of the n_coef coefficients (section 4.2).
__global__ void kan_recon_final_kernel(const double* __restrict__ part, int n_blocks, double n_coef,
                                       double* __restrict__ sums) {
  __shared__ double tot[3];
  if (threadIdx.x < 3) {
    double t = 0.0;
    for (int q = 0; q < n_blocks; ++q) t += part[(long long)q * 3 + threadIdx.x];
    sums[threadIdx.x] = t;
    tot[threadIdx.x] = t;
  }
  __syncthreads();
  if (threadIdx.x == 0) sums[3] = 1.0 - tot[0] / (tot[2] - tot[1] * tot[1] / n_coef);
}

}  // namespace

size_t assign_centroid_bytes(int K) { return centroid_bytes(K); }
int recon_blocks(long long E) {
  const long long b = (E + 255) / 256;
  return (int)(b < 1024 ? b : 1024);
}

namespace {
size_t round256(size_t n) { return (n + 255) / 256 * 256; }
constexpr int kFilterTiles = 256;                 // tiles of a part (both sides at the head of the whole search)
// Operands of all shapes in LDS: 40 KB at most, four workgroups of a CU.  512 shapes and 65,536 / 131,072 / 358,400 edges 9.2 /
// 11.0 / 21.0 us so, 9.9 / 14.1 / 29.3 with the waves sharing their edges; 640 shapes 10.7 / 13.3 / 25.4 against 10.3 / 15.1 /
// 32.6.  (700 shapes, three workgroups of a CU: 2^18 edges 24.1 against 22.9 with waves on their own.)
constexpr int kLocalShapes = 640;
constexpr long long kLocalMaxWork = 500000000;
constexpr unsigned kLocalWorkgroups = 1024;       // what is resident
// Every workgroup builds them, which takes longer than shared edges do where a CU has one workgroup of these: 4,096 / 32,768
// edges x 384 shapes 8.0 / 7.9 against 7.9 / 8.4 us, x 448 8.5 / 8.5 against 8.3 / 8.7, x 512 8.9 / 9.4 against 8.2 / 8.4; and with
// two where a workgroup has not a row for every thread once more: 65,536 x 512 9.2 against 9.9, 46,948 x 627 11.0 against 10.1.
bool local_ok(long long E, int K) {
  if (E * K >= kLocalMaxWork || K > kLocalShapes) return false;
  return E > (1ll << 16) || K <= 384 || (E > (1ll << 15) && K <= 512);
}
// Waves on their own with operands from memory, four tiles of edges each, from 3 * 2^18 edges.  Against operands in LDS (from
// kLocalMaxWork): 2^20 / 1,536,000 edges x 300 shapes 34.5 / 47.3 us against 35.7 / 50.9, 953,281 x 305 34.8 against 33.1, 786,432 x
// 640 45.2 against 48.7.  Against shared edges: 665,600 / 786,432 edges x 4,096 205 / 210 against 194 / 223; with fewer shapes the
// first edges come to more of the time: 229,376 x 641 21 against 24, 196,608 / 2^18 x 768 24 / 24 against 23 / 28, 2^18 / 358,400 x
// 1,000 30 / 38 against 32 / 41, 358,400 / 402,408 / 524,288 x 1,500 52 / 61 / 65 against 52 / 59 / 72, 358,400 / 524,288 x 2,048
// 64 / 83 against 63 / 88.
constexpr long long kOwnMinEdges = 3ll << 18;
bool own_ok(long long E, int K) { return E >= kOwnMinEdges || (E >= (7ll << 15) && E >= 320ll * K); }

enum class Search { kLocal, kOwn, kWhole };
Search search_of(long long E, int K) { return local_ok(E, K) ? Search::kLocal : (own_ok(E, K) ? Search::kOwn : Search::kWhole); }

// Parts of the codebook: by the work of the fullest CU.  A step of a workgroup (eight tiles of shapes, 128 edges) takes 0.58 us
// alone on its CU, 0.92 for two there, 0.47 each for more; the first ones, with a new best in nearly every tile, as long as
// eight more; the second launch 3 us.  2^13 edges x 65,536 shapes in 4 / 8 / 16 parts 55 / 47 / 54 us, 24,000 in 2 / 4 / 6 110 /
// 102 / 115, 32,768 in 1 / 2 / 4 151 / 118 / 126, 65,536 in 1 / 2 217 / 217.
int whole_parts_of(long long E, int K, double* us) {
  const long long groups = (E + kWholeEdges - 1) / kWholeEdges;
  const int n_tiles = (K + 31) / 32;
  int best = 1;
  double least = 0.0;
  for (int parts = 1; parts <= std::min(32, std::max(1, n_tiles / kWholeWaves)); ++parts) {
    const long long n = (groups * parts + 255) / 256;        // workgroups of the fullest CU
    const int steps = ((n_tiles + parts - 1) / parts + kWholeWaves - 1) / kWholeWaves;
    const double t = (steps + 8) * (n == 1 ? 0.58 : (n == 2 ? 0.92 : 0.47 * (double)n)) + (parts > 1 ? 3.0 : 0.0);
    if (parts == 1 || t < least) {
      least = t;
      best = parts;
    }
  }
  if (us) *us = least;
  return best;
}
int whole_parts(long long E, int K) { return search_of(E, K) == Search::kWhole ? whole_parts_of(E, K, nullptr) : 1; }
size_t whole_bytes(long long E, int K, int parts) {
  return round256(centroid_bytes(K)) + (parts > 1 ? (size_t)parts * (size_t)E * sizeof(uint2) : 0);
}
}  // namespace
size_t assign_whole_bytes(long long E, int K) { return whole_bytes(E, K, whole_parts(E, K)); }

// The bounded search pays where its cells, launches and bound tests (90 us and more that hardly depend on the edges) are small
// next to the scores they save, for grids that fit their codebook and at little loss for those that do not.  Bounded search with
// 2 % / 5 % / 15 % noise per coefficient / unrelated grids against the whole search (which hardly cares), us:
//     K = 65,536   2^20 edges  332 / 491 / 885 / 908                  2^16 edges  5 %: 160 against 217
//                  2^15 edges  119 / 159 / 225 / 218  against 118
//     K = 32,768   2^17 edges  105 / 130 / 193 / 192                  2^16 edges  98 / 121 / 173 / 169  against 125
//     K = 16,384   2^20 edges  203 / 286 / 552 / 561                  2^18 edges  102 / 131 / 210 / 216
//                  2^17 edges  85 / 103 / 152 / 154   against 124     98,304      5 %: 100 against 97
//     K = 8,192    2^20 edges  184 / 243 / 445 / 443                  2^19 edges  124 / 159 / 266 / 263
//                  2^18 edges  96 / 117 / 178 / 177
//     K = 4,096    2^20 edges  168 / 211 / 355 / 362  against 282
//     K = 119,045  34,440 edges  171 / 220 / -         against 267    K = 131,072  66,030 edges  - / - / 374  against 480
//     K = 262,144  16,524 edges  - / 448 / 634         against 283    33,304  - / - / 588  against 530
//     K = 330,923  13,760 edges  - / 513 / 758         against 266
// The call does not know the noise.  The bounded search is taken where it is ahead with 5 %: 72 us + 1.28 ns a shape + 0.125 to 0.38
// ns an edge, growing by 0.047 as the shapes double from 8,192 on (15 % off at most in 19 of 20 of 1,116 calls), against the
// whole search's steps above, whose time jumps with the workgroups of the fullest CU (98,304 edges are three of them there, 98,944
// four: 16,384 and 17,688 shapes, bounded / whole 100 / 97 and 106 / 123 us).  Near that line grids with 15 % lose up to half (43,168 x
// 65,536 shapes), so a plain line in front of it keeps calls whole where they would lose that for little: (E - 25000) K >= 1.2e9 from 16,384
// shapes on, 2^32 scores from 8,192 on.  In 1,179 calls of 8,192 to 331,338 shapes the search taken is behind the better one by 0.9 % on
// average with 5 %, 2.4 % with 2 % and 1.0 % with 15 % (the plain line alone 1.6, 2.4 and 2.6: it took few edges against very many
// shapes, 13,760 x 330,923 513 / 266).  Grids that fit their codebook better would gain below it (34,020 edges x 65,536 shapes with 2 %
// 122 / 159); a caller who knows of a poor fit passes the smaller workspace and gets the whole search.
bool assign_bounded_ok(long long E, int K) {
  if (K < 8192 || cell_layout(1, K).groups_max > kCellMaxGroups) return false;
  if (K < 16384) return E * K >= (1ll << 32);
  if ((E - 25000) * K < 1200000000ll) return false;
  if (E >= kOwnMinEdges) return true;
  double whole;
  whole_parts_of(E, K, &whole);
  return 72.0 + 1.28e-3 * K + (double)E * (1.25e-4 + 4.7e-5 * std::log2(K / 8192.0)) < whole;
}
size_t assign_bounded_bytes(long long E, int K) { return cell_layout(E, K).bytes; }

hipError_t launch_assign_bounded(const float* coef, long long E, const float* cb, int K, int idx_u32, void* idx,
                                 float* gain, float* bias, void* ws, hipStream_t s) {
  const CellLayout g = cell_layout(E, K);
  char* w = (char*)ws;
  CellArgs a;
  a.coef = coef;
  a.cb = cb;
  a.E = E;
  a.K = K;
  a.M = g.M;
  a.sub = g.sub;
  a.shape_wgs = (K + kEdgesPerWg - 1) / kEdgesPerWg;
  a.centres = (uint4*)(w + g.centres);
  a.frag = (uint4*)(w + g.frag);
  a.ids = (uint32_t*)(w + g.ids);
  a.cell_bound = (uint4*)(w + g.cell_bound);
  a.bound = (uint4*)(w + g.bound);
  a.sorted[0] = (uint32_t*)(w + g.member);
  a.sorted[1] = (uint32_t*)(w + g.perm);
  for (int p = 0; p < 2; ++p) {
    a.bins[p] = g.bins[p];
    a.groups[p] = g.groups[p];
    a.chunk[p] = g.chunk[p];
    a.key[p] = (uint16_t*)(w + g.key[p]);
    a.hist[p] = (uint32_t*)(w + g.hist[p]);
    a.total[p] = (uint32_t*)(w + g.total[p]);
    a.first[p] = (uint32_t*)(w + g.first[p]);
  }
  a.first_group = (uint32_t*)(w + g.first_group);
  a.wg_least = (unsigned long long*)(w + g.wg_least);
  a.left = (uint8_t*)(w + g.left);
  a.least = (uint32_t*)(w + g.least);
  a.idx = idx;
  a.gain = gain;
  a.bias = bias;
  const unsigned edge_wgs = (unsigned)((E + kEdgesPerWg - 1) / kEdgesPerWg);
  const dim3 sort_grid((unsigned)(g.groups[0] > g.groups[1] ? g.groups[0] : g.groups[1]), 2);
  const size_t cells_lds = (size_t)g.bins[1] * 4;
  hipLaunchKernelGGL(kan_cell_centres_kernel, dim3((unsigned)((g.M * 2 + 255) / 256)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(kan_cells_kernel, dim3((unsigned)a.shape_wgs + edge_wgs), dim3(kAssignThreads), 0, s, a);
  hipLaunchKernelGGL(kan_cell_count_kernel, sort_grid, dim3(kSortThreads), cells_lds, s, a);
  hipLaunchKernelGGL(kan_cell_chunks_kernel, dim3((unsigned)((g.bins[1] + 63) / 64), 2), dim3(256), 0, s, a);
  hipLaunchKernelGGL(kan_cell_scan_kernel, dim3(1), dim3(kSortThreads), 0, s, a);
  hipLaunchKernelGGL(kan_cell_place_kernel, sort_grid, dim3(kSortThreads), cells_lds, s, a);
  hipLaunchKernelGGL(kan_cell_build_kernel, dim3((unsigned)(g.M + (K + kBuildChunk - 1) / kBuildChunk)), dim3(kBuildThreads), 0, s, a);
  const dim3 grid((unsigned)((E + 127) / 128));
  if (idx_u32) hipLaunchKernelGGL(kan_assign_bounded_kernel<uint32_t>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(kan_assign_bounded_kernel<uint16_t>, grid, dim3(256), 0, s, a);
  RestArgs rest = {};
  rest.coef = coef;
  rest.cent = a.frag;
  rest.E = E;
  rest.list = a.sorted[1];
  rest.left = a.left;
  rest.groups = a.first_group + g.M;
  rest.ids = a.ids;
  rest.idx = idx;
  const dim3 rest_grid((unsigned)std::min<long long>((E + 127) / 128, kRestWorkgroups));
  if (idx_u32) hipLaunchKernelGGL(kan_assign_rest_kernel<uint32_t>, rest_grid, dim3(kWholeWaves * kWave), 0, s, rest);
  else hipLaunchKernelGGL(kan_assign_rest_kernel<uint16_t>, rest_grid, dim3(kWholeWaves * kWave), 0, s, rest);
  return hipGetLastError();
}

hipError_t launch_assign(const float* coef, long long E, const float* cb, int K, int idx_u32, void* idx, float* gain,
                         float* bias, void* ws, size_t ws_bytes, hipStream_t s) {
  WholeArgs a = {};
  a.coef = coef;
  a.cent = (const uint4*)ws;
  a.E = E;
  a.n_tiles = (K + 31) / 32;
  a.idx = idx;
  a.gain = gain;
  a.bias = bias;
  auto own = [&](auto tiles, auto local, unsigned most, size_t lds) {
    constexpr int kOwn = kAssignThreads / kWave * 32 * tiles.value;
    const dim3 grid((unsigned)std::min<long long>((E + kOwn - 1) / kOwn, most)), block(kAssignThreads);
    if (idx_u32) hipLaunchKernelGGL((kan_assign_own_kernel<uint32_t, tiles.value, local.value>), grid, block, lds, s, a, cb, K);
    else hipLaunchKernelGGL((kan_assign_own_kernel<uint16_t, tiles.value, local.value>), grid, block, lds, s, a, cb, K);
    return hipGetLastError();
  };
  using std::integral_constant;
  const Search search = search_of(E, K);
  if (search == Search::kLocal)
    return own(integral_constant<int, 2>(), std::true_type(), kLocalWorkgroups, (size_t)a.n_tiles * 2 * 64 * sizeof(uint4));
  const long long recs = (long long)a.n_tiles * 2 * 64;
  hipLaunchKernelGGL(kan_assign_prep_kernel, dim3((unsigned)((recs + 255) / 256)), dim3(256), 0, s, cb, K, a.n_tiles, (uint4*)ws);
  if (search == Search::kOwn) return own(integral_constant<int, 4>(), std::false_type(), 1u << 30, 0);
  a.parts = ws_bytes < assign_whole_bytes(E, K) ? 1 : whole_parts(E, K);
  a.part_tiles = (a.n_tiles + a.parts - 1) / a.parts;
  a.parts = (a.n_tiles + a.part_tiles - 1) / a.part_tiles;
  a.found = (uint2*)((char*)ws + round256(centroid_bytes(K)));
  const dim3 grid((unsigned)((E + kWholeEdges - 1) / kWholeEdges * a.parts)), join((unsigned)((E + 255) / 256));
  const dim3 block(kWholeWaves * kWave);
  const bool filter = a.part_tiles >= kFilterTiles;
  if (idx_u32 && filter) hipLaunchKernelGGL((kan_assign_whole_kernel<uint32_t, true>), grid, block, 0, s, a);
  else if (idx_u32) hipLaunchKernelGGL((kan_assign_whole_kernel<uint32_t, false>), grid, block, 0, s, a);
  else if (filter) hipLaunchKernelGGL((kan_assign_whole_kernel<uint16_t, true>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((kan_assign_whole_kernel<uint16_t, false>), grid, block, 0, s, a);
  if (a.parts > 1) {
    if (idx_u32) hipLaunchKernelGGL(kan_assign_join_kernel<uint32_t>, join, dim3(256), 0, s, a.found, a.parts, E, (uint32_t*)idx);
    else hipLaunchKernelGGL(kan_assign_join_kernel<uint16_t>, join, dim3(256), 0, s, a.found, a.parts, E, (uint16_t*)idx);
  }
  return hipGetLastError();
}

hipError_t launch_recon_sums(const float* coef, long long E, const float* cb, int idx_u32, const void* idx,
                             const float* gain, const float* bias, double* part, double* sums, hipStream_t s) {
  const int nb = recon_blocks(E);
  if (idx_u32)
    hipLaunchKernelGGL(kan_recon_partial_kernel<uint32_t>, dim3(nb), dim3(256), 0, s, coef, cb, (const uint32_t*)idx,
                       gain, bias, E, part);
  else
    hipLaunchKernelGGL(kan_recon_partial_kernel<uint16_t>, dim3(nb), dim3(256), 0, s, coef, cb, (const uint16_t*)idx,
                       gain, bias, E, part);
  hipLaunchKernelGGL(kan_recon_final_kernel, dim3(1), dim3(64), 0, s, (const double*)part, nb, (double)E * kG, sums);
  return hipGetLastError();
}

}  // namespace kan
