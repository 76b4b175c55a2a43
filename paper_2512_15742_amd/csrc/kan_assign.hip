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

// That is the whole search (kan_assign_kernel).  Large codebooks take the bounded search further down, which
// finds the same shapes from a small part of the scores.

#include <algorithm>

#include "kan_device.hpp"
#include "kan_internal.hpp"
#include "kan_mfma_common.hpp"

namespace kan {
namespace {

constexpr int kAssignThreads = 256;
constexpr int kEdgeTilesPerWave = 4;                                   // 4 x 32 edges per wave
constexpr int kEdgesPerWg = (kAssignThreads / kWave) * kEdgeTilesPerWave * 32;   // 512
constexpr long long kSplitMaxEdges = 1ll << 17;                         // whole search: up to here eight waves share their edges
constexpr int kSlots = 32;                                             // contraction length

__device__ __forceinline__ void split_h(float v, _Float16& hi, _Float16& lo) {
  hi = (_Float16)v;
  lo = (_Float16)(v - (float)hi);
}

// Slots s0 .. s0+7 of a shape's operand.  Without a shape (rows past the last one) the norm term is minus infinity,
// so that the row never wins, whatever the norms of the shapes.  Both searches take these, and the products in this
// order: a score has the same bits in either.
__device__ __forceinline__ uint4 shape_slots(const float* __restrict__ cb, long long c, bool there, int s0) {
  h16x8 v;
  float row[kG], nrm = 0.f;
#pragma unroll
  for (int m = 0; m < kG; ++m) {
    row[m] = there ? cb[c * kG + m] : 0.f;
    nrm = fmaf(row[m], row[m], nrm);
  }
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
  out[rec] = shape_slots(cb, c, c < K, ks * 16 + (lane >> 5) * 8);
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
// The first register that holds it.
__device__ __forceinline__ int row_of(const f32x16& v, float m) {
  int r_best = 15;
#pragma unroll
  for (int r = 14; r >= 0; --r) r_best = v[r] == m ? r : r_best;
  return r_best;
}

struct AssignArgs {
  const float* coef;        // [E][10]
  const uint4* cent;        // prepared centroid operands
  long long E;
  // LIST: behind the bounded search, on its tiles.  The edges in its order, and of every 32 whether they are left (their
  // gains and biases are there already); the number of tiles and the shape of every row
  const uint32_t* list;
  const uint8_t* left;      // [4 * ceil(E / 128)]
  const uint32_t *tiles, *ids;
  int n_tiles;              // ceil(K / 32)
  void* idx;
  float* gain;
  float* bias;
};

// SPLIT = 1: four waves with 128 edges of their own each.  SPLIT > 1: that many waves share 128 edges and take the
// centroid tiles in turn: with few edges a wave's chain of tiles is what takes the time (K = 4,096 and 2^11 / 2^16 /
// 2^17 edges 21 / 34 / 58 us with eight waves against 85 / 89 / 91 us, with 2^18 edges 104 against 107, above it loses).
template <typename IdxT, int SPLIT, bool LIST>
__global__ __launch_bounds__(SPLIT > 1 ? SPLIT * kWave : kAssignThreads, 4) void kan_assign_kernel(const AssignArgs a) {
  static_assert(!LIST || SPLIT > 1, "a workgroup's edges are four tiles of the list");
  constexpr int kThreads = SPLIT > 1 ? SPLIT * kWave : kAssignThreads;
  constexpr int kEdges = SPLIT > 1 ? kEdgeTilesPerWave * 32 : kEdgesPerWg;
  // edge-side operands of the workgroup's edges: [edge][32 slots] fp16
  __shared__ __attribute__((aligned(16))) _Float16 sB[kEdges * kSlots];
  __shared__ float s_best[SPLIT > 1 ? SPLIT : 1][SPLIT > 1 ? kEdges : 1];
  __shared__ int s_id[SPLIT > 1 ? SPLIT : 1][SPLIT > 1 ? kEdges : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int first_tile = SPLIT > 1 ? 0 : wave * kEdgeTilesPerWave;        // of the wave's edges
  const long long E = a.E;
  auto edge_at = [&](long long at) { return LIST ? (long long)a.list[at] : at; };
  // One workgroup's share: the edges from e_wg on, LIST: of these the tiles with their byte set in `tiles`.
  auto serve = [&](long long e_wg, uint32_t tiles) {
    // ---- step 1: bias = mean, gain = norm of the centred grid, n = centred / gain ------------
    for (int q = tid; q < kEdges; q += kThreads) {
      const long long at = e_wg + q, e = edge_at(min(at, E - 1));
      float c[kG], mean, g;
      normalise(a.coef + e * kG, c, mean, g);
      if (!LIST && at < E) {
        a.gain[e] = g;
        a.bias[e] = mean;
      }
      _Float16* p = sB + q * kSlots;
#pragma unroll
      for (int m = 0; m < kG; ++m) {
        _Float16 hi, lo;
        split_h(c[m], hi, lo);
        p[m] = hi;
        p[11 + m] = hi;
        p[21 + m] = lo;
      }
      p[10] = (_Float16)1.0f;
      p[31] = (_Float16)1.0f;
    }
    __syncthreads();

    // ---- this wave's edge fragments (MFMA B operand: column = lane & 31, slots (lane/32)*8..+8) --
    h16x8 fb[kEdgeTilesPerWave][2];
#pragma unroll
    for (int nb = 0; nb < kEdgeTilesPerWave; ++nb)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const int q = (first_tile + nb) * 32 + (lane & 31);
        fb[nb][ks] = *(const h16x8*)(sB + q * kSlots + ks * 16 + (lane >> 5) * 8);
      }

    float best[kEdgeTilesPerWave];
    int best_tile[kEdgeTilesPerWave], best_row[kEdgeTilesPerWave];
#pragma unroll
    for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
      best[nb] = -3.0e38f;
      best_tile[nb] = 0;
      best_row[nb] = 0;
    }

    // ---- step 3: stream the centroid tiles (two tiles in flight) -----------------------------------
    const int n_tiles = LIST ? (int)*a.tiles : a.n_tiles;
    const uint4* cp = a.cent + lane;
    auto load_tile = [&](int t, uint4 (&fa)[2]) {
      const int tc = t < n_tiles ? t : n_tiles - 1;        // past the end: a harmless re-read
      fa[0] = cp[(long long)(tc * 2) * 64];
      fa[1] = cp[(long long)(tc * 2 + 1) * 64];
    };
    f32x16 zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.f;
    auto score_tile = [&](int t, const uint4 (&fa)[2]) {
      const h16x8 a0 = __builtin_bit_cast(h16x8, fa[0]), a1 = __builtin_bit_cast(h16x8, fa[1]);
#pragma unroll
      for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
        if (LIST && !((tiles >> (8 * nb)) & 1u)) continue;
        f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, fb[nb][0], zero, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, fb[nb][1], acc, 0, 0, 0);
        const float m = max_of(acc);
        // A new best is rare (the t-th tile improves a lane's running maximum with probability
        // ~1/t), so the row is looked for only then.  Strictly greater: the earliest tile, and in
        // it the lowest register, keeps a tie.  (LIST: the lowest id, whatever tile it lies in.)
        if constexpr (LIST) {
          if (m >= best[nb]) {
            const int r = row_of(acc, m), id = (int)a.ids[t * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)];
            if (m > best[nb] || (uint32_t)id < (uint32_t)best_tile[nb]) best_tile[nb] = id;
            best[nb] = m;
          }
        } else if (m > best[nb]) {
          best[nb] = m;
          best_tile[nb] = t;
          best_row[nb] = row_of(acc, m);
        }
      }
    };
    uint4 fa0[2], fa1[2];
    const int t0 = SPLIT > 1 ? wave : 0;
    load_tile(t0, fa0);
    load_tile(t0 + SPLIT, fa1);
    for (int t = t0; t < n_tiles; t += 2 * SPLIT) {
      score_tile(t, fa0);
      load_tile(t + 2 * SPLIT, fa0);
      if (t + SPLIT < n_tiles) score_tile(t + SPLIT, fa1);
      load_tile(t + 3 * SPLIT, fa1);
    }

    // ---- the two half-waves hold different rows of the same edges: keep the better one ------------
#pragma unroll
    for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
      const int r = best_row[nb];
      // D layout of the 32x32 MFMA: register r of a lane is row 8*(r/4) + 4*(lane/32) + r%4
      int id = LIST ? best_tile[nb] : best_tile[nb] * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      float sc = best[nb];
      const float sc_o = __shfl_xor(sc, 32, kWave);
      const int id_o = __shfl_xor(id, 32, kWave);
      if (sc_o > sc || (sc_o == sc && id_o < id)) {
        id = id_o;
        sc = sc_o;
      }
      const int q = (first_tile + nb) * 32 + (lane & 31);
      if constexpr (SPLIT > 1) {
        if (lane < 32) {
          s_best[wave][q] = sc;
          s_id[wave][q] = id;
        }
      } else {
        const long long at = e_wg + q;
        if (lane < 32 && at < E) ((IdxT*)a.idx)[at] = (IdxT)id;
      }
    }
    if constexpr (SPLIT > 1) {
      __syncthreads();
      const long long at = e_wg + tid;
      if (tid < kEdges && at < E && (!LIST || ((tiles >> (8 * (tid >> 5))) & 1u))) {
        float sc = s_best[0][tid];
        int id = s_id[0][tid];
#pragma unroll
        for (int w = 1; w < SPLIT; ++w) {
          const float o = s_best[w][tid];
          const int io = s_id[w][tid];
          if (o > sc || (o == sc && io < id)) {
            sc = o;
            id = io;
          }
        }
        ((IdxT*)a.idx)[edge_at(at)] = (IdxT)id;
      }
    }
  };
  if constexpr (LIST) {
    const long long groups = (E + kEdges - 1) / kEdges;
    for (long long g0 = blockIdx.x; g0 < groups; g0 += (long long)kWave * gridDim.x) {
      const long long mine = g0 + (long long)lane * gridDim.x;
      const uint32_t flags = mine < groups ? ((const uint32_t*)a.left)[mine] : 0u;
      for (unsigned long long m = __ballot(flags != 0); m; m &= m - 1) {
        const int l = __ffsll(m) - 1;
        serve((g0 + (long long)l * gridDim.x) * kEdges, (uint32_t)__builtin_amdgcn_readlane((int)flags, l));
        __syncthreads();
      }
    }
  } else {
    serve((long long)blockIdx.x * kEdges, 0u);
  }
}

// ---- bounded search -------------------------------------------------------------------------------
// The codebook is cut into cells (the shapes nearest to one of M = K / 64 sampled shapes, the cell's centre c)
// and a cell into tiles of 32 shapes sorted by their distance to c.  A tile whose shapes all lie within R of c can be
// left out for an edge n that knows a shape at distance d already when |n - c| > R + d; in scores (|n| = 1)
//     n . c - |c|^2 / 2 + R^2 / 2 + R d  <  (1 - d^2) / 2 .
// The left side is a product of an edge's vector (n, 1, d) with a tile's vector (c, (R^2 - |c|^2) / 2, R), so one
// v_mfma_f32_32x32x16_f16 tests 32 edges against 32 tiles, the right side included; what the fp16 operands
// round away is covered by a margin.  The edges are sorted by their nearest centre, so that the 32 of a wave ask for
// about the same tiles, and a wave scores every tile that any of its edges asks for:
//     (1) the tiles of the edges' own cells: seven of ten edges with 5 % noise find their shape here;
//     (2) the tiles within R + min(d, the wave's mean d): finds nearly all of the others, whose d of step 1 alone
//         would ask for a large part of the codebook;
//     (3) where an edge is left with a larger d: what that one still asks for.
// The scores are those of the whole search, bit for bit, no tile that can hold the best one is left out and equal
// scores go to the lowest id: the result is the whole search's, whichever edges share a wave (the sort places them in
// no particular order) and whichever of them are handed over: a wave that would visit more than kRestShare of the tiles
// in (2) or in (3) leaves its edges to the whole search.  A visit costs about what a tile costs there, so that is worth
// it only for edges that ask for nearly everything (vectors that the bounds do not hold for, codebooks of one shape):
// grids that fit their codebook poorly ask for less, and stay.  With 25 % noise or unrelated grids, 2^20 edges: 234 of
// 330 tiles for K = 8,192, 356 of 630 for 16,384, 636 of 2,500 for 65,536.  With 0.7 of the tiles for both steps
// together and the left edges compacted by one counter, unrelated grids took 1003 us for K = 8,192 against 528 of the
// whole search alone and 471 against 292 for K = 16,384, 2^18 edges (a few waves left behind there were one chain
// through all tiles, 340 us); now 553 and 252.
//
// What bounds it: instructions issued and operands.  A wave of the search makes (tiles / 32) bound tests and visits
// about 250 of 2,500 tiles (65,536 shapes, 5 % noise; 15 % noise: 600), each 1 KB of operands, one matrix and about ten
// vector instructions; the counters show the address units busy for 65 % of the time, the matrix pipe for a third.
// What that took, 2048 x 512 edges against 65,536 shapes: two instructions a visit and tiles picked from bit masks by
// scalar code 1057 us, one instruction a visit 1084, more loads in flight 998, tiles listed in LDS and taken in
// pairs 818, the second instruction in place of vector arithmetic for near scores 761, six waves per SIMD
// 690; cells of 64 instead of 32 shapes (the choice of the cells 154 -> 87 us).  The whole search takes 3.8 ms.

constexpr int kCellShapes = 64;                   // shapes per cell on average
constexpr int kCellMaxTiles = 16384;              // (a wave marks the tiles it has visited in LDS)
constexpr float kRestShare = 0.9f, kMeanFactor = 1.0f;          // (0.6 / 0.7: K = 8,192, unrelated grids 1153 / 873 us)
constexpr float kFar = 100.0f;                    // distances above are not bounded in fp16
constexpr int kRestWorkgroups = 1024;             // of the whole search behind it: twice what is resident
constexpr int kAhead = 2;                         // tiles in flight per wave
constexpr int kSortThreads = 1024, kSortGroups = 64;
constexpr int kBuildChunk = 1024;                 // members of a cell that are sorted together

// Where the pieces of the search lie in the workspace.
struct CellLayout {
  int M;                   // cells, a multiple of 32
  int tiles_max;
  int groups[2];           // workgroups of the sort: over the shapes, over the edges
  long long chunk[2];      // items per workgroup
  size_t centres, frag, ids, bound, member, perm, key[2], hist[2], total[2], first[2], first_tile, wg_least, least, left, bytes;
};

size_t centroid_bytes(int K) { return (size_t)((K + 31) / 32) * 2 * 64 * sizeof(uint4); }

CellLayout cell_layout(long long E, int K) {
  CellLayout g;
  g.M = (K / kCellShapes + 31) / 32 * 32;
  g.tiles_max = (K + 31) / 32 + g.M;
  size_t at = 0;
  auto take = [&](size_t bytes) {
    const size_t here = at;
    at += (bytes + 255) / 256 * 256;
    return here;
  };
  g.centres = take((size_t)g.M * 2 * sizeof(uint4));
  g.frag = take((size_t)g.tiles_max * 2 * 64 * sizeof(uint4));
  g.ids = take((size_t)g.tiles_max * 32 * 4);
  g.bound = take((size_t)((g.tiles_max + 31) / 32) * 64 * sizeof(uint4));
  g.member = take((size_t)K * 4);
  g.perm = take((size_t)E * 4);
  for (int p = 0; p < 2; ++p) {
    const long long n = p ? E : K;
    const long long groups = (n + kSortThreads - 1) / kSortThreads;
    g.groups[p] = (int)(groups < kSortGroups ? groups : kSortGroups);
    g.chunk[p] = (n + g.groups[p] - 1) / g.groups[p];
    g.key[p] = take((size_t)n * 2);
    g.hist[p] = take((size_t)g.groups[p] * (g.M + 1) * 4);
    g.total[p] = take((size_t)(g.M + 1) * 4);
    g.first[p] = take((size_t)(g.M + 1) * 4);
  }
  g.first_tile = take((size_t)(g.M + 1) * 4);
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
  int K, M;
  int shape_wgs;                 // kan_cells_kernel: workgroups over the shapes, in front of those over the edges
  int groups[2];
  long long chunk[2];
  uint4* centres;                // operands of the centres
  uint4* frag;                   // operands of the tiles
  uint32_t* ids;                 // shape of every tile row
  uint4* bound;                  // bound operands of the tiles
  uint32_t* sorted[2];           // shapes, edges in the order of their cells
  uint16_t* key[2];              // cell of every shape, edge (M: an edge without direction)
  uint32_t *hist[2], *total[2], *first[2];
  uint32_t* first_tile;          // [M + 1]
  unsigned long long* wg_least;
  uint8_t* left;                 // [4 * ceil(E / 128)] waves whose edges are left to the whole search
  uint32_t* least;               // shape of the smallest norm: the nearest to an edge of gain 0
  void* idx;
  float *gain, *bias;
};

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
  const float* c = centre_row(a, (rec >> 6) * 32 + (rec & 31));
  float nrm = 0.f;
#pragma unroll
  for (int k = 0; k < kG; ++k) nrm = fmaf(c[k], c[k], nrm);
  const float hn = -0.5f * nrm, hi = fp16_of(hn);
  const float v0[8] = {c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7]};
  const float v1[8] = {c[8], c[9], hi, hn - hi, 0.f, 0.f, 0.f, 0.f};
  a.centres[rec] = (rec & 32) ? pack_slots(v1) : pack_slots(v0);
}

// Nearest centre of every shape and every edge; gains and biases of the edges.  Any cell is a valid one, so the
// choice is cheap: the maxima of four rows each, the group's number in the low two bits of the mantissa, one running
// maximum - sixteen vector instructions per 32 x 32 scores - and the four rows of the winning group
// are told apart at the end.
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
  float best[kEdgeTilesPerWave];
  int best_tile[kEdgeTilesPerWave];
#pragma unroll
  for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
    const int q = (wave * kEdgeTilesPerWave + nb) * 32 + (lane & 31);
    fb[nb] = __builtin_bit_cast(h16x8, sB[q * 2 + (lane >> 5)]);
    best[nb] = -3.0e38f;
    best_tile[nb] = 0;
  }
  f32x16 zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
  const uint4* cp = a.centres + lane;
  const int n_tiles = a.M / 32;
  uint4 next = cp[0];
  for (int t = 0; t < n_tiles; ++t) {
    const h16x8 fa = __builtin_bit_cast(h16x8, next);
    next = cp[min(t + 1, n_tiles - 1) * 64];
#pragma unroll
    for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
      f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa, fb[nb], zero, 0, 0, 0);
      float m = best[nb];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float v = fmaxf(max3(acc[q], acc[q + 4], acc[q + 8]), acc[q + 12]);
        m = fmaxf(m, __uint_as_float((__float_as_uint(v) & ~3u) | (uint32_t)q));
      }
      best_tile[nb] = m > best[nb] ? t : best_tile[nb];
      best[nb] = m;
    }
  }
#pragma unroll
  for (int nb = 0; nb < kEdgeTilesPerWave; ++nb) {
    const float sc_o = __shfl_xor(best[nb], 32, kWave);
    const int tile_o = __shfl_xor(best_tile[nb], 32, kWave);
    const bool other = sc_o > best[nb] || (sc_o == best[nb] && lane >= 32);
    const int grp = (int)(__float_as_uint(other ? sc_o : best[nb]) & 3u), tile = other ? tile_o : best_tile[nb];
    const int row0 = tile * 32 + 4 * ((lane >> 5) ^ (int)other) + grp;          // rows row0 + 8 k
    const int q = (wave * kEdgeTilesPerWave + nb) * 32 + (lane & 31);
    // this half's two of the four rows
    float top = -3.0e38f;
    int id = row0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int m = row0 + 8 * (2 * (lane >> 5) + k);
      const float* c = centre_row(a, m);
      const _Float16* v = (const _Float16*)(sB + q * 2);
      float dot = 0.f, nrm = 0.f;
#pragma unroll
      for (int z = 0; z < kG; ++z) {
        dot = fmaf((float)v[z], c[z], dot);
        nrm = fmaf(c[z], c[z], nrm);
      }
      dot -= 0.5f * nrm;
      id = dot > top ? m : id;
      top = fmaxf(top, dot);
    }
    const float top_o = __shfl_xor(top, 32, kWave);
    const int id_o = __shfl_xor(id, 32, kWave);
    if (top_o > top) id = id_o;
    if (lane < 32 && first + q < n) key[first + q] = (uint16_t)(s_flat[q] ? a.M : id);
  }
}

// Counting sort of shapes (blockIdx.y = 0) and edges (1) by cell, in chunks: cells counted per chunk, added up over the
// chunks, over the cells, items put in their places.  No order is kept within a cell of a chunk.
__global__ __launch_bounds__(kSortThreads) void kan_cell_count_kernel(const CellArgs a) {
  extern __shared__ uint32_t h[];
  const int p = blockIdx.y, g = blockIdx.x;
  if (g >= a.groups[p]) return;
  for (int m = threadIdx.x; m <= a.M; m += kSortThreads) h[m] = 0;
  __syncthreads();
  const long long n = p ? a.E : a.K, begin = g * a.chunk[p], end = min(n, begin + a.chunk[p]);
  for (long long i = begin + threadIdx.x; i < end; i += kSortThreads) atomicAdd(&h[a.key[p][i]], 1u);
  __syncthreads();
  for (int m = threadIdx.x; m <= a.M; m += kSortThreads) a.hist[p][(long long)g * (a.M + 1) + m] = h[m];
}

__global__ __launch_bounds__(256) void kan_cell_chunks_kernel(const CellArgs a) {
  const int p = blockIdx.y, m = blockIdx.x * 256 + threadIdx.x;
  if (m > a.M) return;
  uint32_t* h = a.hist[p] + m;
  uint32_t sum = 0;
  for (int g0 = 0; g0 < a.groups[p]; g0 += 16) {
    uint32_t v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = g0 + k < a.groups[p] ? h[(long long)(g0 + k) * (a.M + 1)] : 0;
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (g0 + k < a.groups[p]) {
        h[(long long)(g0 + k) * (a.M + 1)] = sum;
        sum += v[k];
      }
  }
  a.total[p][m] = sum;
}

// One workgroup: running sums over the cells (shapes, tiles, edges) and the shape of the smallest norm.
__global__ __launch_bounds__(kSortThreads) void kan_cell_scan_kernel(const CellArgs a) {
  __shared__ uint32_t part[kSortThreads];
  __shared__ unsigned long long least;
  const int tid = threadIdx.x;
  if (tid == 0) least = ~0ull;
  __syncthreads();
  unsigned long long l = ~0ull;
  for (int k = tid; k < a.shape_wgs; k += kSortThreads) l = min(l, a.wg_least[k]);
  atomicMin(&least, l);
  const int per = (a.M + 1 + kSortThreads - 1) / kSortThreads, m0 = tid * per, m1 = min(a.M + 1, m0 + per);
  for (int pass = 0; pass < 3; ++pass) {       // shapes, tiles, edges
    const uint32_t* total = a.total[pass == 2 ? 1 : 0];
    uint32_t* out = pass == 1 ? a.first_tile : a.first[pass == 2 ? 1 : 0];
    auto item = [&](int m) { return pass == 1 ? (total[m] + 31) / 32 : total[m]; };
    uint32_t sum = 0;
    for (int m = m0; m < m1; ++m) sum += item(m);
    __syncthreads();
    part[tid] = sum;
    __syncthreads();
    for (int o = 1; o < kSortThreads; o <<= 1) {
      const uint32_t v = tid >= o ? part[tid - o] : 0;
      __syncthreads();
      part[tid] += v;
      __syncthreads();
    }
    uint32_t run = part[tid] - sum;
    for (int m = m0; m < m1; ++m) {
      out[m] = run;
      run += item(m);
    }
  }
  if (tid == 0) {
    *a.least = (uint32_t)least;
  }
}

__global__ __launch_bounds__(kSortThreads) void kan_cell_place_kernel(const CellArgs a) {
  extern __shared__ uint32_t at[];
  const int p = blockIdx.y, g = blockIdx.x;
  if (g >= a.groups[p]) return;
  for (int m = threadIdx.x; m <= a.M; m += kSortThreads)
    at[m] = a.first[p][m] + a.hist[p][(long long)g * (a.M + 1) + m];
  __syncthreads();
  const long long n = p ? a.E : a.K, begin = g * a.chunk[p], end = min(n, begin + a.chunk[p]);
  for (long long i = begin + threadIdx.x; i < end; i += kSortThreads)
    a.sorted[p][atomicAdd(&at[a.key[p][i]], 1u)] = (uint32_t)i;
}

// Tiles of one cell: members sorted by distance to the centre (then by id), operands of the search and of the bound.
// The first M workgroups take the first kBuildChunk members of a cell each.  Shapes that coincide (the unused rows of a
// trained codebook) all fall into one cell: the workgroups behind start at every kBuildChunk-th shape in the order of
// the cells and take the further chunk of its cell that begins there or next (one workgroup for the whole cell: with
// 30 % of 65,536 rows unused 658 us, now 35).
__global__ __launch_bounds__(256) void kan_cell_build_kernel(const CellArgs a) {
  __shared__ unsigned long long sorted[kBuildChunk];       // {squared distance to the centre, id}
  __shared__ uint32_t row_id[kBuildChunk];                 // a tile's rows by id
  const int tid = threadIdx.x;
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
  const float* cr = centre_row(a, m);
  float c[kG], cn = 0.f;
#pragma unroll
  for (int k = 0; k < kG; ++k) {
    c[k] = cr[k];
    cn = fmaf(c[k], c[k], cn);
  }
  const int n = (int)a.total[0][m];
  const uint32_t* member = a.sorted[0] + a.first[0][m];
  if (n0 < n) {
    const int nc = min(kBuildChunk, n - n0), tile0 = (int)a.first_tile[m] + n0 / 32, tiles = (nc + 31) / 32;
    int full = 32;
    while (full < nc) full <<= 1;
    for (int i = tid; i < full; i += 256) {
      if (i >= nc) {
        sorted[i] = ~0ull;
        continue;
      }
      const uint32_t k = member[n0 + i];
      float d2 = 0.f;
#pragma unroll
      for (int q = 0; q < kG; ++q) {
        const float d = a.cb[(long long)k * kG + q] - c[q];
        d2 = fmaf(d, d, d2);
      }
      if (!(d2 >= 0.f)) d2 = 3.0e38f;           // (a row that is no number sorts last and is never skipped)
      sorted[i] = ((unsigned long long)__float_as_uint(d2) << 32) | k;
    }
    __syncthreads();
    for (int size = 2; size <= full; size <<= 1)           // bitonic
      for (int stride = size >> 1; stride > 0; stride >>= 1) {
        for (int i = tid; i < full / 2; i += 256) {
          const int lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
          const unsigned long long u = sorted[lo], v = sorted[hi];
          if ((u > v) == ((lo & size) == 0)) {
            sorted[lo] = v;
            sorted[hi] = u;
          }
        }
        __syncthreads();
      }
    // Within a tile by id: of equal scores a lane keeps the first row, which is then the lowest id, as in the whole search.
    for (int i = tid; i < nc; i += 256) {
      const uint32_t id = (uint32_t)sorted[i];
      int at = i & ~31;
#pragma unroll
      for (int o = 0; o < 32; ++o) at += (uint32_t)sorted[(i & ~31) + o] < id;      // (past the last one: the largest id)
      row_id[at] = id;
    }
    __syncthreads();
    for (int rec = tid; rec < tiles * 128; rec += 256) {
      const int row = rec >> 2, part = rec & 3, ks = part >> 1, half = part & 1;       // (a row's four records)
      const int tile = tile0 + (row >> 5), r = row & 31;
      const uint32_t k = row < nc ? row_id[row] : 0xffffffffu;
      a.frag[((long long)tile * 2 + ks) * 64 + half * 32 + r] = shape_slots(a.cb, k, row < nc, ks * 16 + half * 8);
      if (part == 0) a.ids[tile * 32 + r] = k;
    }
    for (int t = tid; t < tiles; t += 256) {
      const float far = __uint_as_float((uint32_t)(sorted[min(nc, t * 32 + 32) - 1] >> 32));
      const float R = fp16_up(sqrtf(far) * 1.00001f);
      // (fp16 operands: n and c are off by 2^-11 of themselves each, or flushed below 6e-5)
      float cst = 0.5f * (R * R - cn) + 1.5e-3f * sqrtf(cn) + 1e-4f;
      if (!(cn < 1e5f) || !(R < 300.f) || !(fabsf(cst) < 6e4f)) cst = 6e4f;      // beyond fp16: always visited
      const float hi = fp16_of(cst), Rf = R < 300.f ? R : 300.f;
      const float v0[8] = {c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7]};
      const float v1[8] = {c[8], c[9], hi, cst - hi, Rf, 1.f, 1.f, 0.f};
      uint4* rec = a.bound + (long long)((tile0 + t) >> 5) * 64 + ((tile0 + t) & 31);
      rec[0] = pack_slots(v0);
      rec[32] = pack_slots(v1);
    }
  }
  if (blockIdx.x == 0 && tid < 32) {             // rows of the last bound operand past the last tile: never visited
    const int T = (int)a.first_tile[a.M], t = (T & ~31) + tid;
    if (t >= T && (T & 31)) {
      const float v0[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      const float v1[8] = {0.f, 0.f, -6e4f, 0.f, 0.f, 0.f, 0.f, 0.f};
      uint4* rec = a.bound + (long long)(t >> 5) * 64 + (t & 31);
      rec[0] = pack_slots(v0);
      rec[32] = pack_slots(v1);
    }
  }
}

// What the second product can add to the score of a shape at distance d or less of an edge (|n| = 1): its norm is at
// most 1 + d, the low parts are at most 2^-11 of what they complete, on either side of n . C and in |C|^2 / 2.
__device__ __forceinline__ float first_product_slack(float d) {
  const float r = 1.001f + d;
  return d <= kFar ? fmaf(r, fmaf(r, 2.45e-4f, 9.8e-4f), 1e-5f) : INFINITY;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}

template <typename IdxT>
__global__ __launch_bounds__(256, 6) void kan_assign_bounded_kernel(const CellArgs a) {
  __shared__ uint32_t s_seen[4][kCellMaxTiles / 32];       // tiles visited, a row per wave
  __shared__ uint16_t s_list[4][64 * 32 + 2 * kAhead];     // tiles to visit
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
  // runs of consecutive workgroups on one XCD (workgroups go to the eight in turn): neighbours ask for the same tiles
  const unsigned W = gridDim.x, xcd = blockIdx.x & 7u, q8 = W >> 3, r8 = W & 7u;
  const long long wg = xcd * q8 + min(xcd, r8) + (blockIdx.x >> 3);
  const long long pos = (wg * 4 + wave) * 32 + (lane & 31);
  if ((wg * 4 + wave) * 32 >= a.E) {                       // (no barrier in this kernel)
    if (lane == 0) a.left[wg * 4 + wave] = 0;
    return;
  }
  volatile uint32_t* seen = s_seen[wave];
  volatile uint16_t* list = s_list[wave];
  const int T = (int)a.first_tile[a.M], words = (T + 31) / 32, most = (int)(kRestShare * T);
  for (int w = lane; w < words; w += 64) seen[w] = 0;

  const uint32_t e = a.sorted[1][min(pos, a.E - 1)];
  const int key = a.key[1][e];
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
  uint32_t best_id = 0;
  auto id_of = [&](int t, int r) { return a.ids[t * 32 + 8 * (r >> 2) + 4 * half + (r & 3)]; };
  // The first product of a shape that can win reaches `near` = best - slack (see first_product_slack).
  float slack = 0.f, near = 0.f;
  auto take = [&](float sc, uint32_t id) {       // (equal scores: the lower id)
    if (sc > best || (sc == best && id < best_id)) best_id = id;
    best = fmaxf(best, sc);
    near = best - slack;
  };
  auto leave = [&] {                             // to the whole search
    if (lane == 0) a.left[wg * 4 + wave] = 1;
  };

  // (1) own cells, both instructions of every tile
  int visits = 0;
  bool pending = live;
  for (unsigned long long w; (w = __ballot(pending)) != 0;) {
    const int cell = __builtin_amdgcn_readlane(key, __ffsll(w) - 1);
    pending = pending && key != cell;
    const int t0 = (int)a.first_tile[cell], t1 = (int)a.first_tile[cell + 1];
    visits += t1 - t0;
    if (visits > most) {
      leave();
      return;
    }
    for (int t = t0; t < t1; ++t) {
      const h16x8 f0 = __builtin_bit_cast(h16x8, (a.frag + (long long)t * 128)[lane]);
      const h16x8 f1 = __builtin_bit_cast(h16x8, (a.frag + (long long)t * 128 + 64)[lane]);
      f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(f0, fb[0], zero, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(f1, fb[1], acc, 0, 0, 0);
      const float m = max_of(acc);
      if (m >= best) take(m, id_of(t, row_of(acc, m)));
      if (lane == 0) seen[t >> 5] = seen[t >> 5] | (1u << (t & 31));
    }
  }

  // Distance to the best shape so far (scores are good to 1e-6).  The two lanes of an edge hold different rows:
  // they agree on the better shape first.
  auto distance = [&] {
    const float sc_o = __shfl_xor(best, 32, kWave);
    take(sc_o, (uint32_t)__shfl_xor((int)best_id, 32, kWave));
    float dist = live ? sqrtf(fmaxf(0.f, 1.0f - 2.0f * best) + 4e-6f) : 0.f;
    if (live && !unit) dist = 2.0f * kFar;       // (every tile: the wave goes to the whole search)
    slack = live ? first_product_slack(dist) : -INFINITY;      // (an edge without direction asks for nothing)
    near = best - slack;
    return dist;
  };
  const __amdgpu_buffer_rsrc_t bound_rsrc = buffer_of(a.bound, (size_t)((T + 31) / 32) * 1024);
  const __amdgpu_buffer_rsrc_t frag_rsrc = buffer_of(a.frag, (size_t)T * 2048);
  auto load = [&](const __amdgpu_buffer_rsrc_t& rsrc, int at) {
    return __builtin_bit_cast(h16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, at, 0));
  };
  // A tile whose first product comes near the best score gets the second instruction.
  auto examine = [&](int t, const f32x16& first) {
    const f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(load(frag_rsrc, t * 2048 + 1024), fb[1], first, 0, 0, 0);
    const float m = max_of(acc);
    if (m >= best) take(m, id_of(t, row_of(acc, m)));
  };
  // Every tile not visited yet that an edge with its bit in `who` asks for at distance d.  False: too many.
  // (An instruction of any kind takes its wave's SIMD an issue slot: tiles are listed first, so that a visit is a
  // lane read, a load, a matrix instruction and the maxima of a pair of tiles.)
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
    for (int w0 = 0; w0 < words; w0 += 64) {
      const int w1 = min(words, w0 + 64);
      uint32_t mine = 0;                         // lane w: the tiles of word w0 + w
      h16x8 f[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) f[k] = load(bound_rsrc, min(w0 + k, words - 1) * 1024);
      for (int w = 0; w < w1 - w0; w += kAhead) {        // (past the last word: that one again, struck out below)
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
          // rows: edges, columns: tiles
          const f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(fe, f[k], zero, 0, 0, 0);
          f[k] = load(bound_rsrc, min(w0 + w + k + kAhead, words - 1) * 1024);
          const unsigned long long any = __ballot(!(max_of(acc) <= 0.f));
          mine = lane == w + k ? (uint32_t)any | (uint32_t)(any >> 32) : mine;
        }
      }
      if (w0 + lane < w1) {
        const uint32_t before = seen[w0 + lane];
        mine &= ~before;
        seen[w0 + lane] = before | mine;
      } else {
        mine = 0;
      }
      // the list of these tiles
      int upto = __popc(mine);
      const int own = upto;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(upto, o, kWave);
        upto += lane >= o ? v : 0;
      }
      const int count = __builtin_amdgcn_readlane(upto, 63);
      asked += count;
      if (asked > most) return false;
      if (count == 0) continue;
      int last = 0;
      for (int at = upto - own; mine; ++at) {
        last = (w0 + lane) * 32 + __ffs(mine) - 1;
        mine &= mine - 1;
        list[at] = (uint16_t)last;
      }
      const unsigned long long some = __ballot(own != 0);
      last = __builtin_amdgcn_readlane(last, 63 - __clzll(some));
      if (lane < 2 * kAhead) list[count + lane] = (uint16_t)last;      // (to whole groups, and one ahead: the last again)
      for (int i0 = 0; i0 < count; i0 += 64) {
        const int tiles = list[min(i0 + lane, count)];
        auto tile = [&](int i) { return __builtin_amdgcn_readlane(tiles, i); };
        int t[kAhead];
        const int n_here = min(64, count - i0);
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
          t[k] = tile(k);
          f[k] = load(frag_rsrc, t[k] * 2048);
        }
        for (int i = 0; i < n_here; i += kAhead) {
#pragma unroll
          for (int k = 0; k < kAhead; k += 2) {
            const f32x16 acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[k], fb[0], zero, 0, 0, 0);
            const f32x16 acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[k + 1], fb[0], zero, 0, 0, 0);
            const int u0 = t[k], u1 = t[k + 1];
            t[k] = tile(min(i + k + kAhead, 63));
            t[k + 1] = tile(min(i + k + 1 + kAhead, 63));
            f[k] = load(frag_rsrc, t[k] * 2048);
            f[k + 1] = load(frag_rsrc, t[k + 1] * 2048);
            const float m0 = max_of(acc0), m1 = max_of(acc1);
            if (__ballot(fmaxf(m0, m1) >= near)) {
              if (__ballot(m0 >= near)) examine(u0, acc0);
              if (__ballot(m1 >= near)) examine(u1, acc1);
            }
          }
        }
      }
    }
    return true;
  };

  float d = distance();
  const bool in = live && d <= kFar;
  float sum = in ? d : 0.f, cnt = in ? 1.f : 0.f;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    sum += __shfl_xor(sum, o, kWave);
    cnt += __shfl_xor(cnt, o, kWave);
  }
  const float mean = cnt > 0.f ? kMeanFactor * sum / cnt : 2.0f * kFar;
  bool done = search(live, fminf(d, mean));      // (2)
  if (done) {
    d = distance();
    const bool left = live && d > mean;
    if (__ballot(left)) done = search(left, d);  // (3)
  }
  if (!done) {
    leave();
    return;
  }
  (void)distance();
  if (lane == 0) a.left[wg * 4 + wave] = 0;
  // (an edge without direction: the shape of the smallest norm; one that is no number has no scores and keeps row 0)
  if (lane < 32 && there) {
    if (!live) best_id = a.gain[e] == a.gain[e] ? *a.least : 0u;
    ((IdxT*)a.idx)[e] = (IdxT)best_id;
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
dim3 split_grid(long long E) { return dim3((unsigned)((E + kEdgeTilesPerWave * 32 - 1) / (kEdgeTilesPerWave * 32))); }
}  // namespace

// The bounded search pays where its cells, launches and bound tests are small next to the scores they save, for grids
// that fit their codebook and at little loss for those that do not.  Bounded search with 2 % / 5 % / 15 % noise per
// coefficient / unrelated grids against the whole search (which does not care), us:
//     K = 65,536   2^20 edges  545 / 779 / 1290 / 1332  against 3820      2^16 edges  128 / 167 / 224 / 226  against 312
//     K = 32,768   2^17 edges  110 / 148 / 203 / 212  against 313
//     K = 16,384   2^20 edges  300 / 420 / 688 / 732  against 1024        2^18 edges  132 / 167 / 238 / 252  against 296
//                  2^17 edges  98 / 126 / 160 / 165  against 173          98,304 edges  94 / 112 / 141 / 146  against 132
//     K = 8,192    2^20 edges  252 / 335 / 522 / 553  against 547
// (K = 8,192 and 2^18 edges with 5 % noise 249 against 195; K = 262,144 and 2^20 edges 1.9 against 14.9 ms).
bool assign_bounded_ok(long long E, int K) {
  const long long work = E * K;
  return (work >= (3ll << 29) && K >= 16384 || work >= (1ll << 33) && K >= 8192) && cell_layout(1, K).tiles_max <= kCellMaxTiles;
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
  a.shape_wgs = (K + kEdgesPerWg - 1) / kEdgesPerWg;
  a.centres = (uint4*)(w + g.centres);
  a.frag = (uint4*)(w + g.frag);
  a.ids = (uint32_t*)(w + g.ids);
  a.bound = (uint4*)(w + g.bound);
  a.sorted[0] = (uint32_t*)(w + g.member);
  a.sorted[1] = (uint32_t*)(w + g.perm);
  for (int p = 0; p < 2; ++p) {
    a.groups[p] = g.groups[p];
    a.chunk[p] = g.chunk[p];
    a.key[p] = (uint16_t*)(w + g.key[p]);
    a.hist[p] = (uint32_t*)(w + g.hist[p]);
    a.total[p] = (uint32_t*)(w + g.total[p]);
    a.first[p] = (uint32_t*)(w + g.first[p]);
  }
  a.first_tile = (uint32_t*)(w + g.first_tile);
  a.wg_least = (unsigned long long*)(w + g.wg_least);
  a.left = (uint8_t*)(w + g.left);
  a.least = (uint32_t*)(w + g.least);
  a.idx = idx;
  a.gain = gain;
  a.bias = bias;
  const unsigned edge_wgs = (unsigned)((E + kEdgesPerWg - 1) / kEdgesPerWg);
  const dim3 sort_grid((unsigned)(g.groups[0] > g.groups[1] ? g.groups[0] : g.groups[1]), 2);
  const size_t cells_lds = (size_t)(g.M + 1) * 4;
  hipLaunchKernelGGL(kan_cell_centres_kernel, dim3((unsigned)((g.M * 2 + 255) / 256)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(kan_cells_kernel, dim3((unsigned)a.shape_wgs + edge_wgs), dim3(kAssignThreads), 0, s, a);
  hipLaunchKernelGGL(kan_cell_count_kernel, sort_grid, dim3(kSortThreads), cells_lds, s, a);
  hipLaunchKernelGGL(kan_cell_chunks_kernel, dim3((unsigned)(g.M / 256 + 1), 2), dim3(256), 0, s, a);
  hipLaunchKernelGGL(kan_cell_scan_kernel, dim3(1), dim3(kSortThreads), 0, s, a);
  hipLaunchKernelGGL(kan_cell_place_kernel, sort_grid, dim3(kSortThreads), cells_lds, s, a);
  hipLaunchKernelGGL(kan_cell_build_kernel, dim3((unsigned)(g.M + (K + kBuildChunk - 1) / kBuildChunk)), dim3(256), 0, s, a);
  const dim3 grid((unsigned)((E + 127) / 128));
  if (idx_u32) hipLaunchKernelGGL(kan_assign_bounded_kernel<uint32_t>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(kan_assign_bounded_kernel<uint16_t>, grid, dim3(256), 0, s, a);
  AssignArgs rest = {};
  rest.coef = coef;
  rest.cent = a.frag;
  rest.E = E;
  rest.list = a.sorted[1];
  rest.left = a.left;
  rest.tiles = a.first_tile + g.M;
  rest.ids = a.ids;
  rest.idx = idx;
  const dim3 rest_grid((unsigned)std::min<long long>((E + 127) / 128, kRestWorkgroups));
  if (idx_u32) hipLaunchKernelGGL((kan_assign_kernel<uint32_t, 8, true>), rest_grid, dim3(8 * kWave), 0, s, rest);
  else hipLaunchKernelGGL((kan_assign_kernel<uint16_t, 8, true>), rest_grid, dim3(8 * kWave), 0, s, rest);
  return hipGetLastError();
}

hipError_t launch_assign(const float* coef, long long E, const float* cb, int K, int idx_u32, void* idx, float* gain,
                         float* bias, void* ws, hipStream_t s) {
  AssignArgs a = {};
  a.coef = coef;
  a.cent = (const uint4*)ws;
  a.E = E;
  a.n_tiles = (K + 31) / 32;
  a.idx = idx;
  a.gain = gain;
  a.bias = bias;
  const long long recs = (long long)a.n_tiles * 2 * 64;
  hipLaunchKernelGGL(kan_assign_prep_kernel, dim3((unsigned)((recs + 255) / 256)), dim3(256), 0, s, cb, K, a.n_tiles, (uint4*)ws);
  const dim3 grid((unsigned)((E + kEdgesPerWg - 1) / kEdgesPerWg));
  if (E <= kSplitMaxEdges) {
    if (idx_u32) hipLaunchKernelGGL((kan_assign_kernel<uint32_t, 8, false>), split_grid(E), dim3(8 * kWave), 0, s, a);
    else hipLaunchKernelGGL((kan_assign_kernel<uint16_t, 8, false>), split_grid(E), dim3(8 * kWave), 0, s, a);
  } else {
    if (idx_u32) hipLaunchKernelGGL((kan_assign_kernel<uint32_t, 1, false>), grid, dim3(kAssignThreads), 0, s, a);
    else hipLaunchKernelGGL((kan_assign_kernel<uint16_t, 1, false>), grid, dim3(kAssignThreads), 0, s, a);
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
