// Matrix-core contraction that dequantises its own coefficients (batch above the fused kernel's tiles).
//
// Same contraction and operands as kan_mfma.hip (sparse matrix instruction, k order (m, m + 5)), but no
// coefficient records pass through memory: a workgroup owns 64 outputs, a chunk of inputs and a tall tile of
// samples (128, 256 or 512), gathers and dequantises the edges of a step once and keeps them in LDS for all of
// its samples.  The basis operand goes from memory straight into the registers of the lane that multiplies it.
//
//   samples    wave w of eight owns 32 (or 64) rows; in the 128-sample tile four waves share the rows of the
//              other four and each takes half of the columns
//   edges      1,024 per step of 16 inputs, two per thread: wave w takes inputs 2 w and 2 w + 1, lanes along the
//              outputs, so the ids, gains and biases of a wave's two steps are four rows of 64 elements
//   LDS        two tiles of 64 columns x 20 records x 16 bytes (twice that for split operands)
//
// What bounds it is the CU's vector-memory path: a step gathers 1,024 codewords (2.3 clocks each, whatever their
// width) and brings 160 bytes of basis words per sample row: 1.5 us of the 1.7-1.9 us that a step takes with 256
// samples, 1.8 of 2.5 us with 512 (MFMAs 0.4 and 0.8 us).  That is also why a tile is 64 outputs by as many samples as
// the accumulators allow: per edge 2.3 clocks plus 160 / 58 clocks per row over 64 columns.  Around the steps a
// workgroup spends 4 us until its first MFMA (ids, then codewords, then the tile) and 2-8 us on its partial sums.
// Layer times against the streaming form: at make_wide in kan_api.hip (2048 x 512 fp32 codebook, split operands, batch
// 256: preparation 18.8 + contraction 22.8 us -> 5 + 26 us; 2048 x 1024 Int8, batch 256: 25 + 19 -> 5 + 23 us).
// Tried without gain: the two waves of a SIMD taking multiplication and dequantisation in opposite order (equal within
// 1 %, split form spills), all of a step's loads at its top (2048 x 512 split at batch 256 47 us against 36).
//
// The basis operand in memory ("rotated words"): an input's ten basis values hold four consecutive ones, so of its
// pairs (m, m + 5), m = 0..4, four hold one value each and one holds none.  prep_rot_block stores the five values
// in pair order, 10 bytes per (sample, input), each with the bit "takes coefficient m + 5" in its sign.  They are
// the stored values of the sparse operand as they stand: the sign, which the instruction would multiply by, is
// undone by holding coefficients 5..9 negated, and the position bits are collected from the signs (10 vector
// instructions per 16 bytes, where the 8-byte words of kan_prep_basis need a table read and three permutes per
// input).
#include <type_traits>

#include "kan_device.hpp"
#include "kan_internal.hpp"
#include "kan_mfma_common.hpp"

namespace kan {
namespace {

constexpr int kThreads = 512;
constexpr int kWaves = 8;
constexpr int IT = 16;                           // inputs per step
constexpr int BN = kWideTileN;                   // outputs per workgroup
constexpr int kPlane = BN * 16;                  // one 16-byte record per column
constexpr int kTile = 20 * kPlane;               // records (S, h, a) of a step, S = 0..4
constexpr int kBufferFlags = 0x00020000;         // buffer resource word 3: raw 32-bit data format, no swizzle

// The ids, gains or biases that a wave needs for two steps: four rows of 64 elements of E bytes.  Rows start
// anywhere, so what is fetched are the 16-byte units that hold them (elements of four bytes: units from the row's
// first element on, which is aligned well enough).
template <int E> constexpr int kUnits = E == 4 ? 16 : 4 * E + 1;       // per row

// In the place of the gains' type: the dense layer.  An edge's coefficients are row i n_out + j of the array (64 lanes side by
// side: 2,560 consecutive bytes), there are no ids, gains and biases.  Against records converted in a launch of their
// own (80 bytes an edge written and read for the 40 of the array): 2048 x 512 at batch 256 49.4 -> 30.0 us.
struct dense_t {};

template <typename IdxT, typename GbT, typename CbT, bool SPLIT, int RB, int WM>
__global__ __launch_bounds__(kThreads, 2) void kan_wide_kernel(const WideArgs a) {
  constexpr int WN = kWaves / WM;                // waves along the columns
  constexpr int NB = BN / 32 / WN;               // column blocks per wave
  constexpr int BM = 32 * RB * WM;
  constexpr int EI = (int)sizeof(IdxT), EG = (int)sizeof(GbT);
  constexpr bool kIsDense = std::is_same_v<GbT, dense_t>;
  static_assert(NB >= 1, "");
  __shared__ __attribute__((aligned(16))) unsigned char sB[2][(SPLIT ? 2 : 1) * kTile];     // split form: high records, then low
  __shared__ __attribute__((aligned(16))) unsigned char sMeta[kWaves][kIsDense ? 16 : 3 * 1024];            // ids, gains, biases
  __shared__ float sBias[kWaves][BN];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ln = lane & 31, lh = lane >> 5;
  const int wm = wave % WM, wn = wave / WM;
  // Work items sorted by head, chunk of inputs, tile, cut into eight contiguous runs, one per XCD: the tiles of a
  // chunk share its slice of the basis words, its ids and gains, and a head's codebook in one L2.
  int head, chunk, tile;
  {
    const unsigned T = gridDim.x, C = gridDim.y, W = T * C * gridDim.z;
    const unsigned L = blockIdx.x + T * (blockIdx.y + C * blockIdx.z);
    const unsigned xcd = L & 7u, m = L >> 3, q = W >> 3, r = W & 7u;
    const unsigned item = xcd * q + min(xcd, r) + m;          // XCD x owns q + (x < r) items
    head = (int)(item / (T * C));
    const unsigned rem = item % (T * C);
    chunk = (int)(rem / T);
    tile = (int)(rem % T);
  }
  const int jt = tile % a.n_jt, b0 = (tile / a.n_jt) * BM, j0 = jt * BN;
  const int n_in = a.n_in, n_out = a.n_out, B = a.B;
  const int i_begin = chunk * a.rows_per_chunk;
  const int i_end = min(n_in, i_begin + a.rows_per_chunk);
  const int n_steps = (i_end - i_begin + IT - 1) / IT;
  const int step0 = i_begin / IT;
  const LayerPtrs hp = a.h[head];
  const Q8Params qp = {hp.gain_log2_lo, hp.gain_log2_step, hp.bias_scale};
  const CbT* const cb = (const CbT*)hp.cb;

  // ---- basis operand: rows b0 + (wm RB + rb) 32 + ln, half a = lh of every record
  uint32_t a_off[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
    a_off[rb] = ((uint32_t)lh * (uint32_t)B + (uint32_t)min(b0 + (wm * RB + rb) * 32 + ln, B - 1)) * 16u;
  const uint32_t plane_bytes = 2u * (uint32_t)B * 16u;          // both halves of a record plane
  const char* const Wm = (const char*)(a.W + (long long)head * a.w_head_stride);
  const char* const Wl = SPLIT ? (const char*)(a.W_lo + (long long)head * a.w_head_stride) : nullptr;
  struct AFrag {
    u32x4 h[RB][5];
    u32x4 l[SPLIT ? RB : 1][5];
  };
  auto load_a = [&](int k, int S, AFrag& f) {                     // fragments of group S of step k
    const int step = step0 + min(k, n_steps - 1);                 // past the end: the last step again
    auto part = [&](const char* W, u32x4 (&v)[RB][5]) {
      const char* const p = W + (size_t)(step * 5 + S) * plane_bytes;
      const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)plane_bytes, kBufferFlags);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) v[rb][S] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)a_off[rb], 0, 0);
    };
    part(Wm, f.h);
    if constexpr (SPLIT) part(Wl, f.l);
  };
  // ---- edges: inputs 2 wave, 2 wave + 1 of every step, column j0 + lane
  const bool j_ok = j0 + lane < n_out;
  struct MetaRaw {
    u32x4 i, g, b;
  };
  // the array as a buffer of whole 16-byte units (what lies past its last element reads as zero)
  auto array = [&](const void* p, int E) {
    const uint32_t mis = (uint32_t)(uintptr_t)p & 15u;
    const uint32_t bytes = mis + (uint32_t)n_in * (uint32_t)n_out * (uint32_t)E;
    return __builtin_amdgcn_make_buffer_rsrc((void*)((uintptr_t)p - mis), 0, (int)((bytes + 3u) & ~3u), kBufferFlags);
  };
  auto row_input = [&](int t, int r) { return i_begin + 32 * t + 16 * (r >> 1) + 2 * wave + (r & 1); };      // row r of steps 2 t, 2 t + 1
  auto row_byte = [&](const void* p, auto E_, int i) {             // byte of (input i, column j0) in that buffer
    constexpr int E = decltype(E_)::value;
    return ((uint32_t)(uintptr_t)p & 15u) + ((uint32_t)min(i, n_in - 1) * (uint32_t)n_out + (uint32_t)j0) * (uint32_t)E;
  };
  auto fetch = [&](const void* p, auto E_, int t) {
    constexpr int E = decltype(E_)::value, U = kUnits<E>;
    const int q = min(lane, 4 * U - 1), r = q / U, part = q - r * U;      // (lanes past the last unit repeat it)
    uint32_t at = row_byte(p, E_, row_input(t, r));
    if constexpr (E != 4) at &= ~15u;
    return __builtin_amdgcn_raw_buffer_load_b128(array(p, E), (int)(at + part * 16), 0, 0);
  };
  using EI_ = std::integral_constant<int, EI>;
  using EG_ = std::integral_constant<int, EG>;
  auto meta_issue = [&](int t, MetaRaw& m) {
    if constexpr (kIsDense) return;
    m.i = fetch(hp.idx, EI_{}, t);
    m.g = fetch(hp.gain, EG_{}, t);
    m.b = fetch(hp.bias, EG_{}, t);
  };
  struct Meta {
    uint32_t id[2][2];      // [step of the pair][edge]
    float g[2][2];
  };
  float bsum = 0.f;
  unsigned char* const strip = sMeta[wave];
  auto meta_commit = [&](int t, const MetaRaw& raw, Meta& m) {
    if constexpr (kIsDense) {      // (past the last input or output: one that is there, times zero)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = row_input(t, r);
        m.id[r >> 1][r & 1] = (uint32_t)min(i, i_end - 1) * (uint32_t)n_out + (uint32_t)min(j0 + lane, n_out - 1);
        m.g[r >> 1][r & 1] = i < i_end ? 1.f : 0.f;
      }
      return;
    }
    __builtin_amdgcn_wave_barrier();                             // earlier reads of the strip stay before these writes
    *(u32x4*)(strip + lane * 16) = raw.i;
    *(u32x4*)(strip + 1024 + lane * 16) = raw.g;
    *(u32x4*)(strip + 2048 + lane * 16) = raw.b;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // rows past the last input (the array's last row was read) keep its codeword and have gain 0; steps past the
      // chunk are never multiplied and gather one row
      const int i = row_input(t, r);
      const bool ok = j_ok && i < i_end, live = j_ok && 2 * t + (r >> 1) < n_steps;
      auto at = [&](const void* p, auto E_) {
        constexpr int E = decltype(E_)::value;
        return r * kUnits<E> * 16 + (E == 4 ? 0 : (int)(row_byte(p, E_, i) & 15u)) + lane * E;
      };
      const uint32_t id = *(const IdxT*)(strip + at(hp.idx, EI_{}));
      float g, b;
      if constexpr (EG == 1) {
        g = q8_gain(strip[1024 + at(hp.gain, EG_{})], qp);
        b = q8_bias(strip[2048 + at(hp.bias, EG_{})], qp);
      } else if constexpr (EG == 2) {
        g = half_bits_to_float(*(const uint16_t*)(strip + 1024 + at(hp.gain, EG_{})));
        b = half_bits_to_float(*(const uint16_t*)(strip + 2048 + at(hp.bias, EG_{})));
      } else {
        g = *(const float*)(strip + 1024 + at(hp.gain, EG_{}));
        b = *(const float*)(strip + 2048 + at(hp.bias, EG_{}));
      }
      m.id[r >> 1][r & 1] = live ? id : 0u;
      m.g[r >> 1][r & 1] = ok ? g : 0.f;
      bsum += ok ? b : 0.f;
    }
  };
  struct Rows {
    RawRow<CbT> r[2];
    uint32_t odd;
  };
  auto gather = [&](const uint32_t (&id)[2], Rows& rows) {
    rows.odd = 0u;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      load_row<CbT>(cb, id[e], rows.r[e]);
      rows.odd |= row_odd<CbT>(cb, id[e]) << e;
    }
  };
  // Input 4 S + 2 h' + h of a step (h' = a): S = wave / 2, a = wave % 2, h = the edge.  Coefficient pairs (m, m + 5),
  // the second negated, m = 0..3 in record (S, h, a), m = 4 in words 2 (S % 2) + h of record (4, S / 2, a).
  auto dequant = [&](Rows& rows, const float (&g)[2], unsigned char* t) {
    uint32_t tail[2], tail_lo[2];
    const int S = wave >> 1, ha = wave & 1;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      align_row<CbT>(rows.r[e], (rows.odd >> e) & 1u);
      unsigned char* rec = t + ((S * 2 + e) * 2 + ha) * kPlane + lane * 16;
      uint32_t hi[5], lo[5];
      if constexpr (SPLIT) {
        float c[kG];
        dequant_row_f32<CbT>(rows.r[e], g[e], c);
#pragma unroll
        for (int m = 5; m < kG; ++m) c[m] = -c[m];
        split_pairs(c, hi, lo);
        *(uint4*)(rec + kTile) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        tail_lo[e] = lo[4];
      } else {
        dequant_row_pairs<CbT>(rows.r[e], g[e], hi);
      }
      *(uint4*)rec = make_uint4(hi[0], hi[1], hi[2], hi[3]);
      tail[e] = hi[4];
    }
    unsigned char* rec = t + ((8 + (S >> 1)) * 2 + ha) * kPlane + lane * 16 + (S & 1) * 8;
    *(uint2*)rec = make_uint2(tail[0], tail[1]);
    if constexpr (SPLIT) *(uint2*)(rec + kTile) = make_uint2(tail_lo[0], tail_lo[1]);
  };

  f32x16 acc[RB][NB], acc_x[SPLIT ? RB : 1][SPLIT ? NB : 1];      // (acc_x: the cross products of the split form)
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[rb][nb][r] = 0.f;
        if constexpr (SPLIT) acc_x[rb][nb][r] = 0.f;
      }
  const int col = wn * NB * 32 + ln;
  // The B fragments of group S + 1 are read from LDS while the matrix pipe works on group S; behind it go the loads of
  // the next step's A fragments of the group (into the registers that it has just read) and what `between` adds.
  auto multiply = [&](int k, AFrag& f, const unsigned char* t, auto&& between) {
    struct BFrag {
      u32x4 h[NB][2], l[SPLIT ? NB : 1][2];
    };
    BFrag bf[2];
    const unsigned char* const p = t + lh * 2 * kPlane + col * 16;
    auto read_b = [&](int S, BFrag& o) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          o.h[nb][x] = *(const u32x4*)(p + (S * 4 + x) * kPlane + nb * 512);
          if constexpr (SPLIT) o.l[nb][x] = *(const u32x4*)(p + kTile + (S * 4 + x) * kPlane + nb * 512);
        }
    };
    read_b(0, bf[0]);
    __builtin_amdgcn_s_setprio(2);
#pragma unroll
    for (int S = 0; S < 5; ++S) {
      if (S < 4) read_b(S + 1, bf[(S + 1) & 1]);
      int ix[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) ix[rb] = rot_positions(f.h[rb][S]);
      __builtin_amdgcn_sched_barrier(0);
      const BFrag& o = bf[S & 1];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const h16x16 fb = __builtin_bit_cast(h16x16, o.h[nb]);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          const h16x8 fa = __builtin_bit_cast(h16x8, f.h[rb][S]);
          if constexpr (SPLIT) {
            const h16x16 fbl = __builtin_bit_cast(h16x16, o.l[nb]);
            const h16x8 fal = __builtin_bit_cast(h16x8, f.l[rb][S]);
            acc_x[rb][nb] = __builtin_amdgcn_smfmac_f32_32x32x32_f16(fa, fbl, acc_x[rb][nb], ix[rb], 0, 0);
            acc[rb][nb] = __builtin_amdgcn_smfmac_f32_32x32x32_f16(fa, fb, acc[rb][nb], ix[rb], 0, 0);
            acc_x[rb][nb] = __builtin_amdgcn_smfmac_f32_32x32x32_f16(fal, fb, acc_x[rb][nb], ix[rb], 0, 0);
          } else {
            acc[rb][nb] = __builtin_amdgcn_smfmac_f32_32x32x32_f16(fa, fb, acc[rb][nb], ix[rb], 0, 0);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      load_a(k + 1, S, f);
      between(S);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
  };

  // ---- pipeline.  Top of step k: coefficient tile k is complete; basis words of step k and codewords of step
  // k + 1 are in flight, the ids of step k + 2 at hand.  What a step waits for was requested before the gathers that
  // are to stay in flight behind it, and no more than a few vector-memory instructions follow each other without an
  // MFMA between them: a wave that queues at the address unit issues nothing else (all of a step's loads at its top:
  // 1.1-1.8 us of a 3 us step spent there, 512-sample tile).  Even steps request the ids and gains of steps k + 4,
  // k + 5, odd ones deal them out.
  AFrag af;
  Rows rows[2];
  MetaRaw raw;
  Meta ma;                 // steps k + 2, k + 3 at the top of an even step
  float g1[2];             // gains of step k + 1
  {
    MetaRaw first;
    meta_issue(0, first);
    meta_issue(1, raw);
#pragma unroll
    for (int S = 0; S < 5; ++S) load_a(0, S, af);
    meta_commit(0, first, ma);
  }
  gather(ma.id[0], rows[0]);
  gather(ma.id[1], rows[1]);
  dequant(rows[0], ma.g[0], sB[0]);
  g1[0] = ma.g[1][0];
  g1[1] = ma.g[1][1];
  meta_commit(1, raw, ma);
  int k = 0;
  for (; k + 2 <= n_steps; k += 2) {
    __syncthreads();
    multiply(k, af, sB[0], [&](int S) {
      if (S == 0) meta_issue(k / 2 + 2, raw);
    });
    gather(ma.id[0], rows[0]);
    __builtin_amdgcn_sched_barrier(0);
    dequant(rows[1], g1, sB[1]);
    __syncthreads();
    multiply(k + 1, af, sB[1], [](int) {});
    gather(ma.id[1], rows[1]);
    __builtin_amdgcn_sched_barrier(0);
    dequant(rows[0], ma.g[0], sB[0]);
    g1[0] = ma.g[1][0];
    g1[1] = ma.g[1][1];
    meta_commit(k / 2 + 2, raw, ma);
  }
  if (k < n_steps) {       // an odd step left over
    __syncthreads();
    multiply(k, af, sB[0], [](int) {});
  }

  // ---- epilogue.  D layout of the 32x32 MFMA: lane holds column (lane & 31), rows
  //      8*(r/4) + 4*(lane/32) + r%4 for r = 0..15.  Rows past the last sample are dropped by the buffer's bound. ----
  sBias[wave][lane] = bsum;
  __syncthreads();
  const float scale = sizeof(CbT) == 1 ? hp.scale : 1.0f;
  float* const dst = a.dst + (long long)head * a.dst_head_stride + (long long)chunk * a.dst_chunk_stride + (long long)b0 * n_out;
  const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc((void*)dst, 0, min(BM, B - b0) * n_out * 4, kBufferFlags);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int j = j0 + col + nb * 32;
    float bs = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) bs += sBias[w][col + nb * 32];
    if (j < n_out) {
      const int at = (4 * lh * n_out + j) * 4;
      auto store = [&](auto act) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            float v = acc[rb][nb][r];
            if constexpr (SPLIT) v = fmaf(1.0f / 2048.0f, acc_x[rb][nb][r], v);
            v = act(fmaf(scale, v, bs));
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rd, at, ((wm * RB + rb) * 32 + 8 * (r >> 2) + (r & 3)) * n_out * 4, 0);
          }
      };
      if (a.apply_tanh) store([](float v) { return tanhf(v); });
      else store([](float v) { return v; });
    }
  }
}

template <typename IdxT, typename GbT, typename CbT>
hipError_t launch_variant(const WideArgs& a, bool split, int tile_m, dim3 grid, hipStream_t s) {
  if (split) {
    if (tile_m == 128) hipLaunchKernelGGL((kan_wide_kernel<IdxT, GbT, CbT, true, 1, 4>), grid, dim3(kThreads), 0, s, a);
    else if (tile_m == 256) hipLaunchKernelGGL((kan_wide_kernel<IdxT, GbT, CbT, true, 1, 8>), grid, dim3(kThreads), 0, s, a);
    else return hipErrorInvalidValue;
  } else if constexpr (std::is_same_v<GbT, dense_t>) {
    return hipErrorInvalidValue;
  } else {
    if (tile_m == 128) hipLaunchKernelGGL((kan_wide_kernel<IdxT, GbT, CbT, false, 1, 4>), grid, dim3(kThreads), 0, s, a);
    else if (tile_m == 256) hipLaunchKernelGGL((kan_wide_kernel<IdxT, GbT, CbT, false, 1, 8>), grid, dim3(kThreads), 0, s, a);
    else if (tile_m == 512) hipLaunchKernelGGL((kan_wide_kernel<IdxT, GbT, CbT, false, 2, 8>), grid, dim3(kThreads), 0, s, a);
    else return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

#ifndef KAN_WIDE_U32
#define KAN_WIDE_U32 0          // 1: this translation unit holds the kernels for 32-bit ids
#endif
template <typename IdxT>
hipError_t launch_types(const GatherCfg& c, const WideArgs& a, bool split, int tile_m, dim3 grid, hipStream_t s) {
  const bool half = c.gb_kind == kGbF16;
  if (c.code == kCbI8) {
    if (c.gb_kind == kGbQ8) return launch_variant<IdxT, q8_t, int8_t>(a, split, tile_m, grid, s);
    return half ? launch_variant<IdxT, __half, int8_t>(a, split, tile_m, grid, s) : launch_variant<IdxT, float, int8_t>(a, split, tile_m, grid, s);
  }
  if (c.gb_kind == kGbQ8) return hipErrorInvalidValue;      // byte-coded gain/bias go with Int8 codebooks
  if (c.code == kCbBfp8)
    return half ? launch_variant<IdxT, __half, bfp8_t>(a, split, tile_m, grid, s) : launch_variant<IdxT, float, bfp8_t>(a, split, tile_m, grid, s);
  if (c.code == kCbF16)
    return half ? launch_variant<IdxT, __half, __half>(a, split, tile_m, grid, s) : launch_variant<IdxT, float, __half>(a, split, tile_m, grid, s);
  return half ? launch_variant<IdxT, __half, float>(a, split, tile_m, grid, s) : launch_variant<IdxT, float, float>(a, split, tile_m, grid, s);
}

#if !KAN_WIDE_U32
__global__ __launch_bounds__(256) void kan_prep_rot_kernel(const float* __restrict__ x, long long x_head_stride, int x_parts,
                                                           long long x_part_stride, int x_tanh, RotWords w, int n_in, int B,
                                                           int rule) {
  __shared__ RotTile hi, lo;
  __shared__ __attribute__((aligned(16))) uint32_t sel[kSpans][8];
  const int head = blockIdx.z;
  w.W += (long long)head * w.w_head_stride;
  if (w.W_lo) w.W_lo += (long long)head * w.w_head_stride;
  if (w.P) w.P += (long long)head * w.p_head_stride;
  prep_rot_block(x + (long long)head * x_head_stride, x_parts, x_part_stride, x_tanh, w, n_in, B, rule, blockIdx.x, blockIdx.y,
                 hi, lo, sel);
}
#endif

}  // namespace

#if KAN_WIDE_U32
hipError_t launch_wide_u32(const GatherCfg& c, const WideArgs& a, bool split, int tile_m, dim3 grid, hipStream_t s) {
  return launch_types<uint32_t>(c, a, split, tile_m, grid, s);
}
#else
hipError_t launch_wide_u32(const GatherCfg& c, const WideArgs& a, bool split, int tile_m, dim3 grid, hipStream_t s);

bool wide_takes(int n_in, int n_out, int64_t B, bool dense) {
  if (dense && (long long)n_in * n_out * (kG * 4) > 0x7fffffffll) return false;
  // what the kernel's 32-bit offsets assume: the per-edge arrays, a step of basis words and a tile of the result
  return (long long)n_in * n_out * 4 < 0x7fffff00ll && (long long)B * 128 <= 0x7fffffffll && n_out <= kWideMaxOut;
}

hipError_t launch_wide(const GatherCfg& c, const WideArgs& a, bool split, int tile_m, dim3 grid, hipStream_t s) {
  if (a.B < 1 || !wide_takes(a.n_in, a.n_out, a.B, c.code == kDense) || a.rows_per_chunk < IT || a.rows_per_chunk % IT != 0 ||
      !a.W || (split && !a.W_lo) || (long long)a.n_jt * BN < a.n_out)
    return hipErrorInvalidValue;
  if (c.code == kDense) return split ? launch_variant<uint16_t, dense_t, float>(a, true, tile_m, grid, s) : hipErrorInvalidValue;
  return c.idx_u32 ? launch_wide_u32(c, a, split, tile_m, grid, s) : launch_types<uint16_t>(c, a, split, tile_m, grid, s);
}

hipError_t launch_prep_rot(const float* x, long long x_head_stride, int x_parts, long long x_part_stride, int x_tanh,
                           const RotWords& w, int n_in, int B, int heads, int rule, hipStream_t s) {
  if (x_parts < 1 || !w.W) return hipErrorInvalidValue;
  dim3 grid((n_in + 31) / 32, (B + 31) / 32, heads);
  hipLaunchKernelGGL(kan_prep_rot_kernel, grid, dim3(256), 0, s, x, x_head_stride, x_parts, x_part_stride, x_tanh, w, n_in, B, rule);
  return hipGetLastError();
}
#endif

}  // namespace kan
