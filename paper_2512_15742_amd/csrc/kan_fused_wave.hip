// Fused gather + matrix-core kernel, every wave on its own: Y = Phi * Chat (+ bias).  Precise path, up to 32 samples: fp32
// operands (v_mfma_f32_16x16x4f32).  fp16 path, up to 64 samples (KAN_WAVE_HALF, an object of its own): see HALF below.
//
// At these batches a layer is a chain of latencies and not a stream: metadata, codewords, products, one launch after
// the other.  The form that came before (tiles of 128 outputs by four waves side by side, the basis tile in LDS, a
// barrier per step of 8 inputs; configuration 3 at batch 16: 18.8 us for the first layer) took 15.5 us with every
// gather going to one line and 17 us with all metadata in the caches: clock reads put 2,000 - 2,900 clocks into
// a step of 1,280 clocks of matrix instructions.  So:
//
//   - A wave owns 64 outputs and, of the workgroup's inputs, every fourth group of four; lane (kg, c) = (lane / 16,
//     lane % 16) owns input kg of a step's four and the outputs 4c .. 4c+3.  Its metadata is one load per array
//     (16 lanes side by side: the 128-byte line of a row of two-byte values), nothing passes through LDS.
//   - The four outputs of a lane are column c of four instructions ("block q" = the outputs 4c + q), and all four share
//     the A operand, the weights of (sample c, input kg): the lane evaluates that basis itself and spreads the four
//     weights over ten registers.  No basis tile, no barrier in the loop, and no row of the tile computed twice.
//   - The four waves' sums meet in LDS at the end: a quarter of the partial sums leave for memory, and the next layer
//     (or the reduction) reads a quarter.
//   - Codewords are requested two steps ahead and in front of a step's products, so that the address units - two clocks
//     for every gathered row, a 128-byte line into the vector cache: 7 us of configuration 3's first layer - work while
//     the matrix instructions do (all of a short chunk's rows up front, products behind them: 19.5 us; rows requested
//     behind the products: 18.8; in front of them: 17.2).
//
// Configuration 3 at batch 16, first layer 18.8 -> 17.2 us (of which about 2 pass before every XCD has started, 2 until
// the ids are there), head 30.9 -> 28.7, with an fp32 codebook at batch 8 47.8 -> 36.2; 64-40-20-8 at batch 5 24.3 ->
// 18.6; ten heads of 2048-256-21 at batch 8 61.0 -> 53.8.
//
// HALF: the same lanes with fp16 operands, a lane's ten weights and coefficients as five pairs, four, four and two of them to
// a v_mfma_f32_16x16x16_f16.  (One instruction shape for all: next behind a v_mfma_f32_16x16x32_f16 with the same sums, this one
// takes them before they are written, and the compiler puts no wait between the two - it does not for two of one shape, where
// none is needed.  A chain of whole numbers in one accumulator had every sum wrong, with three other accumulators in between
// none; here, 2.7e7 in place of 0.9.  16x16x32 for the first eight measured the same time, 19.4 and 19.2 us for 2048-1024-256 at 16.)
// Int8 rows take the layer's scale at the end, as in kan_fused.hip.  Blocks of 16 samples share a step's
// coefficients, so 64 samples cost a lane four bases for 256 edges - twice the tiles of kan_fused.hip, whose workgroups share them -,
// and that is what bounds it there, with the address units (146 - 150 G rows/s, the tiles up to 175); at up to 48 samples it is
// the gathers and their latency.  Against the tiles of 128 outputs it has no basis tile, no barrier, tiles of half the
// width (outputs rarely fill 128) and a quarter of the partial sums: 1000-333-21 at batch 37 25.7 -> 19.7 us, its layers 11.7 + 8.4
// -> 9.2 + 7.1; 2048-1024-256 at 16 / 48 28.7 / 39.5 -> 25.6 / 33.8, 507 x 40 at 56 10.8 -> 8.3, 931-128-50, four heads, at 36
// 27.6 -> 17.7, forty of 1748-162-21 at 16 134 -> 82.  Steps are kept apart from two blocks on: what two of them hold did not fit
// into 256 registers (forty of 1748-128-21 with fp32 gains at batch 32 86 -> 69 us, precise 109 -> 95).

#include <type_traits>

#include "kan_device.hpp"
#include "kan_internal.hpp"
#include "kan_mfma_common.hpp"

namespace kan {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 h16x4 __attribute__((ext_vector_type(4)));

#ifdef KAN_WAVE_HALF
constexpr bool kHalf = true;
#else
constexpr bool kHalf = false;
#endif
constexpr int kThreads = 256, kWaves = 4;
constexpr int kCols = kFusedWaveCols;          // outputs per workgroup
static_assert(kCols == 64 && kFusedWaveStep == 4 * kWaves, "lane layout");

// Four consecutive values of a per-edge array as loaded (alignment of one element).
template <typename T> struct Raw4 {
  uint32_t w[sizeof(T)];
};
// NT: read past the caches' keeping (next to codebooks of megabytes, which need the L2: 4096 x 4096 with 262,144 rows
// at batch 31 152 -> 132 us, fp32 rows of configuration 3's head at batch 8 51 -> 36; a stream that an L2 could keep
// from one call to the next loses: configuration 3's first layer at batch 16 17.2 -> 19.3).
template <bool NT, typename T>
__device__ __forceinline__ void load4(const T* p, Raw4<T>& r) {
  if constexpr (NT && sizeof(T) == 4) {
    typedef uint32_t v4 __attribute__((ext_vector_type(4), aligned(4)));
    const v4 v = __builtin_nontemporal_load((const v4*)p);
#pragma unroll
    for (int n = 0; n < 4; ++n) r.w[n] = v[n];
  } else if constexpr (NT && sizeof(T) == 2) {
    typedef uint32_t v2 __attribute__((ext_vector_type(2), aligned(2)));
    const v2 v = __builtin_nontemporal_load((const v2*)p);
    r.w[0] = v.x;
    r.w[1] = v.y;
  } else {
    __builtin_memcpy(r.w, p, 4 * sizeof(T));
  }
}
// Value q of the lane's four, which start `shift` elements into what was loaded (lanes at the end of the array).
template <typename T>
__device__ __forceinline__ T pick(const Raw4<T>& r, int q) {
  T v;
  if constexpr (sizeof(T) == 4) {
    v = __builtin_bit_cast(T, r.w[q]);
  } else if constexpr (sizeof(T) == 2) {
    v = __builtin_bit_cast(T, (uint16_t)(r.w[q >> 1] >> (16 * (q & 1))));
  } else {
    v = __builtin_bit_cast(T, (uint8_t)(r.w[0] >> (8 * q)));
  }
  return v;
}
template <typename T>
__device__ __forceinline__ void shift_down(Raw4<T>& r, int shift) {
  if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int n = 1; n < 4; ++n) {
      const bool on = shift >= n;                // one element down, `shift` times
      r.w[0] = on ? r.w[1] : r.w[0];
      r.w[1] = on ? r.w[2] : r.w[1];
      r.w[2] = on ? r.w[3] : r.w[2];
    }
  } else if constexpr (sizeof(T) == 2) {
    const uint64_t v = (((uint64_t)r.w[1] << 32) | r.w[0]) >> (16 * shift);
    r.w[0] = (uint32_t)v;
    r.w[1] = (uint32_t)(v >> 32);
  } else {
    r.w[0] >>= 8 * shift;
  }
}

__device__ __forceinline__ h16x4 operand(uint32_t lo, uint32_t hi) { return __builtin_bit_cast(h16x4, make_uint2(lo, hi)); }

// Four weights at their places span .. span + 3 among ten: three conditional shifts, by 1, 2 and 4.
__device__ __forceinline__ void spread(float w0, float w1, float w2, float w3, int span, float (&v)[kG]) {
  const bool s1 = span & 1, s2 = span & 2, s4 = span & 4;
  const float a[5] = {s1 ? 0.f : w0, s1 ? w0 : w1, s1 ? w1 : w2, s1 ? w2 : w3, s1 ? w3 : 0.f};
  float b[7];
#pragma unroll
  for (int n = 0; n < 7; ++n) b[n] = s2 ? (n >= 2 ? a[n - 2] : 0.f) : (n < 5 ? a[n] : 0.f);
#pragma unroll
  for (int n = 0; n < kG; ++n) v[n] = s4 ? (n >= 4 ? b[n - 4] : 0.f) : (n < 7 ? b[n] : 0.f);      // (span 6: b[6] is 0)
}

// The same as fp16 pairs, slots 0 .. 9 of an operand (the places as above: a 64-bit shift by one place, selects by two and four).
__device__ __forceinline__ void spread_half(uint32_t w01, uint32_t w23, int span, uint32_t (&v)[5]) {
  const bool s1 = span & 1, s2 = span & 2, s4 = span & 4;
  const uint64_t w = (((uint64_t)w23 << 32) | w01) << (s1 ? 16 : 0);
  const uint32_t a[3] = {(uint32_t)w, (uint32_t)(w >> 32), s1 ? w23 >> 16 : 0u};
  const uint32_t b[4] = {s2 ? 0u : a[0], s2 ? a[0] : a[1], s2 ? a[1] : a[2], s2 ? a[2] : 0u};
  v[0] = s4 ? 0u : b[0];
  v[1] = s4 ? 0u : b[1];
  v[2] = s4 ? b[0] : b[2];
  v[3] = s4 ? b[1] : b[3];
  v[4] = s4 ? b[2] : 0u;
}

// MB: blocks of 16 samples (1 or 2; 1 to 4 with HALF).  HALF: fp16 operands.  CH: the input arrives as the previous layer's partial sums, slices
// [x_parts][B][n_in]; the workgroup adds those of its own inputs in slice order, squashes them and keeps them in
// dynamic shared memory, [sample rows][inputs of the chunk].
template <typename IdxT, typename GbT, typename CbT, int MB, bool CH, bool HALF>
__global__ __launch_bounds__(kThreads, 2) void kan_fused_wave_kernel(const FusedArgs a) {
  constexpr bool kNt = sizeof(IdxT) == 4 || sizeof(CbT) == 4;     // (32-bit ids: more than 65,536 rows)
  constexpr int kLead = 2;                     // steps between the request of codewords and their use
  constexpr bool kEarly = sizeof(CbT) < 4;     // registers for a step's codewords and those of the next three: requested in
  constexpr int kSlots = kEarly ? 4 : 2;       // front of a step's products, else behind them
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kg = lane >> 4, c = lane & 15;
  // Workgroups go to the eight XCDs in turn.  Several heads, or an input in slices: runs of consecutive (head, chunk,
  // tile) items per XCD, so that a codebook, or a line of the slices, enters one L2 only.
  int head = blockIdx.z, chunk = blockIdx.y, tile = blockIdx.x;
  if (gridDim.z > 1 || CH) {
    const unsigned T = gridDim.x, C = gridDim.y, W = T * C * gridDim.z;
    const unsigned L = blockIdx.x + T * (blockIdx.y + C * blockIdx.z);
    const unsigned xcd = L & 7u, m = L >> 3, q = W >> 3, r = W & 7u;
    const unsigned item = xcd * q + min(xcd, r) + m;          // XCD x owns q + (x < r) items
    head = (int)(item / (T * C));
    const unsigned rem = item % (T * C);
    chunk = (int)(rem / T);
    tile = (int)(rem % T);
  }
  const int n_in = a.n_in, n_out = a.n_out, B = a.B;
  const int i_begin = chunk * a.rows_per_chunk, i_end = min(n_in, i_begin + a.rows_per_chunk);
  const int n_steps = (i_end - i_begin + kFusedWaveStep - 1) / kFusedWaveStep;
  const int i_lane = i_begin + 4 * wave + kg;                 // step k: input i_lane + 16 k
  const LayerPtrs hp = a.h[head];
  const IdxT* idx = (const IdxT*)hp.idx;
  const GbT* gain = (const GbT*)hp.gain;
  const GbT* bias = (const GbT*)hp.bias;
  const Q8Params qp = {hp.gain_log2_lo, hp.gain_log2_step, hp.bias_scale};
  const CbT* cb = (const CbT*)hp.cb;
  const float scale = sizeof(CbT) == 1 ? hp.scale : 1.0f;
  const float gmul = HALF ? 1.0f : scale;       // fp16 coefficients: the sums are scaled
  const float* xh = a.x + (long long)head * a.x_head_stride;

  // the lane's four outputs; loads start at most four elements before the end of the arrays
  const int j0 = tile * kCols + 4 * c;
  const long long last4 = (long long)n_in * n_out - 4;

  struct Ids {
    Raw4<IdxT> v;
    int shift;
  };
  struct GainBias {
    Raw4<GbT> g, b;
    int shift;
  };
  // (steps past the end: the chunk's last row again, with no effect)
  auto edge_at = [&](int k, int& shift) {
    const long long e = (long long)min(i_lane + k * kFusedWaveStep, i_end - 1) * n_out + min(j0, n_out - 1);
    const long long at = min(e, last4);
    shift = (int)(e - at);
    return at;
  };
  auto load_ids = [&](int k, Ids& m) { load4<kNt>(idx + edge_at(k, m.shift), m.v); };
  auto load_gb = [&](int k, GainBias& m) {
    const long long at = edge_at(k, m.shift);
    load4<kNt>(gain + at, m.g);
    load4<kNt>(bias + at, m.b);
  };
  auto gather = [&](int k, Ids& m, RawRow<CbT> (&rows)[4], uint32_t& odd) {
    // (outputs past n_out of a lane: what lies behind in the array, a valid row, or a shifted-in zero; steps past the
    // end: row 0 for every lane, one line)
    shift_down(m.v, m.shift);
    odd = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t id = k < n_steps ? (uint32_t)pick(m.v, q) : 0u;
      load_row<CbT>(cb, id, rows[q]);
      odd |= row_odd<CbT>(cb, id) << q;
    }
  };

  // (one block: a pointer per lane, 27.0 against 28.0 us for 2048-1024-256 with byte codes at batch 4; several: offsets, a
  // register each, of at most 64 samples of 2^20 inputs)
  using Row = std::conditional_t<MB == 1, const float*, uint32_t>;
  Row xrow[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int b = min(mb * 16 + c, B - 1);
    if constexpr (MB == 1) xrow[mb] = xh + (long long)b * n_in;
    else xrow[mb] = (uint32_t)b * (uint32_t)n_in;
  }
  extern __shared__ __attribute__((aligned(16))) float sX[];
  const int x_len = i_end - i_begin;
  auto load_x = [&](int k, float (&u)[MB]) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      if constexpr (CH) u[mb] = sX[min(mb * 16 + c, B - 1) * x_len + min(i_lane + k * kFusedWaveStep, i_end - 1) - i_begin];
      else if constexpr (MB == 1) u[mb] = xrow[mb][min(i_lane + k * kFusedWaveStep, i_end - 1)];
      else u[mb] = xh[xrow[mb] + (uint32_t)min(i_lane + k * kFusedWaveStep, i_end - 1)];
    }
  };

  f32x4 acc[MB][4];
  float bsum[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    bsum[q] = 0.f;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb][q] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  Ids ids[4];
  GainBias gb[4];
  RawRow<CbT> rows[kSlots][4];
  uint32_t odd[kSlots];
  float u[4][MB];

  auto take_slices = [&] {
    // Sixteen bytes of one sample row per item; where there are fewer items than threads, the threads of an item
    // take consecutive runs of slices, whose sums are added in run order.
    __shared__ f32x4 s_run[kThreads];
    const int len4 = x_len >> 2, n_items = B * len4;
    const int runs = n_items >= kThreads ? 1 : kThreads / n_items;
    const int per_run = (a.x_parts + runs - 1) / runs;
    for (int q0 = 0; q0 < n_items; q0 += kThreads) {
      const int q = runs > 1 ? tid % n_items : q0 + tid, g = runs > 1 ? tid / n_items : 0;
      const bool live = q < n_items && g < runs;
      const int row = (live ? q : 0) / len4, c4 = (live ? q : 0) - row * len4;
      const float* src = xh + (long long)row * n_in + i_begin + 4 * c4;
      const int p_end = min(a.x_parts, (g + 1) * per_run);
      f32x4 sum = {0.f, 0.f, 0.f, 0.f};
      for (int p0 = g * per_run; p0 < p_end; p0 += 8) {
        f32x4 t[8];
#pragma unroll
        for (int p = 0; p < 8; ++p)               // (slices past the last one: re-reads of it, not added)
          t[p] = *(const f32x4*)(src + (long long)min(p0 + p, a.x_parts - 1) * a.x_part_stride);
#pragma unroll
        for (int p = 0; p < 8; ++p)
          if (p0 + p < p_end) sum += t[p];
      }
      bool owner = live;
      if (runs > 1) {                             // (uniform; one round then)
        s_run[tid] = sum;
        __syncthreads();
        owner = tid < n_items;
        if (owner)
          for (int r = 1; r < runs; ++r) sum += s_run[r * n_items + tid];
      }
      if (owner) {
        if (a.x_tanh) {
#pragma unroll
          for (int n = 0; n < 4; ++n) sum[n] = tanhf(sum[n]);
        }
        *(f32x4*)(sX + row * x_len + 4 * c4) = sum;
      }
    }
    __syncthreads();
  };

  // The first N steps' loads, the codewords of the first two, and the input.
  auto begin = [&](auto N) {
    constexpr int n = decltype(N)::value;
#pragma unroll
    for (int k = 0; k < n; ++k) load_ids(k, ids[k]);
#pragma unroll
    for (int k = 0; k < n; ++k) load_gb(k, gb[k]);
    if constexpr (!CH) {
#pragma unroll
      for (int k = 0; k < n; ++k) load_x(k, u[k]);
    }
#pragma unroll
    for (int k = 0; k < kLead; ++k) {
      gather(k, ids[k], rows[k], odd[k]);
      if constexpr (n > 2) load_ids(k + 4, ids[k]);
    }
    if constexpr (CH) {
      take_slices();
#pragma unroll
      for (int k = 0; k < n; ++k) load_x(k, u[k]);
    }
  };

  // A step, t = k mod 4.  GATHER, MORE: with the codewords of step k + 2, the other loads of later steps, all of them
  // unconditional (behind a branch around a load the compiler waits for more than is needed next); the last group of
  // steps has none that are not needed.
  auto step = [&](auto GATHER, auto MORE, int k, int t) {
    auto request = [&] {
      if constexpr (decltype(GATHER)::value) gather(k + kLead, ids[(t + kLead) % 4], rows[(t + kLead) % kSlots], odd[(t + kLead) % kSlots]);
    };
    if constexpr (kEarly) request();
    const bool live = i_lane + k * kFusedWaveStep < i_end;
    GainBias& m = gb[t];
    shift_down(m.g, m.shift);
    shift_down(m.b, m.shift);
    // A: the weights of (sample c, input kg), at their places among ten; none for inputs past the end
    float w[HALF ? 1 : MB][kG];
    if constexpr (!HALF) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const BasisW bw = basis_fast(u[t][mb], a.rule);
        spread(live ? bw.w0 : 0.f, live ? bw.w1 : 0.f, live ? bw.w2 : 0.f, live ? bw.w3 : 0.f, bw.span, w[mb]);
      }
    }
    uint32_t ch[HALF ? 4 : 1][5];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float g, b;
      if constexpr (sizeof(GbT) == 1) {
        g = q8_gain(pick(m.g, q).v, qp);
        b = q8_bias(pick(m.b, q).v, qp);
      } else if constexpr (sizeof(GbT) == 2) {
        g = __half2float(pick(m.g, q));
        b = __half2float(pick(m.b, q));
      } else {
        g = pick(m.g, q);
        b = pick(m.b, q);
      }
      bsum[q] += live ? b : 0.f;
      align_row<CbT>(rows[t % kSlots][q], (odd[t % kSlots] >> q) & 1u);
      if constexpr (HALF) {
        dequant_row<CbT>(rows[t % kSlots][q], g * gmul, ch[q]);
      } else {
        float cf[kG];
        dequant_row_f32<CbT>(rows[t % kSlots][q], g * gmul, cf);
#pragma unroll
        for (int n = 0; n < kG; ++n)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
            acc[mb][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[mb][n], cf[n], acc[mb][q], 0, 0, 0);
      }
    }
    if constexpr (HALF) {                         // four, four and two coefficients of the four inputs at a time
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const BasisW bw = basis_fast(u[t][mb], a.rule);
        const uint32_t w01 = pack_h2(bw.w0, bw.w1), w23 = pack_h2(bw.w2, bw.w3);
        uint32_t wh[5];
        spread_half(live ? w01 : 0u, live ? w23 : 0u, bw.span, wh);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc[mb][q] = __builtin_amdgcn_mfma_f32_16x16x16f16(operand(wh[0], wh[1]), operand(ch[q][0], ch[q][1]), acc[mb][q], 0, 0, 0);
          acc[mb][q] = __builtin_amdgcn_mfma_f32_16x16x16f16(operand(wh[2], wh[3]), operand(ch[q][2], ch[q][3]), acc[mb][q], 0, 0, 0);
          acc[mb][q] = __builtin_amdgcn_mfma_f32_16x16x16f16(operand(wh[4], 0u), operand(ch[q][4], 0u), acc[mb][q], 0, 0, 0);
        }
      }
    }
    if constexpr (!kEarly) request();
    if constexpr (decltype(MORE)::value) {
      load_gb(k + 4, m);
      load_x(k + 4, u[t]);
      load_ids(k + kLead + 4, ids[(t + kLead) % 4]);
    }
    if constexpr (MB > 1) __builtin_amdgcn_sched_barrier(0);              // (what two steps hold does not fit)
  };
  constexpr auto yes = std::true_type{};
  constexpr auto no = std::false_type{};
  if (n_steps <= 2) {                             // (short chunks: nothing is loaded that is not needed)
    begin(std::integral_constant<int, 2>{});
    step(no, no, 0, 0);
    if (n_steps > 1) step(no, no, 1, 1);
  } else {
    begin(std::integral_constant<int, 4>{});
    int k = 0;
    for (; k + 4 < n_steps; k += 4) {
      step(yes, yes, k, 0);
      step(yes, yes, k + 1, 1);
      step(yes, yes, k + 2, 2);
      step(yes, yes, k + 3, 3);
    }
    step(yes, no, k, 0);
    if (k + 1 < n_steps) {
      step(yes, no, k + 1, 1);
      if (k + 2 < n_steps) {
        step(no, no, k + 2, 2);
        if (k + 3 < n_steps) step(no, no, k + 3, 3);
      }
    }
  }

  // ---- sums of the waves.  A lane's accumulators are (sample 4 kg + r, output 4c + q): wave w finishes the
  //      samples of r = w, four consecutive outputs per lane -------------------------------------------------
  __shared__ f32x4 s_red[kWaves][MB][4][64];
#pragma unroll
  for (int q = 0; q < 4; ++q) {                   // the biases of all inputs of the wave
    bsum[q] += __shfl_xor(bsum[q], 16);
    bsum[q] += __shfl_xor(bsum[q], 32);
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      s_red[wave][mb][r][lane] =
          HALF ? f32x4{fmaf(scale, acc[mb][0][r], bsum[0]), fmaf(scale, acc[mb][1][r], bsum[1]),
                       fmaf(scale, acc[mb][2][r], bsum[2]), fmaf(scale, acc[mb][3][r], bsum[3])}
               : f32x4{acc[mb][0][r] + bsum[0], acc[mb][1][r] + bsum[1], acc[mb][2][r] + bsum[2], acc[mb][3][r] + bsum[3]};
  __syncthreads();
  float* dst = a.dst + (long long)head * a.dst_head_stride + (long long)chunk * a.dst_chunk_stride;
  const bool whole = n_out % 4 == 0 && ((uintptr_t)dst & 15) == 0;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    f32x4 v = s_red[0][mb][wave][lane];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += s_red[w][mb][wave][lane];
    const int b = mb * 16 + 4 * kg + wave;
    if (a.apply_tanh) {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = tanhf(v[q]);
    }
    if (b < B && j0 < n_out) {
      float* o = dst + (long long)b * n_out + j0;
      if (whole) {
        *(f32x4*)o = v;
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (j0 + q < n_out) o[q] = v[q];
      }
    }
  }
}

template <typename IdxT, typename GbT, typename CbT, int MB>
hipError_t launch_blocks(const FusedArgs& a, dim3 grid, hipStream_t s) {
  const bool ch = a.x_parts > 1;
  const size_t lds = ch ? (size_t)a.B * a.rows_per_chunk * 4 : 0;
  if (ch) hipLaunchKernelGGL((kan_fused_wave_kernel<IdxT, GbT, CbT, MB, true, kHalf>), grid, dim3(kThreads), lds, s, a);
  else hipLaunchKernelGGL((kan_fused_wave_kernel<IdxT, GbT, CbT, MB, false, kHalf>), grid, dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

template <typename IdxT, typename GbT, typename CbT>
hipError_t launch_variant(const FusedArgs& a, dim3 grid, hipStream_t s) {
  if (a.B <= 16) return launch_blocks<IdxT, GbT, CbT, 1>(a, grid, s);
  if (a.B <= 32) return launch_blocks<IdxT, GbT, CbT, 2>(a, grid, s);
  if constexpr (kHalf) {
    if (a.B <= 48) return launch_blocks<IdxT, GbT, CbT, 3>(a, grid, s);
    return launch_blocks<IdxT, GbT, CbT, 4>(a, grid, s);
  }
  return hipErrorInvalidValue;
}

template <typename IdxT>
hipError_t launch_types(const GatherCfg& c, const FusedArgs& a, dim3 grid, hipStream_t s) {
  if (c.code == kCbI8) {
    if (c.gb_kind == kGbQ8) return launch_variant<IdxT, q8_t, int8_t>(a, grid, s);
    return c.gb_kind == kGbF16 ? launch_variant<IdxT, __half, int8_t>(a, grid, s) : launch_variant<IdxT, float, int8_t>(a, grid, s);
  }
  if (c.gb_kind == kGbQ8) return hipErrorInvalidValue;      // byte-coded gain/bias go with Int8 codebooks
  if (c.code == kCbBfp8)
    return c.gb_kind == kGbF16 ? launch_variant<IdxT, __half, bfp8_t>(a, grid, s) : launch_variant<IdxT, float, bfp8_t>(a, grid, s);
  if (c.code == kCbF16)
    return c.gb_kind == kGbF16 ? launch_variant<IdxT, __half, __half>(a, grid, s) : launch_variant<IdxT, float, __half>(a, grid, s);
  return c.gb_kind == kGbF16 ? launch_variant<IdxT, __half, float>(a, grid, s) : launch_variant<IdxT, float, float>(a, grid, s);
}

}  // namespace

#ifdef KAN_WAVE_HALF
hipError_t launch_fused_wave_half(const GatherCfg& c, const FusedArgs& a, dim3 grid, hipStream_t s) {
#else
hipError_t launch_fused_wave(const GatherCfg& c, const FusedArgs& a, dim3 grid, hipStream_t s) {
#endif
  if (c.code == kDense || a.B < 1 || a.B > (kHalf ? 64 : 32) || (long long)a.n_in * a.n_out < 4 || a.rows_per_chunk % kFusedWaveStep != 0)
    return hipErrorInvalidValue;
  // what the 16-byte loads of the slices and the inputs in LDS assume
  if (a.x_parts > 1 && (a.x_parts > kFusedChainMaxParts || a.n_in % 4 != 0 || a.x_part_stride % 4 != 0 || a.x_head_stride % 4 != 0 ||
                        (uintptr_t)a.x % 16 != 0 || (long long)a.B * a.rows_per_chunk > kFusedWaveChainFloats))
    return hipErrorInvalidValue;
  return c.idx_u32 ? launch_types<uint32_t>(c, a, grid, s) : launch_types<uint16_t>(c, a, grid, s);
}

}  // namespace kan
