// Dense-coefficient baseline at up to 64 samples per tile: one pass over coef[in][out][10] (40 bytes per
// edge, the only traffic that counts), straight from memory into the operand registers of the matrix
// instruction, no LDS copy and no converted copy in memory.
//
//   y[b][j] = sum over (i, m) of B_m(x_bi) * coef[i][j][m]: a product with (in x 10) terms per output.
//
// The order of these terms is free as long as both operands agree on it, so a lane takes whole grids: lane
// (g, c) = (lane / 16, lane % 16) of a 16-column tile loads the ten coefficients of its own edge (input 4g + t,
// column c) - 40 consecutive bytes, sixteen lanes side by side: 640 consecutive bytes - and they are the
// operand as they are.
//
// What bounds it: the stream of coefficients.  All of a wave's loads for two groups of 16 inputs are in flight
// before the first weight is computed, so that a launch of two groups per wave asks for its whole share of
// the stream at once.  (The three loads of a grid touch the same lines: with non-temporal loads, whose lines the
// vector cache drops, 2048 x 512 at batch 16 takes 17.7 instead of 13.2 us.)
// Measured, call by call on three sets of coefficients, against the fp32 FMA kernel (to batch 16) and the converted
// records + streaming contraction (above) that came before: 2048 x 512 (42 MB) at batch 1 / 16 / 32 / 64 / 128
// 12.4 / 13.1 / 17.7 / 21.4 / 29.7 against 19.4 / 34.3 / 33.7 / 35.0 / 38.8 us; 4096 x 1024 at batch 16 / 64 37.9 / 62.1
// against 96.9 / 110 us; 64 x 32 at batch 16 / 64 4.6 / 11.2 against 11.2 / 21.1 us.
//
// Two forms:
//   kan_dense_kernel        up to 16 samples, fp32 operands (v_mfma_f32_16x16x4f32: lane group g brings one of
//                           the four terms).  The lane that needs a weight computes it: lane (g, s) evaluates the
//                           basis of (sample s, input 4g + t) and spreads the four weights over ten registers.
//                           Weights in fp64, rounded once to fp32 (error 3.0e-8 against 1.3e-7 with fp32
//                           polynomials; behind the stream they cost less than 0.2 us: 2048 x 512 at batch
//                           16 14.2 -> 14.3 us back to back, 4096 x 1024 38.0 -> 38.15).
//                           No LDS, no barrier before the sums of the four waves (spread over the inputs) meet.
//   kan_dense_split_kernel  17 samples and more, operands in high and low fp16 parts (v_mfma_f32_16x16x32_f16,
//                           three products: 22 significant bits), tiles of 32 or 64 samples.  The weights of a
//                           group are built once for the four waves that share it (64 columns), in LDS,
//                           in the order in which the instruction reads them.

#include "kan_device.hpp"
#include "kan_internal.hpp"
#include "kan_mfma_common.hpp"

namespace kan {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));     // a grid starts at a multiple of 8 bytes
typedef float f32x2_a8 __attribute__((ext_vector_type(2), aligned(8)));

constexpr int kStepIn = 16;               // inputs per step of a wave (four per lane group)

// The grids of this lane's edges of one step: inputs i0 + 4g + t.  Rows from i_end on re-read the chunk's last row
// (their weights are zero).
struct Grids {
  float c[4][kG];
};
__device__ __forceinline__ void load_grids(const float* col, long long row_stride, int i0, int i_end, Grids& r) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const float* p = col + (long long)min(i0 + t, i_end - 1) * row_stride;
    const f32x4 a = *(const f32x4_a8*)p, b = *(const f32x4_a8*)(p + 4);
    const f32x2_a8 d = *(const f32x2_a8*)(p + 8);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      r.c[t][m] = a[m];
      r.c[t][4 + m] = b[m];
    }
    r.c[t][8] = d.x;
    r.c[t][9] = d.y;
  }
}

// Span and weights of basis_eval (evaluated in fp64, rounded once) in half its instructions: t = (7x + 7) / 2 and the
// local coordinate are exact in fp64, and the polynomials are written for fma.
__device__ __forceinline__ BasisW basis_fp64(float xf) {
  const double t = fma((double)fminf(fmaxf(xf, -1.0f), 1.0f), 3.5, 3.5);
  BasisW r;
  r.span = min((int)t, kSpans - 1);
  const double u = t - (double)r.span, om = 1.0 - u, u2 = u * u;
  r.w0 = (float)(om * om * (om * (1.0 / 6.0)));
  r.w1 = (float)fma(u2, fma(u, 0.5, -1.0), 2.0 / 3.0);
  r.w2 = (float)fma(u, fma(u, fma(u, -0.5, 0.5), 0.5), 1.0 / 6.0);
  r.w3 = (float)(u2 * (u * (1.0 / 6.0)));
  return r;
}

// The four weights at their places among ten, zeros elsewhere.
__device__ __forceinline__ void spread_weights(const BasisW& w, float (&v)[kG]) {
#pragma unroll
  for (int m = 0; m < kG; ++m) {
    float r = 0.f;
    r = w.span == m ? w.w0 : r;
    r = w.span == m - 1 ? w.w1 : r;
    r = w.span == m - 2 ? w.w2 : r;
    r = w.span == m - 3 ? w.w3 : r;
    v[m] = r;
  }
}

// Four waves interleaved over the inputs of the chunk, 16 columns, up to 16 samples.
__global__ __launch_bounds__(256, 2) void kan_dense_kernel(const DenseArgs a) {
  __shared__ f32x4 red[3][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, c = lane & 15;
  const int jt = blockIdx.x % a.n_jt, b0 = (blockIdx.x / a.n_jt) * 16;
  const int i_begin = blockIdx.y * a.rows_per_chunk + wave * kStepIn;
  const int i_end = min(a.n_in, (int)(blockIdx.y + 1) * a.rows_per_chunk);
  const int j = jt * 16 + c;
  const float* col = a.coef + (long long)min(j, a.n_out - 1) * kG;
  const long long row_stride = (long long)a.n_out * kG;
  const float* xrow = a.x + (long long)min(b0 + c, a.B - 1) * a.n_in;
  constexpr int kHop = 4 * kStepIn;       // inputs between two steps of a wave

  f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
  Grids buf[2];
  float xs[2][4];
  auto load = [&](int i0, int s) {
#pragma unroll
    for (int t = 0; t < 4; ++t) xs[s][t] = xrow[min(i0 + 4 * g + t, i_end - 1)];
    load_grids(col, row_stride, i0 + 4 * g, i_end, buf[s]);
  };
  auto step = [&](int i0, int s) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      BasisW w = basis_fp64(xs[s][t]);
      if (i0 + 4 * g + t >= i_end) w = {0.f, 0.f, 0.f, 0.f, 0};
      float v[kG];
      spread_weights(w, v);
#pragma unroll
      for (int m = 0; m < kG; m += 2) {
        acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(v[m], buf[s].c[t][m], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(v[m + 1], buf[s].c[t][m + 1], acc1, 0, 0, 0);
      }
    }
  };
  if (i_begin < i_end) {
    load(i_begin, 0);
    load(i_begin + kHop, 1);              // (past the end: the last row again)
    for (int i0 = i_begin; i0 < i_end; i0 += 2 * kHop) {
      step(i0, 0);
      if (i0 + 2 * kHop < i_end) load(i0 + 2 * kHop, 0);
      if (i0 + kHop < i_end) step(i0 + kHop, 1);
      if (i0 + 3 * kHop < i_end) load(i0 + 3 * kHop, 1);
    }
  }
  acc0 += acc1;
  if (wave > 0) red[wave - 1][lane] = acc0;
  __syncthreads();
  if (wave == 0) {
    acc0 += red[0][lane];
    acc0 += red[1][lane];
    acc0 += red[2][lane];
    float* dst = a.dst + (long long)blockIdx.y * a.dst_chunk_stride + j;
#pragma unroll
    for (int r = 0; r < 4; ++r) {         // (column c, sample 4g + r)
      const int b = b0 + 4 * g + r;
      if (b < a.B && j < a.n_out) dst[(long long)b * a.n_out] = acc0[r];
    }
  }
}

// Eight waves: four 16-column tiles x two groups of inputs; MB blocks of 16 samples.
template <int MB>
__global__ __launch_bounds__(512, 2) void kan_dense_split_kernel(const DenseArgs a) {
  // weights of a step, per group of inputs: [term group q][high, low][block of samples][lane] x 16 bytes
  constexpr int kRec = 5 * 2 * MB * 64;
  __shared__ uint4 sw[2][kRec];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, c = lane & 15, cw = wave & 3, grp = wave >> 2;
  const int jt = blockIdx.x % a.n_jt, b0 = (blockIdx.x / a.n_jt) * (16 * MB);
  const int i_first = blockIdx.y * a.rows_per_chunk + grp * kStepIn;
  const int i_end = min(a.n_in, (int)(blockIdx.y + 1) * a.rows_per_chunk);
  const int j = jt * 64 + cw * 16 + c;
  const float* col = a.coef + (long long)min(j, a.n_out - 1) * kG;
  const long long row_stride = (long long)a.n_out * kG;
  constexpr int kHop = 2 * kStepIn;

  f32x4 acc[MB], acx[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) acc[mb] = acx[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
  Grids buf[2];
  float xs[MB];
  uint32_t* const w32 = (uint32_t*)sw[grp];
  auto load_x = [&](int i0) {             // this lane's evaluations: input 4g + (its wave), sample c of every block
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      xs[mb] = a.x[(long long)min(b0 + mb * 16 + c, a.B - 1) * a.n_in + min(i0 + 4 * g + cw, i_end - 1)];
  };
  // Lane (g, c) of the operand holds the 40 terms (t, m) of inputs 4g .. 4g+3 in that order, eight to an
  // instruction: input 4g + t is the dwords 5t .. 5t+4 of its twenty.
  auto build = [&](int i0) {
    const bool live = i0 + 4 * g + cw < i_end;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      BasisW w = basis_fast(xs[mb], kRuleBspline3);
      if (!live) w = {0.f, 0.f, 0.f, 0.f, 0};
      uint32_t h01, l01, h23, l23;
      split_weights(w.w0, w.w1, h01, l01);
      split_weights(w.w2, w.w3, h23, l23);
      const bool odd = w.span & 1;
      const int d0 = w.span >> 1;
      auto spread = [&](uint32_t p01, uint32_t p23, uint32_t (&v)[5]) {
        const uint32_t a0 = odd ? p01 << 16 : p01;
        const uint32_t a1 = odd ? (p01 >> 16) | (p23 << 16) : p23;
        const uint32_t a2 = odd ? p23 >> 16 : 0u;
#pragma unroll
        for (int d = 0; d < 5; ++d) v[d] = d0 == d ? a0 : (d0 == d - 1 ? a1 : (d0 == d - 2 ? a2 : 0u));
      };
      uint32_t hi[5], lo[5];
      spread(h01, h23, hi);
      spread(l01, l23, lo);
#pragma unroll
      for (int d = 0; d < 5; ++d) {
        const int n = 5 * cw + d, q = n >> 2;
        uint32_t* p = w32 + (((q * 2) * MB + mb) * 64 + lane) * 4 + (n & 3);
        p[0] = hi[d];
        p[MB * 64 * 4] = lo[d];
      }
    }
  };
  auto contract = [&](int s) {
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      uint32_t bh[4], bl[4];
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int n = 8 * q + 2 * d;
        const float c0 = buf[s].c[n / kG][n % kG], c1 = buf[s].c[(n + 1) / kG][(n + 1) % kG];
        bh[d] = flush_h2(pack_h2(c0, c1));
        bl[d] = flush_h2(pack_h2((c0 - half_bits_to_float(bh[d] & 0xffffu)) * 2048.0f,
                                 (c1 - half_bits_to_float(bh[d] >> 16)) * 2048.0f));
      }
      const h16x8 b_hi = __builtin_bit_cast(h16x8, make_uint4(bh[0], bh[1], bh[2], bh[3]));
      const h16x8 b_lo = __builtin_bit_cast(h16x8, make_uint4(bl[0], bl[1], bl[2], bl[3]));
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const h16x8 a_hi = __builtin_bit_cast(h16x8, sw[grp][((q * 2) * MB + mb) * 64 + lane]);
        const h16x8 a_lo = __builtin_bit_cast(h16x8, sw[grp][((q * 2 + 1) * MB + mb) * 64 + lane]);
        acx[mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_hi, b_lo, acx[mb], 0, 0, 0);
        acc[mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_hi, b_hi, acc[mb], 0, 0, 0);
        acx[mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_lo, b_hi, acx[mb], 0, 0, 0);
      }
    }
  };
  // Every wave makes the same number of steps (the barriers); steps past the end contribute zeros.
  const int steps = (i_end - (int)(blockIdx.y * a.rows_per_chunk) + kHop - 1) / kHop;
  load_x(i_first);
  load_grids(col, row_stride, i_first + 4 * g, i_end, buf[0]);
  load_grids(col, row_stride, i_first + kHop + 4 * g, i_end, buf[1]);
  auto one = [&](int k, int s) {
    const int i0 = i_first + k * kHop;
    build(i0);
    __syncthreads();
    load_x(i0 + kHop);
    contract(s);
    if (k + 2 < steps) load_grids(col, row_stride, i0 + 2 * kHop + 4 * g, i_end, buf[s]);
    __syncthreads();
  };
  for (int k = 0; k < steps; k += 2) {
    one(k, 0);
    if (k + 1 < steps) one(k + 1, 1);
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) acc[mb] += acx[mb] * (1.0f / 2048.0f);
  f32x4* const red = (f32x4*)sw;          // (behind the loop's last barrier)
  if (grp == 1) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) red[(cw * MB + mb) * 64 + lane] = acc[mb];
  }
  __syncthreads();
  if (grp == 0) {
    float* dst = a.dst + (long long)blockIdx.y * a.dst_chunk_stride + j;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      acc[mb] += red[(cw * MB + mb) * 64 + lane];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int b = b0 + mb * 16 + 4 * g + r;
        if (b < a.B && j < a.n_out) dst[(long long)b * a.n_out] = acc[mb][r];
      }
    }
  }
}

}  // namespace

hipError_t launch_dense(const DenseArgs& a, int tile_m, dim3 grid, hipStream_t s) {
  if (tile_m == 16) hipLaunchKernelGGL(kan_dense_kernel, grid, dim3(256), 0, s, a);
  else if (tile_m == 32) hipLaunchKernelGGL(kan_dense_split_kernel<2>, grid, dim3(512), 0, s, a);
  else if (tile_m == 64) hipLaunchKernelGGL(kan_dense_split_kernel<4>, grid, dim3(512), 0, s, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace kan
