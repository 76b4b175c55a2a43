// Small layers of the matrix-core path (batch > 64): basis, contraction and sum over the inputs in one launch.
//
// The streaming contraction of kan_mfma.hip is made for layers that fill the chip.  A layer of a few thousand
// edges behind it - the usual last layer of a head - ran as three launches (basis words, contraction, reduction of
// partial sums: 4-7 + 8-10 + 2.4-5 us), each of them a latency chain on a part of the chip.  Here a workgroup of
// eight waves owns 32 samples x 32 or 64 outputs and all inputs of the layer:
//   1. the coefficient records of every wave's first step and the bias sums are requested (they depend on nothing);
//   2. the inputs of the 32 samples are loaded - plain, or the slices that the previous layer left, added in slice
//      order and squashed - and kept in LDS;
//   3. wave w takes the steps w, w + 8, ... of 16 inputs: every lane evaluates the basis of eight (sample, input)
//      pairs and forms its own A fragments in registers (the lane of half a needs the inputs with i % 2 = a, and of
//      the other parity one word per quarter, which comes from the lane 32 away), so no Phi tile and no barrier;
//   4. the waves' sums meet in LDS, are added in wave order, and finished outputs leave.
// Operands, their order and the two forms (fp16; high and low parts with three products) are those of kan_mfma.hip.
// Bound by: latency (launch, two dependent reads, the reduction), then by one CU's vector-memory path for the
// records (20 bytes per edge at about 120 B/ns) and its vector ALU for the basis (55 instructions per pair).

#include "kan_device.hpp"
#include "kan_internal.hpp"
#include "kan_mfma_common.hpp"

namespace kan {
namespace {

constexpr int kTailThreads = 512;
constexpr int kTailWaves = kTailThreads / 64;
constexpr int IT = 16;                           // inputs per step, as in kan_mfma.hip
constexpr int kTailXStride = kTailMaxIn + 1;     // (odd: the 32 rows of a column lie in 32 banks)

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// The inputs of samples b0 .. b0 + 31 into xs: the tile's rows are one run of floats in memory, taken in items of four
// (wherever rows end), U items per thread and round, P slices of each in flight, added in slice order.  Loads are
// unconditional (clamped addresses; the last item of the run ends with it and repeats what the one before holds).  A
// tile of eight slices is two trips to memory that way at most (single floats, half the slices at a time, where rows are no multiple
// of four: six; 500-333-21 at batch 128 34.0 -> 29.1 us, 399 x 10 at any batch 19.0 -> 13.5).
template <int U, int P>
__device__ __forceinline__ void stage_inputs(const TailArgs& a, const float* x, int b0, float* xs) {
  const int n = min(32, a.B - b0) * a.n_in, items = (n + 3) >> 2;
  const float* const p = x + (long long)b0 * a.n_in;
  if (n < 4) {                                                          // (a last row of up to three inputs)
    const int t = threadIdx.x;
    if (t < n) {
      float sum = 0.f;
      for (int q = 0; q < a.x_parts; ++q) sum += p[(long long)q * a.x_part_stride + t];
      xs[t / a.n_in * kTailXStride + t % a.n_in] = a.x_tanh ? tanhf(sum) : sum;
    }
    return;
  }
  for (int base = threadIdx.x; base < items; base += U * kTailThreads) {
    int at[U];
    f32x4 sum[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      at[u] = min(4 * (base + u * kTailThreads), n - 4);
      sum[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int p0 = 0; p0 < a.x_parts; p0 += P) {
      f32x4 t[P][U];
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const float* const slice = p + (long long)min(p0 + q, a.x_parts - 1) * a.x_part_stride;
#pragma unroll
        for (int u = 0; u < U; ++u) t[q][u] = *(const f32x4_a4*)(slice + at[u]);
      }
#pragma unroll
      for (int q = 0; q < P; ++q) {
        if (p0 + q < a.x_parts) {
#pragma unroll
          for (int u = 0; u < U; ++u) sum[u] += t[q][u];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (base + u * kTailThreads >= items) continue;
      int row = at[u] / a.n_in, col = at[u] - row * a.n_in;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        xs[row * kTailXStride + col] = a.x_tanh ? tanhf(sum[u][c]) : sum[u][c];
        if (++col == a.n_in) {
          col = 0;
          ++row;
        }
      }
    }
  }
}

// The A fragments of one step for a lane: f[S] and, for the index words, ix (see kan_mfma.hip).
struct TailA {
  h16x8 f[5];
  uint32_t ix[3];
};

template <int NB, bool THREE>
__global__ __launch_bounds__(kTailThreads) void kan_tail_kernel(const TailArgs a) {
  constexpr int BN = 32 * NB;
  constexpr int NP = THREE ? 2 : 1;                 // parts of an operand
  constexpr int kRed = kTailWaves * 32 * BN, kXs = 32 * kTailXStride;
  __shared__ __attribute__((aligned(16))) float buf[kRed > kXs ? kRed : kXs];    // inputs, later the waves' sums
  __shared__ __attribute__((aligned(16))) uint32_t sSel[kSpans][8];
  __shared__ float sBias[BN];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ln = lane & 31, lh = lane >> 5;
  const int head = blockIdx.z, jt = blockIdx.x % a.n_jt, bt = blockIdx.x / a.n_jt;
  const int b0 = bt * 32, j0 = jt * BN;
  const int n_in = a.n_in, n_out = a.n_out;
  const int n_steps = (n_in + IT - 1) / IT;

  const uint4* cf[NP];
  cf[0] = a.cf + (long long)head * a.cf_head_stride;
  if constexpr (THREE) cf[1] = a.cf_lo + (long long)head * a.cf_head_stride;
  uint32_t b_off[NB];
#pragma unroll
  for (int n = 0; n < NB; ++n) b_off[n] = (uint32_t)(lh * 2 * n_out + min(j0 + 32 * n + ln, n_out - 1));
  auto load_b = [&](int step, uint4 (&bf)[NP][NB][5][2]) {
    const uint32_t s0 = (uint32_t)step * 20u * (uint32_t)n_out;
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int S = 0; S < 5; ++S)
#pragma unroll
          for (int h = 0; h < 2; ++h) bf[p][n][S][h] = cf[p][s0 + b_off[n] + (uint32_t)((4 * S + h) * n_out)];
  };
  // (the next step's records travel behind the current step where the registers allow it)
  constexpr bool kTwo = NP * NB == 1;
  uint4 bf0[NP][NB][5][2], bf1[kTwo ? NP : 1][NB][5][2];
  load_b(min(wave, n_steps - 1), bf0);
  fill_sparse_selectors(sSel, tid);
  if (tid < BN) {
    const float* bp = a.bias_partial + (long long)head * a.bp_head_stride + min(j0 + tid, n_out - 1);
    const int nrb = (n_in + kMfmaPrepRows - 1) / kMfmaPrepRows;
    float v[kTailMaxIn / kMfmaPrepRows], bs = 0.f;
#pragma unroll
    for (int r = 0; r < kTailMaxIn / kMfmaPrepRows; ++r) v[r] = bp[(long long)min(r, nrb - 1) * n_out];
#pragma unroll
    for (int r = 0; r < kTailMaxIn / kMfmaPrepRows; ++r) bs += r < nrb ? v[r] : 0.f;
    sBias[tid] = bs;
  }
  {
    const float* x = a.x + (long long)head * a.x_head_stride;
    // (as many items in flight as a thread has, up to 24 and 32 loads: with three items of eight slices whatever the width, two thirds of
    // the loads of 64 inputs were repeats: 864-64-32 at batch 105 24.4 us, 1560-64-16 precise at 182 39.6, 1024-128-64 at 70 27.4, 600-256-16 at 70 31.4,
    // now 21.1, 35.6, 25.8 and 29.7)
    const int own = (8 * n_in + kTailThreads - 1) / kTailThreads;
    if (a.x_parts == 1) {
      if (own <= 2) stage_inputs<2, 1>(a, x, b0, buf);
      else stage_inputs<8, 1>(a, x, b0, buf);
    } else if (own == 1) {
      stage_inputs<1, 8>(a, x, b0, buf);
    } else if (own == 2 && a.x_parts > 4) {
      stage_inputs<2, 8>(a, x, b0, buf);
    } else if (own == 4 || a.x_parts <= 4) {
      stage_inputs<4, 4>(a, x, b0, buf);
    } else {
      stage_inputs<3, 8>(a, x, b0, buf);
    }
    for (int t = tid + (a.B - b0) * n_in; t < 32 * n_in; t += kTailThreads) buf[t / n_in * kTailXStride + t % n_in] = 0.f;   // rows past the last
    const int pad = n_steps * IT - n_in;            // the last step's missing inputs (their coefficients are zeros)
    for (int t = tid; t < 32 * pad; t += kTailThreads) buf[(t / pad) * kTailXStride + n_in + t % pad] = 0.f;
  }
  __syncthreads();

  f32x16 acc[NB], accx[NB];
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[n][r] = accx[n][r] = 0.f;

  auto make_a = [&](int step, TailA (&fa)[NP]) {
    const float* xr = buf + ln * kTailXStride + step * IT + lh;
    uint32_t own[NP][4], bits[4], iw[4];            // pair-4 values, their position bits, index half-words per quarter
    uint32_t st[NP][4][4];
#pragma unroll
    for (int ph = 0; ph < 4; ++ph) {
      uint32_t v4[NP][2];
      iw[ph] = 0;
      bits[ph] = 0;
#pragma unroll
      for (int q = 0; q < 2; ++q) {                 // input 4 ph + lh + 2 q of the step
        const BasisW bw = basis_fast(xr[4 * ph + 2 * q], a.rule);
        uint32_t w01[NP], w23[NP];
        if constexpr (THREE) {
          split_weights(bw.w0, bw.w1, w01[0], w01[1]);
          split_weights(bw.w2, bw.w3, w23[0], w23[1]);
        } else {
          w01[0] = pack_h2(bw.w0, bw.w1);
          w23[0] = pack_h2(bw.w2, bw.w3);
        }
        const uint4 sl = *(const uint4*)&sSel[bw.span][0];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          st[p][ph][2 * q] = __builtin_amdgcn_perm(w23[p], w01[p], sl.x);
          st[p][ph][2 * q + 1] = __builtin_amdgcn_perm(w23[p], w01[p], sl.y);
          v4[p][q] = __builtin_amdgcn_perm(w23[p], w01[p], sl.z);
        }
        iw[ph] |= (sl.w & 0xffu) << (8 * q);
        bits[ph] |= (sl.w >> 8) << q;
      }
#pragma unroll
      for (int p = 0; p < NP; ++p) own[p][ph] = v4[p][0] | (v4[p][1] << 16);
    }
    // Quarter ph of the tail fragment belongs to the lane half ph % 2: it keeps its own two values and takes the
    // other parity's from the lane 32 away.
    uint32_t tail_ix = 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const uint32_t kb = lh ? bits[2 * k + 1] : bits[2 * k], sb = lh ? bits[2 * k] : bits[2 * k + 1];
      const uint32_t rb = (uint32_t)__shfl_xor((int)sb, 32);
      const uint32_t eb = lh ? rb : kb, ob = lh ? kb : rb;            // even, odd inputs of the quarter
      const uint32_t byte = ((eb & 1u) | ((2u + (ob & 1u)) << 2)) | (((eb >> 1) | ((2u + (ob >> 1)) << 2)) << 4);
      tail_ix |= byte << (8 * k);
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const uint32_t kv = lh ? own[p][2 * k + 1] : own[p][2 * k], sv = lh ? own[p][2 * k] : own[p][2 * k + 1];
        const uint32_t rv = (uint32_t)__shfl_xor((int)sv, 32);
        const uint32_t ev = lh ? rv : kv, ov = lh ? kv : rv;
        uint32_t* w = (uint32_t*)&fa[p].f[4];
        w[2 * k] = __builtin_amdgcn_perm(ov, ev, 0x05040100u);        // (even 0, odd 0)
        w[2 * k + 1] = __builtin_amdgcn_perm(ov, ev, 0x07060302u);    // (even 1, odd 1)
      }
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
#pragma unroll
      for (int S = 0; S < 4; ++S) {
        uint32_t* w = (uint32_t*)&fa[p].f[S];
#pragma unroll
        for (int c = 0; c < 4; ++c) w[c] = st[p][S][c];
      }
    }
    fa[0].ix[0] = iw[0] | (iw[1] << 16);
    fa[0].ix[1] = iw[2] | (iw[3] << 16);
    fa[0].ix[2] = tail_ix;
  };
  auto product = [&](const TailA& f, const uint32_t (&ix)[3], const uint4 (&b)[NB][5][2], f32x16 (&c)[NB]) {
#pragma unroll
    for (int S = 0; S < 5; ++S)
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const uint4 two[2] = {b[n][S][0], b[n][S][1]};
        const h16x16 fb = __builtin_bit_cast(h16x16, two);
        const int w = (int)ix[S >> 1];
        if (S == 1 || S == 3) c[n] = __builtin_amdgcn_smfmac_f32_32x32x32_f16(f.f[S], fb, c[n], w, 0, 1);
        else c[n] = __builtin_amdgcn_smfmac_f32_32x32x32_f16(f.f[S], fb, c[n], w, 0, 0);
      }
  };
  auto body = [&](int step, const uint4 (&b)[NP][NB][5][2]) {
    TailA fa[NP];
    make_a(step, fa);
    if constexpr (THREE) {
      product(fa[0], fa[0].ix, b[1], accx);
      product(fa[1], fa[0].ix, b[0], accx);
    }
    product(fa[0], fa[0].ix, b[0], acc);
  };
  if constexpr (kTwo) {
    for (int s = wave; s < n_steps; s += 2 * kTailWaves) {
      load_b(min(s + kTailWaves, n_steps - 1), bf1);
      body(s, bf0);
      if (s + kTailWaves < n_steps) {
        load_b(min(s + 2 * kTailWaves, n_steps - 1), bf0);
        body(s + kTailWaves, bf1);
      }
    }
  } else {
    for (int s = wave; s < n_steps; s += kTailWaves) {
      body(s, bf0);
      if (s + kTailWaves < n_steps) load_b(s + kTailWaves, bf0);
    }
  }

  __syncthreads();                                  // every wave is done with the inputs
  const int nw = min(n_steps, kTailWaves);
  if (wave < nw) {
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) {                // D layout: column lane % 32, row 8 (r / 4) + 4 (lane / 32) + r % 4
        const float v = THREE ? fmaf(1.0f / 2048.0f, accx[n][r], acc[n][r]) : acc[n][r];
        buf[(wave * 32 + 8 * (r >> 2) + 4 * lh + (r & 3)) * BN + 32 * n + ln] = v;
      }
  }
  __syncthreads();
  float* dst = a.dst + (long long)head * a.dst_head_stride;
#pragma unroll
  for (int u = 0; u < 32 * BN / kTailThreads; ++u) {
    const int o = tid + u * kTailThreads, row = o / BN, col = o % BN;
    float s = 0.f;
    for (int w = 0; w < nw; ++w) s += buf[w * 32 * BN + o];
    float v = fmaf(a.scale[head], s, sBias[col]);
    if (a.apply_tanh) v = tanhf(v);
    if (b0 + row < a.B && j0 + col < n_out) dst[(long long)(b0 + row) * n_out + j0 + col] = v;
  }
}

}  // namespace

hipError_t launch_tail(const TailArgs& a, bool split, int tile_n, dim3 grid, hipStream_t s) {
  if (!a.cf || !a.bias_partial || !a.x || !a.dst || (split && !a.cf_lo)) return hipErrorInvalidValue;
  if (a.n_in < 1 || a.n_in > kTailMaxIn || a.B < 1 || a.x_parts < 1 || (long long)a.n_out * kTailMaxIn * 20 > 0x7fffffffLL)
    return hipErrorInvalidValue;
  if (tile_n != 32 && (tile_n != 64 || split)) return hipErrorInvalidValue;
  if ((long long)a.n_jt * tile_n < a.n_out || (long long)(grid.x / (unsigned)a.n_jt) * 32 < a.B) return hipErrorInvalidValue;
  if (split) hipLaunchKernelGGL((kan_tail_kernel<1, true>), grid, dim3(kTailThreads), 0, s, a);
  else if (tile_n == 64) hipLaunchKernelGGL((kan_tail_kernel<2, false>), grid, dim3(kTailThreads), 0, s, a);
  else hipLaunchKernelGGL((kan_tail_kernel<1, false>), grid, dim3(kTailThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace kan
