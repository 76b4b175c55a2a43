// Vector-ALU path of the KAN forward pass for gfx950 (fp32): VQ layers at batch 1 (larger batches go
// to the fused matrix-core kernel).
//
// Mapping.  Lanes own outputs j (JPL consecutive ones each), so the per-edge
// metadata idx/gain/bias[i][j..] of paper Eq. (1) is one contiguous, coalesced,
// read-once stream per i-row, and everything that depends on x_bi alone (the
// interval index and the four basis weights, App. A.1 / section 4.1) is the same
// for all lanes of a wave: it is computed once per i into LDS and broadcast.
// Only the 4 coefficients under the nonzero bases are gathered (from L2), scaled by
// gain (and the Int8 scale) while they are unpacked; bias is summed once per edge
// because the bases sum to 1.
// A workgroup is 4 waves: WJ of them side by side along j, 4/WJ interleaved
// along i, whose partial sums meet in LDS.  Workgroups split i into chunks; the
// chunk partial sums are written out and reduced in a fixed order by
// kan_reduce (deterministic: no atomics).

#include "kan_device.hpp"
#include "kan_internal.hpp"

namespace kan {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kSub = 32;   // i-rows whose basis data is staged in LDS at a time

// SL: the input is still in slices, the previous layer's partial sums.
template <typename IdxT, typename GbT, typename CbT, int CODE, int JPL, bool SL = false>
__global__ __launch_bounds__(kThreads) void kan_gather_kernel(const GatherArgs a, const int wj_count) {
  // LDS: basis data for kSub rows; later reused for the cross-wave sum.
  constexpr int kBasisFloats = kSub * 5;
  constexpr int kRedFloats = (kWaves - 1) * kWave * JPL;
  constexpr int kLdsFloats = kBasisFloats > kRedFloats ? kBasisFloats : kRedFloats;
  __shared__ __attribute__((aligned(16))) float lds[kLdsFloats];
  float4* const sw = (float4*)lds;                       // [kSub] weights
  int* const ss = (int*)(lds + kSub * 4);                // [kSub] spans

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = tid >> 6;
  const int wi_count = kWaves / wj_count;
  const int wj = wave % wj_count;
  const int wi = wave / wj_count;

  int head = blockIdx.z, chunk = blockIdx.y, tile = blockIdx.x;
  const bool by_head = a.by_head != 0;
  if (SL || by_head) {
    // Workgroups go to the eight XCDs in turn (linear id mod 8), each with an L2 of its own.  The output
    // tiles of a chunk read the same slices, and a chunk of 16 rows is half a 128-byte line per slice,
    // whose other half the next chunk reads: runs of consecutive (chunk, tile) items per XCD fetch every
    // line once.
    // Heads whose codebooks together exceed an L2: an XCD takes its heads one behind the other, a few at a time, and a codebook
    // enters one L2 only (all of them on every XCD: fifty heads of 2048-256-21, Int8, at batch 1 403 us, now 150; twenty of
    // fp32 rows 224, now 77; line fills from L2 to the vector caches bound it, 170 G/s of the 255 that gathers alone reach).
    const unsigned T = gridDim.x, C = gridDim.y, W = T * C * gridDim.z;
    const unsigned L = blockIdx.x + T * (blockIdx.y + C * blockIdx.z);
    const unsigned xcd = L & 7u, m = L >> 3, q = W >> 3, r = W & 7u;
    const unsigned item = xcd * q + min(xcd, r) + m;          // XCD x owns q + (x < r) items
    head = __builtin_amdgcn_readfirstlane((int)(item / (T * C)));
    const unsigned rem = item % (T * C);
    chunk = __builtin_amdgcn_readfirstlane((int)(rem / T));
    tile = __builtin_amdgcn_readfirstlane((int)(rem % T));
  }
  const int jt = tile % a.n_jt;
  const int btile = tile / a.n_jt;

  const LayerPtrs hp = a.h[head];
  const int n_in = a.n_in, n_out = a.n_out;
  const int b0 = btile;
  const int i_begin = chunk * a.rows_per_chunk;
  const int i_end = min(n_in, i_begin + a.rows_per_chunk);
  const int j0 = (jt * wj_count + wj) * (kWave * JPL) + lane * JPL;
  const bool j_ok = j0 < n_out;          // n_out % JPL == 0, so the whole group is in range

  const float* xh = a.x + (long long)head * a.x_head_stride;
  const IdxT* idx = (const IdxT*)hp.idx;
  const GbT* gain = (const GbT*)hp.gain;
  const GbT* bias = (const GbT*)hp.bias;
  const Q8Params qp = {hp.gain_log2_lo, hp.gain_log2_step, hp.bias_scale};
  const CbT* cb = (const CbT*)hp.cb;
  const float scale = (CODE == kCbI8) ? hp.scale : 1.0f;

  {
    // Warm this XCD's L2 with the codebook before the random gathers start: the workgroups that share an XCD (linear
    // id mod 8; by head: those of the head, which sit on one XCD or two) each stream one slice of it, coalesced.
    if (a.warm_slice > 0) {
      const unsigned wg = by_head ? (unsigned)tile + gridDim.x * (unsigned)chunk
                                  : (blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)) >> 3;
      const long long lo = (long long)wg * a.warm_slice, hi = min(lo + a.warm_slice, a.cb_bytes - 16);
      uint32_t v = 0;
      for (long long off = lo + tid * 16; off < hi; off += kThreads * 16) {
        uint4 q;
        __builtin_memcpy(&q, (const uint8_t*)cb + off, 16);
        v ^= q.x ^ q.y ^ q.z ^ q.w;
      }
      asm volatile("" ::"v"(v));      // keep the loads; the value is not used
    }
  }

  float acc[JPL], bsum[JPL];
#pragma unroll
  for (int p = 0; p < JPL; ++p) acc[p] = bsum[p] = 0.f;

  // SL: the kRuns threads that share a row take consecutive runs of slices, up to 16 loads in
  // flight each; their sums are added in run order when the row's basis data is built.
  constexpr int kRuns = kThreads / kSub;
  __shared__ float sxr[SL ? kRuns : 1][SL ? kSub : 1];

  for (int s0 = i_begin; s0 < i_end; s0 += kSub) {
    const int rows = min(kSub, i_end - s0);
    __syncthreads();
    if constexpr (SL) {
      const int r = tid % kSub, g = tid / kSub;
      const int per_run = (a.x_parts + kRuns - 1) / kRuns;
      const int p_begin = min(g * per_run, a.x_parts), p_end = min(a.x_parts, p_begin + per_run);
      const float* src = xh + (long long)b0 * n_in + s0 + min(r, rows - 1);
      float sum = 0.f;
      for (int p0 = p_begin; p0 < p_end; p0 += 16) {
        float t[16];
#pragma unroll
        for (int pp = 0; pp < 16; ++pp)               // (slices past the last one are re-reads of it, added as zero)
          t[pp] = src[(long long)min(p0 + pp, a.x_parts - 1) * a.x_part_stride];
#pragma unroll
        for (int pp = 0; pp < 16; ++pp) sum += (p0 + pp < p_end) ? t[pp] : 0.f;
      }
      sxr[g][r] = sum;
      __syncthreads();
    }
    // ---- span + weights of this sub-chunk's rows ----------------------------------
    if (tid < kSub) {
      const int r = tid;
      BasisW bw = {0.f, 0.f, 0.f, 0.f, 0};
      if constexpr (SL) {
        float xv = sxr[0][r];
#pragma unroll
        for (int g = 1; g < kRuns; ++g) xv += sxr[g][r];
        if (r < rows) bw = basis_eval_rule(a.x_tanh ? tanhf(xv) : xv, a.rule);
      } else {
        if (r < rows && b0 < a.B) bw = basis_eval_rule(xh[(long long)b0 * n_in + s0 + r], a.rule);
      }
      sw[r] = make_float4(bw.w0, bw.w1, bw.w2, bw.w3);
      ss[r] = bw.span;
    }
    __syncthreads();

    // Only the 4 coefficients under the nonzero bases are fetched.  Rows are taken four at a time
    // so that all metadata loads, then all gathers, are in flight together (rows past the end are
    // clamped and contribute nothing).
    constexpr int R = 4;
    if (j_ok) {
      for (int r0 = wi; r0 < rows; r0 += wi_count * R) {
        uint32_t id[R][JPL];
        float g[R][JPL], bv[R][JPL];
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const int r = min(r0 + q * wi_count, rows - 1);
          const long long e = (long long)(s0 + r) * n_out + j0;
          load_idx<IdxT, JPL>(idx + e, id[q]);
          load_gain<GbT, JPL>(gain + e, qp, g[q]);
          load_bias<GbT, JPL>(bias + e, qp, bv[q]);
        }
        typename WindowRaw<CbT>::type raw[R][JPL];
        int sp[R];
        float4 w[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const int r = min(r0 + q * wi_count, rows - 1);
          sp[q] = ss[r];
          w[q] = sw[r];
#pragma unroll
          for (int p = 0; p < JPL; ++p) raw[q][p] = load_window<CbT>(cb, id[q][p], sp[q]);
        }
        // (left to itself the compiler uses the first windows before it has asked for the last: 4096 x 4096, fp16 rows, 160 us, now
        // 144; 1024 x 512 11.0, now 9.8)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const float live = (r0 + q * wi_count < rows) ? 1.0f : 0.0f;
#pragma unroll
          for (int p = 0; p < JPL; ++p) {
            float c[4];
            dequant_window<CbT>(raw[q][p], live * g[q][p] * scale, c);
            float v = acc[p];
            v = fmaf(w[q].x, c[0], v);
            v = fmaf(w[q].y, c[1], v);
            v = fmaf(w[q].z, c[2], v);
            v = fmaf(w[q].w, c[3], v);
            acc[p] = v;
            bsum[p] = fmaf(live, bv[q][p], bsum[p]);
          }
        }
      }
    }
  }

  // ---- sum over the waves interleaved along i ------------------------------------
  if (wi_count > 1) {
    __syncthreads();
    float* red = lds;    // [(wi-1)][wj][JPL][lane]
    if (wi > 0) {
      float* dstp = red + (((wi - 1) * wj_count + wj) * JPL) * kWave + lane;
#pragma unroll
      for (int p = 0; p < JPL; ++p) dstp[p * kWave] = acc[p];
    }
    __syncthreads();
    if (wi == 0) {
      for (int o = 1; o < wi_count; ++o) {
        const float* srcp = red + (((o - 1) * wj_count + wj) * JPL) * kWave + lane;
#pragma unroll
        for (int p = 0; p < JPL; ++p) acc[p] += srcp[p * kWave];
      }
    }
    __syncthreads();   // bias sums travel in a second pass through the same buffer
    if (wi > 0) {
      float* dstp = red + (((wi - 1) * wj_count + wj) * JPL) * kWave + lane;
#pragma unroll
      for (int p = 0; p < JPL; ++p) dstp[p * kWave] = bsum[p];
    }
    __syncthreads();
    if (wi == 0) {
      for (int o = 1; o < wi_count; ++o) {
        const float* srcp = red + (((o - 1) * wj_count + wj) * JPL) * kWave + lane;
#pragma unroll
        for (int p = 0; p < JPL; ++p) bsum[p] += srcp[p * kWave];
      }
    }
  }

  // ---- write y, the hidden activation, or this chunk's partial sums -------------
  if (wi == 0 && j_ok) {
    float* dst = a.dst + (long long)head * a.dst_head_stride + (long long)chunk * a.dst_chunk_stride;
    if (b0 < a.B) {
      float* o = dst + (long long)b0 * n_out + j0;
#pragma unroll
      for (int p = 0; p < JPL; ++p) {
        float v = acc[p] + bsum[p];
        if (a.apply_tanh) v = tanhf(v);
        o[p] = v;
      }
    }
  }
}

template <typename IdxT, typename GbT, typename CbT, int CODE, int JPL>
hipError_t launch_one(const GatherCfg& c, const GatherArgs& a, dim3 grid, hipStream_t s) {
  if (a.x_parts > 1)
    hipLaunchKernelGGL((kan_gather_kernel<IdxT, GbT, CbT, CODE, JPL, true>), grid, dim3(kThreads), 0, s, a, c.wj);
  else
    hipLaunchKernelGGL((kan_gather_kernel<IdxT, GbT, CbT, CODE, JPL>), grid, dim3(kThreads), 0, s, a, c.wj);
  return hipGetLastError();
}

template <typename IdxT, typename GbT, typename CbT, int CODE>
hipError_t launch_jpl(const GatherCfg& c, const GatherArgs& a, dim3 grid, hipStream_t s) {
  switch (c.jpl) {
    case 1: return launch_one<IdxT, GbT, CbT, CODE, 1>(c, a, grid, s);
    case 2: return launch_one<IdxT, GbT, CbT, CODE, 2>(c, a, grid, s);
    case 4: return launch_one<IdxT, GbT, CbT, CODE, 4>(c, a, grid, s);
    case 8: return launch_one<IdxT, GbT, CbT, CODE, 8>(c, a, grid, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename IdxT>
hipError_t launch_types(const GatherCfg& c, const GatherArgs& a, dim3 grid, hipStream_t s) {
  if (c.code == kCbI8) {
    if (c.gb_kind == kGbQ8) return launch_jpl<IdxT, q8_t, int8_t, kCbI8>(c, a, grid, s);
    return c.gb_kind == kGbF16 ? launch_jpl<IdxT, __half, int8_t, kCbI8>(c, a, grid, s)
                               : launch_jpl<IdxT, float, int8_t, kCbI8>(c, a, grid, s);
  }
  if (c.gb_kind == kGbQ8) return hipErrorInvalidValue;      // byte-coded gain/bias go with Int8 codebooks
  if (c.code == kCbBfp8)
    return c.gb_kind == kGbF16 ? launch_jpl<IdxT, __half, bfp8_t, kCbBfp8>(c, a, grid, s)
                               : launch_jpl<IdxT, float, bfp8_t, kCbBfp8>(c, a, grid, s);
  if (c.code == kCbF16)
    return c.gb_kind == kGbF16 ? launch_jpl<IdxT, __half, __half, kCbF16>(c, a, grid, s)
                               : launch_jpl<IdxT, float, __half, kCbF16>(c, a, grid, s);
  return c.gb_kind == kGbF16 ? launch_jpl<IdxT, __half, float, kCbF32>(c, a, grid, s)
                             : launch_jpl<IdxT, float, float, kCbF32>(c, a, grid, s);
}

}  // namespace

hipError_t launch_gather(const GatherCfg& c, const GatherArgs& a, dim3 grid, hipStream_t s) {
  if (c.bt != 1 || a.x_parts > kGatherChainMaxParts) return hipErrorInvalidValue;
  GatherArgs g = a;
  g.by_head = gather_by_head((int)grid.z, a.cb_bytes);
  // The codebook is brought into L2 ahead where several heads gather 64 times and more from each of its lines (fifty heads of
  // 2048-256 150 against 155 us, five 35.0 / 36.8).  With fewer edges the gathers themselves are the faster way: twenty heads
  // of 1024-128, 25 to a line, 27.1 / 26.1, and second layers of 256 x 21 took 13 to 35 us for their share, now 6 to 10.
  // One head, whose codebook all eight XCDs read, is the better without at any size: 2048-1024-256 23.7 / 22.7, 1024 x 512
  // 9.8 / 9.0, 4096 x 4096 144.8 / 139.4.
  if (grid.z > 1 && (long long)a.n_in * a.n_out * 2 >= a.cb_bytes) {
    const long long wgs = (long long)grid.x * grid.y;
    const long long sharers = g.by_head ? wgs : (wgs * grid.z + 7) / 8;
    g.warm_slice = ((a.cb_bytes + sharers - 1) / sharers + 4095) / 4096 * 4096;
  } else {
    g.warm_slice = 0;
  }
  return c.idx_u32 ? launch_types<uint32_t>(c, g, grid, s) : launch_types<uint16_t>(c, g, grid, s);
}

}  // namespace kan
