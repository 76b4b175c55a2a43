// Pieces shared by the matrix-core kernels: fp16 packing, the raw codeword of an edge and
// its dequantisation into fp16 pairs (Int8: packed-half arithmetic; fp32: multiply, round).
#pragma once

#include "kan_device.hpp"
#include "kan_internal.hpp"

namespace kan {

typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 h16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 h16x16 __attribute__((ext_vector_type(16)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint32_t pack_h2(float a, float b) {
  h16x2 v = {(_Float16)a, (_Float16)b};
  return __builtin_bit_cast(uint32_t, v);
}

// fp16 pair (g*q[p], g*q[p+1]) from bytes p, p+1 of w, where w holds q + 128 as
// unsigned bytes: 0x6400 | byte is the half 1024 + byte, so subtracting 1152 is
// exact and leaves q.
template <int P>
__device__ __forceinline__ uint32_t dq_pair(uint32_t w, h16x2 g2) {
  const uint32_t sel = 0x04000400u | ((uint32_t)(P + 1) << 16) | (uint32_t)P;
  const uint32_t m = __builtin_amdgcn_perm(0x64646464u, w, sel);
  const h16x2 off = {(_Float16)-1152.0f, (_Float16)-1152.0f};
  const h16x2 v = (__builtin_bit_cast(h16x2, m) + off) * g2;
  return __builtin_bit_cast(uint32_t, v);
}

// Both halves of a packed fp16 pair with subnormals set to zero.  The split form does this to
// its high parts itself, before it forms the low parts from what is left, so that the sum of
// the parts does not depend on how conversions and matrix instructions treat subnormals.
__device__ __forceinline__ uint32_t flush_h2(uint32_t v) {
  if ((v & 0x7c00u) == 0u) v &= 0xffff8000u;
  if ((v & 0x7c000000u) == 0u) v &= 0x8000ffffu;
  return v;
}

// Split form of the precise path: a number v travels as two fp16 parts, v = hi + lo / 2048 with
// hi = fp16(v) and lo = fp16((v - hi) * 2048): 22 significant bits; the factor keeps the low
// parts out of the fp16 subnormals.  Ten coefficients in consecutive pairs (2m, 2m + 1).
__device__ __forceinline__ void split_consecutive(const float (&c)[kG], uint32_t (&hi)[5], uint32_t (&lo)[5]) {
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    hi[m] = flush_h2(pack_h2(c[2 * m], c[2 * m + 1]));
    lo[m] = flush_h2(pack_h2((c[2 * m] - half_bits_to_float(hi[m] & 0xffffu)) * 2048.0f,
                             (c[2 * m + 1] - half_bits_to_float(hi[m] >> 16)) * 2048.0f));
  }
}

// Ten fp32 coefficients as high and low fp16 parts, in pairs (m, m + 5): c = hi + lo / 2048.
__device__ __forceinline__ void split_pairs(const float (&c)[kG], uint32_t (&hi)[5], uint32_t (&lo)[5]) {
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    hi[m] = flush_h2(pack_h2(c[m], c[m + 5]));
    lo[m] = flush_h2(pack_h2((c[m] - half_bits_to_float(hi[m] & 0xffffu)) * 2048.0f,
                             (c[m + 5] - half_bits_to_float(hi[m] >> 16)) * 2048.0f));
  }
}

// A pair of basis weights (never negative) in split form: the high parts cut to fp16 towards zero
// (so that the low parts are never negative either), no subnormal high parts.
__device__ __forceinline__ void split_weights(float wa, float wb, uint32_t& hi, uint32_t& lo) {
  const uint32_t h = pack_h2(wa, wb);
  uint32_t ha = h & 0xffffu, hb = h >> 16;
  if (half_bits_to_float(ha) > wa) ha -= 1u;                   // one fp16 step down (w > 0 there)
  if (half_bits_to_float(hb) > wb) hb -= 1u;
  if ((ha & 0x7c00u) == 0u) ha = 0u;
  if ((hb & 0x7c00u) == 0u) hb = 0u;
  hi = ha | (hb << 16);
  lo = flush_h2(pack_h2((wa - half_bits_to_float(ha)) * 2048.0f, (wb - half_bits_to_float(hb)) * 2048.0f)) & 0x7fff7fffu;
}

// Raw codeword of one edge as loaded from the codebook.
template <typename CbT> struct RawRow;
template <> struct RawRow<int8_t> { uint32_t a, b, d; };
template <> struct RawRow<__half> { uint32_t w[kG / 2]; };
template <> struct RawRow<float> { float c[kG]; };
template <> struct RawRow<bfp8_t> { uint32_t a, b, d; };           // d: mantissas 8, 9, exponent byte, zero

// One row = one to three load instructions per lane, as wide as they come: every vector-memory
// instruction of a divergent gather costs the CU's address and tag pipeline a slot per lane,
// whether it brings 2 bytes or 16.  The loads are raw buffer loads (exact widths whatever the
// alignment of the row; the resource spans the address space from the codebook's base, so no
// range check cuts a row short):
//   Int8 (10 bytes, 2-byte aligned): the three aligned dwords that hold the row, shifted into
//     place (0 or 2 bytes).  Every dword touched holds at least one byte of the row, so the load
//     never leaves the pages of the codebook, whatever its size.
//   fp16 (20 bytes, 4-byte aligned): 16 + 4.   fp32 (40 bytes, 8-byte aligned): 16 + 16 + 8.
constexpr int kRowBufferFlags = 0x00020000;       // buffer resource word 3: raw 32-bit data, no swizzle

// For Int8 rows the shift is applied when the row is used (align_row), so that a row in flight
// costs three registers and one bit: row_odd() is that bit, and callers keep the bits of the
// rows of a step in one word.
template <typename CbT>
__device__ __forceinline__ uint32_t row_odd(const CbT* cb, uint32_t id) {
  if constexpr (sizeof(CbT) == 1) return ((uint32_t)((uintptr_t)cb >> 1) + id) & 1u;    // (base + 10 id) / 2 mod 2
  else return 0u;
}

template <typename CbT>
__device__ __forceinline__ void load_row(const CbT* cb, uint32_t id, RawRow<CbT>& r) {
  typedef unsigned int bu32x2 __attribute__((ext_vector_type(2)));
  typedef unsigned int bu32x3 __attribute__((ext_vector_type(3)));
  typedef unsigned int bu32x4 __attribute__((ext_vector_type(4)));
  if constexpr (kIsBfp8<CbT>) {                                   // twelve bytes, 4-byte aligned: one load
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)cb, 0, 0x7fffffff, kRowBufferFlags);
    const bu32x3 v = __builtin_amdgcn_raw_buffer_load_b96(rs, (int)(id * 12u), 0, 0);
    r.a = v.x;
    r.b = v.y;
    r.d = v.z;
  } else if constexpr (sizeof(CbT) == 1) {
    const uint32_t mis = (uint32_t)(uintptr_t)cb & 3u;           // 0 or 2: the base within its dword
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)((uintptr_t)cb - mis), 0, 0x7fffffff, kRowBufferFlags);
    const uint32_t at = id * (uint32_t)kG + mis;                 // byte offset of the row from the aligned base
    const bu32x3 v = __builtin_amdgcn_raw_buffer_load_b96(rs, (int)(at & ~3u), 0, 0);
    r.a = v.x;                                                   // still to be shifted: align_row
    r.b = v.y;
    r.d = v.z;
  } else if constexpr (sizeof(CbT) == 2) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)cb, 0, 0x7fffffff, kRowBufferFlags);
    const int at = (int)(id * (uint32_t)(kG * 2));
    const bu32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, at, 0, 0);
    r.w[0] = v.x;
    r.w[1] = v.y;
    r.w[2] = v.z;
    r.w[3] = v.w;
    r.w[4] = __builtin_amdgcn_raw_buffer_load_b32(rs, at, 16, 0);
  } else {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)cb, 0, 0x7fffffff, kRowBufferFlags);
    const int at = (int)(id * (uint32_t)(kG * 4));
    const bu32x4 v0 = __builtin_amdgcn_raw_buffer_load_b128(rs, at, 0, 0);
    const bu32x4 v1 = __builtin_amdgcn_raw_buffer_load_b128(rs, at, 16, 0);
    const bu32x2 v2 = __builtin_amdgcn_raw_buffer_load_b64(rs, at, 32, 0);
    r.c[0] = __uint_as_float(v0.x); r.c[1] = __uint_as_float(v0.y); r.c[2] = __uint_as_float(v0.z); r.c[3] = __uint_as_float(v0.w);
    r.c[4] = __uint_as_float(v1.x); r.c[5] = __uint_as_float(v1.y); r.c[6] = __uint_as_float(v1.z); r.c[7] = __uint_as_float(v1.w);
    r.c[8] = __uint_as_float(v2.x); r.c[9] = __uint_as_float(v2.y);
  }
}

// The row as it lies in memory: bytes 0..3 in a, 4..7 in b, 8..9 in the low half of d (odd: the
// row starts in the upper half of its first dword).  No-op for the other row types.
template <typename CbT>
__device__ __forceinline__ void align_row(RawRow<CbT>& r, uint32_t odd) {
  if constexpr (sizeof(CbT) == 1) {
    const uint32_t sh = odd * 2u;
    const uint32_t a = __builtin_amdgcn_alignbyte(r.b, r.a, sh);
    const uint32_t b = __builtin_amdgcn_alignbyte(r.d, r.b, sh);
    const uint32_t d = __builtin_amdgcn_alignbyte(0u, r.d, sh) & 0xffffu;
    r.a = a;
    r.b = b;
    r.d = d;
  }
}

// w[0..3] = fp16 pairs of g*coef 0..7, w[4] = g*coef 8, 9.
template <typename CbT>
__device__ __forceinline__ void dequant_row(const RawRow<CbT>& r, float g, uint32_t (&w)[5]) {
  if constexpr (sizeof(CbT) == 1 || kIsBfp8<CbT>) {
    float gs = g;
    if constexpr (kIsBfp8<CbT>) gs = g * bfp8_row_scale(r.d);      // the row's own power of two goes with the gain
    const _Float16 gh = (_Float16)gs;
    const h16x2 g2 = {gh, gh};
    const uint32_t a = r.a ^ 0x80808080u, b = r.b ^ 0x80808080u, d = r.d ^ 0x00008080u;
    w[0] = dq_pair<0>(a, g2);
    w[1] = dq_pair<2>(a, g2);
    w[2] = dq_pair<0>(b, g2);
    w[3] = dq_pair<2>(b, g2);
    w[4] = dq_pair<0>(d, g2);
  } else if constexpr (sizeof(CbT) == 2) {
#pragma unroll
    for (int m = 0; m < 5; ++m)
      w[m] = pack_h2(g * half_bits_to_float(r.w[m] & 0xffffu), g * half_bits_to_float(r.w[m] >> 16));
  } else {
#pragma unroll
    for (int m = 0; m < 5; ++m) w[m] = pack_h2(g * r.c[2 * m], g * r.c[2 * m + 1]);
  }
}

// Position bits of the four value pairs of an A fragment of rotated words: pair t holds its values' bits in bits 15 and 31
// of word t, the sparse instruction takes them from bits 4 t and 4 t + 2 (bit 4 t + 3 set: the second value is one of
// elements 2, 3 of its group).
__device__ __forceinline__ int rot_positions(const u32x4 v) {
  uint32_t u = v.w & 0x80008000u;
  u |= (v.z >> 4) & 0x08000800u;
  u |= (v.y >> 8) & 0x00800080u;
  u |= (v.x >> 12) & 0x00080008u;
  return (int)((u >> 3) | (u >> 17) | 0x8888u);
}

// w[m] = fp16 pair (g*coef m, -g*coef m + 5), m = 0..4: the pairs of the sparse operand whose stored values carry
// "takes the second of the pair" in their sign (kan_wide.hip).
template <typename CbT>
__device__ __forceinline__ void dequant_row_pairs(const RawRow<CbT>& r, float g, uint32_t (&w)[5]) {
  if constexpr (sizeof(CbT) == 1 || kIsBfp8<CbT>) {
    float gs = g;
    if constexpr (kIsBfp8<CbT>) gs = g * bfp8_row_scale(r.d);
    const _Float16 gh = (_Float16)gs;
    const h16x2 g2 = {gh, -gh}, off = {(_Float16)-1152.0f, (_Float16)-1152.0f};
    const uint32_t q[5] = {__builtin_amdgcn_perm(r.b, r.a, 0x0c050c00u), __builtin_amdgcn_perm(r.b, r.a, 0x0c060c01u),
                           __builtin_amdgcn_perm(r.b, r.a, 0x0c070c02u), __builtin_amdgcn_perm(r.d, r.a, 0x0c040c03u),
                           __builtin_amdgcn_perm(r.d, r.b, 0x0c050c00u)};
#pragma unroll
    for (int m = 0; m < 5; ++m)        // 0x6480 ^ byte: the half 1152 + q
      w[m] = __builtin_bit_cast(uint32_t, (__builtin_bit_cast(h16x2, q[m] ^ 0x64806480u) + off) * g2);
  } else if constexpr (sizeof(CbT) == 2) {
    auto coef = [&](int m) { return g * half_bits_to_float((r.w[m >> 1] >> (16 * (m & 1))) & 0xffffu); };
#pragma unroll
    for (int m = 0; m < 5; ++m) w[m] = pack_h2(coef(m), -coef(m + 5));
  } else {
#pragma unroll
    for (int m = 0; m < 5; ++m) w[m] = pack_h2(g * r.c[m], -(g * r.c[m + 5]));
  }
}

// c[m] = g * coef m as fp32 (matrix-core path with fp32 operands).
template <typename CbT>
__device__ __forceinline__ void dequant_row_f32(const RawRow<CbT>& r, float g, float (&c)[kG]) {
  if constexpr (sizeof(CbT) == 1 || kIsBfp8<CbT>) {
    if constexpr (kIsBfp8<CbT>) g *= bfp8_row_scale(r.d);          // the row's own power of two goes with the gain
    const float off = -128.0f * g;
    float t[4];
    dequant4(r.a, g, off, &c[0]);
    dequant4(r.b, g, off, &c[4]);
    dequant4(r.d, g, off, t);
    c[8] = t[0];
    c[9] = t[1];
  } else if constexpr (sizeof(CbT) == 2) {
#pragma unroll
    for (int m = 0; m < kG / 2; ++m) {
      c[2 * m] = g * half_bits_to_float(r.w[m] & 0xffffu);
      c[2 * m + 1] = g * half_bits_to_float(r.w[m] >> 16);
    }
  } else {
#pragma unroll
    for (int m = 0; m < kG; ++m) c[m] = g * r.c[m];
  }
}

// Byte-permute selectors that place the four fp16 weights {w23:w01} of one input at
// half-word slots l..l+3 of its ten: entry [l][k], k = 0..4, builds slots 2k, 2k+1;
// selector byte 0x0c yields 0.  56 threads fill the 7 x 8 table.
__device__ __forceinline__ void fill_weight_selectors(uint32_t (*sel)[8], int tid) {
  if (tid < kSpans * 8) {
    const int l = tid >> 3, k = tid & 7;
    uint32_t v = 0x0c0c0c0cu;
    if (k < 5) {
      const int r0 = 2 * k - l, r1 = 2 * k + 1 - l;
      const uint32_t lo = (r0 >= 0 && r0 <= 3) ? (uint32_t)((2 * r0) | ((2 * r0 + 1) << 8)) : 0x0c0cu;
      const uint32_t hi = (r1 >= 0 && r1 <= 3) ? (uint32_t)((2 * r1) | ((2 * r1 + 1) << 8)) : 0x0c0cu;
      v = lo | (hi << 16);
    }
    sel[l][k] = v;
  }
}

// Span (0..6) and the two weight words from a packed basis word (kan_prep_basis, fp16 form).
__device__ __forceinline__ void unpack_basis(uint2 u, uint32_t& l, uint32_t& w01, uint32_t& w23) {
  l = ((u.x >> 15) & 1u) | ((u.x >> 30) & 2u) | ((u.y >> 13) & 4u);
  w01 = u.x & 0x7fff7fffu;
  w23 = u.y & 0x7fff7fffu;
}

// An input's basis word for a sample = { half2(w0, w1), half2(w2, w3) } with span bit 0, 1, 2 in the
// sign bits of w0, w1, w2 (the weights are never negative).
__device__ __forceinline__ uint2 basis_words(const BasisW& bw) {
  const uint32_t l = (uint32_t)bw.span;
  return make_uint2(pack_h2(bw.w0, bw.w1) | ((l & 1u) << 15) | ((l & 2u) << 30), pack_h2(bw.w2, bw.w3) | ((l & 4u) << 13));
}
// Split form: the high parts are the weights cut to fp16 towards zero, so that the low parts (w - hi) * 2048
// are never negative and their sign bits are free for the span too.
__device__ __forceinline__ void basis_words_split(const BasisW& bw, uint2& v, uint2& lo) {
  const uint32_t l = (uint32_t)bw.span;
  const uint32_t sx = ((l & 1u) << 15) | ((l & 2u) << 30), sy = (l & 4u) << 13;
  split_weights(bw.w0, bw.w1, v.x, lo.x);
  split_weights(bw.w2, bw.w3, v.y, lo.y);
  v.x |= sx;
  v.y |= sy;
  lo.x |= sx;
  lo.y |= sy;
}

// Per span l: byte-permute selectors that pick, from the four fp16 weights {w23:w01} of an
// input, the stored values of its pairs (m, m+5): word 0 pairs 0 and 1, word 1 pairs 2 and 3,
// word 2 pair 4 (high half zero); word 3 the index byte of the input's two full groups
// (nibble = position of the first value | position of the second << 2) and, in bit 8, whether
// pair 4 takes coefficient 9: one 16-byte table read per input.  Selector byte 0x0c yields 0.
__device__ __forceinline__ void fill_sparse_selectors(uint32_t (*sel)[8], int tid) {
  if (tid < kSpans) {
    const int l = tid;
    uint32_t half_sel[5], hi[5];
#pragma unroll
    for (int p = 0; p < 5; ++p) {
      int k = -1;
      hi[p] = 0;
      if (p >= l && p <= l + 3) k = p - l;
      else if (p + 5 >= l && p + 5 <= l + 3) { k = p + 5 - l; hi[p] = 1; }
      half_sel[p] = k >= 0 ? (uint32_t)((2 * k) | ((2 * k + 1) << 8)) : 0x0c0cu;
    }
    sel[l][0] = half_sel[0] | (half_sel[1] << 16);
    sel[l][1] = half_sel[2] | (half_sel[3] << 16);
    sel[l][2] = half_sel[4] | 0x0c0c0000u;
    sel[l][3] = (hi[0] | ((2u + hi[1]) << 2)) | ((hi[2] | ((2u + hi[3]) << 2)) << 4) | (hi[4] << 8);
    sel[l][4] = sel[l][5] = sel[l][6] = sel[l][7] = 0;
  }
}

// ---- basis operand of a block of 32 samples x 32 inputs (256 threads: 32 x 8) ---------------------------------
// The inputs of the thread's four elements (sample 32 by + ty + 8 r, input 32 bx + tx): x itself, or (x_parts > 1) the
// previous layer's partial sums, added here in the order of the slices.  Every load is unconditional (clamped
// addresses): the slices of all four are in flight together instead of one element's after the other's arithmetic.
__device__ __forceinline__ void load_block_inputs(const float* __restrict__ xh, const int x_parts, const long long x_part_stride,
                                                  const int n_in, const int B, const int bx, const int by, float (&xs)[4]) {
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const float* xp[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    xp[r] = xh + (long long)min(by * 32 + ty + 8 * r, B - 1) * n_in + min(bx * 32 + tx, n_in - 1);
    xs[r] = xp[r][0];
  }
  for (int p0 = 1; p0 < x_parts; p0 += 8) {           // eight slices in flight per element, added in order
    float t[8][4];
#pragma unroll
    for (int pp = 0; pp < 8; ++pp) {
      const long long off = (long long)min(p0 + pp, x_parts - 1) * x_part_stride;
#pragma unroll
      for (int r = 0; r < 4; ++r) t[pp][r] = xp[r][off];
    }
#pragma unroll
    for (int pp = 0; pp < 8; ++pp)
#pragma unroll
      for (int r = 0; r < 4; ++r) xs[r] += p0 + pp < x_parts ? t[pp][r] : 0.f;
  }
}

// Rotated words (what kan_wide.hip and kan_stream.hip multiply): the values of an input's pairs (m, m + 5) in order of m,
// each with the bit "coefficient m + 5" in its sign.  Input 4 S + 2 a + h of a step of 16: pairs 0..3 (8 bytes) in half h
// of the 16-byte item W[step][S][a][sample], pair 4 (2 bytes) in place 2 S + h of the item W[step][4][a][sample].
struct RotTile {
  uint2 w[32][33];
  uint16_t z[32][34];
};
__device__ __forceinline__ void prep_rot_block(const float* __restrict__ xh, const int x_parts, const long long x_part_stride,
                                               const int x_tanh, const RotWords& out, const int n_in, const int B, const int rule,
                                               const int bx, const int by, RotTile& hi, RotTile& lo, uint32_t (*sel)[8]) {
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  float xs[4];
  load_block_inputs(xh, x_parts, x_part_stride, n_in, B, bx, by, xs);
  fill_sparse_selectors(sel, threadIdx.x);
  __syncthreads();
  const bool split = out.W_lo != nullptr;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int s = ty + 8 * r;
    const bool live = by * 32 + s < B && bx * 32 + tx < n_in;      // inputs past the last one: zeros
    float xv = xs[r];
    if (x_tanh) xv = tanhf(xv);
    const BasisW bw = basis_fast(xv, rule);
    const uint4 sl = *(const uint4*)&sel[bw.span][0];
    const uint32_t s0 = ((sl.w & 1u) << 15) | ((sl.w & 4u) << 29), s1 = ((sl.w & 16u) << 11) | ((sl.w & 64u) << 25);
    const uint32_t sz = (sl.w & 256u) << 7;
    auto place = [&](uint32_t w01, uint32_t w23, RotTile& t) {
      t.w[s][tx] = live ? make_uint2(__builtin_amdgcn_perm(w23, w01, sl.x) | s0, __builtin_amdgcn_perm(w23, w01, sl.y) | s1)
                        : make_uint2(0u, 0u);
      t.z[s][tx] = live ? (uint16_t)(__builtin_amdgcn_perm(w23, w01, sl.z) | sz) : (uint16_t)0;
    };
    if (split) {
      uint32_t h01, h23, l01, l23;
      split_weights(bw.w0, bw.w1, h01, l01);
      split_weights(bw.w2, bw.w3, h23, l23);
      place(h01, h23, hi);
      place(l01, l23, lo);
    } else {
      place(pack_h2(bw.w0, bw.w1), pack_h2(bw.w2, bw.w3), hi);
    }
  }
  __syncthreads();
  const int n_steps = (n_in + 15) / 16;
  const long long rows = out.P ? rot_rows(B) : B;
  for (int it = threadIdx.x; it < 32 * 20; it += 256) {            // 16-byte items: 2 steps x 2 halves x 5, 32 samples each
    const int s = it & 31, rest = it >> 5, q = rest % 5, a = (rest / 5) & 1, s2 = rest / 10;
    const int b = by * 32 + s, step = bx * 2 + s2;
    if (b >= B || step >= n_steps) continue;
    const long long row = out.P ? rot_row(b) : b, item = ((long long)step * 5 + q) * 2 + a;
    auto write = [&](const RotTile& t, uint4* W) {
      const int i0 = 16 * s2 + 2 * a;
      u32x4 v;
      if (q < 4) {
        const uint2 e0 = t.w[s][i0 + 4 * q], e1 = t.w[s][i0 + 4 * q + 1];
        v = u32x4{e0.x, e0.y, e1.x, e1.y};
      } else {
#pragma unroll
        for (int S = 0; S < 4; ++S) v[S] = (uint32_t)t.z[s][i0 + 4 * S] | ((uint32_t)t.z[s][i0 + 4 * S + 1] << 16);
      }
      *(u32x4*)(W + item * rows + row) = v;
      return v;
    };
    const u32x4 v = write(hi, out.W);
    if (out.P) out.P[item * rows + b] = (uint16_t)rot_positions(v);
    if (split) write(lo, out.W_lo);
  }
}

}  // namespace kan
