// Small-batch path over a prepared layer: the codebook lives in LDS.
//
// At batch 1 a layer is one pass over its per-edge metadata (paper section 4.2: the
// memory-bound regime) plus one codeword lookup per edge (Eq. (1)).  Lookups that go to L2
// are limited by the rate at which a CU can issue divergent addresses, far below what the
// metadata stream could sustain; lookups in LDS are not.  The 655 KB Int8 codebook does not
// fit the 160 KB LDS of a CU, but an eighth of it does, so the edges are regrouped once
// (kan_vq_prepare) by bucket = idx / 8192 (fp16 and block-floating-point rows: idx / 4096, fp32 rows:
// idx / 2048; half of that for layers
// with more than 2048 inputs) and every workgroup serves one bucket: it copies the bucket's
// codeword rows into LDS, builds the span/basis table of all inputs of its sample there as
// well, and streams its block of the bucket's edges.
//
// Inside a bucket the edges are ordered by output j, then input i (layers of more than 2^20 edges: by LDS bank,
// kan_prepare_order_kernel).  A workgroup owns the
// block of edges of a run of outputs and reads it flat, 512 edges per wave and pass (a lane holds
// 8 consecutive ones: 16-byte loads whose addresses depend on nothing but the block's bounds); a
// wave turns its products of a pass into running sums that start anew with every segment (the edges
// of one output), so what a segment has of the pass stands at its last edge and holds nothing of its
// neighbours: neither their rounding nor their overflow, infinities and NaN.  (As differences of running
// sums over the whole pass, an output next to one of a thousand times its terms was off by 5e-6 to 2e-5
// of its own.)  Two ways: blocks of up to 17 passes
// (batch 1 to 2 on a layer of two million edges) keep the running sums of all of them and add after one barrier;
// in larger blocks each of the 16 waves takes a sixteenth of the passes and adds pass by pass
// without any barrier.  A segment that reaches into several waves' runs is put
// together at the end in the order of the waves, the per-bucket sums are added by the fixed-order
// reduction kernel or by the next bucket layer itself: reproducible bits.
// The bias of an edge needs no lookup at all: the four bases sum to 1 on [-1,1], so
// sum_i bias_ij is a per-output constant computed at preparation time.
//
// This file also holds the column kernel for small prepared layers (one workgroup per output and
// sample, windows gathered from L2, no partial sums) and the preparation kernels (count, scan,
// fill, bias sums, block tables).

#include <type_traits>

#include "kan_device.hpp"
#include "kan_internal.hpp"

namespace kan {
namespace {

constexpr int kWaves = kBucketThreads / kWave;     // 16
constexpr int kEpt = 8;                            // consecutive edges per thread and pass
constexpr int kPass = kWave * kEpt;                // 512 edges per wave and pass

// Raw records of one pass: edges e0 .. e0 + 7 of the thread (16-byte loads; the eight gains
// are 32 bytes as fp32 - two loads -, 16 as fp16, 8 as byte codes).  GK is the GbKind.
template <int GK>
struct PassRegs {
  u32x4 i, q;
  typename std::conditional<GK == kGbQ8, u32x2, u32x4>::type g0;
  typename std::conditional<GK == kGbF32, u32x4, char>::type g1;
};

__device__ __forceinline__ float bias_to_float(float b, const Q8Params&) { return b; }
__device__ __forceinline__ float bias_to_float(__half b, const Q8Params&) { return __half2float(b); }
__device__ __forceinline__ float bias_to_float(q8_t b, const Q8Params& qp) { return q8_bias(b.v, qp); }

__device__ __forceinline__ uint32_t dword_of(const u32x4& v, int n) {
  return n == 0 ? v.x : (n == 1 ? v.y : (n == 2 ? v.z : v.w));
}
__device__ __forceinline__ uint32_t u16_of(const u32x4& v, int u) {   // u = 0..7
  const uint32_t w = dword_of(v, u >> 1);
  return (u & 1) ? (w >> 16) : (w & 0xffffu);
}
template <int GK>
__device__ __forceinline__ float gain_of(const PassRegs<GK>& c, int u, const Q8Params& qp) {
  if constexpr (GK == kGbF16) {
    return __half2float(__ushort_as_half((uint16_t)u16_of(c.g0, u)));
  } else if constexpr (GK == kGbQ8) {
    const uint32_t w = u < 4 ? c.g0.x : c.g0.y;
    return q8_gain((w >> (8 * (u & 3))) & 0xffu, qp);
  } else {
    return __uint_as_float(u < 4 ? dword_of(c.g0, u) : dword_of(c.g1, u - 4));
  }
}

// Sum over the 64 lanes of a wave, delivered in lane 63, with data-parallel-primitive moves
// (register crossbar: a few clocks each) instead of LDS permutes (a dependent chain of six
// LDS round trips per segment).  The order of the additions is fixed.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add(float v) {
  const int moved = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, false);
  return v + __int_as_float(moved);
}

__device__ __forceinline__ float masked(float v, uint32_t m) { return __uint_as_float(__float_as_uint(v) & m); }

// What another lane holds; 0 where there is no such lane.
template <int CTRL>
__device__ __forceinline__ float dpp_moved(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

__device__ __forceinline__ float wave_sum_to_last_lane(float v) {
  v = dpp_add<0xB1, 0xf>(v);       // quad_perm [1,0,3,2]: neighbours
  v = dpp_add<0x4E, 0xf>(v);       // quad_perm [2,3,0,1]: every lane holds its quad's sum
  v = dpp_add<0x141, 0xf>(v);      // row_half_mirror: sums of 8
  v = dpp_add<0x140, 0xf>(v);      // row_mirror: every lane holds its row's sum (16 lanes)
  v = dpp_add<0x142, 0xa>(v);      // row_bcast 15 into rows 1 and 3: sums of 32 in rows 1, 3
  v = dpp_add<0x143, 0xc>(v);      // row_bcast 31 into rows 2 and 3: lane 63 holds the sum of 64
  return v;
}

// Every global load below is unconditional (addresses are clamped into valid memory instead
// of being predicated): with no branch around a load the compiler counts outstanding loads
// exactly, so each wait covers only the loads whose data is needed next, and table
// building, record traffic and arithmetic overlap.
//
// MAXIN: inputs the basis table holds (2048 or 4096); the bucket shrinks to make room.
template <int GK, int CODE, int MAXIN>
__global__ __launch_bounds__(kBucketThreads) void kan_bucket_kernel(const BucketArgs a) {
  constexpr int kCbBytes = bucket_bytes(MAXIN);
  // bytes from one bucket's rows to the next's in the codebook: the whole LDS share, except for the 12-byte
  // block-floating-point rows (a power of two of them per bucket: 4096 or 2048)
  constexpr int kCbStride = CODE == kCbBfp8 ? kCbBytes / 20 * 12 : kCbBytes;
  constexpr int kXPerThread = MAXIN / kBucketThreads;
  constexpr int kEntryBytes = CODE == kCbF32 ? 4 : (CODE == kCbF16 ? 2 : 1);
  constexpr int kRowBytes = CODE == kCbBfp8 ? 12 : 10 * kEntryBytes;
  constexpr int kWindow = CODE == kCbF32 ? 4 : (CODE == kCbF16 ? 3 : 2);      // dwords that hold four entries of a row
  constexpr int kCbPerThread = (kCbBytes / 16 + kBucketThreads - 1) / kBucketThreads;   // 16-byte units per thread
  // The bucket's rows (+ 16 bytes read-ahead, + 16 spare) and the basis table {w0, w1, w2, where in LDS the entry of row 0 lies
  // that the window begins with}; w3 = 1 - w0 - w1 - w2.  The table lies where the offset field of an LDS instruction (16 bits)
  // reaches, the rows' address is part of the table: neither lookup takes an addition.
  constexpr int kCbLds = kCbBytes + 32, kBasLds = MAXIN * 16, kCbAt = kCbLds < kBasLds ? 0 : kBasLds, kBasAt = kCbLds < kBasLds ? kCbLds : 0;
  static_assert(kBasAt < 65536 && kCbLds % 16 == 0 && kBasLds % 16 == 0, "offset of 16 bits");
  __shared__ __attribute__((aligned(16))) char tables[kCbLds + kBasLds];
  char* const cb = tables + kCbAt;
  float4* const bas = (float4*)(tables + kBasAt);
  // running sums of the products of a wave's pass (and of a 17th): of each lane's eight, and at the end of each lane of all before it
  __shared__ __attribute__((aligned(16))) float prod[kWaves + 1][kPass];
  __shared__ float upto[kWaves + 1][kWave];
  __shared__ float res[kBucketMaxJw];           // sums of this workgroup's segments: what the wave in whose run a segment begins has of it ...
  __shared__ uint32_t segl[kBucketMaxJw + 1];   // first edge of every segment of the block (+ end)
  __shared__ __attribute__((aligned(16))) float head_sum[kWaves];            // ... and what each wave has of the segment that began before its run
  __shared__ __attribute__((aligned(16))) int head_seg[kWaves];              // (-1: none did)
  __shared__ uint32_t starts[kWaves + 1][kPass / 32];                        // a bit per edge of prod: the first of its segment

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hd = blockIdx.z, b = blockIdx.y;
  const BucketHead H = a.h[hd];
  const char* prep = (const char*)H.prepared;
  // the block of this workgroup: outputs [j0, j1) of one bucket, edges [blk_lo, blk_hi)
  const uint32_t* __restrict__ ent = (const uint32_t*)(prep + a.off_blk) + (size_t)blockIdx.x * kBucketEntryWords;
  const int bucket = (int)ent[0];
  const int j0 = (int)ent[1], j1 = (int)ent[2];
  const uint32_t blk_lo = ent[3], blk_hi = ent[4];
  const int njw = j1 - j0;
  const uint32_t* __restrict__ seg = (const uint32_t*)(prep + a.off_seg) + (size_t)bucket * a.n_out;
  const uint16_t* __restrict__ pi = (const uint16_t*)(prep + a.off_i);
  const uint16_t* __restrict__ pq = (const uint16_t*)(prep + a.off_q);
  const char* __restrict__ pg = prep + a.off_g;
  constexpr int kGainBytes = gb_bytes(GK);
  const Q8Params qp = {H.gain_log2_lo, H.gain_log2_step, 0.f};

  // No segment starts yet.  The barrier waits beside the scalar loads above, which everything below needs (behind the
  // vector loads the waves would wait until the address units have taken the last wave's, 0.4 us).
  if (tid < (kWaves + 1) * (kPass / 32)) starts[0][tid] = 0u;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();

  // Loads are issued in the order their data is needed (they return in order): the inputs
  // of the sample, the codebook bucket, the segment table; then, after the basis table has
  // been built from the inputs, two passes of records.

  // ---- (1) inputs: x itself, or the previous layer's per-bucket sums still to be added
  //          (fixed order) and squashed ----------------------------------------------------
  float xv[kXPerThread];
  {
    const float* xr = a.x + (long long)hd * a.x_head_stride + (long long)b * a.n_in;
    int xi[kXPerThread];
#pragma unroll
    for (int r = 0; r < kXPerThread; ++r) {
      xi[r] = min(tid + r * kBucketThreads, a.n_in - 1);
      xv[r] = xr[xi[r]];
    }
    // further slices eight at a time, all their loads in flight together; the additions keep
    // the order p = 1, 2, ... (slices past the last one are re-reads of it, added as zero)
    for (int p0 = 1; p0 < a.x_parts; p0 += 8) {
      float t[8][kXPerThread];
#pragma unroll
      for (int pp = 0; pp < 8; ++pp) {
        const float* xp = xr + (long long)min(p0 + pp, a.x_parts - 1) * a.x_part_stride;
#pragma unroll
        for (int r = 0; r < kXPerThread; ++r) t[pp][r] = xp[xi[r]];
      }
#pragma unroll
      for (int pp = 0; pp < 8; ++pp)
#pragma unroll
        for (int r = 0; r < kXPerThread; ++r) xv[r] += (p0 + pp < a.x_parts) ? t[pp][r] : 0.f;
    }
  }

  // ---- (2) codebook bucket, 16 bytes per thread and round.  The workgroups of a bucket
  //          start at different offsets so that they do not all ask the same L2 channel
  //          for the same line at the same moment ------------------------------------------
  const long long cb_start = (long long)bucket * kCbStride;
  const long long cb_rest = a.cb_bytes - cb_start;
  const int cb_nbytes = (int)(cb_rest < kCbStride ? cb_rest : kCbStride);
  const char* cb_src = (const char*)H.cb + cb_start;
  const int n16 = cb_nbytes >> 4;
  const int cb_tail = cb_nbytes & 15;
  const int rot = (int)((long long)blockIdx.x * n16 / gridDim.x);
  // a bucket shorter than 16 bytes, or without tail bytes: the (unused) load goes to the
  // prepared buffer, which always has that many bytes
  const u32x4* cb_src16 = n16 > 0 ? (const u32x4*)cb_src : (const u32x4*)prep;
  const uint8_t* cb_tailp = cb_tail > 0 ? (const uint8_t*)cb_src + n16 * 16 + min(tid, cb_tail - 1)
                                        : (const uint8_t*)prep;
  // (plain arrays with compile-time indices only; every element is assigned unconditionally,
  // so they live in registers)
  int cbu[kCbPerThread];
  u32x4 cbv[kCbPerThread];
#pragma unroll
  for (int r = 0; r < kCbPerThread; ++r) {
    const int t = tid + r * kBucketThreads;
    int u = t + rot;
    if (u >= n16) u -= n16;
    cbu[r] = t < n16 ? u : kCbBytes / 16;          // no unit: the spare slot behind the bucket
    cbv[r] = cb_src16[t < n16 ? u : 0];
  }
  const uint8_t cb_tailv = *cb_tailp;

  // ---- (3) segment table of the block ---------------------------------------------------------
  const uint32_t sv0 = seg[j0 + min(tid, njw)];
  const uint32_t sv1 = seg[j0 + min(tid + kBucketThreads, njw)];

  __builtin_amdgcn_sched_barrier(0);   // keep the loads above in this order, ahead of their uses

  // ---- span + weights of every input -> LDS ---------------------------------------------------
  {
#pragma unroll
    for (int r = 0; r < kXPerThread; ++r) {
      if (r * kBucketThreads < a.n_in) {        // uniform: rounds past the last input are skipped
        const int i = tid + r * kBucketThreads;
        const float xin = a.x_tanh ? tanhf(xv[r]) : xv[r];
        const BasisW w = basis_eval_rule(xin, a.rule);
        // (threads past the last input of the round write entries nobody reads)
        bas[i] = make_float4(w.w0, w.w1, w.w2, __uint_as_float((uint32_t)(kCbAt + w.span * kEntryBytes)));
      }
    }
  }
  // ---- (4) records (their addresses need the block's bounds, two dependent scalar loads that
  //          have had the basis evaluation above to arrive).  A wave's run is a number of whole
  //          passes from blk_lo rounded down to a multiple of 8, so that every lane's group of 8
  //          is 16-byte aligned: dealt out evenly, except that the first wave takes the last of
  //          17 (blocks end where a segment does, so those of a chip filled with blocks of 16
  //          passes are a little more or a little less).  Groups past the block re-read its last
  //          group; the arrays are padded, so a group that straddles the end of the last block
  //          stays inside the buffer. ----------------------------------------------------------------
  const uint32_t base = blk_lo & ~7u;
  const uint32_t last_group = blk_hi > 0u ? (blk_hi - 1u) & ~7u : 0u;
  const uint32_t n_edges = blk_hi > blk_lo ? blk_hi - base : 0u, passes = (n_edges + kPass - 1u) / kPass;
  const bool one_pass = passes <= (uint32_t)kWaves + 1u;
  const uint32_t first = one_pass ? (uint32_t)wave : (uint32_t)wave * passes / kWaves;
  const uint32_t w_lo = base + min(first * (uint32_t)kPass, n_edges);
  const uint32_t w_hi = one_pass ? base + n_edges : base + min((uint32_t)(wave + 1) * passes / kWaves * (uint32_t)kPass, n_edges);
  const int n_pass = (int)((w_hi - w_lo + kPass - 1u) / kPass);
  auto load_pass = [&](PassRegs<GK>& c, int p) {
    const uint32_t e0 = min(w_lo + (uint32_t)p * kPass + (uint32_t)lane * kEpt, last_group);
    c.i = __builtin_nontemporal_load((const u32x4*)(pi + e0));
    c.q = __builtin_nontemporal_load((const u32x4*)(pq + e0));
    if constexpr (GK == kGbQ8) c.g0 = __builtin_nontemporal_load((const u32x2*)(pg + (size_t)e0 * kGainBytes));
    else c.g0 = __builtin_nontemporal_load((const u32x4*)(pg + (size_t)e0 * kGainBytes));
    if constexpr (GK == kGbF32) c.g1 = __builtin_nontemporal_load((const u32x4*)(pg + (size_t)e0 * kGainBytes) + 1);
  };
  PassRegs<GK> A, B;
  load_pass(A, 0);
  load_pass(B, one_pass ? kWaves : 1);

  __builtin_amdgcn_sched_barrier(0);

  // ---- codebook rows, segment table -> LDS (unconditional stores: a store inside a branch
  //      would pull its load into the branch, behind all the others) ------------------------------
  {
#pragma unroll
    for (int r = 0; r < kCbPerThread; ++r) ((u32x4*)cb)[cbu[r]] = cbv[r];
    ((uint8_t*)cb)[tid < cb_tail ? n16 * 16 + tid : kCbBytes + 16 + (tid & 15)] = cb_tailv;
  }
  segl[min(tid, njw)] = sv0;
  segl[min(tid + kBucketThreads, njw)] = sv1;
  static_assert(kBucketMaxJw <= kBucketThreads, "a thread per segment");
  if (one_pass && tid < njw && sv0 < blk_hi) atomicOr(&starts[0][(sv0 - base) >> 5], 1u << ((sv0 - base) & 31u));
  for (int t = tid; t < njw; t += kBucketThreads) res[t] = 0.f;
  if (lane == 0) head_sum[wave] = 0.f;
  __syncthreads();

  // No barrier from here to the end of the passes: the waves drift apart, and one's LDS reads, arithmetic and waits for
  // records run beside another's.  (With passes of 8,192 edges for the whole workgroup and two barriers each, the sums in
  // between cost 0.8 us a pass: 4096 x 4096, K = 262,144, batch 2 61.4 -> 53.6 us.)
  int seg_now = 0, head = -1;      // set by find_segment: the wave's first segment not ended, and if it began before the run
  static_assert(kBucketMaxJw <= kWave * 16, "two rounds find a segment");
  const uint32_t start = max(w_lo, blk_lo);
  const uint32_t sixteenth = segl[min((lane + 1) * 16, njw)];
  auto find_segment = [&] {        // (rounds of 64 and 16 lanes over at most 1024)
    seg_now = 16 * (int)__popcll(__builtin_amdgcn_ballot_w64((lane + 1) * 16 <= njw && sixteenth <= start));
    seg_now += (int)__popcll(__builtin_amdgcn_ballot_w64(lane < 16 && seg_now + lane < njw && segl[min(seg_now + lane + 1, njw)] <= start));
    head = seg_now < njw && segl[min(seg_now, njw)] < start ? seg_now : -1;
  };
  const int lanes_to_row = lane & 16 ? (lane & 15) + 1 : kWave, lanes_to_half = lane & 32 ? lane - 31 : kWave;
  // Running sums of the products of the lane's 8 edges, anew from every segment's first edge (bit u of f: the lane's edge
  // u is one) -> prod[strip], and of all the lanes' up to this one's last edge, anew likewise -> upto[strip].  Edges outside the block (groups that straddle its ends, re-read groups) are looked up like the
  // others: what they give, numbers or not, stands in front of the block's first segment or behind its last.
  auto products = [&](const PassRegs<GK>& c, const uint32_t f, const int strip) {
    const uint32_t go_on = ~f;
    float4 w[kEpt];
    uint32_t at[kEpt], win[kEpt][kWindow];       // a window's first byte, the aligned dwords that hold it
    uint32_t third[kEpt];                        // block floating point: the row's third dword, with its power of two
    auto read_basis = [&](int u0) {
#pragma unroll
      for (int u = u0; u < u0 + kEpt / 2; ++u) w[u] = bas[u16_of(c.i, u)];
    };
    auto read_window = [&](int u0) {
#pragma unroll
      for (int u = u0; u < u0 + kEpt / 2; ++u) {
        at[u] = u16_of(c.q, u) * (uint32_t)kRowBytes + __float_as_uint(w[u].w);
        // (LDS serves unaligned reads as well, at less than half the rate: 2048 x 1024 at batch 1 10.0 against 12.3 us)
        const uint32_t* const d = (const uint32_t*)(tables + (at[u] & ~3u));
#pragma unroll
        for (int n = 0; n < kWindow; ++n) win[u][n] = d[n];
        if constexpr (CODE == kCbBfp8) third[u] = ((const uint32_t*)cb)[u16_of(c.q, u) * 3u + 2u];
      }
    };
    float sums[kEpt];
    auto add_products = [&](int u0) {
#pragma unroll
      for (int u = u0; u < u0 + kEpt / 2; ++u) {
        float c0, c1, c2, c3;
        if constexpr (CODE == kCbI8 || CODE == kCbBfp8) {
          const int v = (int)__builtin_amdgcn_alignbyte(win[u][1], win[u][0], at[u]);      // (shifts by its low two bits)
          c0 = (float)(int8_t)v;
          c1 = (float)(int8_t)(v >> 8);
          c2 = (float)(int8_t)(v >> 16);
          c3 = (float)(int8_t)(v >> 24);
        } else if constexpr (CODE == kCbF16) {
          const uint32_t lo = __builtin_amdgcn_alignbyte(win[u][1], win[u][0], at[u]);
          const uint32_t hi = __builtin_amdgcn_alignbyte(win[u][2], win[u][1], at[u]);
          c0 = half_bits_to_float(lo & 0xffffu);
          c1 = half_bits_to_float(lo >> 16);
          c2 = half_bits_to_float(hi & 0xffffu);
          c3 = half_bits_to_float(hi >> 16);
        } else {
          c0 = __uint_as_float(win[u][0]);
          c1 = __uint_as_float(win[u][1]);
          c2 = __uint_as_float(win[u][2]);
          c3 = __uint_as_float(win[u][3]);
        }
        // sum_k w_k c_k with w3 = 1 - w0 - w1 - w2 (the bases sum to 1)
        float s = c3;
        s = fmaf(w[u].z, c2 - c3, s);
        s = fmaf(w[u].y, c1 - c3, s);
        s = fmaf(w[u].x, c0 - c3, s);
        if constexpr (CODE == kCbBfp8) s *= bfp8_row_scale(third[u]);
        uint32_t go;                             // all ones unless the edge starts a segment (written as C++, the compiler compares and selects)
        asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(go) : "v"(go_on), "n"(u));
        sums[u] = u > 0 ? fmaf(gain_of<GK>(c, u, qp), s, masked(sums[u - 1], go)) : gain_of<GK>(c, u, qp) * s;
      }
    };
    // Four edges' reads are in flight beside four edges' arithmetic.  Left to itself the compiler made it an LDS round trip
    // per edge (2048 x 1024 at batch 1 10.0 against 9.6 us); two trips for all eight, or two or one edge at a time, are
    // slower by 1-4 %.
    read_basis(0);
    __builtin_amdgcn_sched_barrier(0);
    read_window(0);
    read_basis(kEpt / 2);
    __builtin_amdgcn_sched_barrier(0);
    add_products(0);
    read_window(kEpt / 2);
    add_products(kEpt / 2);
    // Inclusive scan of the lanes' last sums over the wave.  A lane in which a segment starts takes nothing from the lanes
    // before it; `open` is how many lanes back the nearest such lane is (this one: 0; none among 32: 32).
    float v = sums[kEpt - 1];
    const uint32_t back = (uint32_t)((__builtin_amdgcn_ballot_w64(f != 0u) << (kWave - 1 - lane)) >> 32);
    const int open = back != 0u ? __builtin_clz(back) : 32;
    auto add = [&](float moved, int lanes) { v += open >= lanes ? moved : 0.f; };
    add(dpp_moved<0x111>(v), 1);         // row_shr 1, 2, 4, 8: within rows of 16 lanes
    add(dpp_moved<0x112>(v), 2);
    add(dpp_moved<0x114>(v), 4);
    add(dpp_moved<0x118>(v), 8);
    add(dpp_moved<0x142>(v), lanes_to_row);      // row_bcast 15: rows 1 and 3 add the sum of the row before
    add(dpp_moved<0x143>(v), lanes_to_half);     // row_bcast 31: rows 2 and 3 add the sum of the first half
    upto[strip][lane] = v;
    ((float4*)prod[strip])[lane * 2] = make_float4(sums[0], sums[1], sums[2], sums[3]);
    ((float4*)prod[strip])[lane * 2 + 1] = make_float4(sums[4], sums[5], sums[6], sums[7]);
  };
  // What the segment of edges [lo, hi) of that strip has.
  auto piece = [&](const int strip, uint32_t lo, uint32_t hi) {
    const uint32_t l = (hi - 1u) / kEpt;
    const float own = prod[strip][hi - 1u], before = upto[strip][l > 0u ? l - 1u : 0u];
    return lo < l * kEpt ? own + before : own;
  };
  auto starts_of_lane = [&](int strip) { return (uint32_t)((const uint8_t*)starts[strip])[lane]; };

  // What the segments have of pass p, a lane per segment; the bounds of the first 64 are read ahead.
  uint32_t s0 = 0u, s1 = 0u;
  auto read_bounds = [&] {
    s0 = segl[min(seg_now + lane, njw)];
    s1 = segl[min(seg_now + lane + 1, njw)];
  };
  auto pass = [&](PassRegs<GK>& c, int p) {
    uint32_t* const st = starts[wave];
    const uint32_t pa = w_lo + (uint32_t)p * kPass, pe = min(pa + (uint32_t)kPass, w_hi);
    if (lane < kPass / 32) st[lane] = 0u;
    __builtin_amdgcn_wave_barrier();
    uint32_t from = s0;
    for (int jj = seg_now + lane;;) {          // (64 segments that start before the pass ends: there may be more)
      const bool before_end = jj < njw && from < pe;
      if (before_end && from > pa) atomicOr(&st[(from - pa) >> 5], 1u << ((from - pa) & 31u));
      if (__popcll(__builtin_amdgcn_ballot_w64(before_end)) < kWave) break;
      jj += kWave;
      from = segl[min(jj, njw)];
    }
    __builtin_amdgcn_wave_barrier();
    products(c, starts_of_lane(wave), wave);
    load_pass(c, p + 2);
    __builtin_amdgcn_wave_barrier();
    for (;;) {
      const int jj = seg_now + lane;
      const uint32_t lo = max(s0, pa), hi = min(s1, pe);
      // (one wave adds to an element, in the order of its passes)
      if (jj < njw && lo < hi) atomicAdd(jj == head ? &head_sum[wave] : &res[jj], piece(wave, lo - pa, hi - pa));
      const int ended = (int)__popcll(__builtin_amdgcn_ballot_w64(jj < njw && s1 <= pe));
      seg_now += ended;
      read_bounds();
      if (ended < kWave) break;
    }
    __builtin_amdgcn_wave_barrier();
  };

  if (one_pass) {
    // The strips lie behind one another, so a thread can take a segment's sum from the strips of all waves, without the
    // search for the segments of a run: 1500 x 1100, K = 20,000, batch 1 (segments of 500 edges, a wave's run) 13.1 -> 11.5 us;
    // 2048 x 1024 x 256 at batch 1, whose first layer's blocks are 16 passes and a little, 13.8 -> 12.0 with the 17th strip.
    if (n_pass > 0) products(A, starts_of_lane(wave), wave);
    if (n_pass > kWaves) products(B, starts_of_lane(kWaves), kWaves);
  } else {
    // two passes are always in flight: a slot is refilled as soon as it has been consumed
    // (after the last pass the refills are harmless re-reads)
    find_segment();
    read_bounds();
    for (int p = 0; p < n_pass; p += 2) {
      pass(A, p);
      if (p + 1 >= n_pass) break;
      pass(B, p + 1);
    }
    if (lane == 0) head_seg[wave] = head;
  }
  __syncthreads();
  // what the waves have of segments that began before their runs, in the order of the waves
  if (!one_pass && wave == 0) {
    const int seg_of = lane < kWaves ? head_seg[lane] : -1;
    float sum = head_sum[lane & (kWaves - 1)];
    const int other = __shfl_up(seg_of, 1, 64);
    const bool first = lane == 0 || seg_of != other;
    if (__builtin_amdgcn_ballot_w64(seg_of >= 0 && !first) != 0) {  // a segment that takes up whole runs
      const int own = __float_as_int(sum);
      sum = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w)
        sum += seg_of == __builtin_amdgcn_readlane(seg_of, w) ? __int_as_float(__builtin_amdgcn_readlane(own, w)) : 0.f;
    }
    if (seg_of >= 0 && first) res[seg_of] += sum;
  }
  if (!one_pass && njw > kWave) __syncthreads();  // (else the same wave reads them)
  // a segment's sum where the passes are at most 17
  auto sum_of_strips = [&](int t) {
    const uint32_t lo = segl[t] - base, hi = segl[t + 1] - base;
    if (lo >= hi) return 0.f;
    const uint32_t last = (hi - 1u) / kPass, at = last * kPass;
    float sum = piece((int)last, max(lo, at) - at, hi - at);
    for (uint32_t w = lo / kPass; w < last; ++w) sum += upto[w][kWave - 1];
    return sum;
  };

  // ---- segment sums -> memory (coalesced): scale, bias sum (first bucket only), activation ----
  float* dst = a.dst + (long long)hd * a.dst_head_stride + (long long)bucket * a.dst_chunk_stride +
               (long long)b * a.n_out;
  const float* bias_sum = (const float*)(prep + a.off_bias);
  const float scale = CODE == kCbI8 ? H.scale : 1.0f;
  for (int t = tid; t < njw; t += kBucketThreads) {
    const float sum = res[t] + (one_pass ? sum_of_strips(t) : 0.f);
    float v = scale * sum + (bucket == 0 ? bias_sum[j0 + t] : 0.0f);
    if (a.apply_tanh && a.n_buckets == 1) v = tanhf(v);
    dst[j0 + t] = v;
  }
}

// ---- column kernel: small prepared layers ------------------------------------------------
// A layer of a few hundred thousand edges gives a bucket workgroup a thousand edges or fewer:
// what it does then is wait - for 80 KB of codeword rows to reach its LDS, for its block
// bounds, for a reduction launch behind it.  Such a layer is served by one workgroup per
// (output j, sample) instead.  The prepared buffer of a small layer also holds ids and gains
// transposed ([output][input]), so thread t owns inputs t, t + 256, ... of the sample: it loads
// x, id and gain of its edges at once (coalesced, nothing depends on anything), evaluates the
// basis of its own inputs, fetches each edge's four-coefficient window straight from the
// codebook in L2 (Eq. (1); a thousand gathers per CU are a microsecond) and adds the products
// in a fixed order: per thread by ascending input, then across the lanes, then the waves.
// It writes the finished output - bias sum, activation - so no reduction pass follows.
// PER: edges per thread and round, 8 (2048 inputs per round) or 4 for layers of at most 1024 inputs, whose
// upper four slots would only re-read the last input (the address units see every load, used or not).

template <int GK, typename CbT, int PER>
__global__ __launch_bounds__(kColumnThreads) void kan_column_kernel(const BucketArgs a) {
  __shared__ float wave_sum[kColumnThreads / kWave];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int j = blockIdx.x, b = blockIdx.y, head = blockIdx.z;
  const BucketHead H = a.h[head];
  const char* prep = (const char*)H.prepared;
  constexpr int kGainBytes = gb_bytes(GK);
  const uint32_t* __restrict__ ti = (const uint32_t*)(prep + a.off_ti) + (size_t)j * a.n_in;
  const char* __restrict__ tg = prep + a.off_tg + (size_t)j * a.n_in * kGainBytes;
  const Q8Params qp = {H.gain_log2_lo, H.gain_log2_step, 0.f};
  const CbT* __restrict__ cbk = (const CbT*)H.cb;
  const float* xr = a.x + (long long)head * a.x_head_stride + (long long)b * a.n_in;
  const float bias_sum = ((const float*)(prep + a.off_bias))[j];

  float acc = 0.f;
  for (int i0 = 0; i0 < a.n_in; i0 += kColumnThreads * PER) {       // one round for up to 256 * PER inputs
    // ---- everything the round needs from memory except the windows: unconditional loads,
    //      clamped addresses (inputs past the end re-read the last one and count as zero) ----
    int xi[PER];
    float xv[PER], gain[PER];
    uint32_t row[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      xi[r] = min(i0 + tid + r * kColumnThreads, a.n_in - 1);
      xv[r] = xr[xi[r]];
      row[r] = ti[xi[r]];
      if constexpr (GK == kGbF16) gain[r] = __half2float(((const __half*)tg)[xi[r]]);
      else if constexpr (GK == kGbQ8) gain[r] = q8_gain(((const uint8_t*)tg)[xi[r]], qp);
      else gain[r] = ((const float*)tg)[xi[r]];
    }
    // the input is x itself, or the previous layer's per-bucket sums still to be added (in order) and squashed
    for (int p0 = 1; p0 < a.x_parts; p0 += 8) {
      float t[8][PER];
#pragma unroll
      for (int pp = 0; pp < 8; ++pp) {
        const float* xp = xr + (long long)min(p0 + pp, a.x_parts - 1) * a.x_part_stride;
#pragma unroll
        for (int r = 0; r < PER; ++r) t[pp][r] = xp[xi[r]];
      }
#pragma unroll
      for (int pp = 0; pp < 8; ++pp)
#pragma unroll
        for (int r = 0; r < PER; ++r) xv[r] += (p0 + pp < a.x_parts) ? t[pp][r] : 0.f;
    }
    // ---- basis of the thread's own inputs, then the windows of its edges ----------------------
    BasisW w[PER];
    typename WindowRaw<CbT>::type raw[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      w[r] = basis_eval_rule(a.x_tanh ? tanhf(xv[r]) : xv[r], a.rule);
      raw[r] = load_window<CbT>(cbk, row[r], w[r].span);
    }
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      float c[4];
      dequant_window<CbT>(raw[r], 1.0f, c);
      // sum_k w_k c_k with w3 = 1 - w0 - w1 - w2 (the bases sum to 1)
      float sv = c[3];
      sv = fmaf(w[r].w2, c[2] - c[3], sv);
      sv = fmaf(w[r].w1, c[1] - c[3], sv);
      sv = fmaf(w[r].w0, c[0] - c[3], sv);
      acc += (i0 + tid + r * kColumnThreads < a.n_in) ? gain[r] * sv : 0.f;
    }
  }
  acc = wave_sum_to_last_lane(acc);
  if (lane == kWave - 1) wave_sum[wave] = acc;
  __syncthreads();
  if (tid == 0) {
    const float scale = sizeof(CbT) == 1 ? H.scale : 1.0f;
    float v = scale * ((wave_sum[0] + wave_sum[1]) + (wave_sum[2] + wave_sum[3])) + bias_sum;
    if (a.apply_tanh) v = tanhf(v);
    a.dst[(long long)head * a.dst_head_stride + (long long)b * a.n_out + j] = v;
  }
}

// ---- preparation ------------------------------------------------------------------------
// The regrouping is a counting sort of the edges by (bucket, output j), input i ascending
// inside a run, and at the same time a transposition: the layer stores consecutive outputs side
// by side, the prepared layout consecutive inputs.  It is done tile by tile (kPrepareRows inputs x
// kPrepareCols outputs per workgroup), so that both the reads (rows of the tile) and the writes
// (runs of one (bucket, output) within the tile's row block) move whole runs of bytes:
//   count   per tile: edges per (bucket, output) -> tcnt[row block][bucket][output] and, added
//           up over the row blocks with integer atomics, the segment lengths; bias sums per
//           (row block, output) in fp64
//   scan    exclusive prefix over the segment lengths (bucket-major) -> segment table
//   fill    per tile: the tile's idx and gain staged in LDS; a wave takes a column, and for
//           every 64 rows ranks its lanes within their bucket (ballots) behind the edges of the
//           earlier row blocks and rows
//   order   layers of more than 2^20 edges: the records of a segment by the LDS banks of their inputs
//   bias    per output: the row blocks' sums added in order, rounded once to fp32

template <typename IdxT, typename GbT>
__global__ __launch_bounds__(256) void kan_prepare_count_kernel(const IdxT* __restrict__ idx,
                                                                const GbT* __restrict__ bias, int n_in, int n_out,
                                                                int rows_shift, int n_buckets,
                                                                uint32_t* __restrict__ seg, uint16_t* __restrict__ tcnt,
                                                                double* __restrict__ tbias, Q8Params qp) {
  extern __shared__ uint32_t cnt[];                 // [n_buckets][kPrepareCols]
  __shared__ double bsum[4][kPrepareCols];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = blockIdx.x * kPrepareCols + lane;
  const int i0 = blockIdx.y * kPrepareRows + wave * (kPrepareRows / 4);
  for (int t = threadIdx.x; t < n_buckets * kPrepareCols; t += 256) cnt[t] = 0u;
  __syncthreads();
  double bs = 0.0;
  if (j < n_out) {
    const int i1 = min(i0 + kPrepareRows / 4, n_in);
    for (int i = i0; i < i1; ++i) {
      const size_t e = (size_t)i * n_out + j;
      const uint32_t b = min((uint32_t)idx[e] >> rows_shift, (uint32_t)(n_buckets - 1));
      atomicAdd(&cnt[b * kPrepareCols + lane], 1u);            // (waves share a column: integer, order-free)
      bs += (double)bias_to_float(bias[e], qp);
    }
  }
  bsum[wave][lane] = bs;
  __syncthreads();
  for (int t = threadIdx.x; t < n_buckets * kPrepareCols; t += 256) {
    const int b = t / kPrepareCols, jj = blockIdx.x * kPrepareCols + (t % kPrepareCols);
    if (jj < n_out) {
      const uint32_t c = cnt[t];
      tcnt[((size_t)blockIdx.y * n_buckets + b) * n_out + jj] = (uint16_t)c;
      if (c) atomicAdd(&seg[(size_t)b * n_out + jj], c);
    }
  }
  if (wave == 0 && j < n_out)
    tbias[(size_t)blockIdx.y * n_out + j] = ((bsum[0][lane] + bsum[1][lane]) + bsum[2][lane]) + bsum[3][lane];
}

__global__ __launch_bounds__(256) void kan_prepare_zero_kernel(uint32_t* __restrict__ p, long long n) {
  for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (long long)gridDim.x * blockDim.x) p[t] = 0u;
}

__global__ __launch_bounds__(256) void kan_prepare_bias_kernel(const double* __restrict__ tbias, int n_row_blocks, int n_out,
                                                               float* __restrict__ bias_sum) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_out) return;
  double s = 0.0;
  for (int r = 0; r < n_row_blocks; ++r) s += tbias[(size_t)r * n_out + j];
  bias_sum[j] = (float)s;
}

// In-place exclusive scan of n counts by one workgroup; seg[n] = total.
__global__ __launch_bounds__(1024) void kan_prepare_scan_kernel(uint32_t* __restrict__ seg, long long n) {
  __shared__ uint32_t part[1024];
  const int t = threadIdx.x;
  const long long per = (n + 1023) / 1024;
  const long long lo = t * per, hi = lo + per < n ? lo + per : n;
  uint32_t s = 0;
  for (long long p = lo; p < hi; ++p) s += seg[p];
  part[t] = s;
  __syncthreads();
  if (t == 0) {
    uint32_t run = 0;
    for (int q = 0; q < 1024; ++q) {
      const uint32_t v = part[q];
      part[q] = run;
      run += v;
    }
    seg[n] = run;
  }
  __syncthreads();
  uint32_t run = part[t];
  for (long long p = lo; p < hi; ++p) {
    const uint32_t v = seg[p];
    seg[p] = run;
    run += v;
  }
}

template <typename IdxT, typename GbT>
__global__ __launch_bounds__(256) void kan_prepare_fill_kernel(const IdxT* __restrict__ idx, const GbT* __restrict__ gain,
                                                               int n_in, int n_out, int rows_shift, int n_buckets,
                                                               const uint32_t* __restrict__ seg,
                                                               const uint16_t* __restrict__ tcnt,
                                                               uint16_t* __restrict__ pi, uint16_t* __restrict__ pq,
                                                               GbT* __restrict__ pg, uint32_t* __restrict__ ti,
                                                               GbT* __restrict__ tgo) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  // tile of ids and gains, [row][column], then the running position of every bucket, one table per wave
  IdxT* tid_ = (IdxT*)lds_raw;
  GbT* tg = (GbT*)(lds_raw + (size_t)kPrepareRows * kPrepareCols * sizeof(IdxT));
  uint32_t* base = (uint32_t*)(lds_raw + (size_t)kPrepareRows * kPrepareCols * (sizeof(IdxT) + sizeof(GbT)));
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j0 = blockIdx.x * kPrepareCols, i0 = blockIdx.y * kPrepareRows;
  const int rows = min(kPrepareRows, n_in - i0), cols = min(kPrepareCols, n_out - j0);
  for (int r = wave; r < rows; r += 4) {                     // a wave reads a row of the tile
    if (lane < cols) {
      const size_t e = (size_t)(i0 + r) * n_out + j0 + lane;
      tid_[r * kPrepareCols + lane] = idx[e];
      tg[r * kPrepareCols + lane] = gain[e];
    }
  }
  __syncthreads();
  uint32_t* wbase = base + (size_t)wave * n_buckets;
  const uint32_t mask = (1u << rows_shift) - 1u;
  const unsigned long long lt = (1ull << lane) - 1ull;
  for (int c = wave; c < cols; c += 4) {                     // a wave takes a column
    const int j = j0 + c;
    // where this row block's edges of (bucket, j) start: the segment's start plus the earlier row blocks
    for (int b = lane; b < n_buckets; b += 64) {
      uint32_t at = seg[(size_t)b * n_out + j];
      for (int rb = 0; rb < (int)blockIdx.y; ++rb) at += tcnt[((size_t)rb * n_buckets + b) * n_out + j];
      wbase[b] = at;
    }
    __builtin_amdgcn_wave_barrier();
    for (int r0 = 0; r0 < rows; r0 += 64) {
      const int r = r0 + lane;
      const bool live = r < rows;
      const uint32_t id = live ? (uint32_t)tid_[r * kPrepareCols + c] : 0u;
      if (ti && live) {        // small layers: ids and gains once more, the inputs of an output side by side
        ti[(size_t)j * n_in + i0 + r] = id;
        tgo[(size_t)j * n_in + i0 + r] = tg[r * kPrepareCols + c];
      }
      const uint32_t b = min(id >> rows_shift, (uint32_t)(n_buckets - 1));
      unsigned long long todo = __builtin_amdgcn_ballot_w64(live);
      uint32_t pos = 0;
      while (todo) {                                         // one round per bucket present among the 64 rows
        const int first = __ffsll((long long)todo) - 1;
        const uint32_t kb = __shfl(b, first);
        const unsigned long long same = __builtin_amdgcn_ballot_w64(live && b == kb) & todo;
        const uint32_t start = wbase[kb];
        if (live && b == kb) pos = start + (uint32_t)__popcll(same & lt);
        __builtin_amdgcn_wave_barrier();
        if (lane == first) wbase[kb] = start + (uint32_t)__popcll(same);
        __builtin_amdgcn_wave_barrier();
        todo &= ~same;
      }
      if (live) {
        pi[pos] = (uint16_t)(i0 + r);
        pq[pos] = (uint16_t)(id & mask);
        pg[pos] = tg[r * kPrepareCols + c];
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Order within the segments of layers that only the bucket kernel serves.  For every u < 8, the lanes of a wave read the basis
// entries of the edges at 8 l + u of its pass, sixteen bytes each: as the inputs fall, most of them meet others in their LDS
// banks (half of the time that the LDS was busy).  So position e is given an edge whose input is e / 8 modulo 16, the
// banks of sixteen lanes side by side, if the segment has one left, else one of e / 8 modulo 8, else any.  A wave per
// segment, 512 edges at a time.  2048 x 1024 at batch 1 9.68 -> 9.45 us, 2048 x 2048 at 2 17.7 -> 17.0, 2048-1024-256 at 1 / 4
// 12.5 / 23.1 -> 12.2 / 22.3, 4096 x 4096 at 1 29.1 -> 28.5.
template <typename GbT>
__global__ __launch_bounds__(256) void kan_prepare_order_kernel(const uint32_t* __restrict__ seg, long long n_seg, uint16_t* pi,
                                                                uint16_t* pq, GbT* pg) {
  constexpr int kClasses = 16, kRounds = 8, kBlock = kRounds * kWave;
  __shared__ uint32_t s_taken[4][kClasses];                  // places of a class that are given away
  __shared__ __attribute__((aligned(8))) uint8_t s_filled[4][kBlock];
  __shared__ uint16_t s_spare[4][kBlock];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long s = (long long)blockIdx.x * 4 + wave;
  if (s >= n_seg) return;
  uint32_t* taken = s_taken[wave];
  uint8_t* filled = s_filled[wave];
  uint16_t* spare = s_spare[wave];
  const unsigned long long below = (1ull << lane) - 1ull;
  for (uint32_t lo = seg[s], end = seg[s + 1]; lo < end; lo += kBlock) {
    const uint32_t hi = min(end, lo + (uint32_t)kBlock);
    uint32_t in[kRounds], q[kRounds], to[kRounds];
    GbT g[kRounds];
    bool left[kRounds];                                      // edges without a place yet
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const uint32_t e = min(lo + (uint32_t)(r * kWave + lane), hi - 1u);
      in[r] = pi[e];
      q[r] = pq[e];
      g[r] = pg[e];
      left[r] = lo + (uint32_t)(r * kWave + lane) < hi;
      to[r] = 0u;
    }
    if (lane < kClasses) taken[lane] = 0u;
    *(uint2*)(filled + 8 * lane) = make_uint2(0u, 0u);
    __builtin_amdgcn_wave_barrier();
    // places of class c in front of position e, and the k-th of the block
    auto before = [](uint32_t e, uint32_t c) { return (e >> 7) * 8u + min((uint32_t)max((int)(e & 127u) - (int)(8u * c), 0), 8u); };
    for (uint32_t other = 0; other <= 8u; other += 8u) {     // the edge's own class, then the one that shares half of its banks
#pragma unroll
      for (int r = 0; r < kRounds; ++r) {
        const uint32_t c = (in[r] ^ other) & (kClasses - 1u);
        unsigned long long same = __builtin_amdgcn_ballot_w64(left[r]);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const unsigned long long ones = __builtin_amdgcn_ballot_w64((c >> b) & 1u);
          same &= (c >> b) & 1u ? ones : ~ones;
        }
        const uint32_t first = before(lo, c), places = before(hi, c) - first;
        const uint32_t k = taken[c] + (uint32_t)__popcll(same & below), n = (uint32_t)__popcll(same);
        __builtin_amdgcn_wave_barrier();
        if (left[r] && (same & below) == 0ull) taken[c] = min(taken[c] + n, places);
        if (left[r] && k < places) {
          to[r] = ((first + k) >> 3) * 128u + 8u * c + ((first + k) & 7u);
          filled[to[r] - lo] = 1;
          left[r] = false;
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
    // the places that are left, in order
    const uint2 mine = *(const uint2*)(filled + 8 * lane);
    uint32_t free8 = 0u;
#pragma unroll
    for (int t = 0; t < 8; ++t)
      free8 |= lo + 8u * lane + t < hi && !(((t < 4 ? mine.x : mine.y) >> (8 * (t & 3))) & 1u) ? 1u << t : 0u;
    int upto = __popc(free8);
    const int own = upto;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int v = __shfl_up(upto, o, kWave);
      upto += lane >= o ? v : 0;
    }
    for (int at = upto - own; free8; ++at, free8 &= free8 - 1u) spare[at] = (uint16_t)(8 * lane + __ffs(free8) - 1);
    __builtin_amdgcn_wave_barrier();
    uint32_t next = 0u;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const unsigned long long rest = __builtin_amdgcn_ballot_w64(left[r]);
      if (left[r]) to[r] = lo + spare[next + (uint32_t)__popcll(rest & below)];
      next += (uint32_t)__popcll(rest);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // every lane holds its edges: their places are written over
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
      if (lo + (uint32_t)(r * kWave + lane) < hi) {
        pi[to[r]] = (uint16_t)in[r];
        pq[to[r]] = (uint16_t)q[r];
        pg[to[r]] = g[r];
      }
    __builtin_amdgcn_wave_barrier();
  }
}

// Blocks per bucket for a table of W blocks (prefix sums -> cnt[0 .. n_buckets]): every bucket
// gets min_blocks, the rest goes in proportion to the edges (cumulative rounding).
__global__ void kan_prepare_block_counts_kernel(const uint32_t* __restrict__ seg, int n_out, int n_buckets,
                                                int min_blocks, int W, uint32_t* __restrict__ cnt) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  const unsigned long long E = seg[(size_t)n_buckets * n_out];
  const unsigned long long spare = (unsigned long long)(W - (long long)n_buckets * min_blocks);
  unsigned long long given = 0;
  uint32_t run = 0;
  cnt[0] = 0;
  for (int b = 0; b < n_buckets; ++b) {
    const unsigned long long upto = seg[(size_t)(b + 1) * n_out];          // edges of buckets 0..b
    const unsigned long long target = E > 0 ? (spare * upto + E / 2) / E : 0;
    run += (uint32_t)min_blocks + (uint32_t)(target - given);
    given = target;
    cnt[b + 1] = run;
  }
}

// The entries of one bucket (thread = bucket): its outputs are cut into its blocks so that
// the blocks hold about equal numbers of edges, never more than kBucketMaxJw outputs each
// (the cuts are made one after the other so that the limit holds for every block).
//
// Where a block sits in the table decides its XCD (workgroups go to the 8 XCDs in turn): the
// bucket-sorted list of blocks is dealt out in 8 contiguous runs, run x taking the positions
// x, x + 8, ..., so that an XCD serves few buckets and its L2 holds only their rows (with 8
// equal buckets: one bucket per XCD, the codebook crosses the fabric once).
__device__ __forceinline__ int bucket_table_position(int s, int W) {
  const int base = W >> 3, rem = W & 7;
  int x = 0, start = 0;
  while (x < 7) {
    const int c = base + (x < rem ? 1 : 0);
    if (s < start + c) break;
    start += c;
    ++x;
  }
  return (s - start) * 8 + x;
}

__global__ __launch_bounds__(256) void kan_prepare_blocks_kernel(const uint32_t* __restrict__ seg, int n_out,
                                                                 int n_buckets, const uint32_t* __restrict__ cnt,
                                                                 uint32_t* __restrict__ table) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= n_buckets) return;
  const int W = (int)cnt[n_buckets];
  const int first = (int)cnt[b], nb = (int)(cnt[b + 1] - cnt[b]);
  const uint32_t* sb = seg + (size_t)b * n_out;     // sb[0 .. n_out] are valid (the prefix runs on)
  const unsigned long long e0 = sb[0], eb = sb[n_out] - sb[0];
  int j0 = 0;
  for (int q = 0; q < nb; ++q) {
    int j1 = n_out;
    if (q + 1 < nb) {
      const unsigned long long target = e0 + eb * (unsigned long long)(q + 1) / (unsigned long long)nb;
      int a = 0, c = n_out;                          // smallest j with sb[j] >= target
      while (a < c) {
        const int mid = (a + c) >> 1;
        if (sb[mid] >= target) c = mid; else a = mid + 1;
      }
      const int lo_c = max(j0, n_out - (nb - q - 1) * kBucketMaxJw);   // the blocks after this one can take the rest
      const int hi_c = min(j0 + kBucketMaxJw, n_out);
      j1 = min(max(a, lo_c), hi_c);
    }
    uint32_t* e = table + (size_t)bucket_table_position(first + q, W) * kBucketEntryWords;
    e[0] = (uint32_t)b;
    e[1] = (uint32_t)j0;
    e[2] = (uint32_t)j1;
    e[3] = sb[j0];
    e[4] = sb[j1];
    e[5] = e[6] = e[7] = 0u;
    j0 = j1;
  }
}

template <typename IdxT, typename GbT>
hipError_t prepare_typed(const LayerPtrs& h, int n_in, int n_out, const BucketGeom& g, void* prepared,
                         hipStream_t s) {
  char* p = (char*)prepared;
  uint32_t* seg = (uint32_t*)(p + g.off_seg);
  uint16_t* tcnt = (uint16_t*)(p + g.off_tcnt);
  double* tbias = (double*)(p + g.off_tbias);
  const long long n_seg = (long long)g.n_buckets * n_out;
  const Q8Params qp = {h.gain_log2_lo, h.gain_log2_step, h.bias_scale};
  dim3 grid((unsigned)((n_out + kPrepareCols - 1) / kPrepareCols), (unsigned)g.n_row_blocks);
  const size_t lds_count = (size_t)g.n_buckets * kPrepareCols * sizeof(uint32_t);
  const size_t lds_fill = (size_t)kPrepareRows * kPrepareCols * (sizeof(IdxT) + sizeof(GbT)) + (size_t)4 * g.n_buckets * sizeof(uint32_t);
  if (lds_count > 64 * 1024 || lds_fill > 150 * 1024) return hipErrorInvalidValue;     // (n_buckets <= 256 fits)
  // (dynamic LDS beyond 64 KB has to be asked for; the tile of 4-byte ids and 4-byte gains takes 128 KB)
  hipError_t err = hipFuncSetAttribute((const void*)kan_prepare_fill_kernel<IdxT, GbT>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_fill);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(kan_prepare_zero_kernel, dim3((unsigned)((n_seg + 1 + 255) / 256 > 1024 ? 1024 : (n_seg + 1 + 255) / 256)),
                     dim3(256), 0, s, seg, n_seg + 1);
  hipLaunchKernelGGL((kan_prepare_count_kernel<IdxT, GbT>), grid, dim3(256), lds_count, s, (const IdxT*)h.idx,
                     (const GbT*)h.bias, n_in, n_out, g.rows_shift, g.n_buckets, seg, tcnt, tbias, qp);
  hipLaunchKernelGGL(kan_prepare_scan_kernel, dim3(1), dim3(1024), 0, s, seg, n_seg);
  hipLaunchKernelGGL((kan_prepare_fill_kernel<IdxT, GbT>), grid, dim3(256), lds_fill, s, (const IdxT*)h.idx,
                     (const GbT*)h.gain, n_in, n_out, g.rows_shift, g.n_buckets, (const uint32_t*)seg,
                     (const uint16_t*)tcnt, (uint16_t*)(p + g.off_i), (uint16_t*)(p + g.off_q), (GbT*)(p + g.off_g),
                     g.off_ti ? (uint32_t*)(p + g.off_ti) : nullptr, g.off_tg ? (GbT*)(p + g.off_tg) : nullptr);
  if ((long long)n_in * n_out > kColumnMaxEdges)
    hipLaunchKernelGGL(kan_prepare_order_kernel<GbT>, dim3((unsigned)((n_seg + 3) / 4)), dim3(256), 0, s, (const uint32_t*)seg, n_seg,
                       (uint16_t*)(p + g.off_i), (uint16_t*)(p + g.off_q), (GbT*)(p + g.off_g));
  hipLaunchKernelGGL(kan_prepare_bias_kernel, dim3((unsigned)((n_out + 255) / 256)), dim3(256), 0, s, (const double*)tbias,
                     g.n_row_blocks, n_out, (float*)(p + g.off_bias));
  const int min_blocks = (n_out + kBucketMaxJw - 1) / kBucketMaxJw;
  for (int t = 0; t < kBucketTables; ++t) {
    uint32_t* cnt = (uint32_t*)(p + g.off_cnt) + (size_t)t * (g.n_buckets + 1);
    uint32_t* table = (uint32_t*)(p + g.off_blk) + (size_t)g.tab_first[t] * kBucketEntryWords;
    hipLaunchKernelGGL(kan_prepare_block_counts_kernel, dim3(1), dim3(64), 0, s, (const uint32_t*)seg, n_out,
                       g.n_buckets, min_blocks, g.tab_w[t], cnt);
    hipLaunchKernelGGL(kan_prepare_blocks_kernel, dim3((unsigned)((g.n_buckets + 255) / 256)), dim3(256), 0, s,
                       (const uint32_t*)seg, n_out, g.n_buckets, (const uint32_t*)cnt, table);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_bucket_prepare(const LayerPtrs& h, int idx_u32, int gb_kind, int n_in, int n_out,
                                 const BucketGeom& g, void* prepared, hipStream_t s) {
  if (idx_u32) {
    if (gb_kind == kGbQ8) return prepare_typed<uint32_t, q8_t>(h, n_in, n_out, g, prepared, s);
    if (gb_kind == kGbF16) return prepare_typed<uint32_t, __half>(h, n_in, n_out, g, prepared, s);
    return prepare_typed<uint32_t, float>(h, n_in, n_out, g, prepared, s);
  }
  if (gb_kind == kGbQ8) return prepare_typed<uint16_t, q8_t>(h, n_in, n_out, g, prepared, s);
  if (gb_kind == kGbF16) return prepare_typed<uint16_t, __half>(h, n_in, n_out, g, prepared, s);
  return prepare_typed<uint16_t, float>(h, n_in, n_out, g, prepared, s);
}

hipError_t launch_bucket(int code, int gb_kind, const BucketArgs& a, int blocks, int heads, hipStream_t s) {
  if (a.n_in > kBucketMaxIn || a.n_buckets < 1 || blocks < a.n_buckets) return hipErrorInvalidValue;
  if (code != kCbI8 && code != kCbF16 && code != kCbF32 && code != kCbBfp8) return hipErrorInvalidValue;
  if (gb_kind == kGbQ8 && code != kCbI8) return hipErrorInvalidValue;      // byte-coded gains go with Int8 codebooks
  dim3 grid((unsigned)blocks, (unsigned)a.B, (unsigned)heads);
  dim3 block(kBucketThreads);
  const bool wide = a.n_in > 2048;
#define KAN_LAUNCH_BUCKET(GK, CODE)                                                                    \
  do {                                                                                                 \
    if (wide) hipLaunchKernelGGL((kan_bucket_kernel<GK, CODE, 4096>), grid, block, 0, s, a);           \
    else hipLaunchKernelGGL((kan_bucket_kernel<GK, CODE, 2048>), grid, block, 0, s, a);                \
  } while (0)
  if (code == kCbI8) {
    if (gb_kind == kGbQ8) KAN_LAUNCH_BUCKET(kGbQ8, kCbI8);
    else if (gb_kind == kGbF16) KAN_LAUNCH_BUCKET(kGbF16, kCbI8);
    else KAN_LAUNCH_BUCKET(kGbF32, kCbI8);
  } else if (code == kCbF16) {
    if (gb_kind == kGbF16) KAN_LAUNCH_BUCKET(kGbF16, kCbF16);
    else KAN_LAUNCH_BUCKET(kGbF32, kCbF16);
  } else if (code == kCbBfp8) {
    if (gb_kind == kGbF16) KAN_LAUNCH_BUCKET(kGbF16, kCbBfp8);
    else KAN_LAUNCH_BUCKET(kGbF32, kCbBfp8);
  } else {
    if (gb_kind == kGbF16) KAN_LAUNCH_BUCKET(kGbF16, kCbF32);
    else KAN_LAUNCH_BUCKET(kGbF32, kCbF32);
  }
#undef KAN_LAUNCH_BUCKET
  return hipGetLastError();
}

hipError_t launch_column(int code, int gb_kind, const BucketArgs& a, int heads, hipStream_t s) {
  if ((long long)a.n_in * a.n_out > kColumnMaxEdges || a.off_ti <= 0 || a.off_tg <= 0) return hipErrorInvalidValue;
  if (code != kCbI8 && code != kCbF16 && code != kCbF32 && code != kCbBfp8) return hipErrorInvalidValue;
  if (gb_kind == kGbQ8 && code != kCbI8) return hipErrorInvalidValue;
  dim3 grid((unsigned)a.n_out, (unsigned)a.B, (unsigned)heads);
  dim3 block(kColumnThreads);
#define KAN_LAUNCH_COLUMN(GK, CB)                                                                                  \
  do {                                                                                                             \
    if (a.n_in <= 4 * kColumnThreads) hipLaunchKernelGGL((kan_column_kernel<GK, CB, 4>), grid, block, 0, s, a);    \
    else hipLaunchKernelGGL((kan_column_kernel<GK, CB, 8>), grid, block, 0, s, a);                                 \
  } while (0)
  if (code == kCbI8) {
    if (gb_kind == kGbQ8) KAN_LAUNCH_COLUMN(kGbQ8, int8_t);
    else if (gb_kind == kGbF16) KAN_LAUNCH_COLUMN(kGbF16, int8_t);
    else KAN_LAUNCH_COLUMN(kGbF32, int8_t);
  } else if (code == kCbF16) {
    if (gb_kind == kGbF16) KAN_LAUNCH_COLUMN(kGbF16, __half);
    else KAN_LAUNCH_COLUMN(kGbF32, __half);
  } else if (code == kCbBfp8) {
    if (gb_kind == kGbF16) KAN_LAUNCH_COLUMN(kGbF16, bfp8_t);
    else KAN_LAUNCH_COLUMN(kGbF32, bfp8_t);
  } else {
    if (gb_kind == kGbF16) KAN_LAUNCH_COLUMN(kGbF16, float);
    else KAN_LAUNCH_COLUMN(kGbF32, float);
  }
#undef KAN_LAUNCH_COLUMN
  return hipGetLastError();
}

}  // namespace kan
