// Streaming contraction of large batches: tiles of 256 samples x 256 outputs, one workgroup of eight waves per CU.
//
// Same operands as kan_mfma.hip (sparse matrix instruction, k order (m, m + 5)) in the form of kan_wide.hip: rotated
// basis words (each stored value carries "takes coefficient m + 5" in its sign) and coefficient records with
// coefficients 5..9 negated.  Both are laid out in the order in which the instruction's lanes take them, so nothing is
// rearranged on the way: the memory pipeline copies them straight into LDS (buffer_load ... lds, no registers, no
// vector instructions) and a lane's fragment is one 16-byte LDS read.
//
// A step of 16 inputs is five groups S (one sparse MFMA of K = 32 per 32 x 32 block each); a group needs 8 KB of basis
// words, 16 KB of records and 1 KB of position bits and keeps every SIMD's matrix pipe busy for 16 MFMAs.  Groups run
// through a ring of six slots; one barrier per group.  Wave (wm, wn) of 2 x 4 owns 128 x 64 results: 4 + 4 fragment
// reads of 1 KB per 8 MFMAs.
//
// What bounds it is most likely power: 4096 x 4096 at batch 8192 takes 1.34-1.45 ms over the cards (tiles of 128 x 256 with
// the basis tile built in LDS by the waves, kan_mfma.hip: 1.73).  On a card where it took 1.44 the counters read 2.12 M
// clocks, 1.47 GHz (the preparation launch in front ran at 2.16), the matrix pipe busy for 58 % of them (60.5 where it took
// 1.39), LDS 31 %: 1.0 of the 1.3 PFLOP/s that a large dense product reaches here.  What each part costs there:
// without the copies 1.07 ms (with position bits computed for free), without copies and LDS reads 0.93.  Position bits
// computed from the fragments' signs instead of read (40 vector instructions per 8 MFMAs) 1.49; reads, copies and MFMAs
// in blocks instead of in turn 1.56; planes padded by half a bank row: no change (the counters show no conflicts).
#include <type_traits>

#include "kan_device.hpp"
#include "kan_internal.hpp"
#include "kan_mfma_common.hpp"

namespace kan {
namespace {

constexpr int kThreads = 512;
constexpr int BM = kStreamTile, BN = kStreamTile;
constexpr int IT = 16;                           // inputs per step
constexpr int RB = 4, NB = 2;                    // 32 x 32 blocks per wave
constexpr int kAPlane = BM * 16, kBPlane = BN * 16;
constexpr int kABytes = 2 * kAPlane;             // basis words of a group: planes a = 0, 1
constexpr int kPosAt = kABytes + 4 * kBPlane;     // behind the records (planes (h, a)): position bits
constexpr int kSlot = kPosAt + 2 * BM * 2;
constexpr int kSlots = 6;
constexpr int kLoads = 3;                        // 1 KB copies per wave and group: 24 for the six planes (and one by wave s % 8 of group s)
constexpr int kBufferFlags = 0x00020000;         // buffer resource word 3: raw 32-bit data format, no swizzle

// 64 lanes x 16 bytes from the buffer r at each lane's `off` into LDS at `lds`, `lds` + 16, ...  The compiler does not
// count these copies: the waits are explicit (copies_done); the s_nop is the wait state between a write of M0 and its use
// by such a load.
__device__ __forceinline__ void copy_to_lds(const u32x4 r, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(off), "s"(r) : "memory", "m0");
}
// All but the newest N of this wave's copies have landed, and its own LDS reads are done.
template <int N>
__device__ __forceinline__ void copies_done() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ u32x4 buffer_of(const void* p, uint32_t bytes) {
  const uint64_t a = (uint64_t)(uintptr_t)p;
  u32x4 r = {(uint32_t)a, (uint32_t)(a >> 32), bytes, (uint32_t)kBufferFlags};
  return r;
}

template <bool THREE>
__global__ __launch_bounds__(kThreads, 2) void kan_stream_kernel(const StreamArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char sRing[kSlots * kSlot];
  __shared__ float sBias[BN];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, lh = lane >> 5;
  const int wm = wave & 1, wn = wave >> 1;
  const int head = blockIdx.z;
  // Runs of consecutive work items per XCD (chunk, then patches of 8 x 4 tiles: 32 workgroups that an XCD runs at a
  // time and that share eight slices of the basis words and four of the records).
  int chunk, bt, jt;
  {
    const unsigned T = gridDim.x, W = T * gridDim.y;
    const unsigned L = blockIdx.x + T * blockIdx.y;
    const unsigned xcd = L & 7u, m = L >> 3, q = W >> 3, r = W & 7u;
    const unsigned item = xcd * q + min(xcd, r) + m;
    chunk = (int)(item / T);
    const int seq = (int)(item % T), njt = a.n_jt, nbt = (int)T / njt;
    if (njt % 4 == 0 && nbt % 8 == 0) {
      const int patch = seq >> 5, w = seq & 31, per_row = njt / 4;
      bt = (patch / per_row) * 8 + (w >> 2);
      jt = (patch % per_row) * 4 + (w & 3);
    } else {
      jt = seq % njt;
      bt = seq / njt;
    }
  }
  const int b0 = bt * BM, j0 = jt * BN;
  const int n_in = a.n_in, n_out = a.n_out, B = a.B;
  const int i_begin = chunk * a.rows_per_chunk;
  const int i_end = min(n_in, i_begin + a.rows_per_chunk);
  const int groups = (i_end - i_begin + IT - 1) / IT * 5;        // groups of the chunk
  const int total = THREE ? 3 * groups : groups;
  const size_t g0 = (size_t)(i_begin / IT) * 5;

  // ---- copies of a group (rows past the last sample are whatever the workspace holds: their results are dropped): wave w
  // takes rows (w % 4) 64 .. of basis plane w / 4 and chunks 2 w, 2 w + 1 of the records
  // (chunk c: plane c / 4, columns (c % 4) 64 ..).
  const uint32_t rows = (uint32_t)rot_rows(B), a_plane = 2u * rows * 16u, b_plane = 4u * (uint32_t)n_out * 16u;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)sRing;
  const uint32_t a_off = ((uint32_t)(wave >> 2) * rows + (uint32_t)(b0 + (wave & 3) * 64 + lane)) * 16u;
  const uint32_t a_lds = lds0 + (uint32_t)((wave >> 2) * kAPlane + (wave & 3) * 1024);
  uint32_t b_off[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int c = 2 * wave + u;
    b_off[u] = ((uint32_t)(c >> 2) * (uint32_t)n_out + (uint32_t)min(j0 + (c & 3) * 64 + lane, n_out - 1)) * 16u;
  }
  const uint32_t b_lds = lds0 + (uint32_t)(kABytes + (wave >> 1) * kBPlane + (wave & 1) * 2048);
  const char* const Wm = (const char*)(a.W + (long long)head * a.w_head_stride);
  const char* const Pm = (const char*)(a.P + (long long)head * a.p_head_stride);
  const uint32_t p_plane = rows * 2u, p_off = (uint32_t)lh * p_plane + (uint32_t)b0 * 2u + (uint32_t)ln * 16u;
  const char* const Wl = THREE ? (const char*)(a.W_lo + (long long)head * a.w_head_stride) : nullptr;
  const char* const Cm = (const char*)(a.cf + (long long)head * a.cf_head_stride);
  const char* const Cl = THREE ? (const char*)(a.cf_lo + (long long)head * a.cf_head_stride) : nullptr;
  // Group s of the kernel.  Split form: the cross products (W, low records), (low W, records) first, which carry a
  // factor 2048, then the main product on top.
  struct CopySrc {
    u32x4 a, b, p;
    uint32_t slot;
  };
  auto copy_src = [&](int s) {
    const int v = min(s, total - 1);                              // past the end: the last group again, never read
    const int pass = THREE ? (v >= 2 * groups ? 2 : (v >= groups ? 1 : 0)) : 0;
    const size_t g = g0 + (size_t)(v - pass * groups);
    CopySrc c;
    c.a = buffer_of((THREE && pass == 1 ? Wl : Wm) + g * a_plane, a_plane);
    c.b = buffer_of((THREE && pass == 0 ? Cl : Cm) + g * b_plane, b_plane);
    c.p = buffer_of(Pm + g * (2 * p_plane), 2 * p_plane);
    c.slot = (uint32_t)(s % kSlots) * (uint32_t)kSlot;
    return c;
  };
  auto copy_part = [&](const CopySrc& c, int u) {
    if (u == 0) copy_to_lds(c.a, a_off, a_lds + c.slot);
    else copy_to_lds(c.b, b_off[u - 1], b_lds + c.slot + (u - 1) * 1024);
  };
  // (one more copy in flight in one of the waves: its waits then cover one copy more than they need)
  auto copy_positions = [&](const CopySrc& c, int s) {
    if (wave == (s & 7)) copy_to_lds(c.p, p_off, lds0 + c.slot + kPosAt);
  };

  struct Frags {
    u32x4 a[RB], b[NB][2];
    uint2 pos;               // of row blocks 0, 1 / 2, 3
  };
  const uint32_t ra0 = (uint32_t)(lh * kAPlane + (wm * (32 * RB) + ln) * 16);
  const uint32_t rb0 = (uint32_t)(kABytes + lh * 2 * kBPlane + (wn * (32 * NB) + ln) * 16);
  auto read_a = [&](const unsigned char* slot, int rb, Frags& f) { f.a[rb] = *(const u32x4*)(slot + ra0 + rb * 512); };
  auto read_b = [&](const unsigned char* slot, int u, Frags& f) {
    f.b[u >> 1][u & 1] = *(const u32x4*)(slot + rb0 + (u & 1) * kBPlane + (u >> 1) * 512);
  };

  const uint32_t rp0 = (uint32_t)(kPosAt + (lh * BM + wm * (32 * RB) + ln * RB) * 2);
  auto read_pos = [&](const unsigned char* slot, Frags& f) { f.pos = *(const uint2*)(slot + rp0); };

  f32x16 acc[RB][NB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[rb][nb][r] = 0.f;

#pragma unroll
  for (int s = 0; s < kSlots; ++s) {
    const CopySrc src = copy_src(s);
#pragma unroll
    for (int u = 0; u < kLoads; ++u) copy_part(src, u);
    copy_positions(src, s);
  }
  {      // bias sums of the tile's columns, parked in LDS until the epilogue
    const float* bp = a.bias_partial + (long long)head * a.bp_head_stride + min(j0 + (tid & (BN - 1)), n_out - 1);
    const int rb_end = (i_end + kMfmaPrepRows - 1) / kMfmaPrepRows;
    float bs = 0.f;
    if (tid < BN) {
      for (int r0 = i_begin / kMfmaPrepRows; r0 < rb_end; r0 += 8) {
        float t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = bp[(long long)min(r0 + u, rb_end - 1) * n_out];
#pragma unroll
        for (int u = 0; u < 8; ++u) bs += r0 + u < rb_end ? t[u] : 0.f;
      }
      sBias[tid] = bs;
    }
  }
  copies_done<(kSlots - 1) * kLoads>();
  __builtin_amdgcn_s_barrier();
  Frags f[2];
  read_pos(sRing, f[0]);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) read_a(sRing, rb, f[0]);
#pragma unroll
  for (int u = 0; u < 2 * NB; ++u) read_b(sRing, u, f[0]);
  static_assert(RB == 4 && RB == 2 * NB, "eight MFMAs, eight fragment reads per group");

  // Group s: its fragments are in registers.  Behind the barrier every wave's copies of group s + 1 have
  // landed and nobody reads slot s % kSlots any more, which takes group s + kSlots.
  auto group = [&](auto P, int s) {
    constexpr int p = decltype(P)::value;
    if (THREE && s == 2 * groups) {       // the cross products are complete
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[rb][nb][r] *= 1.0f / 2048.0f;
    }
    copies_done<(kSlots - 2) * kLoads>();
    __builtin_amdgcn_s_barrier();
    const CopySrc src = copy_src(s + kSlots);
    const unsigned char* const next = sRing + ((s + 1) % kSlots) * kSlot;
    __builtin_amdgcn_sched_barrier(0);
    // One MFMA, one fragment read of the next group, and so on: a wave that hands the LDS or the memory pipeline several
    // instructions in a row waits until the other seven waves' are through, and issues no MFMA meanwhile (all eight
    // reads ahead of the MFMAs: 1.56 ms for 4096 x 4096 at batch 8192).
    __builtin_amdgcn_s_setprio(2);
#pragma unroll
    for (int i = 0; i < RB * NB; ++i) {
      const int rb = i / NB, nb = i % NB;
      const h16x8 fa = __builtin_bit_cast(h16x8, f[p].a[rb]);
      const h16x16 fb = __builtin_bit_cast(h16x16, f[p].b[nb]);
      const int ix = (int)(rb < 2 ? f[p].pos.x : f[p].pos.y);
      if (rb & 1) acc[rb][nb] = __builtin_amdgcn_smfmac_f32_32x32x32_f16(fa, fb, acc[rb][nb], ix, 0, 1);
      else acc[rb][nb] = __builtin_amdgcn_smfmac_f32_32x32x32_f16(fa, fb, acc[rb][nb], ix, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      // (the last reads go out two MFMAs before the end, so that the wait in front of the next barrier finds them done)
      constexpr int first[9] = {0, 1, 2, 4, 6, 7, 8, 8, 8};
      for (int u = first[i]; u < first[i + 1]; ++u) {
        if (u < RB) read_a(next, u, f[p ^ 1]);
        else read_b(next, u - RB, f[p ^ 1]);
      }
      if (i % 2 == 0 && i / 2 < kLoads) copy_part(src, i / 2);
      if (i == 0) read_pos(next, f[p ^ 1]);
      if (i == 6) copy_positions(src, s + kSlots);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
  };
  int s = 0;
  for (; s + 2 <= total; s += 2) {
    group(std::integral_constant<int, 0>{}, s);
    group(std::integral_constant<int, 1>{}, s + 1);
  }
  if (s < total) group(std::integral_constant<int, 0>{}, s);
  copies_done<0>();

  // ---- epilogue.  D layout of the 32x32 MFMA: lane holds column (lane & 31), rows
  //      m = 8*(r/4) + 4*(lane/32) + r%4 for r = 0..15: samples 4 m + rb of the wave's 128.  Rows past the last sample are dropped by the buffer's bound. ----
  const float scale = a.scale[head];
  float* const dst = a.dst + (long long)head * a.dst_head_stride + (long long)chunk * a.dst_chunk_stride + (long long)b0 * n_out;
  const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc((void*)dst, 0, min(BM, B - b0) * n_out * 4, kBufferFlags);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int c = wn * (32 * NB) + nb * 32 + ln, j = j0 + c;
    const float bs = sBias[c];
    if (j < n_out) {
      const int at = (16 * lh * n_out + j) * 4;
      auto store = [&](auto act) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(act(fmaf(scale, acc[rb][nb][r], bs))), rd, at,
                                                  (wm * (32 * RB) + (8 * (r >> 2) + (r & 3)) * RB + rb) * n_out * 4, 0);
      };
      if (a.apply_tanh) store([](float v) { return tanhf(v); });
      else store([](float v) { return v; });
    }
  }
}

}  // namespace

bool stream_takes(int n_out, int64_t B) {      // a group of either operand and a tile of the result: 32-bit offsets
  return B <= (1 << 24) && n_out <= kWideMaxOut;
}

hipError_t launch_stream(const StreamArgs& a, bool split, dim3 grid, hipStream_t s) {
  if (a.B < 1 || !stream_takes(a.n_out, a.B) || a.rows_per_chunk < kMfmaPrepRows || a.rows_per_chunk % kMfmaPrepRows != 0 ||
      !a.W || !a.cf || (split && (!a.W_lo || !a.cf_lo)) || (long long)a.n_jt * BN < a.n_out)
    return hipErrorInvalidValue;
  if (split) hipLaunchKernelGGL((kan_stream_kernel<true>), grid, dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL((kan_stream_kernel<false>), grid, dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace kan
