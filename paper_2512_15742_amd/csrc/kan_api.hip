// C-ABI of the library (include/kan.h): host-side validation, launch planning
// and dispatch.  All arithmetic of the method runs in the kernels; this file
// only decides which kernels run, with what grid, and where their scratch data
// lives inside the caller's workspace.

#include "../../include/kan.h"

#include <hip/hip_runtime.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "kan_internal.hpp"

// Scratch memory of kan_vq_head_forward_static: one array per GPU, held from the moment the
// library's code is loaded on that GPU until the process ends.  In host code this name is only
// a handle for hipGetSymbolAddress; the address the kernels get is looked up per device.
static __device__ __align__(256) unsigned char scratch[KAN_STATIC_SCRATCH_BYTES];

namespace kan {
namespace {

// Device address of `scratch` on the current device (looked up on the first call per device).
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mutex;

kan_status static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return KAN_ERR_LAUNCH;
  if (dev < 0 || dev >= kMaxDevices) return KAN_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return KAN_ERR_LAUNCH;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return KAN_OK;
}

// ---- per-kernel event timing ---------------------------------------------------
struct Prof {
  bool on = false;
  int cap = 0, n = 0;
  std::vector<hipEvent_t> ev;
  std::vector<const char*> names;
  std::vector<int> layer;     // 1-based layer of a head call the launch belongs to, 0: none
  int cur_layer = 0;
} g_prof;

template <typename F>
kan_status run(const char* name, hipStream_t s, F&& f) {
  hipError_t err;
  if (g_prof.on && g_prof.n < g_prof.cap) {
    const int n = g_prof.n++;
    g_prof.names[n] = name;
    g_prof.layer[n] = g_prof.cur_layer;
    (void)hipEventRecord(g_prof.ev[2 * n], s);
    err = f();
    (void)hipEventRecord(g_prof.ev[2 * n + 1], s);
  } else {
    err = f();
  }
  return err == hipSuccess ? KAN_OK : KAN_ERR_LAUNCH;
}

// ---- validation ------------------------------------------------------------------
constexpr int64_t kMaxDim = 1 << 20;
constexpr int64_t kMaxBatch = 1 << 24;

inline bool aligned(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }
inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

int gb_kind_of(const kan_vq_layer& L) {
  return L.gb_dtype == KAN_F32 ? kGbF32 : (L.gb_dtype == KAN_F16 ? kGbF16 : kGbQ8);
}

int code_of(const kan_vq_layer& L) {
  return L.cb_dtype == KAN_I8 ? kCbI8 : (L.cb_dtype == KAN_F16 ? kCbF16 : (L.cb_dtype == KAN_BFP8 ? kCbBfp8 : kCbF32));
}

kan_status validate_layer(const kan_vq_layer* L) {
  if (!L) return KAN_ERR_NULL;
  if (L->G != 10 || L->degree != 3) return KAN_ERR_UNSUPPORTED;
  if (L->rule != KAN_RULE_BSPLINE3 && L->rule != KAN_RULE_PLI2) return KAN_ERR_UNSUPPORTED;
  if (L->in < 1 || L->out < 1 || L->in > kMaxDim || L->out > kMaxDim || L->K < 1) return KAN_ERR_SHAPE;
  if (L->idx_dtype != KAN_U16 && L->idx_dtype != KAN_U32) return KAN_ERR_DTYPE;
  if (L->gb_dtype != KAN_F32 && L->gb_dtype != KAN_F16 && L->gb_dtype != KAN_Q8) return KAN_ERR_DTYPE;
  if (L->cb_dtype != KAN_F32 && L->cb_dtype != KAN_F16 && L->cb_dtype != KAN_I8 && L->cb_dtype != KAN_BFP8) return KAN_ERR_DTYPE;
  if (L->idx_dtype == KAN_U16 && L->K > 65536) return KAN_ERR_SHAPE;
  // byte-coded gain/bias belong to the fully quantised format: one-byte codebook entries too
  if (L->gb_dtype == KAN_Q8 && L->cb_dtype != KAN_I8) return KAN_ERR_UNSUPPORTED;
  if (L->flags & ~KAN_LAYER_NO_COLUMN) return KAN_ERR_UNSUPPORTED;
  if (!L->idx || !L->gain || !L->bias || !L->codebook) return KAN_ERR_NULL;
  const size_t idx_sz = L->idx_dtype == KAN_U16 ? 2 : 4;
  const size_t gb_sz = L->gb_dtype == KAN_F32 ? 4 : (L->gb_dtype == KAN_F16 ? 2 : 1);
  if (!aligned(L->idx, idx_sz) || !aligned(L->gain, gb_sz) || !aligned(L->bias, gb_sz)) return KAN_ERR_SHAPE;
  if (!aligned(L->codebook, L->cb_dtype == KAN_F32 ? 8 : (L->cb_dtype == KAN_I8 ? 2 : 4))) return KAN_ERR_SHAPE;
  return KAN_OK;
}

// ---- planning -----------------------------------------------------------------------
// Everything below is a pure function of shapes, dtypes, batch, head count and
// pointer alignment, so the workspace query and the forward call always agree.

enum PlanKind { kPlanGather = 0, kPlanMfma = 1, kPlanFused16 = 2, kPlanFused32 = 3, kPlanBucket = 4, kPlanColumn = 5, kPlanDense = 6, kPlanFusedWave = 7, kPlanTail = 8 };

struct LayerPlan {
  GatherCfg cfg;
  int n_jt, n_bt, n_chunks, rows_per_chunk;
  int tile_n = 0;              // matrix-core path: outputs per workgroup tile (128: four waves, 256: eight)
  int kind;          // PlanKind
  bool half = false; // kPlanFusedWave with fp16 operands
  bool tiles_ahead = false;    // kPlanFused16, kPlanFused32 in the place of the wave-by-wave kernel, because it is the faster one, but by little enough to give way
  bool one_head = false;       // kPlanFusedWave whose chunks depend on the workgroups that heads taken one at a time get
  bool wide = false; // kPlanMfma whose workgroups dequantise their own coefficients (kan_wide.hip): cfg.bt samples x tile_n outputs
  bool stream = false;   // kPlanMfma on tiles of 256 x 256 with both operands copied to LDS (kan_stream.hip)
  bool rot() const { return wide || stream; }      // basis words in the rotated form
  bool mfma;         // kind == kPlanMfma (coefficient + basis preparation, streaming contraction) or kPlanTail (coefficient preparation, one launch)
  int products = 1;  // 3: both operands in high and low fp16 parts, hi*hi + hi*lo + lo*hi (three passes inside the kernel)
  const char* name;
};

constexpr int kCUs = 256;
constexpr int kTargetWorkgroups = 512;    // two workgroups of 4 waves per CU
constexpr int kEnoughWorkgroups = 384;
constexpr long long kFusedMinEdgesForResidency = 1 << 17;   // several heads: workgroups for the sake of L2 from this many edges per head
constexpr int kGatherMinWgsPerHead = 32, kGatherMinRowsPerHead = 16;

// Geometry for one choice of outputs-per-lane.  The four waves of a workgroup are
// interleaved along i whenever the layer has rows for them (their sums meet in LDS), so a
// workgroup spans 64*jpl outputs and parallelism comes from output tiles first; i is split
// into chunks only as far as the partial sums stay small next to the parameter stream
// (n_chunks * B * out * 4 bytes <= a quarter of in * out * bytes_per_edge).
// head_cb: bytes of a head's codebook where the XCDs take the heads one behind the other (gather_by_head), 0 where they do
// not.  An XCD holds 128 or 160 workgroups: with one for every 8 KB of the codebook it works on as many heads as its L2 holds
// codebooks.  Fifty heads of 2048-256-21 at batch 1, Int8, 11 / 32 / 64 workgroups each: 234 / 173 / 165 us, twenty 94 / 83 / 74,
// of fp32 rows with 11 / 64 / 128 171 / 130 / 109; thirty of 1000-200-60 with 5,000 shapes 9 / 32 / 64 69 / 59 / 64 (chunks of 16
// inputs there: one pass of the four waves).
void gather_geometry(LayerPlan& p, int n_in, int n_out, int64_t B, int n_heads, int jpl, int bytes_per_edge, long long head_cb) {
  p.cfg.jpl = jpl;
  const int lanes_j = (n_out + jpl - 1) / jpl;
  p.cfg.wj = n_in >= 16 ? 1 : (lanes_j > 128 ? 4 : (lanes_j > 64 ? 2 : 1));
  const int wi = 4 / p.cfg.wj;
  p.n_jt = (lanes_j + 64 * p.cfg.wj - 1) / (64 * p.cfg.wj);
  p.n_bt = (int)((B + p.cfg.bt - 1) / p.cfg.bt);
  const long long base = (long long)n_heads * p.n_jt * p.n_bt;
  long long chunks = (kTargetWorkgroups + base - 1) / (base > 0 ? base : 1);
  if (head_cb > 0) {
    const long long want = std::max<long long>(kGatherMinWgsPerHead, head_cb >> 13) / p.n_jt;
    chunks = std::max(chunks, std::min<long long>(want, n_in / kGatherMinRowsPerHead));
  }
  const long long max_by_rows = n_in / (wi * 4);
  const long long max_by_bytes = (long long)n_in * bytes_per_edge / (16 * (B > 0 ? B : 1));
  if (chunks > max_by_rows) chunks = max_by_rows;
  if (chunks > max_by_bytes) chunks = max_by_bytes;
  if (chunks < 1) chunks = 1;
  int rows = (int)((n_in + chunks - 1) / chunks);
  const int unit = head_cb > 0 ? kGatherMinRowsPerHead : wi;
  rows = (rows + unit - 1) / unit * unit;
  p.rows_per_chunk = rows;
  p.n_chunks = (n_in + rows - 1) / rows;
}

// VQ layers at batch 1.  compact: no finer chunks for the sake of L2, for calls that fit the static scratch only so.
LayerPlan plan_gather(int n_in, int n_out, int64_t B, int n_heads, int idx_u32, int gb_kind, int code,
                      bool vec_ok, long long cb_bytes, bool compact) {
  LayerPlan p;
  const bool by_head = !compact && (long long)n_in * n_out >= kFusedMinEdgesForResidency && gather_by_head(n_heads, cb_bytes);
  const long long head_cb = by_head ? cb_bytes : 0;
  p.mfma = false;
  p.kind = kPlanGather;
  p.cfg.idx_u32 = idx_u32;
  p.cfg.gb_kind = gb_kind;
  p.cfg.code = code;
  p.cfg.bt = 1;
  p.name = "kan_gather_bt1";
  const int bytes_per_edge = (idx_u32 ? 4 : 2) + 2 * gb_bytes(gb_kind);
  const int jpl_max = 8;
  // Widest per-lane vector that divides the row and still gives the chip enough workgroups;
  // narrower vectors mean more output tiles (load width does not matter to the stream).
  int best = 1;
  long long best_wgs = -1;
  for (int c = vec_ok ? jpl_max : 1; c >= 1; c >>= 1) {
    if (n_out % c != 0 || (c > 1 && n_out / c < 64)) continue;
    gather_geometry(p, n_in, n_out, B, n_heads, c, bytes_per_edge, head_cb);
    const long long wgs = (long long)n_heads * p.n_jt * p.n_bt * p.n_chunks;
    if (wgs >= kEnoughWorkgroups) { best = c; break; }
    if (wgs > best_wgs) { best = c; best_wgs = wgs; }
  }
  gather_geometry(p, n_in, n_out, B, n_heads, best, bytes_per_edge, head_cb);
  return p;
}

// Matrix-core path: tiles of 64 or 128 samples x 128 outputs (128 x 256 for eight waves), i split so that
// every CU has two workgroups of four waves (or one of eight).
constexpr int kMfmaTileN = 128;
constexpr int kMfmaRowsStep = kMfmaPrepRows;   // chunk boundaries coincide with partial bias sums
constexpr int kMfmaTargetWorkgroups = 512;
// A chunk of inputs is at least two steps: a layer that leaves CUs idle is a latency chain (first loads 3 us, then a
// step per 1-1.5 us of memory latency), and the slices of more chunks cost its consumer less than the steps (with
// 64 inputs against 32: a 160-64-31-11 head at batch 72 34.0 / 30.4 us, 1832-96-25-20 at 2846 63.9 / 59.5,
// 1085-512-117 precise at 772 77.8 / 74.9, 2048-1024-256 at 1024 88.7 / 88.6).
constexpr int kMfmaMinRows = 32, kMfmaMinRowsCompact = 64;    // (64: see plan_head)
// (config 3 at batch 65-128, whose first layer is cut into 32 chunks: 55.3-56.4 us with the 32 slices handed
// on against 56.7-57.4 us with a reduction launch)
constexpr int kMaxChainedSlices = 32;   // more slices than this go through the reduction pass (more loads in flight per output)
constexpr int kMfmaMaxSteps = 256;            // steps of 16 inputs per workgroup of the streaming contraction
constexpr int64_t kHalfFusedMaxBatch = 64;   // fp16 path: fused kernel up to here, streaming contraction above
constexpr int64_t kFusedTwoTilesMaxBatch = 128;            // ... and up to here (both paths) for layers of at least
constexpr long long kFusedTwoTilesMinEdges = 1ll << 22;    // this many edges whose codeword rows are one gather each
constexpr long long kFusedSmallLayerEdges = 1 << 19;   // fused kernels: layers up to here may write partial sums four times as large as their stream
// Precise path, 2 to 32 samples: calls that fit the static scratch only compact take the tiles of 128 outputs, with their smaller
// partial sums, for launches of more than this many edges.
constexpr long long kFusedTilesCompactMinEdges = 6ll << 20;
constexpr int kFusedMinWgsPerHead = 20;      // fused kernels, several heads: workgroups per head (L2 residency of the codebooks)
// ... of the wave-by-wave kernel's fp16 form from kFusedLargeCodebook on, three of which do not fit an L2 beside each other, where
// the heads' together take half of all L2s: an XCD works on one head at a time.  20 / 40 / 64 workgroups per head, us: twenty of
// 2048-256-21 with 65,536 fp32 rows at batch 40 / 64 156 / 123 / 121, 185 / 147 / 146, fp16 rows 94 / 88 / 88, 105 / 101 / 103,
// 40,000 of them 112 / 103 / 103, thirty of 1000-200-21 fp16 rows at 16 / 40 80 / 75 / 75, 90 / 90 / 81, fifty of 2048-72-21 at 16
// 107 / - / 82.  Smaller codebooks and fewer heads lose (forty of 1748-162-21, 65,536 Int8 rows, at 48 100 / 99 / 109; ten of
// 512-300-40, fp16 rows, at 40 33 / - / 35), but of fp32 rows, whose longer steps do not mind more sums (twenty of 2048-256-21 with
// 15,000 at 40 116 / 113 / 112, 22 of 1280-224-21 with 6,195 87.6 / 93.4 / 82.3; 25 of 512-300-40 at 16 65 / - / 56, at 40
// 74 / - / 77).  What 64 workgroups write may take a call past the static scratch: see plan_head.
constexpr int kFusedOneHeadWgs = 64;
constexpr long long kFusedLargeCodebook = 768 * 1024;
// Precise path: from this batch on the split-operand matrix-core form.  Its time hardly depends on
// the batch below 128 (config 3: 96 us, config 2: 44 us) while the fused fp32 kernel's doubles with
// its second tile of 64 samples (config 3: 97 us at 64, 113 at 80; config 2: 33 and 57).
constexpr int64_t kSplitMinBatch = 65;
// Dense baseline: fp32 operands up to 16 samples (one tile of the fp32 instruction), split operands above.  Three forms for
// these, chosen by what they cost: one pass over the coefficients per tile of 32 or 64 samples (kan_dense.hip), beyond 64 samples the
// contraction that converts its own coefficients for 128 or 256 samples at a time (kan_wide.hip), converted records (kan_mfma.hip).
// One pass / kan_wide / records, us:
//   1024 x 256 at 256 / 300   18.3 / 21.3 / 28.7,  23.2 / 20.7 / 27.5     300 x 64 at 128 / 300   11.3 / 16.2 / -,  11.5 / 19.3 / 24.9
//   500 x 333 at 128 / 300    12.9 / 16.0 / -,     19.6 / 19.1 / 26.2     256 x 500 at 256        13.8 / 17.8 / 28.5
//   2048 x 200 at 128 / 160   20.8 / 20.9 / -,     30.2 / 24.2 / 34.6     2784 x 88 at 194        26.6 / 32.8 / 35.8
//   64 x 2481 at 202          15.7 / 19.2 / 28.2   192 x 64 at 4979       36.2 / 28.5 / 33.2      160 x 1820 at 92  18.7 / 17.7 / 28.0
// kan_wide / records from batch 1024 on, where one pass is left to the smallest layers (two tile steps a CU):
//   2048 x 512 at 1024 / 2048 / 3000 69.4 / 93.7, 122 / 128, 197 / 180; 1024 x 256 at 3000 / 4096 63.3 / 82.5, 79.3 / 84.5; 2048 x 1024 at 1300
//   177 / 171, 4096 x 1024 at 1300 344 / 330; 128 x 2993 at 2601 87 / 64, 352 x 512 at 9186 134 / 107, 192 x 544 at 13,756 91 / 132, 800 x 544 at 2861 87 / 124: what
//   decides is how well the last round of workgroups is filled.
// Layers whose tiles of 64 outputs would be half empty, which make_wide leaves: one pass as long as it is ahead of the records,
// whose time grows from 20 us by 93 a million edges and 12 a million inputs.
constexpr int64_t kDenseSplitMinBatch = 17;
constexpr int64_t kDenseManySamples = 1024;
constexpr long long kDenseOnePassMaxSteps = 512;        // tiles of 64 x 64 times steps of 32 inputs
constexpr long long kDenseWideMaxWork = 1ll << 31;      // edges x samples; records from there (2048 x 1024 at 1300, 4096 x 1024 at 1300, 2048 x 512 at 3000 above)
constexpr long long kDenseSmallSums = 2ll << 20;        // bytes of partial sums that any layer may write
constexpr int64_t kAutoMfmaBatch = 32;    // KAN_PATH_AUTO switches to the matrix cores from here (measured crossover 16-32)

LayerPlan plan_mfma(int n_in, int n_out, int64_t B, int n_heads, int idx_u32, int gb_kind, int code, bool split3 = false,
                    int min_rows = kMfmaMinRows) {
  LayerPlan p;
  p.mfma = true;
  p.kind = kPlanMfma;
  p.name = "kan_mfma";
  p.cfg.jpl = 1;
  p.cfg.wj = 1;
  p.cfg.idx_u32 = idx_u32;
  p.cfg.gb_kind = gb_kind;
  p.cfg.code = code;
  // (finer chunks only as far as the next layer still takes the slices as they are)
  long long max_chunks = n_in / min_rows;
  if (max_chunks > kMaxChainedSlices) max_chunks = std::max<long long>(kMaxChainedSlices, n_in / kMfmaMinRowsCompact);
  // Tiles of 128 outputs by 128 samples (half the coefficient bytes per MFMA through the
  // vector cache), unless their grid would need more than eight chunks of inputs to give
  // every CU two workgroups (64-sample tiles then halve the chunks and with them the
  // partial sums written and read back), or would be padded with many more empty rows.
  p.n_jt = (n_out + kMfmaTileN - 1) / kMfmaTileN;
  const long long big = (long long)n_heads * p.n_jt * ((B + 127) / 128);
  const long long rows128 = (B + 127) / 128 * 128, rows64 = (B + 63) / 64 * 64;     // sample rows the tiles cover
  p.cfg.bt = (big * 8 >= kMfmaTargetWorkgroups && rows128 * 10 <= rows64 * 11) ? 128 : 64;
  p.n_bt = (int)((B + p.cfg.bt - 1) / p.cfg.bt);
  // 128-sample tiles come 256 outputs wide, for one workgroup of eight waves per CU instead of two of four:
  // the eight waves read one Phi tile, so it is built (and its basis words are loaded) once per CU and step, not
  // twice (config 3 at batch 1024: layer 1 43.3 -> 38.2 us, at 4096 139 -> 121.6; config 5 2.22 -> 2.01 ms; the
  // split form at batch 1024 103 -> 89.6 us), unless the wider tiles would pad the outputs by more than an eighth.
  p.tile_n = kMfmaTileN;
  if (p.cfg.bt == 128 && (long long)((n_out + 255) / 256 * 256) * 8 <= (long long)p.n_jt * kMfmaTileN * 9) {
    p.tile_n = 2 * kMfmaTileN;
    p.n_jt = (n_out + p.tile_n - 1) / p.tile_n;
  }
  const long long base = (long long)n_heads * p.n_jt * p.n_bt * (p.tile_n / kMfmaTileN);   // in workgroups of four waves
  long long chunks = kMfmaTargetWorkgroups / (base > 0 ? base : 1);
  // A workgroup that lives for hundreds of steps drifts away from the others of its XCD, which work on
  // the same rows and columns of the operands, by more steps than that XCD's L2 holds: operands are then
  // fetched again and again (config 5 with patches of 8 x 8 tiles and 256 steps: 15 GB for 0.6 GB of
  // operands, L2 hit rate 46 %, 2.56 ms; capped at 128 steps 2.27 ms + 65 us for the reduction).  With the
  // patches of 32 sample tiles x 2 output tiles the kernel uses now (64 workgroups share two slices of the
  // coefficient records, the larger operand) the uncapped form is the faster one: 2.50 against 2.62 ms per
  // step, no partial sums, no reduction.  The cap remains for layers of more than 4096 inputs.
  const long long by_steps = ((n_in + 15) / 16 + kMfmaMaxSteps - 1) / kMfmaMaxSteps;
  if (chunks < by_steps) chunks = by_steps;
  if (chunks > max_chunks) chunks = max_chunks;
  if (chunks < 1) chunks = 1;
  int rows = (int)((n_in + chunks - 1) / chunks);
  rows = (rows + kMfmaRowsStep - 1) / kMfmaRowsStep * kMfmaRowsStep;
  p.rows_per_chunk = rows;
  p.n_chunks = (n_in + rows - 1) / rows;
  if (split3) {
    p.products = 3;
    p.name = "kan_mfma_split";
  }
  return p;
}

// Contraction whose workgroups gather and dequantise their own coefficients (kan_wide.hip): tiles of 64 outputs by 128,
// 256 or 512 samples (256 at most for split operands).  A row of tiles gathers every edge once more, the streaming form
// writes and reads 20 (40) bytes per edge once; times of a layer in us, streaming form (fused kernel's two tiles: *) /
// this one:
//                        batch 128      256         512          768           1024          1536
//   256 x 256   fp16   16.2 / 15.6   15.9 / 16.9   17.8 / 20.3
//   2048 x 256  fp16   20.5 / 20.5   23.7 / 24.4   28.9 / 27.3   30.3 / 35.5
//   2048 x 512  fp16   27.8 / 23.9   30.7 / 24.9   34.5 / 33.3   42.7 / 43.8   45.6 / 49.7
//   2048 x 1024 fp16   37.0 / 27.4   43.3 / 30.6   50.6 / 45.7   64.1 / 65.6   65.0 / 61.7
//   4096 x 1024 fp16   57.7*/ 39.2   69.8 / 44.4   90.6 / 74.0    117 / 113     109 / 105     152 / 152
//   4096 x 4096 fp16    176*/ 111     216 / 124     272 / 170     376 / 305     378 / 313     590 / 529
//   2048 x 512  split  37.4 / 30.6   43.0 / 33.0   56.7 / 47.3   80.0 / 62.5   85.7 / 77.1
//   2048 x 1024 split  59.9 / 37.1   70.7 / 44.3   98.7 / 69.7    136 / 100     125 / 124
//   4096 x 1024 split  88.9*/ 55.5    135 / 70.0    200 / 121     266 / 184     226 / 232     333 / 413
//   4096 x 4096 split   312*/ 169     431 / 212     575 / 400     873 / 687     875 / 792    1501 / 1397
// and with ten heads of 2048-256-21 at batch 128 114 / 61 (fp16), 206 / 87 (split).  The lines are drawn through this table,
// where one size gains and the next loses on their far side.
// Beyond them it is ahead for single heads of one- and two-byte codebook rows (parameters from the memory-side cache):
//   - batch 513 to 900, more than 512 outputs, fp16, at 520 / 640 / 768 / 900: 1024 x 1024 36.2 / 39.2 / 41.0 / 45.0 against
//     34.1 / 35.0 / 36.2 / 38.0, 2048 x 1024 58.8 / 62.8 / 67.3 / 66.6 against 52.0 / 53.3 / 55.3 / 58.8, 1500 x 1100
//     79.9 / 80.5 / 61.0 / 86.0 against 46.5 / 47.6 / 50.3 / 53.1 (kan_mfma.hip pads 1100 outputs to 1280), 1900 x 1100 at 900
//     101.6 against 62.0; fp32 rows 2048 x 1024 at 1024 74.8 against 75.8;
//   - up to batch 1024 where the next layer adds the slices (2048-1024-256 at 640 / 1024 83.0 / 90.9 against 79.8 / 87.6).  From
//     there to batch 1500 it is 9 to 23 % behind where the records' tiles of 256 outputs are full (900 to 1024, 1281 to 1536 and 1793
//     to 2048 outputs, by 14 % at most on average, 11 % ahead elsewhere), so the line stays;
//   - layers of 2^18 edges with 512 outputs and more, up to batch 256 fp16 and 768 split: 512 x 512 fp16 at 80 / 256 / 400
//     16.0 / 17.6 / 20.1 against 14.6 / 16.9 / 20.7, split at 80 / 256 / 700 21.2 / 22.9 / 31.4 against 18.3 / 21.5 / 27.9, 1024 x 512
//     fp16 at 80 / 256 19.6 / 22.1 against 17.3 / 19.1, split at 256 / 700 30.6 / 45.9 against 24.2 / 37.9, 700 x 900 split at 128 / 512
//     31.8 / 44.0 against 21.0 / 34.8, 300 x 1000 split at 80 / 700 25.9 / 34.8 against 19.2 / 29.1.  Layers of few outputs
//     for their inputs lose (2048 x 128 split at 400 29.7 against 32.3, fp16 21.4 against 25.5), smaller ones gain 1 to 5 %;
//     fp16 ones that take a layer's slices lose, their records being written beside the first layer's (2048-700-512-30 at 250
//     58.1 against 60.1).
// Above these batches the sizes disagree again (fp16 at 1536 2048 x 1024 87.6 / 86.3, at 2048 100 / 105.5; 4096 x 1024 at 1200 134 /
// 141; split at 1536 2048 x 1024 176 / 195).
constexpr long long kWideMinEdges = 1ll << 20;        // over the heads of a launch
constexpr int64_t kWideMinBatch = 65, kWideMaxBatchHalf = 512, kWideMaxBatchHalfLarge = 1024, kWideMaxBatchSplit = 768;
constexpr long long kWideLargeEdges = 1ll << 22;      // ... for kWideMaxBatchHalfLarge
constexpr int64_t kWideMaxBatchHalfManyOut = 900;     // ... above kWideManyOut outputs
constexpr int kWideManyOut = 512;
constexpr long long kWideSmallEdges = 1ll << 18;      // from kWideManyOut outputs on
constexpr int64_t kWideSmallMaxBatchHalf = 256;

// Largest batch at which that kernel is the faster one, 0: at none.
int64_t wide_max_batch(int n_in, int n_out, int n_heads, int code, bool split3, int x_parts, bool reduced) {
  const long long edges = (long long)n_in * n_out * n_heads;
  const bool beyond = n_heads == 1 && code != kCbF32;
  if (edges < kWideMinEdges)
    return !beyond || edges < kWideSmallEdges || n_out < kWideManyOut ? 0 : (split3 ? kWideMaxBatchSplit : (x_parts > 1 ? 0 : kWideSmallMaxBatchHalf));
  if (split3) return kWideMaxBatchSplit;
  if (edges >= kWideLargeEdges || (beyond && !reduced)) return kWideMaxBatchHalfLarge;
  return beyond && n_out > kWideManyOut ? kWideMaxBatchHalfManyOut : kWideMaxBatchHalf;
}

// Turns plan p of such a layer into one for that kernel where it is the faster one.
bool make_wide(LayerPlan& p, int n_in, int n_out, int64_t B, int n_heads, bool split3, int x_parts, bool reduced) {
  const bool dense = p.cfg.code == kDense;
  if (!dense && (B < kWideMinBatch || B > wide_max_batch(n_in, n_out, n_heads, p.cfg.code, split3, x_parts, reduced))) return false;
  if (!wide_takes(n_in, n_out, B, dense)) return false;
  const int n_jt = (n_out + kWideTileN - 1) / kWideTileN;
  if ((long long)n_jt * kWideTileN * 2 > 3ll * n_out) return false;        // (tiles half empty)
  const int tile = B <= 128 ? 128 : (B <= 256 || split3 ? 256 : 512), n_bt = (int)((B + tile - 1) / tile);
  // Chunks of inputs: the fewest rounds of one workgroup per CU.  In units of a step (about 2 us): what a workgroup takes
  // outside its steps is about five, the partial sums cost 8 bytes per chunk, sample and output at 4 TB/s.
  const long long base = (long long)n_heads * n_jt * n_bt, steps = (n_in + 15) / 16;
  long long best = 1;
  double best_cost = 0.0;
  for (long long c = 1; c <= kMaxChainedSlices && (c == 1 || c * 2 <= steps); ++c) {
    const double rounds = (double)((base * c + 255) / 256);
    const double cost = rounds * ((double)((steps + c - 1) / c) + 5.0) + (c > 1 ? 1e-6 * (double)(c * n_heads * B * n_out) : 0.0);
    if (c == 1 || cost < best_cost) {
      best = c;
      best_cost = cost;
    }
  }
  p.kind = kPlanMfma;
  p.mfma = true;
  p.wide = true;
  p.name = split3 ? "kan_wide_split" : "kan_wide";
  p.products = split3 ? 3 : 1;
  p.cfg.bt = tile;
  p.tile_n = kWideTileN;
  p.n_jt = n_jt;
  p.n_bt = n_bt;
  p.rows_per_chunk = (int)((steps + best - 1) / best) * 16;
  p.n_chunks = (n_in + p.rows_per_chunk - 1) / p.rows_per_chunk;
  return true;
}

// Large contractions on tiles of 256 x 256 with both operands copied to LDS by the memory pipeline (kan_stream.hip), in
// place of the tiles of kan_mfma.hip.  The line is the work, in tiles times steps of 16 inputs: a workgroup is alone on its
// CU and its partial sums are 256 KB.  Layer times in us, kan_mfma.hip / this:
//                        batch 1024      1536         2048         3072         4096         8192
//   1024 x 512  fp16                                 41 / 46      49 / 56      58 / 66      98 / 105   (256 .. 4,096 tile-steps)
//   2048 x 1024 fp16     66 / 78      84 / 86      98 / 101     135 / 128    162 / 158    279 / 274   (2,048 .. 16,384)
//   4096 x 1024 fp16                 155 / 150    182 / 172     254 / 231    317 / 290    572 / 519   (6,144 at 1536)
//   512 x 4096  fp16                  79 / 79      80 / 85      123 / 104    139 / 123    256 / 220   (6,144 at 3072)
//   4096 x 4096 fp16                 597 / 469    600 / 518     992 / 765   1076 / 864   1965 / 1589
//   2048 x 1024 split   136 / 160    176 / 176    211 / 205     319 / 283                             (6,144 at 3072)
//   4096 x 4096 split   886 / 766   1511 / 1123  1494 / 1287   2639 / 1973
constexpr long long kStreamMinTileSteps = 6144;
constexpr int kStreamMinOut = 513;                  // (two tiles across: 1024 x 512 is slower up to batch 8192)

bool make_stream(LayerPlan& p, int n_in, int n_out, int64_t B, int n_heads, bool split3) {
  if (n_out < kStreamMinOut || !stream_takes(n_out, B)) return false;
  const int n_jt = (n_out + kStreamTile - 1) / kStreamTile, n_bt = (int)((B + kStreamTile - 1) / kStreamTile);
  if ((long long)n_jt * kStreamTile * 8 > 9ll * n_out) return false;            // (tiles an eighth empty)
  if ((long long)n_jt * n_bt * n_heads * ((n_in + 15) / 16) < kStreamMinTileSteps) return false;
  const long long base = (long long)n_heads * n_jt * n_bt, steps = (n_in + 15) / 16;
  long long best = 1;
  double best_cost = 0.0;
  for (long long c = 1; c <= kMaxChainedSlices && (c == 1 || c * 4 <= steps); ++c) {
    const double rounds = (double)((base * c + 255) / 256);
    const double cost = rounds * ((double)((steps + c - 1) / c) + 5.0) + (c > 1 ? 1e-6 * (double)(c * n_heads * B * n_out) : 0.0);
    if (c == 1 || cost < best_cost) {
      best = c;
      best_cost = cost;
    }
  }
  p.stream = true;
  p.name = split3 ? "kan_stream_split" : "kan_stream";
  p.cfg.bt = kStreamTile;
  p.tile_n = kStreamTile;
  p.n_jt = n_jt;
  p.n_bt = n_bt;
  p.rows_per_chunk = (int)(((steps + best - 1) / best * 16 + kMfmaPrepRows - 1) / kMfmaPrepRows * kMfmaPrepRows);
  p.n_chunks = (n_in + p.rows_per_chunk - 1) / p.rows_per_chunk;
  return true;
}

// Small layers take one launch (kan_tail.hip) in place of basis words, contraction and reduction.  A workgroup
// evaluates the basis of all inputs for its 32 samples and reads the records of its outputs, so the line is where
// that takes longer than the launches it saves: kTailMaxIn inputs (416-32 at batch 1166 17.9 -> 14.6 us, 475-52-13 at
// 65 25.2 -> 26.6 without the limit), 32,768 edges (318-192-108 at batch 474 30.8 -> 25.5 us, 128-256 at
// 225 16.4 -> 12.0; 8 or 16 thousand lose half of that), eight workgroups per CU (288-38-19 at batch 6842 34.6 ->
// 21.8 us, with four 29.5), and 4,096 slices x inputs to add (2,048 where three or more output tiles add them again):
// 1696-224-15 at batch 315 (26 slices) 39.3 -> 43.5 us, 800-159-147 at 137 (25 slices) 33.9 -> 38.8 without it.
// Tiles of 32 outputs, of 64 once those of 32 would be more than one per CU (the basis is then evaluated once for both).
constexpr long long kTailMaxEdges = 32768;
constexpr long long kTailMaxWorkgroups = 2048;
constexpr long long kTailSlicedInputs = 4096, kTailSlicedInputsManyTiles = 2048;

// x_parts: slices the layer's input may come in.
LayerPlan plan_matrix(int n_in, int n_out, int64_t B, int n_heads, int idx_u32, int gb_kind, int code, bool split3,
                      int x_parts, int min_rows, bool wide, bool reduced) {
  LayerPlan p = plan_mfma(n_in, n_out, B, n_heads, idx_u32, gb_kind, code, split3, min_rows);
  const long long n_bt = (B + 31) / 32;
  const int tile_n = split3 || n_out <= 32 || (n_out + 31) / 32 * n_bt * n_heads <= 256 ? 32 : 64;
  const long long n_jt = (n_out + tile_n - 1) / tile_n;
  if (n_in > kTailMaxIn || (long long)n_in * n_out > kTailMaxEdges || n_jt * n_bt * n_heads > kTailMaxWorkgroups ||
      (x_parts > 1 && (long long)x_parts * n_in > (n_jt > 2 ? kTailSlicedInputsManyTiles : kTailSlicedInputs))) {
    if (wide && !make_wide(p, n_in, n_out, B, n_heads, split3, x_parts, reduced)) make_stream(p, n_in, n_out, B, n_heads, split3);
    return p;
  }
  p.kind = kPlanTail;
  p.cfg.bt = 32;
  p.tile_n = tile_n;
  p.n_jt = (int)n_jt;
  p.n_bt = (int)n_bt;
  p.n_chunks = 1;
  p.rows_per_chunk = n_in;
  return p;
}

// Fused gather + matrix-core kernel: batch tiles of 32 (B <= 32) or 64 samples, output tiles
// of 128.  With one batch tile every edge is gathered once and the work is bound by the
// gather rate of the CUs' address units, so every CU should be busy: i is split while the
// partial sums stay below the size of the parameter stream.
// compact: the smaller partial sums of the first count of chunks, for calls that fit the static scratch only so.
// reduced: nobody but a launch of kan_reduce adds the slices (the last layer, or one whose successor does not take them).
// The launch and its pass over the sums are then part of what a cut costs; in the units of cost_of below:
constexpr double kFusedReduceSteps = 1.0, kFusedReduceStepsHalf = 2.8;
LayerPlan plan_fused(int n_in, int n_out, int64_t B, int n_heads, int idx_u32, int gb_kind, int code, bool f32, bool compact,
                     bool reduced) {
  LayerPlan p;
  p.mfma = false;
  p.kind = f32 ? kPlanFused32 : kPlanFused16;
  p.name = f32 ? "kan_fused_f32" : "kan_fused_f16";
  p.cfg.bt = B <= 32 ? 32 : 64;
  p.cfg.jpl = 1;
  p.cfg.wj = 4;
  p.cfg.idx_u32 = idx_u32;
  p.cfg.gb_kind = gb_kind;
  p.cfg.code = code;
  p.n_jt = (n_out + kFusedTileN - 1) / kFusedTileN;
  p.n_bt = (int)((B + p.cfg.bt - 1) / p.cfg.bt);
  const int bytes_per_edge = (idx_u32 ? 4 : 2) + 2 * gb_bytes(gb_kind);
  const long long base = (long long)n_heads * p.n_jt * p.n_bt;
  // (64-sample tiles: with a workgroup per CU and twice the steps each, the metadata of the next
  // steps is in flight behind the gathers of the current one: config 3 at batch 64 57.8 -> 51.1 us
  // on the fp16 path, 96.7 -> 82.9 us on the precise path; 32-sample tiles are better off with two)
  // Two per CU again where the chunks stay long even so: at least 8 steps each for the precise form
  // (4096 x 4096 with K = 262,144 at batch 64: 338 -> 249 us; 4096 x 1024: 67.6 -> 56.5; 2048 x 2048:
  // 65.6 -> 56.2; 8192 x 512: 67.6 -> 60.4), at least 16 for the fp16 form (4096 x 4096: 124 -> 119 us;
  // with 8 steps each it loses: 4096 x 1024 37.8 -> 42 us, 2048 x 2048 36.8 -> 40).
  long long target = p.cfg.bt == 64 ? kTargetWorkgroups / 2 : kTargetWorkgroups;
  if (p.cfg.bt == 64 && (long long)(n_in / 8) * base >= (f32 ? 16 : 32) * target) target *= 2;
  long long chunks = (target + base - 1) / (base > 0 ? base : 1);
  // Several heads in one launch: the kernel gives every XCD a contiguous run of heads, and an XCD
  // (64 resident workgroups) should work on at most two or three heads at a time so that their
  // codebooks stay in its L2: at least kFusedMinWgsPerHead workgroups per head.
  // (layers whose whole codebook traffic is small gain nothing from it: their workgroups would
  // only get shorter)
  long long resident = 1;
  if (n_heads > 1 && (long long)n_in * n_out >= kFusedMinEdgesForResidency) {
    const long long per_head = (long long)p.n_jt * p.n_bt;
    resident = (kFusedMinWgsPerHead + per_head - 1) / per_head;
    if (chunks < resident) chunks = resident;
  }
  // At least two steps each; the precise form, whose steps are longer, takes single ones up to kMaxChainedSlices of
  // them, with a reduction behind them too (500-128-64-10 at batch 37, every layer reduced, 43.5 -> 37 us; in the fp16
  // form 4096 x 64 at batch 24 loses, 11.4 -> 13.4).
  // (rounded down, which leaves chunks of three steps, where a reduction follows: 1000-333-21 fp16 at batch 37 26.4 us, 26.6
  // with more slices; 22.7 against 26.2 at batch 24, whose next layer adds them itself)
  long long max_by_rows = compact || (!f32 && p.cfg.bt == 64) ? n_in / 16 : (n_in + 15) / 16;
  if (f32 && !compact) max_by_rows = std::max(max_by_rows, std::min<long long>((n_in + 7) / 8, kMaxChainedSlices));
  // Partial sums up to the size of the parameter stream (n_in * bytes_per_edge / 4 B chunks of 4 B bytes per output) -
  // up to four times that for small layers, whose launch is a latency chain and not a stream: capped at the stream's
  // size, config 3's second layer (262,144 edges) ran on 48 workgroups at batch 64 and took 17-28 us; with four times it runs on 128 and takes
  // 12.5-14.7 us (the head at batch 32 / 48 / 64: 39.9 / 57.5 / 60.0 against 46.7 / 62.8 / 71.5 us precise, 30.3 /
  // 41.0 / 43.8 against 36.9 / 43.5 / 47.6 us fp16; at batch 32 its chunks also become short enough to take the
  // first layer's partial sums as they are).  Layers of a million edges and more gain nothing from it.
  const long long max_by_bytes =
      (long long)n_in * bytes_per_edge / ((long long)n_in * n_out <= kFusedSmallLayerEdges ? B : 4 * B);
  if (chunks > max_by_rows) chunks = max_by_rows;
  if (chunks > max_by_bytes) chunks = max_by_bytes;
  if (chunks < 1) chunks = 1;
  // A few workgroups more than the CUs hold in whole rounds: the fullest CU then has a round of long chunks for itself
  // (ten heads of 2048-256-21 at batch 64 on 260 workgroups of 20 steps: 72.6 us fp16, 105.4 precise; on 500 of 11 59.1
  // and 86.4).  Cost as for the wave-by-wave kernel below: steps on the fullest CU, and the partial sums.
  const int steps = (n_in + 7) / 8;
  const auto cost_of = [&](int per) {
    const long long wgs = base * ((steps + per - 1) / per);
    return per * std::max((double)((wgs + kCUs - 1) / kCUs), 1.5) + 1.28e-4 * (double)(wgs * p.cfg.bt);
  };
  int per = (int)((steps + chunks - 1) / chunks);
  const int planned = per;
  const long long wgs = base * ((steps + per - 1) / per), rounds = (wgs + kCUs - 1) / kCUs;
  if (!compact && rounds > 1 && rounds * kCUs * 8 > wgs * 9) {
    const long long most = std::min(max_by_rows, max_by_bytes);
    for (long long r = rounds - 1; r <= 2 * rounds; ++r) {
      const long long want = r * kCUs / base;
      if (want < resident || want > most) continue;
      const int other = (int)((steps + want - 1) / want);
      if (cost_of(other) < cost_of(per) && cost_of(other) < 0.9 * cost_of(planned)) per = other;
    }
  }
  // A cut that only a reduction launch undoes, against none (whole us, one chunk / cut):
  //   precise  24 x 21 at batch 37 10.9 / 7.9,  26 x 684, 12 heads, at 34 14.5 / 12.5,  25 x 217, 8 heads, at 40 14.3 / 11.5,
  //            31 x 3724, 7 heads, at 48 15.8 / 21.3,  21 x 303, 39 heads, at 54 12.1 / 15.7,  73 x 1749, 21 heads, at 45 45.9 / 49.9
  //   fp16     24 x 128 at 16 5.3 / 6.1,  25 x 727 at 31 7.4 / 6.9,  31 x 327, 35 heads, at 30 8.0 / 9.1,
  //            30 x 3297, 8 heads, at 10 8.0 / 9.9,  147 x 866, 46 heads, at 36 37.5 / 44.4
  if (!compact && reduced && resident == 1 && per < steps) {
    const auto sums = [&](int q) { return 1.28e-4 * (double)(n_heads * (long long)p.n_jt * ((steps + q - 1) / q) * B); };
    const auto work = [&](int q) { return q * std::max((double)((base * ((steps + q - 1) / q) + kCUs - 1) / kCUs), 1.5); };
    const double whole = work(steps) + sums(steps), cut = work(per) + 2 * sums(per) + (f32 ? kFusedReduceSteps : kFusedReduceStepsHalf);
    if (cut >= (planned == steps ? 0.9 : 1.0) * whole) per = steps;       // (0.9: as for the choice of rounds above)
  }
  p.rows_per_chunk = 8 * per;
  p.n_chunks = (steps + per - 1) / per;
  return p;
}

// Precise path up to 32 samples: tiles of 64 outputs, the four waves of a workgroup over its inputs.  The chunk's
// steps of 16 inputs are chosen by what they cost, in steps of a busy CU (1 us, its address units bound): the fullest
// CU's workgroups times their steps (a lone workgroup's step takes as long as 1.75: latencies without a neighbour
// behind them), and the partial sums, written here and read by the next layer or the reduction.  Filling the chip with
// at least 512 workgroups of two steps or more, as before, left one CU with three workgroups of ten steps where
// 520 were launched (ten heads of 2048-256-21 at batch 4 / 16 / 32: 54.6 / 55.5 / 75 us, now 41.6 / 46.0 / 59.3;
// twenty of 1024-128-50 at 16 38.7 -> 30.5), and small layers with a second step that takes longer than
// the slices it saves (64-32 at batch 16 7.5 -> 6.5 on the GPU - the call is bound by the host, 9.6 before and after -,
// 1000-333-21 24.3 -> 20.9, 2048-1024-256 at batch 4 28.2 -> 26.7).
// Not more chunks than the next layer takes as they are, unless two steps each would be too many already; chunks of a
// single step for up to kFusedWaveStepBytes of partial sums, beyond which a caller's workspace would grow with them.
// (Eight waves to a workgroup for half the slices: 2048-1024-256 at batch 16 30.2 against 28.6 us.)
// compact: the smaller partial sums of the former rule, for calls that fit the static scratch only so.  spare: one chunk where the
// cut saves less than a tenth, likewise.
// reduced: nobody but a launch of kan_reduce adds the slices (as in plan_fused).  The launch takes about 2.7 us, in units
// of the cost above: 3.3 where a CU has one workgroup, of 16 samples at most, 2.0 with the longer steps of more samples, 1.3
// where one chunk is several rounds of workgroups.  One chunk / cut, us: 32 x 128 at batch 4 / 16 / 31 4.7 / 5.4, 4.8 / 5.7,
// 6.6 / 6.8, 48 x 128 6.3 / 5.5, 6.5 / 5.7, 9.2 / 6.8; several heads: 34 x 387, 13 of them, at 16 7.2 / 8.0; 38 x 1139, 8, at 4
// 6.9 / 7.8; 48 x 512, 20, at 16 6.8 / 9.6; 64 x 669, 21, at 8 8.0 / 9.9; 82 x 2736, 19, at 24 46.0 / 47.2; 72 x 385, 47, at 5
// 14.9 / 13.9; 97 x 1650, 13, at 8 19.0 / 18.0.
constexpr long long kFusedWaveStepBytes = 512 * 1024;
LayerPlan plan_fused_wave(int n_in, int n_out, int64_t B, int n_heads, int idx_u32, int gb_kind, int code, long long cb_bytes, int large_wgs, bool half, bool compact,
                          bool reduced, bool spare) {
  LayerPlan p;
  p.mfma = false;
  p.kind = kPlanFusedWave;
  p.half = half;
  p.name = half ? "kan_fused_wave_f16" : "kan_fused_wave";
  p.cfg = GatherCfg{32, 1, 1, idx_u32, gb_kind, code};
  p.n_jt = (n_out + kFusedWaveCols - 1) / kFusedWaveCols;
  p.n_bt = 1;
  const int bytes_per_edge = (idx_u32 ? 4 : 2) + 2 * gb_bytes(gb_kind);
  const long long base = (long long)n_heads * p.n_jt;
  const int steps = (n_in + kFusedWaveStep - 1) / kFusedWaveStep;
  // partial sums up to the size of the parameter stream (four times that for small layers, as above)
  const long long max_by_bytes =
      (long long)n_in * bytes_per_edge / ((long long)n_in * n_out <= kFusedSmallLayerEdges ? B : 4 * B);
  long long max_by_count = steps > 2 * kFusedChainMaxParts ? steps : kFusedChainMaxParts;
  if ((long long)steps * n_heads * B * n_out * 4 > kFusedWaveStepBytes) max_by_count = std::min<long long>(max_by_count, (steps + 1) / 2);
  if (compact) max_by_count = std::min<long long>(n_in / (2 * kFusedWaveStep), (kTargetWorkgroups + base - 1) / base);
  const long long most = std::max(1ll, std::min({max_by_count, max_by_bytes, (long long)steps}));
  const double reduction = !reduced ? 0.0 : (base > kCUs ? 1.3 : (B > 16 ? 2.0 : 3.3));
  // Several heads, fp16 form: an XCD works on two or three at a time, as in plan_fused (2048-65-21 at batch 64, forty heads
  // 95.8 -> 82.1 us, fifty 114.5 -> 109.8; 2048-128-21 at 24, fifty 97.4 -> 89.6; fifty of 1024-128-21 at 64 lose, 71 -> 75).
  // The precise form gains at batch 8 and loses at 24 (fifty of 2048-65-21 93.9 -> 89.7, 120 -> 123).
  p.one_head = code == kCbF32 || (cb_bytes > kFusedLargeCodebook && n_heads * cb_bytes > 4 * kL2Bytes);
  const int head_wgs = p.one_head ? large_wgs : kFusedMinWgsPerHead;
  const bool by_head = half && !compact && n_heads > 1 && (long long)n_in * n_out > kFusedMinEdgesForResidency;
  const long long resident = by_head ? std::min<long long>(most, (head_wgs + p.n_jt - 1) / p.n_jt) : 1;
  p.one_head = p.one_head && by_head;
  // A workgroup for more than half of the CUs and none with two: a cut that a reduction launch undoes for a tenth at least, as in
  // plan_fused.  Mean time of one chunk over that of the cut (2,592 launches) with 64 to 95 / 96 / 128 / 160 / 192 / 224 to 256 / 257 / 288 /
  // 320 / 352 / 384 and more workgroups: 1.01 / 0.98 / 0.88 / 0.86 / 0.84 / 0.85 / 1.09 / 1.07 / 1.06 / 1.05 / 1.09; with two and three of them - the last layers of
  // single heads - 1.1 to 1.2 (271-48-152, fp32 rows, at batch 13 18.7 / 15.5 us, 160-44-96 at 5 17.3 / 14.7).
  const bool whole_line = reduced && (spare || (2 * base > kCUs && base <= kCUs));
  double least = 0;
  for (int per_cu = 0; per_cu <= 8; ++per_cu) {          // one chunk; the fewest steps with at most so many workgroups on a CU
    const long long want = compact ? most : std::clamp<long long>((long long)per_cu * kCUs / base, resident, most);
    const int per = (int)((steps + want - 1) / want), chunks = (steps + per - 1) / per;
    const long long wgs = base * chunks;
    const double cost = per * std::max((double)((wgs + kCUs - 1) / kCUs), 1.75) + 1.28e-4 * (double)(wgs * B) +
                        (chunks > 1 ? reduction : 0.0);
    if (least > 0 && cost >= (whole_line && p.n_chunks == 1 ? 0.9 : 1.0) * least) continue;
    least = cost;
    p.rows_per_chunk = per * kFusedWaveStep;
    p.n_chunks = chunks;
  }
  return p;
}

// Which of the two fused kernels a layer of up to 64 samples takes: the wave-by-wave kernel is ahead in short chains, the one on tiles of
// 128 outputs, whose waves share a step's basis and ask for twice the run of a row at once, where its workgroups have many
// steps - from how many on depends on storage types, 16-byte metadata loads (outputs in sixteens) and blocks of 16 samples -
// and the fullest CU has about the same to do.  Lines drawn through 32,492 launches on the fp16 path and 22,878 on the precise one
// (2^18 to 24 * 2^20 edges, one to fifty heads) by the sum of the logarithms of tiles / wave by wave from a line on.
// What the fullest CU has to do, missing outputs included, in steps of 1024 edges (8 x 128 or 16 x 64).
long long fullest_cu(const LayerPlan& p, int n_heads) {
  const long long wgs = (long long)n_heads * p.n_jt * p.n_bt * p.n_chunks;
  return (wgs + kCUs - 1) / kCUs * (p.rows_per_chunk / (p.kind == kPlanFusedWave ? kFusedWaveStep : 8));
}
// (1.02 / 1.06 / 1.1 / 1.2 / 1.3: sums of -131 / -142 / -144 / -141 / -138 on the fp16 path, -16.2 / -16.7 / -15.7 / -13.8 / -13.7 on the precise one)
bool tiles_fill(const LayerPlan& tiles, const LayerPlan& wave, int n_heads) { return fullest_cu(tiles, n_heads) * 12 <= fullest_cu(wave, n_heads) * 13; }
constexpr long long kFusedSmallCodebook = 16 * 1024;      // stays in the vector caches, where the wave-by-wave kernel's gathers cost least (tiles 1.1 - 1.4; at 49 to 64 samples no line: two-byte gains 0.87 - 0.95)

// Precise path, 2 to 32 samples.  Mean time of the tiles over that of the wave-by-wave kernel from the line on, parameters from
// memory / from the caches, one head, two-byte gains, outputs in sixteens:
//   one-byte rows, 32-bit ids    2-16 samples 0.96 / 0.96, 17-32 0.96 / 0.95
//   one-byte rows, 16-bit ids    2-16 0.89 / -, 17-32 0.97 / 1.01;   fp16 rows 2-16 0.89 / 1.08;   fp32 rows 2-16 0.97 / 0.97
// Elsewhere: several heads 0.98 - 1.06 / 1.15, fp32 gains 1.16 / 1.25, one-byte gains 1.04 / 1.10, fp32 rows 1.03 / 1.05, outputs in other
// than sixteens 1.13 - 1.4, half-empty tiles 1.3 - 2.  For instance, us, tiles / wave by wave: 7848 x 1536, fp16 rows, at batch 16 84 / 100,
// 4096 x 2048 with fp32 gains at 4 / 32 70.8 / 62.3, 90.2 / 74.2, 3072 x 2200 at 16 65.9 / 56.3, 2600 x 2500 62.5 / 54.4, forty heads of 1748-97-21
// 77.3 / 60.3.
bool precise_tiles_ahead(int n_out, int64_t B, int n_heads, int idx_u32, int gb_kind, int code, long long cb_bytes, const LayerPlan& tiles, const LayerPlan& wave) {
  if (n_heads > 1 || gb_kind != kGbF16 || n_out % 16 != 0 || cb_bytes < kFusedSmallCodebook || !tiles_fill(tiles, wave, n_heads)) return false;
  const int steps = tiles.rows_per_chunk / 8;
  if (code == kCbF16 || code == kCbF32) return !idx_u32 && B <= 16 && steps >= 12;
  return steps >= (idx_u32 ? 5 : (B > 16 ? 10 : 31));
}

// fp16 path up to 64 samples: least steps of the tiles, 0: never.  Mean ratios as above:
//   one head, two-byte gains, one-byte rows   1-16 samples 0.91 / 0.92 (32-bit ids)      17-32 0.86 / 1.06, 0.90 / 0.89 (32-bit)
//                                             33-48 0.86 / 1.04, 0.93 / 0.89 (32-bit)    49-64 0.86 / 0.99, 0.92 / 0.89 (32-bit)
//   several heads, likewise                   17-32 0.88 / 1.06    33-48 0.85 / 1.01     49-64 0.80 / 0.95
//   four-byte gains                           33-48 0.93 / 0.90 (32-bit)                 49-64 0.86 / 1.08, 0.85 / 0.87 (32-bit)
//   fp16 rows, two-byte gains, one head       1-16 0.83 / 1.06     17-32 0.81 / 1.02     33-48 0.82 / 1.03     49-64 0.85 / 1.01, several 0.84 / 1.05
//   fp32 rows                                 1-16 0.95 / 0.95, 17-32 0.88 / 0.86 (two-byte gains, 16-bit ids)   49-64 0.96 / 0.94, fp32 gains 0.88 / 0.87
// One-byte gains never gain.  fp32 rows of several heads that do not fit the L2s of all XCDs together: the wave-by-wave kernel takes these
// heads one at a time (tiles 1.09 - 1.32).  fp32 rows on 65 to 96 outputs: it fetches for the lanes past the last output as well
// (tiles 0.53 - 0.95, these heads included).  The line before - 49 samples and more, from 2^20 edges, on whole tiles, and one case of 32-bit
// ids - took 30 % of the launches of more than 3 * 2^20 edges with parameters from memory more than 3 % longer than the tiles and 9 % of
// those from the caches, this one 16 and 3.5 % (1.2 and 5.4 % longer than wave by wave).  For instance, us, tiles / wave by wave: 8192 x 1760 at batch 17
// 66 / 87, 4712 x 3200, fp16 rows, at 64 105 / 145, 4096 x 4096, fp32 gains, 32-bit ids, at 64 126 / 146, 4096 x 4095 at 8 116 / 127,
// nine heads of 8192 x 65, fp32 rows, at 64 81 / 128; 1000-333-21 at 37 25.7 / 19.7, 2048-1024-256 at 16 / 48 28.7 / 25.6, 39.5 / 33.8,
// 931-128-50, four heads, at 36 27.6 / 17.7.
int half_tiles_min_steps(int n_out, int64_t B, int n_heads, int idx_u32, int gb_kind, int code, long long cb_bytes) {
  const bool bytes = code == kCbI8 || code == kCbBfp8, sixteens = n_out % 16 == 0, one = n_heads == 1;
  const int blocks = (int)((B + 15) / 16);
  const bool ids32 = idx_u32 && one;       // (several heads as with 16-bit ids: ten of 2048-256 at batch 8 / 48 48 / 38, 61 / 53 us)
  if (gb_kind == kGbQ8 || (cb_bytes < kFusedSmallCodebook && !(blocks == 4 && gb_kind == kGbF16))) return 0;
  if (code == kCbF32) {
    if (n_out > 64 && n_out <= 96) return 6;
    if (!one && n_heads * cb_bytes > 8 * kL2Bytes) return 0;
    if (blocks == 4) return 5;
    if (blocks == 3 || gb_kind == kGbF32 || idx_u32) return 0;
    if (blocks == 2) return sixteens ? 5 : (one ? 9 : 0);
    return one && sixteens ? 6 : 0;
  }
  if (gb_kind == kGbF32) {
    if (!bytes || (blocks < 4 && !ids32)) return 0;
    if (blocks == 4) return ids32 ? (sixteens ? 9 : 4) : (sixteens || one ? 14 : 5);
    return blocks == 3 ? 17 : 0;
  }
  if (!bytes) return idx_u32 || !sixteens ? 0 : (blocks == 4 ? 12 : (one ? 15 : 0));
  if (blocks == 4) return sixteens ? 9 : (one ? (ids32 ? 4 : 9) : 22);
  if (ids32) return blocks == 3 ? (sixteens ? 19 : 16) : (sixteens ? 5 : 12);
  return sixteens && blocks > 1 ? 12 : 0;
}
bool half_tiles_ahead(int n_out, int64_t B, int n_heads, int idx_u32, int gb_kind, int code, long long cb_bytes, const LayerPlan& tiles, const LayerPlan& wave) {
  const int least = half_tiles_min_steps(n_out, B, n_heads, idx_u32, gb_kind, code, cb_bytes);
  return least > 0 && tiles.rows_per_chunk >= 8 * least && tiles_fill(tiles, wave, n_heads);
}
// ... and by so much that a call is not moved off the tiles to fit the static scratch: 49 samples and more, workgroups of half the
// columns each that fill nine tenths of the CUs' rounds (of fp32 rows three quarters), 2^20 edges in one head or 6 * 2^20 in several (us,
// tiles / wave by wave: fifty heads of 2048-256-21 191 / 204, of 2048-65-21 95 / 110, fp32 rows 2048 x 2048 52 / 58).
bool half_tiles_far_ahead(int n_out, int64_t B, int n_heads, int gb_kind, int code, const LayerPlan& tiles, long long edges) {
  const long long wgs = (long long)n_heads * tiles.n_jt * tiles.n_bt * tiles.n_chunks, slots = (wgs + kCUs - 1) / kCUs * kCUs;
  const bool even = (n_out + 63) / 64 == 2 * ((n_out + 127) / 128), large = n_heads == 1 ? edges >= 1 << 20 : edges * n_heads > 6 << 20;
  if (B <= 48 || !even || !large) return false;
  return code == kCbF32 ? wgs * 4 >= slots * 3 : gb_kind == kGbF16 && code != kCbF16 && wgs * 10 >= slots * 9;
}

// Bucket path (prepared layers): one workgroup per (bucket, slice of the outputs, sample).
// A workgroup occupies a whole CU (LDS), so the slices are cut to give every CU one: the
// cuts come from the block table that the preparation made for this many (samples x heads).
constexpr int64_t kBucketMaxBatch = 4;
// A pass over the records per sample costs in proportion to the edges, the fused kernel's single pass for up to
// 16 samples does not: on the largest layers the fourth sample tips it (4096 x 4096, K = 262,144, batch 2 / 3 / 4:
// 61 / 89 / 117 us against 105-109 us fused; 4096 x 1024 and 2048 x 2048: 21 / 28 / 30-31 against 33-35 us).
constexpr long long kBucketThreeSamplesMinEdges = 1ll << 23;
constexpr int64_t bucket_max_batch(long long edges) { return edges >= kBucketThreeSamplesMinEdges ? 3 : kBucketMaxBatch; }

LayerPlan plan_bucket(const kan_vq_layer& L, int64_t B, int n_heads) {
  LayerPlan p;
  p.mfma = false;
  p.kind = kPlanBucket;
  p.name = "kan_bucket";
  p.cfg.bt = 1;
  p.cfg.jpl = 1;
  p.cfg.wj = 1;
  p.cfg.idx_u32 = L.idx_dtype == KAN_U32;
  p.cfg.gb_kind = gb_kind_of(L);
  p.cfg.code = code_of(L);
  const BucketGeom g = bucket_geometry(L.in, L.out, L.K, code_of(L), gb_kind_of(L));
  p.n_jt = g.tab_w[bucket_table_for((long long)B * n_heads)];       // blocks of the table a full group of heads uses
  p.n_bt = (int)B;
  p.n_chunks = g.n_buckets;          // the per-bucket sums are the partial sums
  p.rows_per_chunk = L.in;
  return p;
}

// Small prepared layers: one workgroup per (output, sample) reads the output's ids and gains from the
// transposed copy in the prepared buffer, gathers from L2 and writes finished outputs (no bucket
// copies, no partial sums, no reduction launch).  It is ahead of the bucket kernel while the layer's
// edges x samples stay within about 2^20 (measured, a layer alone, cold, column against bucket kernel:
// 1024 x 256 at batch 1 / 2 / 4: 11.0 / 9.6 / 9.6 against 14.7 / 13.3 / 13.2 us; 1024 x 512: 10.9 / 9.7 /
// 13.1 against 14.9 / 13.5 / 13.1; 1024 x 1024: 10.8 / 13.3 / 22.2 against 14.5 / 12.9 / 15.0; 2048 x 1024:
// 14.0 / 21.6 / 38.3 against 14.4 / 15.6 / 20.0); config 3's head with it on the second layer: 21.8 -> 15.8 us
// at batch 1, 24.2 -> 20.9 at batch 2.
constexpr long long kColumnMaxWork = 1ll << 20;     // edges x samples

bool layer_column_ok(const kan_vq_layer& L) {
  if (L.flags & KAN_LAYER_NO_COLUMN) return false;
  return (long long)L.in * L.out <= kColumnMaxEdges;
}

LayerPlan plan_column(const kan_vq_layer& L, int64_t B) {
  LayerPlan p;
  p.mfma = false;
  p.kind = kPlanColumn;
  p.name = "kan_column";
  p.cfg.bt = 1;
  p.cfg.jpl = 1;
  p.cfg.wj = 1;
  p.cfg.idx_u32 = L.idx_dtype == KAN_U32;
  p.cfg.gb_kind = gb_kind_of(L);
  p.cfg.code = code_of(L);
  p.n_jt = L.out;
  p.n_bt = (int)B;
  p.n_chunks = 1;
  p.rows_per_chunk = L.in;
  return p;
}

bool layer_prepared_ok(const kan_vq_layer& L) {
  return L.prepared != nullptr && aligned(L.prepared, 256) && aligned(L.codebook, 16) && L.in <= kBucketMaxIn &&
         (long long)L.in * L.out <= (1ll << 31);
}

// Which kernels serve a layer:
//   precise path, prepared layers, B <= kBucketMaxBatch (3 for layers of 2^23 edges or more): the bucket kernel
//     (codebook in LDS);
//   precise path (KAN_PATH_GATHER, and AUTO below batch 32): B = 1 the window-gather kernel,
//     B = 2 .. 32 the wave-by-wave kernel (the tiles of the fused kernel where precise_tiles_ahead), above the
//     fused kernel (the fp32 FMA kernel remains the dense baseline's), from kSplitMinBatch the preparation + streaming contraction of the
//     fp16 path on operands split into high and low fp16 parts, the contraction making
//     three passes (hi*lo, lo*hi, hi*hi: fp32-grade sums at matrix-core speed);
//   fp16 path (KAN_PATH_MFMA, and AUTO from batch 32): up to kHalfFusedMaxBatch the wave-by-wave kernel with
//     fp16 operands, or the fused kernel on tiles (half_tiles_ahead), above that coefficient/basis preparation + the streaming
//     contraction (small layers, on either path: coefficient preparation + one launch, plan_matrix);
//   from batch 65, layers of a million edges and more: the contraction that gathers and dequantises its own
//     coefficients (make_wide), large products the one on tiles of 256 x 256 (make_stream), either path;
//   layers of kFusedTwoTilesMinEdges edges or more (not fp32 codebooks) keep the fused kernel up to
//     kFusedTwoTilesMaxBatch on either path where make_wide does not take them.
LayerPlan plan_vq(const kan_vq_layer& L, int64_t B, int n_heads, bool vec_ok, bool prepared_ok, int32_t path,
                  bool column_ok, int x_parts = 1, int min_rows = kMfmaMinRows, bool wide = true, bool reduced = true,
                  int large_wgs = kFusedOneHeadWgs, bool spare = false) {
  const int code = code_of(L);
  const int u32 = L.idx_dtype == KAN_U32, gbk = gb_kind_of(L);
  const long long cb_bytes = (long long)L.K * cb_row_bytes(code);
  const bool half_path = path == KAN_PATH_MFMA || (path == KAN_PATH_AUTO && B >= kAutoMfmaBatch);
  // Large layers stay on the fused kernel for a second batch tile: gathering every row twice costs less
  // than preparing the records of 4 M edges or more and contracting them (4096 x 4096, K = 262,144, batch
  // 96-128: 288-290 -> 210-213 us on the fp16 path, 587 -> 474-478 us precise; 4096 x 1024: 60.8 -> 57.2 and
  // 103 -> 90-95 us; a 2048 x 1024 layer gains at batch 96 and loses at 128, config 3's head 57.5 -> 61.0 us,
  // fp32 rows - three loads per gather - lose: config 2 at batch 128 32.4 -> 35.7 us; at batch 192 all lose).
  // make_wide takes such launches over in turn (4096 x 4096 at batch 128 176 -> 111 us); the plan of two tiles is left
  // for calls that fit the static scratch only without its basis words.
  const bool two_tiles = (long long)L.in * L.out >= kFusedTwoTilesMinEdges && code != kCbF32;
  const int64_t fused_max = two_tiles ? kFusedTwoTilesMaxBatch : kHalfFusedMaxBatch;
  if (half_path) {
    // one batch tile: every edge is needed once, so nothing is staged in memory (the streaming
    // path would write 20 bytes per edge and read them back for no reuse)
    const bool compact = min_rows != kMfmaMinRows;
    if (B <= kHalfFusedMaxBatch && (long long)L.in * L.out >= 4 && !compact) {
      const LayerPlan wave = plan_fused_wave(L.in, L.out, B, n_heads, u32, gbk, code, cb_bytes, large_wgs, true, false, reduced, spare);
      LayerPlan p = plan_fused(L.in, L.out, B, n_heads, u32, gbk, code, false, false, reduced);
      p.tiles_ahead = !half_tiles_far_ahead(L.out, B, n_heads, gbk, code, p, (long long)L.in * L.out);
      return half_tiles_ahead(L.out, B, n_heads, u32, gbk, code, cb_bytes, p, wave) && !(spare && p.tiles_ahead) ? p : wave;
    }
    if (B <= fused_max) {
      LayerPlan p = plan_fused(L.in, L.out, B, n_heads, u32, gbk, code, false, compact, reduced);
      if (wide) make_wide(p, L.in, L.out, B, n_heads, false, x_parts, reduced);
      return p;
    }
    return plan_matrix(L.in, L.out, B, n_heads, u32, gbk, code, false, x_parts, min_rows, wide, reduced);
  }
  if (prepared_ok && B <= bucket_max_batch((long long)L.in * L.out))
    return column_ok && (long long)L.in * L.out * B <= kColumnMaxWork ? plan_column(L, B) : plan_bucket(L, B, n_heads);
  // large batches: the fp16 machinery with both operands split into high and low parts
  if (B >= kSplitMinBatch && B > fused_max) return plan_matrix(L.in, L.out, B, n_heads, u32, gbk, code, true, x_parts, min_rows, wide, reduced);
  const long long edges = (long long)L.in * L.out;
  const bool compact = min_rows != kMfmaMinRows;
  if (B >= 2 && B <= 32 && edges >= 4) {
    const LayerPlan wave = plan_fused_wave(L.in, L.out, B, n_heads, u32, gbk, code, cb_bytes, large_wgs, false, compact, reduced, spare);
    LayerPlan p = plan_fused(L.in, L.out, B, n_heads, u32, gbk, code, true, compact, reduced);
    p.tiles_ahead = !compact;
    const bool tiles = compact ? edges * n_heads > kFusedTilesCompactMinEdges
                               : !spare && precise_tiles_ahead(L.out, B, n_heads, u32, gbk, code, cb_bytes, p, wave);
    return tiles ? p : wave;
  }
  if (B > 32) {
    LayerPlan p = plan_fused(L.in, L.out, B, n_heads, u32, gbk, code, true, compact, reduced);
    if (wide) make_wide(p, L.in, L.out, B, n_heads, true, x_parts, reduced);
    return p;
  }
  return plan_gather(L.in, L.out, B, n_heads, u32, gbk, code, vec_ok, cb_bytes, compact);
}

bool layer_vec_ok(const kan_vq_layer& L) {
  return aligned(L.idx, 16) && aligned(L.gain, 16) && aligned(L.bias, 16);
}

size_t partial_bytes(const LayerPlan& p, int n_out, int64_t B, int heads_in_group) {
  if (p.n_chunks <= 1) return 0;
  return round_up((size_t)heads_in_group * p.n_chunks * (size_t)B * n_out * sizeof(float), 256);
}

// Scratch regions inside the caller's workspace (each a multiple of 256 bytes;
// sized for the largest layer and for one group of heads).
struct WsLayout {
  size_t hidden = 0;    // one of two ping-pong hidden-activation buffers, [n_heads][B][out]
  size_t partial = 0;   // partial sums: of layers 1, 3, .. where a layer hands its sums on (the next one's go to the
  size_t partial2 = 0;  //   other buffer), else of all / of layers 2, 4, .. where a layer hands its sums on, else empty
  std::vector<char> handed;   // layer l leaves its partial sums to layer l + 1
  size_t cf = 0;        // matrix-core path: fp16 coefficient fragments, a region per layer (layers after the
  size_t bp = 0;        //   first are prepared beside the first one's work) / partial bias sums, likewise
  std::vector<size_t> cf_off, bp_off;   // start of each layer's region within cf / bp
  size_t u = 0;         // matrix-core path: packed basis weights + span
  int n_layers = 1;
  size_t total() const { return (n_layers > 1 ? 2 * hidden : 0) + partial + partial2 + cf + bp + u; }
};

size_t mfma_cf_records(int n_in, int n_out) { return (size_t)((n_in + 15) / 16) * 20 * (size_t)n_out; }
size_t mfma_bp_floats(int n_in, int n_out) { return (size_t)((n_in + kMfmaPrepRows - 1) / kMfmaPrepRows) * n_out; }

// Pointers of the scratch regions for the current call.
struct WsPtrs {
  float* hid[2];
  float* partial;
  float* partial2;
  uint4* cf;
  float* bp;
  uint2* u;
};

// One layer of a group of heads.  `a` carries x, shapes and the per-head pointers;
// `final_dst` receives act(y).  Gather path: main kernel, then (if i was split) the
// fixed-order reduction.  Matrix-core path: coefficient and basis preparation first.
// How a layer receives its input and hands on its output when it is chained to its
// neighbours: the partial sums of layer l (per bucket, or per chunk of inputs) are added and
// squashed by layer l+1 itself: by the bucket kernel while it loads x, or by the basis
// preparation of the matrix-core path.
struct Chain {
  int in_parts = 1;              // slices of the input to add (1: plain x)
  long long in_part_stride = 0;
  int in_tanh = 0;
  bool out = false;              // leave the partial sums for the next layer (no reduction pass)
  float* partial = nullptr;      // where this layer's partial sums go (default: w.partial)
  // matrix-core path: stages the head's first launch has already covered
  bool coef_done = false;
  bool basis_done = false;
};

// Matrix-core path, stage 1: coefficient records (and bias sums) of one layer of a group of heads.
// Depends on the layer's parameters only, not on x.
kan_status run_prep_coef(const LayerPlan& p, const GatherArgs& a, int heads, const WsPtrs& w, PrepCoefArgs* out,
                         bool launch, hipStream_t s) {
  PrepCoefArgs& pc = *out;
  memset(&pc, 0, sizeof(pc));
  pc.cf = w.cf;
  pc.cf_head_stride = (long long)mfma_cf_records(a.n_in, a.n_out);
  pc.cf_lo = p.products == 3 ? w.cf + (long long)heads * pc.cf_head_stride : nullptr;
  pc.bias_partial = w.bp;
  pc.bp_head_stride = (long long)mfma_bp_floats(a.n_in, a.n_out);
  pc.n_in = a.n_in;
  pc.n_out = a.n_out;
  pc.rot = p.stream;
  memcpy(pc.h, a.h, sizeof(pc.h));
  if (!launch) return KAN_OK;
  if (p.cfg.code == kDense)
    return run("kan_prep_dense", s, [&] { return launch_prep_dense((const float*)a.h[0].cb, pc.cf, pc.cf_lo, a.n_in, a.n_out, s); });
  return run("kan_prep_coef", s, [&] { return launch_prep_coef(p.cfg, pc, heads, s); });
}

// Stage 2: packed basis weights and spans of the layer's input (x, or the previous layer's
// partial sums added and squashed).
struct BasisBufs {
  uint2* u_lo;
  long long u_stride;
};

// The same in the rotated form (kan_wide.hip, kan_stream.hip).
RotWords rot_words(const LayerPlan& p, const GatherArgs& a, int heads, bool x_shared, const WsPtrs& w) {
  const long long items = (long long)((a.n_in + 15) / 16) * 10 * (p.stream ? rot_rows(a.B) : a.B);
  RotWords r;
  r.W = (uint4*)w.u;
  r.W_lo = p.products == 3 ? r.W + (x_shared ? 1 : heads) * items : nullptr;
  r.w_head_stride = x_shared ? 0 : items;
  r.P = p.stream ? (uint16_t*)((uint4*)w.u + (p.products == 3 ? 2 : 1) * (x_shared ? 1 : heads) * items) : nullptr;
  r.p_head_stride = x_shared ? 0 : (long long)((a.n_in + 15) / 16) * 10 * rot_rows(a.B);
  return r;
}
kan_status run_prep_rot(const RotWords& r, const GatherArgs& a, int heads, bool x_shared, const Chain& chain, hipStream_t s) {
  if (chain.basis_done) return KAN_OK;
  return run("kan_prep_basis", s, [&] {
    return launch_prep_rot(a.x, a.x_head_stride, chain.in_parts, chain.in_part_stride, chain.in_tanh, r, a.n_in, a.B,
                           x_shared ? 1 : heads, a.rule, s);
  });
}
kan_status run_wide(const LayerPlan& p, const GatherArgs& a, int heads, bool x_shared, float* dst, long long dst_head_stride,
                    long long dst_chunk_stride, int apply_tanh, const WsPtrs& w, const Chain& chain, hipStream_t s) {
  const RotWords r = rot_words(p, a, heads, x_shared, w);
  const kan_status st = run_prep_rot(r, a, heads, x_shared, chain, s);
  if (st != KAN_OK) return st;
  WideArgs m;
  memset(&m, 0, sizeof(m));
  m.W = r.W;
  m.W_lo = r.W_lo;
  m.w_head_stride = r.w_head_stride;
  m.dst = dst;
  m.dst_head_stride = dst_head_stride;
  m.dst_chunk_stride = dst_chunk_stride;
  m.n_in = a.n_in;
  m.n_out = a.n_out;
  m.B = a.B;
  m.rows_per_chunk = p.rows_per_chunk;
  m.n_jt = p.n_jt;
  m.apply_tanh = apply_tanh;
  memcpy(m.h, a.h, sizeof(m.h));
  dim3 grid((unsigned)(p.n_jt * p.n_bt), (unsigned)p.n_chunks, (unsigned)heads);
  return run(p.name, s, [&] { return launch_wide(p.cfg, m, p.products == 3, p.cfg.bt, grid, s); });
}
kan_status run_prep_basis(const LayerPlan& p, const GatherArgs& a, int heads, bool x_shared, const WsPtrs& w,
                          const Chain& chain, BasisBufs* out, bool launch, hipStream_t s) {
  const long long u_elems = (long long)((a.n_in + 15) / 16 * 16) * a.B;
  out->u_stride = x_shared ? 0 : u_elems;
  out->u_lo = p.products == 3 ? w.u + (x_shared ? 1 : heads) * u_elems : nullptr;
  if (!launch) return KAN_OK;
  return run("kan_prep_basis", s, [&] {
    return launch_prep_basis(a.x, a.x_head_stride, chain.in_parts, chain.in_part_stride, chain.in_tanh, w.u, out->u_lo,
                             out->u_stride, a.n_in, a.B, x_shared ? 1 : heads, a.rule, s);
  });
}

kan_status run_layer_group(const LayerPlan& p, GatherArgs& a, const void* const* prepared, int heads,
                           bool x_shared, float* final_dst, long long final_head_stride, const WsPtrs& w,
                           int apply_tanh, hipStream_t s, const Chain& chain = Chain()) {
  const long long count = (long long)a.B * a.n_out;
  const bool split = p.n_chunks > 1;
  float* const partial = chain.partial ? chain.partial : w.partial;
  float* dst = split ? partial : final_dst;
  const long long dst_head_stride = split ? count * p.n_chunks : final_head_stride;
  const long long dst_chunk_stride = split ? count : 0;
  const int tanh_in_kernel = split ? 0 : apply_tanh;
  auto reduce = [&] {
    return run("kan_reduce", s, [&] {
      return launch_reduce(partial, dst_head_stride, count, p.n_chunks, final_dst, final_head_stride, count, heads, apply_tanh, s);
    });
  };
  kan_status st;
  if (p.wide) {
    st = run_wide(p, a, heads, x_shared, dst, dst_head_stride, dst_chunk_stride, tanh_in_kernel, w, chain, s);
  } else if (p.mfma) {
    PrepCoefArgs pc;
    const bool split3 = p.products == 3;
    st = run_prep_coef(p, a, heads, w, &pc, !chain.coef_done, s);
    if (st != KAN_OK) return st;
    if (p.kind == kPlanTail) {
      TailArgs t;
      memset(&t, 0, sizeof(t));
      t.cf = pc.cf;
      t.cf_lo = pc.cf_lo;
      t.cf_head_stride = pc.cf_head_stride;
      t.bias_partial = pc.bias_partial;
      t.bp_head_stride = pc.bp_head_stride;
      t.x = a.x;
      t.x_head_stride = a.x_head_stride;
      t.x_part_stride = chain.in_part_stride;
      t.x_parts = chain.in_parts;
      t.x_tanh = chain.in_tanh;
      t.dst = final_dst;
      t.dst_head_stride = final_head_stride;
      t.n_in = a.n_in;
      t.n_out = a.n_out;
      t.B = a.B;
      t.n_jt = p.n_jt;
      t.apply_tanh = apply_tanh;
      t.rule = a.rule;
      for (int h = 0; h < heads; ++h) t.scale[h] = p.cfg.code == kCbI8 ? a.h[h].scale : 1.0f;
      return run(p.name, s, [&] { return launch_tail(t, split3, p.tile_n, dim3((unsigned)(p.n_jt * p.n_bt), 1, (unsigned)heads), s); });
    }
    if (p.stream) {
      const RotWords r = rot_words(p, a, heads, x_shared, w);
      st = run_prep_rot(r, a, heads, x_shared, chain, s);
      if (st != KAN_OK) return st;
      StreamArgs m;
      memset(&m, 0, sizeof(m));
      m.cf = pc.cf;
      m.cf_lo = pc.cf_lo;
      m.cf_head_stride = pc.cf_head_stride;
      m.W = r.W;
      m.W_lo = r.W_lo;
      m.w_head_stride = r.w_head_stride;
      m.P = r.P;
      m.p_head_stride = r.p_head_stride;
      m.bias_partial = pc.bias_partial;
      m.bp_head_stride = pc.bp_head_stride;
      m.dst = dst;
      m.dst_head_stride = dst_head_stride;
      m.dst_chunk_stride = dst_chunk_stride;
      m.n_in = a.n_in;
      m.n_out = a.n_out;
      m.B = a.B;
      m.rows_per_chunk = p.rows_per_chunk;
      m.n_jt = p.n_jt;
      m.apply_tanh = tanh_in_kernel;
      for (int h = 0; h < heads; ++h) m.scale[h] = p.cfg.code == kCbI8 ? a.h[h].scale : 1.0f;
      dim3 grid((unsigned)(p.n_jt * p.n_bt), (unsigned)p.n_chunks, (unsigned)heads);
      st = run(p.name, s, [&] { return launch_stream(m, split3, grid, s); });
      return st != KAN_OK || !split || chain.out ? st : reduce();
    }
    BasisBufs bb;
    st = run_prep_basis(p, a, heads, x_shared, w, chain, &bb, !chain.basis_done, s);
    if (st != KAN_OK) return st;
    uint2* const u_lo = bb.u_lo;
    const long long u_stride = bb.u_stride;
    MfmaArgs m;
    memset(&m, 0, sizeof(m));
    m.cf = w.cf;
    m.cf_head_stride = pc.cf_head_stride;
    m.W = w.u;
    m.w_head_stride = u_stride;
    // (the dense form has no bias sums: the kernel still reads the rows it would add, so it is
    // given valid memory - the coefficient records, which are larger - and told not to add them)
    m.bias_partial = p.cfg.code == kDense ? (const float*)w.cf : w.bp;
    m.bp_head_stride = pc.bp_head_stride;
    m.dst = dst;
    m.dst_head_stride = dst_head_stride;
    m.dst_chunk_stride = dst_chunk_stride;
    m.n_in = a.n_in;
    m.n_out = a.n_out;
    m.B = a.B;
    m.rows_per_chunk = p.rows_per_chunk;
    m.n_jt = p.n_jt;
    m.apply_tanh = tanh_in_kernel;
    m.bias_on = p.cfg.code == kDense ? 0 : 1;            // the dense form has no bias
    for (int h = 0; h < heads; ++h) m.scale[h] = p.cfg.code == kCbI8 ? a.h[h].scale : 1.0f;
    if (split3) {                                        // hi*lo and lo*hi first, scaled by 1/2048, then hi*hi on top
      m.passes = 3;
      m.cf_lo = pc.cf_lo;
      m.W_lo = u_lo;
      m.lo_scale = 1.0f / 2048.0f;
    } else {
      m.passes = 1;
    }
    dim3 grid((unsigned)(p.n_jt * p.n_bt), (unsigned)p.n_chunks, (unsigned)heads);
    st = run(p.name, s, [&] { return launch_mfma(m, p.cfg.bt, p.tile_n ? p.tile_n : kMfmaTileN, grid, s); });
  } else if (p.kind == kPlanBucket || p.kind == kPlanColumn) {
    const BucketGeom g = bucket_geometry(a.n_in, a.n_out, (int)(a.cb_bytes / cb_row_bytes(p.cfg.code)), p.cfg.code,
                                         p.cfg.gb_kind);
    BucketArgs k;
    memset(&k, 0, sizeof(k));
    k.x = a.x;
    k.x_head_stride = a.x_head_stride;
    k.x_parts = chain.in_parts;
    k.x_part_stride = chain.in_part_stride;
    k.x_tanh = chain.in_tanh;
    k.dst = dst;
    k.dst_head_stride = dst_head_stride;
    k.dst_chunk_stride = dst_chunk_stride;
    k.n_in = a.n_in;
    k.n_out = a.n_out;
    k.B = a.B;
    k.n_buckets = g.n_buckets;
    const int table = bucket_table_for((long long)a.B * heads);     // by the heads of this very launch
    k.off_blk = (long long)(g.off_blk + (size_t)g.tab_first[table] * kBucketEntryWords * 4);
    k.rows_shift = g.rows_shift;
    k.cb_bytes = a.cb_bytes;
    k.apply_tanh = tanh_in_kernel;
    k.rule = a.rule;
    k.off_seg = (long long)g.off_seg;
    k.off_bias = (long long)g.off_bias;
    k.off_i = (long long)g.off_i;
    k.off_q = (long long)g.off_q;
    k.off_g = (long long)g.off_g;
    k.off_ti = (long long)g.off_ti;
    k.off_tg = (long long)g.off_tg;
    for (int h = 0; h < heads; ++h) {
      k.h[h].prepared = prepared[h];
      k.h[h].cb = a.h[h].cb;
      k.h[h].scale = a.h[h].scale;
      k.h[h].gain_log2_lo = a.h[h].gain_log2_lo;
      k.h[h].gain_log2_step = a.h[h].gain_log2_step;
    }
    if (p.kind == kPlanColumn) st = run(p.name, s, [&] { return launch_column(p.cfg.code, p.cfg.gb_kind, k, heads, s); });
    else st = run(p.name, s, [&] { return launch_bucket(p.cfg.code, p.cfg.gb_kind, k, g.tab_w[table], heads, s); });
  } else if (p.kind == kPlanFused16 || p.kind == kPlanFused32 || p.kind == kPlanFusedWave) {
    const bool f32 = p.kind == kPlanFused32;
    FusedArgs f;
    memset(&f, 0, sizeof(f));
    f.x = a.x;
    f.x_head_stride = a.x_head_stride;
    f.dst = dst;
    f.dst_head_stride = dst_head_stride;
    f.dst_chunk_stride = dst_chunk_stride;
    f.n_in = a.n_in;
    f.n_out = a.n_out;
    f.B = a.B;
    f.rows_per_chunk = p.rows_per_chunk;
    f.n_jt = p.n_jt;
    f.apply_tanh = tanh_in_kernel;
    f.rule = a.rule;
    f.x_parts = chain.in_parts;
    f.x_part_stride = chain.in_part_stride;
    f.x_tanh = chain.in_tanh;
    memcpy(f.h, a.h, sizeof(f.h));
    dim3 grid((unsigned)(p.n_jt * p.n_bt), (unsigned)p.n_chunks, (unsigned)heads);
    if (p.kind == kPlanFusedWave) st = run(p.name, s, [&] { return p.half ? launch_fused_wave_half(p.cfg, f, grid, s) : launch_fused_wave(p.cfg, f, grid, s); });
    else if (chain.in_parts > 1) st = run(p.name, s, [&] { return launch_fused_chained(p.cfg, f, f32, grid, s); });
    else st = run(p.name, s, [&] { return launch_fused(p.cfg, f, f32, grid, s); });
  } else if (p.kind == kPlanDense) {
    DenseArgs d;
    d.coef = (const float*)a.h[0].cb;
    d.x = a.x;
    d.dst = dst;
    d.dst_chunk_stride = dst_chunk_stride;
    d.n_in = a.n_in;
    d.n_out = a.n_out;
    d.B = a.B;
    d.rows_per_chunk = p.rows_per_chunk;
    d.n_jt = p.n_jt;
    dim3 grid((unsigned)(p.n_jt * p.n_bt), (unsigned)p.n_chunks);
    st = run(p.name, s, [&] { return launch_dense(d, p.cfg.bt, grid, s); });
  } else {
    a.dst = dst;
    a.dst_head_stride = dst_head_stride;
    a.dst_chunk_stride = dst_chunk_stride;
    a.apply_tanh = tanh_in_kernel;
    a.x_parts = chain.in_parts;
    a.x_part_stride = chain.in_part_stride;
    a.x_tanh = chain.in_tanh;
    dim3 grid((unsigned)(p.n_jt * p.n_bt), (unsigned)p.n_chunks, (unsigned)heads);
    st = run(p.name, s, [&] { return launch_gather(p.cfg, a, grid, s); });
  }
  return st != KAN_OK || !split || chain.out ? st : reduce();
}

kan_status check_path(int32_t path) {
  if (path == KAN_PATH_AUTO || path == KAN_PATH_GATHER || path == KAN_PATH_MFMA) return KAN_OK;
  return KAN_ERR_UNSUPPORTED;
}

// Layer l leaves its partial sums to layer l+1 (one group of heads only: the buffers are
// sized for one group).  Consumers: the bucket kernel (after a bucket layer), the basis
// preparation of the matrix-core path (after any layer that splits its inputs), the fused
// kernel on tiles of 32 samples (after any such layer: see fused_takes_slices; on the precise
// path fifty heads of 256-1280-128 at batch 4 / 16 take 136.7 / 139.8 us so, 138.8 / 145.0 with a
// reduction launch), the wave-by-wave kernel and the vector-ALU kernel at batch 1.
bool fused_takes_slices(const LayerPlan& from, const LayerPlan& to, int n_in, int64_t B);

bool chained(const std::vector<LayerPlan>& plans, int l, int n_heads, const kan_vq_layer* layers, int64_t B) {
  if (l < 0 || l + 1 >= (int)plans.size() || n_heads > kMaxGroup || plans[l].n_chunks <= 1) return false;
  if (plans[l + 1].kind == kPlanBucket || plans[l + 1].kind == kPlanColumn) return plans[l].kind == kPlanBucket;
  if (plans[l + 1].kind == kPlanFusedWave)
    return plans[l].n_chunks <= kFusedChainMaxParts && layers[l + 1].in % 4 == 0 && plans[l + 1].n_jt <= 16 &&
           B * plans[l + 1].rows_per_chunk <= kFusedWaveChainFloats &&
           (long long)plans[l].n_chunks * B * (plans[l + 1].rows_per_chunk / 4) <= 32 * 256;
  if (plans[l + 1].kind == kPlanFused16 || plans[l + 1].kind == kPlanFused32)
    return fused_takes_slices(plans[l], plans[l + 1], layers[l + 1].in, B);
  // the vector-ALU kernel at batch 1: the threads that share a row of the basis table split the
  // slices; few output tiles (each adds the slices again)
  if (plans[l + 1].kind == kPlanGather)
    return plans[l].n_chunks <= kGatherChainMaxParts && plans[l + 1].n_jt <= 4;
  return plans[l + 1].mfma && plans[l].n_chunks <= kMaxChainedSlices;
}

// The fused kernel adds the slices of its own chunk of inputs before its first step when that
// is cheaper than a reduction launch in between: tiles of 32 samples, the chunk's inputs of the
// tile within the kernel's LDS array, 16-byte loads (inputs in fours), at most 32 such loads
// per thread (two rounds in flight; with three, batch 32 of config 3, nothing was gained), and
// few output tiles (every one of them adds the slices again).
bool fused_takes_slices(const LayerPlan& from, const LayerPlan& to, int n_in, int64_t B) {
  if (to.cfg.bt != 32 || from.n_chunks > kFusedChainMaxParts || to.n_jt > 8) return false;
  if (n_in % 4 != 0 || to.rows_per_chunk % 4 != 0 || 32ll * to.rows_per_chunk > kFusedChainFloats) return false;
  const long long rows = B < 32 ? B : 32;
  return (long long)from.n_chunks * rows * (to.rows_per_chunk / 4) <= 32 * 256;
}

// Validates a [n_heads][n_layers] descriptor table; fills per-layer plans and scratch sizes.
kan_status plan_head_rows(const kan_vq_layer* layers, int32_t n_layers, int32_t n_heads, int64_t B, int32_t path,
                          int min_rows, bool hand_on, bool wide, int large_wgs, bool spare, std::vector<LayerPlan>* plans, WsLayout* ws) {
  if (!layers) return KAN_ERR_NULL;
  if (n_layers < 1 || n_heads < 1 || n_layers > 64 || n_heads > (1 << 16)) return KAN_ERR_SHAPE;
  if (B < 0 || B > kMaxBatch) return KAN_ERR_SHAPE;
  kan_status st = check_path(path);
  if (st != KAN_OK) return st;
  for (int h = 0; h < n_heads; ++h)
    for (int l = 0; l < n_layers; ++l) {
      const kan_vq_layer& L = layers[(size_t)h * n_layers + l];
      st = validate_layer(&L);
      if (st != KAN_OK) return st;
      const kan_vq_layer& R = layers[l];
      if (L.in != R.in || L.out != R.out || L.K != R.K || L.idx_dtype != R.idx_dtype ||
          L.gb_dtype != R.gb_dtype || L.cb_dtype != R.cb_dtype || L.rule != R.rule)
        return KAN_ERR_UNSUPPORTED;
      if (l > 0 && L.in != layers[(size_t)h * n_layers + l - 1].out) return KAN_ERR_SHAPE;
    }
  const int group = n_heads < kMaxGroup ? n_heads : kMaxGroup;
  *ws = WsLayout();
  ws->n_layers = n_layers;
  plans->clear();
  auto plan_of = [&](int l, bool reduced) {
    const kan_vq_layer& R = layers[l];
    bool vec_ok = true, prepared_ok = true, column_ok = true;
    for (int h = 0; h < n_heads; ++h) {
      vec_ok = vec_ok && layer_vec_ok(layers[(size_t)h * n_layers + l]);
      prepared_ok = prepared_ok && layer_prepared_ok(layers[(size_t)h * n_layers + l]);
      column_ok = column_ok && layer_column_ok(layers[(size_t)h * n_layers + l]);
    }
    return plan_vq(R, B, group, vec_ok, prepared_ok, path, column_ok, l > 0 ? (*plans)[l - 1].n_chunks : 1, min_rows, wide, reduced, large_wgs, spare);
  };
  const int last = n_layers - 1;
  for (int l = 0; l <= last; ++l) plans->push_back(plan_of(l, l == last));
  // Layers whose slices a reduction launch adds - the last one, others once the plans behind them are known - are whole
  // where that is faster, unless they would then no longer take their predecessor's slices.
  auto hands_on = [&](int l) { return hand_on && chained(*plans, l, n_heads, layers, B); };
  if ((*plans)[last].n_chunks == 1 && last > 0 && (*plans)[last - 1].n_chunks > 1 && !hands_on(last - 1)) {
    const LayerPlan whole = (*plans)[last];
    (*plans)[last] = plan_of(last, false);
    if (!hands_on(last - 1)) (*plans)[last] = whole;
  }
  for (int l = last - 1; l >= 0; --l) {
    if ((*plans)[l].n_chunks <= 1 || hands_on(l)) continue;
    const LayerPlan cut = (*plans)[l];
    const bool takes = hands_on(l - 1);
    (*plans)[l] = plan_of(l, true);
    if (takes && !hands_on(l - 1)) (*plans)[l] = cut;
  }
  for (int l = 0; l < n_layers; ++l) {
    const kan_vq_layer& R = layers[l];
    const LayerPlan& p = (*plans)[l];
    auto grow = [](size_t& dst, size_t v) { if (v > dst) dst = v; };
    grow(l & 1 ? ws->partial2 : ws->partial, partial_bytes(p, R.out, B, group));
    ws->cf_off.push_back(ws->cf);
    ws->bp_off.push_back(ws->bp);
    if (p.mfma && !p.wide) {
      ws->cf += round_up((size_t)(p.products == 3 ? 2 : 1) * group * mfma_cf_records(R.in, R.out) * sizeof(uint4), 256);
      ws->bp += round_up((size_t)group * mfma_bp_floats(R.in, R.out) * sizeof(float), 256);
    }
    if (p.kind == kPlanMfma) {
      const size_t rows = (size_t)(l == 0 ? 1 : group) * (size_t)((R.in + 15) / 16), parts = p.products == 3 ? 2 : 1;
      if (p.stream) grow(ws->u, round_up(rows * 10 * (size_t)rot_rows(B) * (parts * sizeof(uint4) + sizeof(uint16_t)), 256));
      else grow(ws->u, round_up(parts * rows * (p.wide ? 10 * sizeof(uint4) : 16 * sizeof(uint2)) * (size_t)B, 256));
    }
    if (l + 1 < n_layers) grow(ws->hidden, round_up((size_t)n_heads * (size_t)B * R.out * sizeof(float), 256));
  }
  for (int l = 0; l < n_layers; ++l) ws->handed.push_back(hands_on(l));
  if (std::find(ws->handed.begin(), ws->handed.end(), 1) == ws->handed.end()) {      // one buffer does for all
    ws->partial = std::max(ws->partial, ws->partial2);
    ws->partial2 = 0;
  }
  return KAN_OK;
}

// Heads that an XCD takes one at a time get fewer workgroups each before anything else is given up (fifty of 2048-256-21 with
// 65,536 fp32 rows, fp16 path, batch 40, 20 / 32 / 48 workgroups 368 / 333 / 311 us; with 64, which take 33 MB, planned compact 403).
// Tiles of 128 outputs that are ahead of the wave-by-wave kernel are cut finer where an XCD takes few heads at a time: where a call
// does not fit with them, they are the next to go, with cuts of the wave-by-wave kernel that save less than a tenth.
// Finer chunks write more partial sums, a layer that hands its sums on keeps a second buffer of them: a call that fits the
// library's static scratch only with larger chunks, or with a reduction between the layers, is planned so.  Basis words
// take room that the fused kernel does without, rotated ones of whole tiles of 256 samples more than those of kan_mfma.hip: a
// call that would fit without the kernels of kan_wide.hip and kan_stream.hip is planned to fit, with the former where
// possible; one that would not is not slowed down to fit.  The same plan serves callers who bring a workspace of their own:
// what it needs does not depend on the entry point (65536 x 64 at batch 128: two tiles of the fused kernel in 8 MB; 200 x
// 4095 at 7700: kan_mfma in 28.6 MB, kan_stream would take 34).
kan_status plan_head(const kan_vq_layer* layers, int32_t n_layers, int32_t n_heads, int64_t B, int32_t path,
                     std::vector<LayerPlan>* plans, WsLayout* ws) {
  kan_status st = plan_head_rows(layers, n_layers, n_heads, B, path, kMfmaMinRows, true, true, kFusedOneHeadWgs, false, plans, ws);
  if (st != KAN_OK || ws->total() <= (size_t)KAN_STATIC_SCRATCH_BYTES) return st;
  std::vector<LayerPlan> other;
  WsLayout other_ws;
  auto fits = [&](int min_rows, bool hand_on, bool wide, int large_wgs, bool spare) {
    return plan_head_rows(layers, n_layers, n_heads, B, path, min_rows, hand_on, wide, large_wgs, spare, &other, &other_ws) == KAN_OK &&
           other_ws.total() <= (size_t)KAN_STATIC_SCRATCH_BYTES;
  };
  auto take_other = [&] {
    plans->swap(other);
    *ws = other_ws;
    return st;
  };
  auto any = [&](auto of) { return std::any_of(plans->begin(), plans->end(), of); };
  const bool any_wide = any([](const LayerPlan& p) { return p.wide; }), any_tiles = any([](const LayerPlan& p) { return p.tiles_ahead; });
  const bool any_spare = any_tiles || any([](const LayerPlan& p) { return p.kind == kPlanFusedWave && p.n_chunks > 1; });
  const int fewer[] = {kFusedOneHeadWgs * 3 / 4, kFusedOneHeadWgs / 2, kFusedMinWgsPerHead};
  const bool one_head = any([](const LayerPlan& p) { return p.one_head; });
  if (one_head)
    for (const int wgs : fewer)
      if (fits(kMfmaMinRows, true, true, wgs, !any_tiles)) return take_other();      // (no tiles that were not there)
  if (any_spare) {
    if (fits(kMfmaMinRows, true, true, kFusedOneHeadWgs, true)) return take_other();
    if (one_head || any_tiles)
      for (const int wgs : fewer)
        if (fits(kMfmaMinRows, true, true, wgs, true)) return take_other();
  }
  auto forms = [&](bool wide) {      // (the first of them is the plan that does not fit, but without kan_wide.hip)
    return (any_wide && !wide && fits(kMfmaMinRows, true, wide, kFusedMinWgsPerHead, false)) ||
           fits(kMfmaMinRowsCompact, true, wide, kFusedMinWgsPerHead, false) || fits(kMfmaMinRows, false, wide, kFusedMinWgsPerHead, !any_tiles) ||
           (any_spare && fits(kMfmaMinRows, false, wide, kFusedMinWgsPerHead, true)) ||
           fits(kMfmaMinRowsCompact, false, wide, kFusedMinWgsPerHead, false);
  };
  if (!forms(false)) return st;
  if (any_wide && !forms(true)) (void)forms(false);
  return take_other();
}

}  // namespace
}  // namespace kan

using namespace kan;

extern "C" {

const char* kan_status_string(int32_t status) {
  switch (status) {
    case KAN_OK: return "ok";
    case KAN_ERR_NULL: return "required pointer is NULL";
    case KAN_ERR_SHAPE: return "invalid or inconsistent size or alignment";
    case KAN_ERR_DTYPE: return "dtype not allowed for this operand";
    case KAN_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case KAN_ERR_UNSUPPORTED: return "unsupported configuration";
    case KAN_ERR_LAUNCH: return "HIP launch failed";
    default: return "unknown status";
  }
}

kan_status kan_bspline_basis(const float* x, int64_t n, uint8_t* span, float* w, void* stream) {
  if (n < 0) return KAN_ERR_SHAPE;
  if (n == 0) return KAN_OK;
  if (!x || !span || !w) return KAN_ERR_NULL;
  if (!aligned(w, 16) || !aligned(x, 4)) return KAN_ERR_SHAPE;
  hipStream_t s = (hipStream_t)stream;
  return run("kan_basis", s, [&] { return launch_basis(x, n, span, w, s); });
}

kan_status kan_pli_basis(const float* x, int64_t n, uint8_t* index, float* w, void* stream) {
  if (n < 0) return KAN_ERR_SHAPE;
  if (n == 0) return KAN_OK;
  if (!x || !index || !w) return KAN_ERR_NULL;
  if (!aligned(w, 8) || !aligned(x, 4)) return KAN_ERR_SHAPE;
  hipStream_t s = (hipStream_t)stream;
  return run("kan_pli_basis", s, [&] { return launch_pli_basis(x, n, index, w, s); });
}

kan_status kan_basis_window(const float* x, int64_t n, int32_t rule, int32_t variant, uint8_t* start, float* w,
                            void* stream) {
  if (n < 0) return KAN_ERR_SHAPE;
  if (rule != KAN_RULE_BSPLINE3 && rule != KAN_RULE_PLI2) return KAN_ERR_UNSUPPORTED;
  if (variant != 0 && variant != 1) return KAN_ERR_UNSUPPORTED;
  if (n == 0) return KAN_OK;
  if (!x || !start || !w) return KAN_ERR_NULL;
  if (!aligned(w, 16) || !aligned(x, 4)) return KAN_ERR_SHAPE;
  hipStream_t s = (hipStream_t)stream;
  return run("kan_basis_window", s, [&] { return launch_basis_window(x, n, rule, variant, start, w, s); });
}

size_t kan_vq_workspace_bytes(const kan_vq_layer* layers, int32_t n_layers, int32_t n_heads, int64_t B,
                              int32_t path) {
  std::vector<LayerPlan> plans;
  WsLayout wl;
  if (plan_head(layers, n_layers, n_heads, B, path, &plans, &wl) != KAN_OK) return (size_t)-1;
  if (B == 0) return 0;
  return wl.total();
}

namespace {
// The forward of a group of heads.  static_ws: take the scratch regions from the library's own
// per-device array instead of a caller's workspace (ws, ws_bytes are then ignored).
kan_status head_forward(const kan_vq_layer* layers, int32_t n_layers, int32_t n_heads, const float* x, int64_t B,
                        float* y, void* ws, size_t ws_bytes, bool static_ws, int32_t path, void* stream) {
  std::vector<LayerPlan> plans;
  WsLayout wl;
  kan_status st = plan_head(layers, n_layers, n_heads, B, path, &plans, &wl);
  if (st != KAN_OK) return st;
  if (B == 0) return KAN_OK;
  if (!x || !y) return KAN_ERR_NULL;
  if (!aligned(x, 4) || !aligned(y, 4)) return KAN_ERR_SHAPE;
  const size_t need = wl.total();
  if (static_ws) {
    if (need > (size_t)KAN_STATIC_SCRATCH_BYTES) return KAN_ERR_WORKSPACE;     // beyond the fixed array: use kan_vq_head_forward
    ws = nullptr;
    ws_bytes = KAN_STATIC_SCRATCH_BYTES;
    if (need > 0) {
      st = static_scratch(&ws);
      if (st != KAN_OK) return st;
    }
  }
  if (need > 0 && (!ws || !aligned(ws, 256) || ws_bytes < need)) return KAN_ERR_WORKSPACE;

  hipStream_t s = (hipStream_t)stream;
  char* wsp = (char*)ws;
  WsPtrs w;
  const size_t hid2 = n_layers > 1 ? 2 * wl.hidden : 0;
  w.hid[0] = (float*)wsp;
  w.hid[1] = (float*)(wsp + wl.hidden);
  w.partial = (float*)(wsp + hid2);
  w.partial2 = (float*)(wsp + hid2 + wl.partial);
  const size_t after_partial = hid2 + wl.partial + wl.partial2;
  uint4* const cf_base = (uint4*)(wsp + after_partial);
  float* const bp_base = (float*)(wsp + after_partial + wl.cf);
  w.cf = cf_base;
  w.bp = bp_base;
  w.u = (uint2*)(wsp + after_partial + wl.cf + wl.bp);

  auto layer_args = [&](int l, int h0, int heads, const float* src, long long src_head_stride, GatherArgs* out,
                        const void** prepared) {
    const kan_vq_layer& R = layers[l];
    GatherArgs& a = *out;
    memset(&a, 0, sizeof(a));
    a.x = src + (long long)h0 * src_head_stride;
    a.x_head_stride = src_head_stride;
    a.n_in = R.in;
    a.n_out = R.out;
    a.B = (int)B;
    a.rows_per_chunk = plans[l].rows_per_chunk;
    a.n_jt = plans[l].n_jt;
    a.cb_bytes = (long long)R.K * cb_row_bytes(code_of(R));
    a.rule = R.rule;
    for (int h = 0; h < heads; ++h) {
      const kan_vq_layer& L = layers[(size_t)(h0 + h) * n_layers + l];
      a.h[h].idx = L.idx;
      a.h[h].gain = L.gain;
      a.h[h].bias = L.bias;
      a.h[h].cb = L.codebook;
      a.h[h].scale = L.scale;
      a.h[h].gain_log2_lo = L.gain_log2_lo;
      a.h[h].gain_log2_step = L.gain_log2_step;
      a.h[h].bias_scale = L.bias_scale;
      if (prepared) prepared[h] = L.prepared;
    }
  };

  // A single head on the matrix cores: one launch prepares the coefficient records of its
  // matrix-core layers (those stored like the first one, up to kStartJobs) and the first layer's
  // basis words; the layers below then skip these stages.
  std::vector<char> coef_done(n_layers, 0);
  bool basis0_done = false;
  if (n_heads == 1 && plans[0].mfma) {
    PrepStartArgs ps;
    memset(&ps, 0, sizeof(ps));
    const LayerPlan& p0 = plans[0];
    for (int l = 0; l < n_layers && ps.n_jobs < kStartJobs; ++l) {
      const LayerPlan& p = plans[l];
      if (!p.mfma || p.wide || p.stream != p0.stream || p.products != p0.products || p.cfg.code != p0.cfg.code || p.cfg.gb_kind != p0.cfg.gb_kind ||
          p.cfg.idx_u32 != p0.cfg.idx_u32)
        continue;
      GatherArgs a;
      layer_args(l, 0, 1, x, 0, &a, nullptr);
      WsPtrs wl_ptrs = w;
      wl_ptrs.cf = cf_base + wl.cf_off[l] / sizeof(uint4);
      wl_ptrs.bp = bp_base + wl.bp_off[l] / sizeof(float);
      PrepCoefArgs pc;
      (void)run_prep_coef(p, a, 1, wl_ptrs, &pc, false, s);
      PrepStartArgs::Job& job = ps.job[ps.n_jobs++];
      job.cf = pc.cf;
      job.cf_lo = pc.cf_lo;
      job.bp = pc.bias_partial;
      job.n_in = pc.n_in;
      job.n_out = pc.n_out;
      job.h = pc.h[0];
      coef_done[l] = 1;
    }
    GatherArgs a0;
    layer_args(0, 0, 1, x, 0, &a0, nullptr);
    BasisBufs bb;
    (void)run_prep_basis(p0, a0, 1, true, w, Chain(), &bb, false, s);
    ps.rot = p0.rot();
    ps.rot_coef = p0.stream;
    if (p0.rot()) ps.rw = rot_words(p0, a0, 1, true, w);
    ps.x = x;
    ps.W = w.u;
    ps.W_lo = bb.u_lo;
    ps.n_in = p0.kind == kPlanMfma ? a0.n_in : 0;
    ps.B = a0.B;
    ps.rule = a0.rule;
    if (prep_start_blocks(ps) <= kPrepStartMaxBlocks) {
      st = run("kan_prep_start", s, [&] { return launch_prep_start(p0.cfg, ps, p0.products == 3, s); });
      if (st != KAN_OK) return st;
      basis0_done = true;
    } else {                                   // too many workgroups for one grid: the layers launch their own
      coef_done.assign(n_layers, 0);
    }
  }

  struct LayerScope {      // launches of the loop below are timed per layer
    ~LayerScope() { if (g_prof.on) g_prof.cur_layer = 0; }
  } layer_scope;
  for (int l = 0; l < n_layers; ++l) {
    if (g_prof.on) g_prof.cur_layer = l + 1;       // (timing hooks: one thread, nothing else in flight)
    const kan_vq_layer& R = layers[l];
    const bool last = (l + 1 == n_layers);
    w.cf = cf_base + wl.cf_off[l] / sizeof(uint4);
    w.bp = bp_base + wl.bp_off[l] / sizeof(float);
    const float* src = (l == 0) ? x : w.hid[(l - 1) & 1];
    long long src_head_stride = (l == 0) ? 0 : (long long)B * R.in;
    Chain chain;
    chain.partial = (l & 1) ? w.partial2 : w.partial;
    if (!wl.partial2) chain.partial = w.partial;
    chain.out = wl.handed[l];
    if (l > 0 && wl.handed[l - 1]) {
      src = ((l - 1) & 1) ? w.partial2 : w.partial;
      chain.in_parts = plans[l - 1].n_chunks;
      chain.in_part_stride = (long long)B * R.in;
      chain.in_tanh = 1;
      src_head_stride = chain.in_part_stride * chain.in_parts;
    }
    float* dst = last ? y : w.hid[l & 1];
    const long long dst_head_stride = (long long)B * R.out;
    for (int h0 = 0; h0 < n_heads; h0 += kMaxGroup) {
      const int heads = (n_heads - h0) < kMaxGroup ? (n_heads - h0) : kMaxGroup;
      GatherArgs a;
      const void* prepared[kMaxGroup];
      layer_args(l, h0, heads, src, src_head_stride, &a, prepared);
      chain.coef_done = coef_done[l] != 0;
      chain.basis_done = l == 0 && basis0_done;
      st = run_layer_group(plans[l], a, prepared, heads, l == 0, dst + (long long)h0 * dst_head_stride, dst_head_stride, w,
                           last ? 0 : 1, s, chain);
      if (st != KAN_OK) return st;
    }
  }
  return KAN_OK;
}
}  // namespace

kan_status kan_vq_head_forward(const kan_vq_layer* layers, int32_t n_layers, int32_t n_heads, const float* x,
                               int64_t B, float* y, void* ws, size_t ws_bytes, int32_t path, void* stream) {
  return head_forward(layers, n_layers, n_heads, x, B, y, ws, ws_bytes, false, path, stream);
}

kan_status kan_vq_head_forward_static(const kan_vq_layer* layers, int32_t n_layers, int32_t n_heads, const float* x,
                                      int64_t B, float* y, int32_t path, void* stream) {
  return head_forward(layers, n_layers, n_heads, x, B, y, nullptr, 0, true, path, stream);
}

kan_status kan_vq_layer_forward(const kan_vq_layer* L, const float* x, int64_t B, float* y, void* ws,
                                size_t ws_bytes, int32_t path, void* stream) {
  return kan_vq_head_forward(L, 1, 1, x, B, y, ws, ws_bytes, path, stream);
}

// The dense baseline: the one-pass kernels of kan_dense.hip (fp32 operands up to 16 samples, split operands above)
// while reading the coefficients once per tile of 64 samples costs less than converting them, from there the
// split-operand streaming form the precise VQ path uses (a converter of the coefficients in place of gather +
// dequantise).
static LayerPlan plan_dense(int32_t in, int32_t out, int64_t B) {
  const long long edges = (long long)in * out;
  LayerPlan p;
  p.mfma = false;
  p.kind = kPlanDense;
  p.name = B < kDenseSplitMinBatch ? "kan_dense" : "kan_dense_split";
  p.cfg = GatherCfg{B < kDenseSplitMinBatch ? 16 : (B <= 32 ? 32 : 64), 1, 1, 0, 0, kDense};
  const int tile_n = p.cfg.bt == 16 ? 16 : 64, step = p.cfg.bt == 16 ? kDenseStep16 : kDenseStep64;
  p.n_jt = (out + tile_n - 1) / tile_n;
  p.n_bt = (int)((B + p.cfg.bt - 1) / p.cfg.bt);
  // Partial sums below a quarter of the coefficients, of small layers, whose launch is a latency chain, below all of them (300 x 64
  // at batch 64 / 256 11.1 / 31.3 -> 11.1 / 11.4 us, 100 x 100 at 400 25.1 -> 11.6).
  const long long base = (long long)p.n_jt * p.n_bt, steps = ((long long)in + step - 1) / step;
  const long long sums = edges * 40 / (edges <= kFusedSmallLayerEdges ? 1 : 4);
  const long long most = std::max(1ll, std::min(steps, std::max(sums, kDenseSmallSums) / (4 * B * out)));
  if (p.cfg.bt == 16) {          // two workgroups of four waves per CU
    const long long chunks = std::min((kTargetWorkgroups + base - 1) / base, most);
    const int rows = (int)((in + chunks - 1) / chunks);
    p.rows_per_chunk = (rows + step - 1) / step * step;
    p.n_chunks = (in + p.rows_per_chunk - 1) / p.rows_per_chunk;
    return p;
  }
  // One workgroup of eight waves per CU: steps of the rounds that the chunks take, the reduction and the sums (us, fitted
  // to 22,788 launches, 5 % off).  A chunk for every CU that 256 / base, rounded up, asked for made 296 workgroups of 148:
  // 64 x 2347 at batch 253 23.5 us, whole 15.4; 1408 x 3750 at 18 92 -> 64, 384 x 2880 at 39 34 -> 25.
  const bool two = p.cfg.bt == 64;
  double one_pass = 0;
  for (long long r = 0; r <= 4; ++r) {                   // whole; as many as r rounds hold
    const long long c = std::clamp<long long>(r * kCUs / base, 1, most);
    if (r > 0 && c == 1) continue;
    const long long per = ((in + c - 1) / c + step - 1) / step, chunks = (steps + per - 1) / per, rounds = (base * chunks + kCUs - 1) / kCUs;
    const double cost = (two ? 4.5 : 2.9) * (double)(per * rounds) + (two ? 0.8 : 0.9) * (double)per + (two ? 1.1 : 2.3) * (double)rounds +
                        (chunks > 1 ? 2.3 + 3.2e-6 * (double)(chunks * B * out) : 0.0);
    if (r > 0 && cost >= one_pass) continue;
    one_pass = cost;
    p.rows_per_chunk = (int)(per * step);
    p.n_chunks = (int)chunks;
  }
  if (!two || B <= 64) return p;
  one_pass += 2.2 + 4.2e-6 * (double)edges;
  // The other forms, fitted below and from batch 1024 on (6 to 8 % off, records 15; the choice is within 1 % of the best on average).
  const bool many = B >= kDenseManySamples;
  const LayerPlan records = plan_mfma(in, out, B, 1, 0, 0, kDense, true);
  LayerPlan m = records;
  const double inputs = 1e-6 * (double)B * in, outputs = 4e-6 * (double)(B * out);
  const long long tile_steps = base * steps;
  if (make_wide(m, in, out, B, 1, true, 1, true)) {
    const long long per = m.rows_per_chunk / 16, rounds = ((long long)m.n_jt * m.n_bt * m.n_chunks + kCUs - 1) / kCUs;
    const bool tall = m.cfg.bt > 128;
    const double sums_out = m.n_chunks > 1 ? m.n_chunks * outputs : 0.0;
    const double wide = many ? 7.7 + 2.66 * (double)(rounds * per) + 1.4 * (double)rounds + 6.05 * inputs + 0.23 * outputs + 0.26 * sums_out + (m.n_chunks > 1 ? 3.4 : 0.0)
                             : 3.4 + (tall ? 2.5 : 1.85) * (double)(rounds * per) + (tall ? 6.0 : 5.6) * (double)rounds + 6.4 * inputs + 1.8e-6 * (double)edges +
                                   0.39 * sums_out + (m.n_chunks > 1 ? 2.6 : 0.0);
    if (one_pass <= wide && (!many || tile_steps <= kDenseOnePassMaxSteps)) return p;
    if (many) {
      const long long wgs = (long long)records.n_jt * records.n_bt * records.n_chunks, cut = records.n_chunks > 1;
      const double by_records = 11.0 + 33.4e-6 * (double)edges + 5.9 * inputs + 0.6 * outputs + cut * (1.8 + 0.33 * records.n_chunks * outputs) +
                                (2.4 * (double)((wgs + 2 * kCUs - 1) / (2 * kCUs)) + 0.8 * (double)((wgs + kCUs - 1) / kCUs)) * (records.rows_per_chunk / 16);
      if (by_records < wide || B * edges >= kDenseWideMaxWork) m = records;
    }
  } else if (many ? tile_steps <= kDenseOnePassMaxSteps : one_pass <= 0.85 * (19.5 + 92.5e-6 * (double)edges + 11.7 * inputs)) {
    return p;
  }
  m.name = "kan_dense_split";
  return m;
}

static void dense_ws(const LayerPlan& p, int32_t in, int32_t out, int64_t B, size_t* partial, size_t* cf, size_t* u) {
  *partial = partial_bytes(p, out, B, 1);
  *cf = p.mfma && !p.wide ? round_up(2 * mfma_cf_records(in, out) * sizeof(uint4), 256) : 0;
  *u = !p.mfma ? 0 : round_up(2 * (size_t)((in + 15) / 16) * (size_t)B * (p.wide ? 10 * sizeof(uint4) : 16 * sizeof(uint2)), 256);
}

size_t kan_dense_workspace_bytes(int32_t in, int32_t out, int64_t B) {
  if (in < 1 || out < 1 || in > kMaxDim || out > kMaxDim || B < 0 || B > kMaxBatch) return (size_t)-1;
  if (B == 0) return 0;
  size_t partial, cf, u;
  dense_ws(plan_dense(in, out, B), in, out, B, &partial, &cf, &u);
  return partial + cf + u;
}

kan_status kan_dense_layer_forward(const float* coef, int32_t in, int32_t out, int32_t G, const float* x,
                                   int64_t B, float* y, void* ws, size_t ws_bytes, void* stream) {
  if (G != 10) return KAN_ERR_UNSUPPORTED;
  if (in < 1 || out < 1 || in > kMaxDim || out > kMaxDim || B < 0 || B > kMaxBatch) return KAN_ERR_SHAPE;
  if (B == 0) return KAN_OK;
  if (!coef || !x || !y) return KAN_ERR_NULL;
  if (!aligned(coef, 8) || !aligned(x, 4) || !aligned(y, 4)) return KAN_ERR_SHAPE;
  const LayerPlan p = plan_dense(in, out, B);
  size_t partial, cf, u;
  dense_ws(p, in, out, B, &partial, &cf, &u);
  const size_t need = partial + cf + u;
  if (need > 0 && (!ws || !aligned(ws, 256) || ws_bytes < need)) return KAN_ERR_WORKSPACE;
  GatherArgs a;
  memset(&a, 0, sizeof(a));
  a.x = x;
  a.n_in = in;
  a.n_out = out;
  a.B = (int)B;
  a.rows_per_chunk = p.rows_per_chunk;
  a.n_jt = p.n_jt;
  a.h[0].cb = coef;
  a.h[0].scale = 1.0f;
  WsPtrs w;
  memset(&w, 0, sizeof(w));
  w.partial = (float*)ws;
  w.cf = (uint4*)((char*)ws + partial);
  w.u = (uint2*)((char*)ws + partial + cf);
  return run_layer_group(p, a, nullptr, 1, true, y, (long long)B * out, w, 0, (hipStream_t)stream);
}

size_t kan_vq_prepared_bytes(const kan_vq_layer* L) {
  if (validate_layer(L) != KAN_OK) return (size_t)-1;
  if (L->in > kBucketMaxIn || (long long)L->in * L->out > (1ll << 31)) return 0;
  return bucket_geometry(L->in, L->out, L->K, code_of(*L), gb_kind_of(*L)).total;
}

kan_status kan_vq_prepare(const kan_vq_layer* L, void* prepared, size_t prepared_bytes, void* stream) {
  kan_status st = validate_layer(L);
  if (st != KAN_OK) return st;
  if (L->in > kBucketMaxIn) return KAN_ERR_UNSUPPORTED;
  if ((long long)L->in * L->out > (1ll << 31)) return KAN_ERR_UNSUPPORTED;   // 32-bit segment offsets
  const BucketGeom g = bucket_geometry(L->in, L->out, L->K, code_of(*L), gb_kind_of(*L));
  if (!prepared || !aligned(prepared, 256) || prepared_bytes < g.total) return KAN_ERR_WORKSPACE;
  LayerPtrs h = {L->idx, L->gain, L->bias, L->codebook, L->scale, L->gain_log2_lo, L->gain_log2_step, L->bias_scale};
  hipStream_t s = (hipStream_t)stream;
  return run("kan_vq_prepare", s, [&] {
    return launch_bucket_prepare(h, L->idx_dtype == KAN_U32, gb_kind_of(*L), L->in, L->out, g, prepared, s);
  });
}

size_t kan_vq_assign_workspace_bytes(int32_t K) {
  if (K < 1) return (size_t)-1;
  return round_up(assign_centroid_bytes(K), 256);
}

namespace {
kan_status check_assign_shapes(int32_t in, int32_t out, int32_t K, int32_t idx_dtype) {
  if (in < 1 || out < 1 || in > kMaxDim || out > kMaxDim || K < 1) return KAN_ERR_SHAPE;
  if ((long long)in * out > (1ll << 31)) return KAN_ERR_SHAPE;
  if (idx_dtype != KAN_U16 && idx_dtype != KAN_U32) return KAN_ERR_DTYPE;
  if (idx_dtype == KAN_U16 && K > 65536) return KAN_ERR_SHAPE;
  return KAN_OK;
}
}  // namespace

size_t kan_vq_assign_fast_workspace_bytes(int32_t in, int32_t out, int32_t K) {
  if (check_assign_shapes(in, out, K, KAN_U32) != KAN_OK) return (size_t)-1;
  const long long E = (long long)in * out;
  const size_t least = kan_vq_assign_workspace_bytes(K);
  if (!assign_bounded_ok(E, K)) return round_up(assign_whole_bytes(E, K), 256);
  const size_t bounded = round_up(assign_bounded_bytes(E, K), 256);
  return bounded > least ? bounded : least;
}

kan_status kan_vq_assign(const float* coef, int32_t in, int32_t out, const float* codebook, int32_t K,
                         int32_t idx_dtype, void* idx, float* gain, float* bias, void* ws, size_t ws_bytes,
                         void* stream) {
  kan_status st = check_assign_shapes(in, out, K, idx_dtype);
  if (st != KAN_OK) return st;
  if (!coef || !codebook || !idx || !gain || !bias) return KAN_ERR_NULL;
  if (!aligned(coef, 8) || !aligned(codebook, 4) || !aligned(gain, 4) || !aligned(bias, 4) ||
      !aligned(idx, idx_dtype == KAN_U16 ? 2 : 4))
    return KAN_ERR_SHAPE;
  if (!ws || !aligned(ws, 256) || ws_bytes < kan_vq_assign_workspace_bytes(K)) return KAN_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const bool bounded = assign_bounded_ok((long long)in * out, K) && ws_bytes >= kan_vq_assign_fast_workspace_bytes(in, out, K);
  return run("kan_vq_assign", s, [&] {
    if (bounded)
      return launch_assign_bounded(coef, (long long)in * out, codebook, K, idx_dtype == KAN_U32, idx, gain, bias, ws, s);
    return launch_assign(coef, (long long)in * out, codebook, K, idx_dtype == KAN_U32, idx, gain, bias, ws, ws_bytes, s);
  });
}

size_t kan_vq_reconstruction_workspace_bytes(int32_t in, int32_t out) {
  if (in < 1 || out < 1 || in > kMaxDim || out > kMaxDim) return (size_t)-1;
  return round_up((size_t)recon_blocks((long long)in * out) * 3 * sizeof(double), 256);
}

kan_status kan_vq_reconstruction_sums(const float* coef, int32_t in, int32_t out, const float* codebook, int32_t K,
                                      int32_t idx_dtype, const void* idx, const float* gain, const float* bias,
                                      double* sums, void* ws, size_t ws_bytes, void* stream) {
  kan_status st = check_assign_shapes(in, out, K, idx_dtype);
  if (st != KAN_OK) return st;
  if (!coef || !codebook || !idx || !gain || !bias || !sums) return KAN_ERR_NULL;
  if (!aligned(coef, 4) || !aligned(codebook, 4) || !aligned(gain, 4) || !aligned(bias, 4) || !aligned(sums, 8) ||
      !aligned(idx, idx_dtype == KAN_U16 ? 2 : 4))
    return KAN_ERR_SHAPE;
  if (!ws || !aligned(ws, 256) || ws_bytes < kan_vq_reconstruction_workspace_bytes(in, out)) return KAN_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  return run("kan_vq_reconstruction_sums", s, [&] {
    return launch_recon_sums(coef, (long long)in * out, codebook, idx_dtype == KAN_U32, idx, gain, bias, (double*)ws,
                             sums, s);
  });
}

kan_status kan_vq_debug_gather(const kan_vq_layer* L, uint32_t* ids, float* rows, void* stream) {
  kan_status st = validate_layer(L);
  if (st != KAN_OK) return st;
  if (!ids && !rows) return KAN_ERR_NULL;
  LayerPtrs h = {L->idx, L->gain, L->bias, L->codebook, L->scale, 0.f, 0.f, 0.f};
  hipStream_t s = (hipStream_t)stream;
  return run("kan_debug_gather", s, [&] {
    return launch_debug_gather(h, L->idx_dtype == KAN_U32, code_of(*L),
                               (long long)L->in * L->out, ids, rows, s);
  });
}

kan_status kan_vq_count_bad_indices(const kan_vq_layer* L, uint32_t* count, void* stream) {
  kan_status st = validate_layer(L);
  if (st != KAN_OK) return st;
  if (!count) return KAN_ERR_NULL;
  hipStream_t s = (hipStream_t)stream;
  return run("kan_count_bad", s, [&] {
    return launch_count_bad(L->idx, L->idx_dtype == KAN_U32, (long long)L->in * L->out, (uint32_t)L->K,
                            count, s);
  });
}

kan_status kan_vq_coef_range(const kan_vq_layer* L, float* range, void* stream) {
  kan_status st = validate_layer(L);
  if (st != KAN_OK) return st;
  if (!range) return KAN_ERR_NULL;
  if (!aligned(range, 4)) return KAN_ERR_SHAPE;
  LayerPtrs h = {L->idx, L->gain, L->bias, L->codebook, L->scale, L->gain_log2_lo, L->gain_log2_step, L->bias_scale};
  hipStream_t s = (hipStream_t)stream;
  return run("kan_coef_range", s, [&] {
    return launch_coef_range(h, L->idx_dtype == KAN_U32, gb_kind_of(*L), code_of(*L), (long long)L->in * L->out, range, s);
  });
}

const char* kan_vq_planned_kernel(const kan_vq_layer* L, int64_t B, int32_t n_heads, int32_t path) {
  if (validate_layer(L) != KAN_OK || check_path(path) != KAN_OK || B < 1 || n_heads < 1) return "invalid";
  // as a call of such layers is planned, its scratch included (a group of heads is as good as all of them)
  const int group = n_heads < kMaxGroup ? n_heads : kMaxGroup;
  const std::vector<kan_vq_layer> heads((size_t)group, *L);
  std::vector<LayerPlan> plans;
  WsLayout ws;
  if (plan_head(heads.data(), 1, group, std::min<int64_t>(B, kMaxBatch), path, &plans, &ws) != KAN_OK) return "invalid";
  return plans[0].name;
}

const char* kan_dense_planned_kernel(int32_t in, int32_t out, int64_t B) {
  if (in < 1 || out < 1 || in > kMaxDim || out > kMaxDim || B < 1 || B > kMaxBatch) return "invalid";
  return plan_dense(in, out, B).name;
}

kan_status kan_prof_begin(int32_t max_launches) {
  if (max_launches < 1 || max_launches > (1 << 20)) return KAN_ERR_SHAPE;
  if (g_prof.on) return KAN_ERR_UNSUPPORTED;
  g_prof.ev.assign(2 * (size_t)max_launches, nullptr);
  g_prof.names.assign(max_launches, nullptr);
  g_prof.layer.assign(max_launches, 0);
  for (auto& e : g_prof.ev)
    if (hipEventCreate(&e) != hipSuccess) return KAN_ERR_LAUNCH;
  g_prof.cap = max_launches;
  g_prof.n = 0;
  g_prof.on = true;
  return KAN_OK;
}

kan_status kan_prof_end(kan_prof_record* out, int32_t cap, int32_t* n_out) {
  if (!g_prof.on) return KAN_ERR_UNSUPPORTED;
  g_prof.on = false;
  int n_rec = 0;
  kan_status st = KAN_OK;
  for (int n = 0; n < g_prof.n; ++n) {
    float ms = 0.f;
    if (hipEventSynchronize(g_prof.ev[2 * n + 1]) != hipSuccess ||
        hipEventElapsedTime(&ms, g_prof.ev[2 * n], g_prof.ev[2 * n + 1]) != hipSuccess) {
      st = KAN_ERR_LAUNCH;
      break;
    }
    char key[sizeof(out[0].name)];
    if (g_prof.layer[n] > 0) snprintf(key, sizeof(key), "%s@L%d", g_prof.names[n], g_prof.layer[n]);
    else snprintf(key, sizeof(key), "%s", g_prof.names[n]);
    int r = 0;
    for (; r < n_rec; ++r)
      if (strcmp(out[r].name, key) == 0) break;
    if (r == n_rec) {
      if (!out || n_rec >= cap) continue;
      memset(&out[r], 0, sizeof(out[r]));
      memcpy(out[r].name, key, sizeof(key));
      ++n_rec;
    }
    out[r].launches += 1;
    out[r].total_ms += ms;
  }
  for (auto& e : g_prof.ev)
    if (e) (void)hipEventDestroy(e);
  g_prof.ev.clear();
  g_prof.names.clear();
  g_prof.layer.clear();
  g_prof.cur_layer = 0;
  if (n_out) *n_out = n_rec;
  return st;
}

}  // extern "C"
