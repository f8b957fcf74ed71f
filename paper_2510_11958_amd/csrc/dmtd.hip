// C ABI of the DMTD decode path (see include/dmtd.h): context, workspace layout, step
// assembly, hipGraph capture/replay and the host-visible calls.
//
// Two kernel paths share the step assembly:
//  - bf16 models ("packed" path): weights repacked once into MFMA operand order, all
//    projections through the MFMA weight-streaming kernel, activations handed from kernel
//    to kernel as packed bf16 rows plus partial sums of squares for the next RMSNorm;
//  - the fp32 parity model: FMA weight-streaming kernels with the norm computed in-kernel.
#include "../../include/dmtd.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <tuple>
#include <type_traits>
#include <vector>

#include "kernels.hpp"
#include "sched.hpp"

using namespace dmtd;

namespace {

constexpr int kMaxTau = 64;          // steps per decode call (size of the emitted-token buffer)
constexpr int kGemvRows = 4;         // activation rows per FMA weight-streaming pass
constexpr int kMaxRows = 16;         // rows per sequence one pass through the layers may carry
constexpr int kPassRows = 128;       // activation rows (all sequences together) a prefill or whole-sequence pass of an fp32 model carries
// The same for a bf16 model.  Its wide GEMM (gemm_wide.hpp) is bound by the matrix cores, so a pass should fill the chip with
// its tiles whatever the projection: 2048 rows give gate/up 608 tiles of 256 x 256 at 4B shapes (512 whole, 96 in two parts of K), QKV 384 of
// 128 x 256 and O and down 80 (their K is split over the 256 CUs).  The activation buffers of such a pass and 512 rows of logits make a 4B context of one sequence 137 MB
// larger than passes of 128 rows did; with less workspace the passes are shorter.
constexpr int kWideRows = 2048;
constexpr int kHeadRows = 512;       // rows of a whole-sequence pass whose logits are held at a time (0.3 GB at a 152k vocabulary)
// Up to this many rows go through the LDS-tiled kernel in passes of 128, more through the wide GEMM.  All four projections of a layer with their
// finishing launches, us, tiled / wide: 2560 wide, 128 rows 111 / 120, 144 rows 163 / 150, 192 rows 188 / 153; 1024 wide 70 / 76, 100 / 81, 117 / 85.
// The line stems from tiles of 256 rows only (192 rows 191 / 190); with those of 128 the kernels meet at 128 rows.
constexpr int kTiledRows = 192;
// Rows per sequence and in all that a decode step may carry: what the attention's partial results are laid out for.
inline int step_row_capacity(int max_batch) { return max_batch * kMaxRows > kPassRows ? max_batch * kMaxRows : kPassRows; }
inline int step_positions(int batch) { const int r = kPassRows / batch; return r > kMaxRows ? r : kMaxRows; }
// Row capacity of the activation buffers: a decode step's rows, and a prefill pass's (never more than the longest batch has).
// wide: rows of a bf16 model's pass (kWideRows, fewer where the caller's workspace does not hold that many: dmtd_create)
inline int row_capacity(const dmtd_config& c, int wide) {
  long cap = step_row_capacity(c.max_batch);
  if (c.dtype == DMTD_DTYPE_BF16) {
    const long all = (long)c.max_batch * c.max_seq_len;
    cap = std::max(cap, std::min<long>(wide, (all + 15) / 16 * 16));
  }
  return (int)cap;
}
// Packed rows of the late layers, one per sequence: whole groups of 16 where they may be in the wide GEMM's layout, which stores them so
inline size_t late_row_capacity(const dmtd_config& c) { return c.max_batch > kTiledRows ? ((size_t)c.max_batch + 15) / 16 * 16 : (size_t)c.max_batch; }
inline int head_row_capacity(const dmtd_config& c, int wide) {
  return c.dtype == DMTD_DTYPE_BF16 ? std::min(row_capacity(c, wide), std::max(kHeadRows, step_row_capacity(c.max_batch))) : row_capacity(c, wide);
}
// Positions per sequence of a prefill or whole-sequence pass.  Full passes and a short last one rather than equal ones: a full
// pass is 8 row tiles of the wide GEMM, and equal passes would pad each to whole tiles (3 x 701 positions at 4B shapes: 2046 + 57
// rows against 1056 + 1047, which are 5 tiles each).
inline int pass_positions(const dmtd_config& c, int wide, int batch) {
  return c.dtype == DMTD_DTYPE_BF16 ? std::max(wide / batch, kMaxRows) : step_positions(batch);
}
// Entries of a sequence's list of a sampled step
inline int sample_cap(const dmtd_config& c) { return std::min(SAMPLE_CAP, c.vocab); }
constexpr int kMaxPatterns = 64;     // distinct step patterns (which sequences start a cycle, with how many rows) a context keeps on the device
constexpr size_t kPatternStride(size_t max_batch) { return (max_batch * 5 + 255) / 256 * 256; }   // int list [max_batch] + byte mask [max_batch]
constexpr int kMfmaRows = 16;        // activation rows per pass of the one-tile-per-block MFMA kernel
#ifndef DMTD_GEMM_MAXSPLIT
#define DMTD_GEMM_MAXSPLIT 12
#endif
constexpr int kGemmMaxSplit = DMTD_GEMM_MAXSPLIT;   // K splits of the tiled kernel at most (sizes the partial-sum buffer)
#ifndef DMTD_FIT_SMALL_KB
#define DMTD_FIT_SMALL_KB 60
#endif
#ifndef DMTD_GEMM_ROWS
#define DMTD_GEMM_ROWS 128
#endif
constexpr int kGemmRows = DMTD_GEMM_ROWS;   // activation rows per pass of the LDS-tiled MFMA kernel (launches with more than 16 rows)
// Key ranges an O projection's blocks merge by themselves (two kernels: up to 4 and up to 8), and the bytes of partial results
// every block may read for that.  us per step with the merge launch / merged here: 64 KiB 331.6 / 319.9 (2560 wide, 6
// layers, 4 ranges), 350.7 / 333.4 (1024 wide, 12 layers, 2 rows); 128 KiB 330.8 / 326.1 (8 ranges), 354.5 / 346.1; 256 KiB
// 337.3 / 346.4 and 374.4 / 392.3: a block's prologue then takes longer than the launch.
constexpr int kMergeFew = 4, kMergeRanges = 8;
constexpr size_t kMergeBytes = 128 * 1024;
constexpr int kMfmaPF = 10;          // k-steps (64 elements) a wave of the MFMA kernel holds in registers
// Waves that split K for one matrix (NW) and k-steps a wave keeps in flight as a rolling window (PF), per projection;
// NW = 0: the one-round rule of launch_mfma with kMfmaPF.  Defaults from sweeps at 4B shapes on MI355X, us per launch
// with 3 rows / 1 row: gate/up 4 x 2: 18.9 / 18.1 (4 x 4: 19.5 / 19.1), down 16 x 3: 11.3 / 10.7 (16 x 5: 11.3 / 10.9),
// O 8 x 4: 6.3 / 6.2 (16 x 5: 8.0 / 7.3), QKV 8 x 2: 7.6 / 7.5 (one round of 5: 8.0 / 7.7); the LM head measures
// 131 us whatever the shape (it runs at the memory system's rate).  Short windows win since every load of the
// prologue is issued without a wait in between: the first k-step's matrix-core work starts as soon as it lands.
// The macros exist so a sweep can override them at build time.
#ifndef DMTD_GU_NW
#define DMTD_GU_NW 4
#define DMTD_GU_PF 2
#endif
#ifndef DMTD_DN_NW
#define DMTD_DN_NW 16
#define DMTD_DN_PF 3
#endif
#ifndef DMTD_O_NW
#define DMTD_O_NW 8
#define DMTD_O_PF 4
#endif
#ifndef DMTD_LM_NW
#define DMTD_LM_NW 5
#define DMTD_LM_PF 4
#endif
#ifndef DMTD_Q_NW
#define DMTD_Q_NW 8
#define DMTD_Q_PF 2
#endif
constexpr int kMfmaPFQkv = 5;        // the same for the QKV projection: shorter runs put 8 waves on a tile (measured 8.3 us instead of 9.3 us at 4B shapes)

thread_local std::string g_create_error;

// The library's own scratch for dmtd_decode_cycle_noalloc (callers that cannot allocate and hand over no workspace for
// partial results).  One copy per GPU the library runs on, held until the process ends; every context on a GPU shares
// it, so two such calls that overlap on one GPU race.  The name below is a host-side stand-in: the device address is
// taken once per device with hipGetSymbolAddress (dmtd_create) and only that address is ever handed to kernels.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
char* g_scratch_ptr[kMaxDevices] = {};

hipError_t static_scratch_for_current_device(char** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = (char*)p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

struct LayerW {   // tensors of one layer inside the caller's blob
  const void *attn_norm, *q, *k, *v, *q_norm, *k_norm, *o, *mlp_norm, *gate, *up, *down;
};
struct LayerSw {  // the layer's matrices in MFMA operand order (workspace; bf16 models only)
  const bf16_t *qkv, *o, *gate, *up, *down;
};

struct Ws {   // device workspace carve-up (byte offsets)
  size_t kv, kv_layer_stride, kv_v_off;
  size_t h, h_late, qkv, attn, mlp, logits, part_o, part_ml, amax;
  size_t tokens, emitted, forced, state, inv_freq, rope_tab;
  size_t xb, xb_late, ssp, ssp_late, wsw;      // packed path only
  size_t gemm_part;                            // K-split partial sums of the tiled kernel
  size_t patterns;
  size_t sample_count, sample_list, sample_best;   // sampled steps: per sequence the list of entries that may stay in, and the slices' best draws
  size_t pend_enc, enc_tmp;                    // ExDy: stored encoding outputs of pending tokens; of a prefill chunk
  // whole-sequence masked forward: mask, a chunk's logits, the LM head's selection keys for them (written by its kernels, read by
  // nobody: nll_rows_kernel finds the best entry of a row itself), per-position results
  size_t mask, logits_rows, amax_rows, nll, best, loss;
  size_t total;
};

// Activation rows in flight between kernels.  On the packed path xb holds bf16(h * gain of
// the norm that reads the rows next) and ssp the partial sums of h^2 (n_parts of them per row).
struct Rows {
  float* h;
  bf16_t* xb;      // high parts
  bf16_t* xb_lo;   // low parts
  float* ssp;
  int n_parts;
};

}  // namespace

struct dmtd_ctx {
  dmtd_config cfg;
  Sched sched;
  std::string err;
  hipStream_t stream = nullptr;
  int elem = 2;
  bool packed = false;        // bf16 model: MFMA path
  int num_cus = 256;
  int batch = 0;              // batch of the current sequence set (after prefill)
  int wide_rows = kWideRows;  // activation rows of a bf16 model's prefill or whole-sequence pass
  int ssp_ld = 0;             // row capacity of the sum-of-squares buffers
  const char* wbase = nullptr;
  char* ws = nullptr;
  Ws o{};
  const void* embed = nullptr;
  const void* final_norm = nullptr;
  const void* lm_head = nullptr;
  const bf16_t* lm_head_sw = nullptr;
  std::vector<LayerW> layers;
  std::vector<LayerSw> sw;
  std::map<std::tuple<int, int, int, int, int>, hipGraphExec_t> graphs;   // (full, rows, n_late / n_early / sampling, bucket / share_kv, batch)
  std::map<std::vector<int>, hipGraphExec_t> group_graphs;            // several steps in one graph (dmtd_decode)
  bool sampling = false;      // tokens are drawn (dmtd_set_sampling) instead of taken greedily
  bool share_kv = false;      // attention launches: one pass over K/V for all rows of a sequence (long contexts)
  int att_bucket = 512;       // attention launches: context bucket (256 or a multiple of 512) the key ranges are laid out for
  int late_batch = 0;         // a front pass over some sequences: sequences of the whole batch (0: all are in the pass)
  int resid_parts = 0;        // partial sums of squares per row the last residual projection left for the next norm
  const int* fmap = nullptr;  // launches of a front pass over SOME sequences: launch sequence -> sequence slot (device); null = all, in order
  const int* live = nullptr;  // ... and the rows each of them has (host; the launch has room for the largest number); null = all rows of the launch
  const unsigned char* full_mask = nullptr;   // the step's bookkeeping: which sequences close their refill gap (device); null = all or none
  // sequences at different points of their cycles (dmtd_decode_per_seq): per-sequence phase and front position (in the
  // counters' coordinates); while `diverged` the single-phase calls are refused
  std::vector<int> seq_phase, seq_front;
  bool diverged = false;
  std::map<std::vector<int>, int> pattern_ids;      // rows per sequence of a step (0 = late-only) -> slot in the device pattern table
  std::map<std::vector<int>, hipGraphExec_t> mixed_graphs;
  bool fold_qkv = false;      // run_layer: a K-split QKV launch may leave its finishing step to the attention launch that follows
  QkvSrc qkv_pending{};       // ... and says so here (part != nullptr) until that launch picks it up
  bool fold_merge = false;    // run_layer: an attention launch over key ranges may leave their merge to the O projection that follows
  MergeSrc merge_pending{};   // ... and says so here (po != nullptr) until that launch picks it up
  // Scratch of the step kernels (partial results that live for one launch pair): the attention ranges' partial outputs
  // and softmax statistics, the LM head's selection-key cells, the K-split partial sums of the tiled kernel.  They sit
  // in the caller's workspace, except inside dmtd_decode_cycle_noalloc, which points them at the library's own array.
  float* part_o = nullptr;
  float* part_ml = nullptr;
  unsigned long long* amax = nullptr;
  float* gemm_part = nullptr;
  int part_rows = 0;          // rows per sequence the partials are laid out for (stride between ranges: part_rows * query heads per KV head)
  int test_fail_step = -1;    // tests of the failure path: the next decode call reports a launch failure before this step (once)
  char* static_scratch = nullptr;   // this device's copy of the library's own scratch array (address taken at create)
  std::vector<Step> plan_buf;       // dmtd_decode_cycle_noalloc: the call's steps (capacity reserved at create)
};

namespace {

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

bool valid_config(const dmtd_config* c, std::string& why) {
  if (!c) { why = "null config"; return false; }
  if (c->n_layers < 1 || c->hidden < 8 || c->n_q_heads < 1 || c->n_kv_heads < 1 || c->intermediate < 8 || c->vocab < 2) {
    why = "non-positive model dimension"; return false;
  }
  if (c->hidden % 8 || c->intermediate % 8) { why = "hidden and intermediate must be multiples of 8"; return false; }
  if (c->head_dim != 64 && c->head_dim != 128) { why = "head_dim must be 64 or 128"; return false; }
  if (c->n_q_heads % c->n_kv_heads) { why = "n_q_heads must be a multiple of n_kv_heads"; return false; }
  if (c->n_q_heads / c->n_kv_heads > QV_MAX) { why = "too many query heads per KV head"; return false; }
  if (c->dtype != DMTD_DTYPE_F32 && c->dtype != DMTD_DTYPE_BF16) { why = "unknown dtype"; return false; }
  if (c->dtype == DMTD_DTYPE_BF16 && (c->hidden % 64 || c->intermediate % 64)) {
    why = "bf16 models need hidden and intermediate to be multiples of 64"; return false;
  }
  if (c->max_batch < 1 || c->max_seq_len < 2) { why = "max_batch >= 1 and max_seq_len >= 2 required"; return false; }
  if (!(c->rms_eps > 0.f) || !(c->rope_theta > 0.f)) { why = "rms_eps and rope_theta must be positive"; return false; }
  return true;
}

size_t weight_elems(const dmtd_config& c) {
  const size_t d = c.hidden, qd = (size_t)c.n_q_heads * c.head_dim, kd = (size_t)c.n_kv_heads * c.head_dim, ff = c.intermediate;
  const size_t per_layer = d + qd * d + 2 * kd * d + 2 * (size_t)c.head_dim + d * qd + d + 3 * ff * d;
  return (size_t)c.vocab * d + c.n_layers * per_layer + d + (c.tied_embeddings ? 0 : (size_t)c.vocab * d);
}

size_t swizzled_layer_elems(const dmtd_config& c) {
  const size_t d = c.hidden, qd = (size_t)c.n_q_heads * c.head_dim, ff = c.intermediate;
  const size_t nqkv = (size_t)(c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
  return swizzled_elems(nqkv, d) + swizzled_elems(d, qd) + 2 * swizzled_elems(ff, d) + swizzled_elems(d, ff);
}

// Floats the K-split partial sums of one launch may take (gemm_part)
size_t gemm_part_floats(const dmtd_config& c) {
  const size_t nqkv = (size_t)(c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
  return (size_t)kGemmMaxSplit * kGemmRows * std::max({2 * (size_t)c.intermediate, nqkv, (size_t)c.hidden});
}

Ws layout(const dmtd_config& c, int wide = kWideRows) {
  Ws w{};
  const size_t e = c.dtype == DMTD_DTYPE_F32 ? 4 : 2;
  const size_t B = c.max_batch, S = c.max_seq_len, d = c.hidden, hd = c.head_dim;
  const size_t nqkv = (size_t)(c.n_q_heads + 2 * c.n_kv_heads) * hd, qd = (size_t)c.n_q_heads * hd;
  const size_t rows = row_capacity(c, wide), step_rows = step_row_capacity(c.max_batch);
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
  const size_t kv_one = B * c.n_kv_heads * S * hd * e;       // K (or V) of one layer
  w.kv_v_off = align_up(kv_one, 256);
  w.kv_layer_stride = 2 * w.kv_v_off;
  w.kv = take(w.kv_layer_stride * c.n_layers);
  w.h = take(rows * d * 4);
  w.h_late = take(B * d * 4);
  // A whole-sequence pass keeps its logits where the layers' scratch is: nothing of that is alive between the last layer
  // of a chunk and the first of the next
  const size_t scratch = off;
  w.qkv = take(rows * nqkv * 4);
  w.attn = take(rows * qd * 4);                       // fp32 path: fp32 rows; packed path: bf16 rows
  w.mlp = take(rows * (size_t)c.intermediate * 4);    // likewise
  // partial results of the attention key ranges: laid out per sequence for kMaxRows rows in decode steps and for
  // step_positions in prefill (a pass with more positions takes one key range per block); sequences x rows per sequence
  // never exceeds a step's row capacity
  const size_t qv_rows = step_rows * (c.n_q_heads / c.n_kv_heads);
  w.part_o = take(c.n_kv_heads * ATT_MAX_SPLITS * qv_rows * hd * 4);
  w.part_ml = take(c.n_kv_heads * ATT_MAX_SPLITS * qv_rows * 2 * 4);
  if (c.dtype == DMTD_DTYPE_BF16) w.gemm_part = take(gemm_part_floats(c) * 4);
  w.logits_rows = scratch;
  off = std::max(off, align_up(scratch + head_row_capacity(c, wide) * (size_t)c.vocab * 4, 256));
  w.logits = take(B * (size_t)c.vocab * 4);
  w.amax = take((size_t)AMAX_CELLS * B * 8);
  w.tokens = take(B * S * 4);
  w.emitted = take((size_t)kMaxTau * B * 4);
  w.forced = take((size_t)kMaxTau * B * 4);
  w.state = take(kStateDeltaOff + 12 * B);            // counters, sampling parameters, per-sequence (delta, front position) pairs, last prompt positions
  w.patterns = take((size_t)kMaxPatterns * kPatternStride(B));   // sequence lists and masks of steps whose sequences are at different points of their cycles
  w.sample_count = take(B * 4);
  w.sample_list = take(B * sample_cap(c) * sizeof(SampleCand));
  w.sample_best = take(B * ((c.vocab + SAMPLE_SLICE - 1) / SAMPLE_SLICE) * 8);
  w.inv_freq = take((hd / 2) * 8);
  w.pend_enc = take(B * kMaxTau * d * 4);
  w.enc_tmp = take(rows * d * 4);
  w.rope_tab = take(S * (hd / 2) * 8);                 // (cos, sin) per position and frequency
  w.mask = take(S * 4);
  w.amax_rows = take((size_t)AMAX_CELLS * head_row_capacity(c, wide) * 8);
  w.nll = take(B * S * 4);
  w.best = take(B * S * 4);
  w.loss = take(B * 4);
  if (c.dtype == DMTD_DTYPE_BF16) {
    const size_t parts = (d + 15) / 16;
    w.xb = take(rows * d * 2 * 2);                     // high and low planes
    w.xb_late = take(late_row_capacity(c) * d * 2 * 2);
    w.ssp = take(parts * rows * 4);
    w.ssp_late = take(parts * rows * 4);
    // The weight image starts 1 KiB off a multiple of 2 (of the workspace, which torch puts on far larger ones).  Gate/up, us, by the
    // start modulo 2 KiB, 0 / 256 / 512 / 1024 / 1536: 2560 wide, 1 row 17.97 / 17.78 / 17.72 / 17.65 / 17.88, 3 rows 18.74 /
    // 18.48 / 18.45 / 18.30 / 18.59; the other projections and widths differ by less than their spread.
    off = (off + 1024 + 2047) / 2048 * 2048 - 1024;
    w.wsw = take((swizzled_layer_elems(c) * c.n_layers + swizzled_elems(c.vocab, d)) * 2);
  }
  w.total = off;
  return w;
}

#define HIP_TRY(ctx, expr)                                                              \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess) {                                                             \
      (ctx)->err = std::string(#expr) + ": " + hipGetErrorString(e_);                   \
      return DMTD_EHIP;                                                                 \
    }                                                                                   \
  } while (0)

// Whether the packed inputs of a pass with that many rows are in the wide GEMM's blocked layout (packed_at)
int blocked_rows(const dmtd_ctx* c, int rows) { return c->packed && rows > kTiledRows; }

DevState* dev_state(dmtd_ctx* c) { return (DevState*)(c->ws + c->o.state); }
int* sample_count(dmtd_ctx* c) { return (int*)(c->ws + c->o.sample_count); }
int* dev_tokens(dmtd_ctx* c) { return (int*)(c->ws + c->o.tokens); }
const void* norm_gain_for_layer(const dmtd_ctx* c, int l) {   // gain of the norm that opens layer l (the final norm after the last)
  return l < c->cfg.n_layers ? c->layers[l].attn_norm : c->final_norm;
}

// ------------------------------------------------------- fp32 path: FMA weight streaming

template <int M, int EPI, bool NORM>
hipError_t launch_gemv(dmtd_ctx* c, GemvArgs a, int groups) {
  // Short rows go through gemv_direct_kernel, which holds a wave's weights and rows in registers: four chunks of 256 fill 128 of them.
  // us per step of 4 layers, gemv_rows_kernel / here (with the attention of the same change): 256 wide 78.8 / 50, 32000 entries 117 / 79,
  // 16 sequences 291 / 74; 1024 wide, 1 row 174 / 141, 4 to 12 rows 213 / 101; 151936 entries, 2 layers 184 / 171.
  if (a.K <= 1024) {
    constexpr int RPW = EPI == EPI_SWIGLU ? 2 : 4;
    const dim3 grid((a.N + 4 * RPW - 1) / (4 * RPW), groups);
    auto go = [&](auto its) {
      hipLaunchKernelGGL((gemv_direct_kernel<M, EPI, NORM, decltype(its)::value>), grid, dim3(256), 0, c->stream, (const float*)a.W, (const float*)a.W2,
                         a.x, (const float*)a.gain, a.y, a.ldx, a.ldy, a.N, a.K, a.eps, a.amax, a.amax_ld);
      return hipGetLastError();
    };
    if (a.K <= 256) return go(std::integral_constant<int, 1>());
    if (a.K <= 512) return go(std::integral_constant<int, 2>());
    if (a.K <= 768) return go(std::integral_constant<int, 3>());
    return go(std::integral_constant<int, 4>());
  }
  // narrow outputs with long rows: the waves of a block split K
  if constexpr ((EPI == EPI_RESID || EPI == EPI_STORE) && !NORM) {
    if (a.N <= 8192) {
      if (a.K <= 4 * 2 * 512) {
        hipLaunchKernelGGL((gemv_ksplit_kernel<float, M, EPI, 2, 4, 1>), dim3((a.N + 3) / 4, groups), dim3(256), 0, c->stream, a);
        return hipGetLastError();
      }
      if (a.K <= 4 * 5 * 512) {
        hipLaunchKernelGGL((gemv_ksplit_kernel<float, M, EPI, 5, 4, 1>), dim3((a.N + 3) / 4, groups), dim3(256), 0, c->stream, a);
        return hipGetLastError();
      }
    }
  }
  const size_t lds = (size_t)M * a.K * 4;
  auto kern = gemv_rows_kernel<float, M, EPI, NORM, 5>;
  static int occ_cache = -1;
  static size_t occ_lds = 0;
  if (lds > 160 * 1024 - 4096) return hipErrorInvalidValue;
  if (occ_cache < 0 || occ_lds != lds) {
    if (lds > 48 * 1024) {
      hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 4096);
      if (e != hipSuccess) return e;
    }
    int occ = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, 256, lds);
    if (e != hipSuccess) return e;
    occ_cache = occ < 1 ? 1 : occ;
    occ_lds = lds;
  }
  constexpr int RPW = (EPI == EPI_SWIGLU) ? 2 : 4;
  const int tasks = (a.N + RPW - 1) / RPW;
  int blocks = (tasks + 3) / 4;                      // one task per wave ...
  const int cap = c->num_cus * occ_cache;            // ... unless that exceeds what is resident at once
  if (blocks > cap) blocks = cap;
  hipLaunchKernelGGL(kern, dim3(blocks, groups), dim3(256), lds, c->stream, a);
  return hipGetLastError();
}

template <int EPI, bool NORM>
hipError_t gemv_rows(dmtd_ctx* c, GemvArgs a, int rows) {
  // Groups of kGemvRows rows, all full groups in one launch (a group per grid row), the rest in another.  One launch per group
  // had the groups wait for each other on a model whose weights sit in cache: the tiny model's 32-row
  // prompt took 1.0 of a request's 2.6 ms.
  for (int m0 = 0; m0 < rows;) {
    const int groups = (rows - m0) / kGemvRows;
    const int m = groups > 0 ? kGemvRows : rows - m0;
    GemvArgs g = a;
    g.x = a.x + (size_t)m0 * a.ldx;
    g.y = a.y + (size_t)m0 * a.ldy;
    if (a.amax) g.amax = a.amax + m0;
    hipError_t e;
    switch (m) {
      case 1: e = launch_gemv<1, EPI, NORM>(c, g, 1); break;
      case 2: e = launch_gemv<2, EPI, NORM>(c, g, 1); break;
      case 3: e = launch_gemv<3, EPI, NORM>(c, g, 1); break;
      default: e = launch_gemv<4, EPI, NORM>(c, g, groups); break;
    }
    if (e != hipSuccess) return e;
    m0 += groups > 0 ? groups * kGemvRows : m;
  }
  return hipSuccess;
}

// ---------------------------------------------------- packed path: MFMA weight streaming

// Row groups (of rpb rows) of an attention launch with r rows per sequence that have a row in them: what its key ranges are chosen by.
// The groups that a front pass has room for beyond a sequence's own rows leave at once (live_rows); counted with the others they
// left those fewer and longer ranges (512 wide, one KV head, 65k keys, 4 sequences of 1 row beside one of 12: 300 us per step of 6 layers, 284 now).
long row_groups(const dmtd_ctx* c, int r, int rpb) {
  if (!c->live) return (long)c->batch * ((r + rpb - 1) / rpb);
  long n = 0;
  for (int b = 0; b < c->batch; ++b) n += (c->live[b] + rpb - 1) / rpb;
  return n;
}

// nw waves split K for each matrix: the smallest of {2, 4, 8} (SwiGLU: {2, 4, 5}) that lets a wave
// hold its k-range in one round of PF k-steps, else the largest with several rounds.
// More than 16 rows go through the LDS-tiled kernel, up to kGemmRows per pass (each pass streams the matrix once).
// Attention launch shape for r rows per sequence: true = one key range per (row group, KV head, sequence), whose triples
// then fill the chip by themselves (see launch_attention_mfma_t).
bool attention_single_range(const dmtd_ctx* c, int r) {
  const dmtd_config& cf = c->cfg;
  const int gq = cf.n_q_heads / cf.n_kv_heads, rpb = 16 / gq, n_rg = (r + rpb - 1) / rpb;
  const long blocks = (long)cf.n_kv_heads * c->batch * n_rg;
  if (r > c->part_rows || cf.n_kv_heads * row_groups(c, r, rpb) >= c->num_cus) return true;         // more rows than the ranges' partials are laid out for: one range
  // Fewer blocks than CUs, short contexts: a block walks 128 keys in about 1.4 us (2.3 us with 8 blocks on the chip), the merge
  // launch and, with K-split QKV sums, their finishing launch cost 4-9 us.  us per step of 8 layers, one range / ranges + merge:
  // 64 blocks (batch 8), 2560 wide: 100 keys 485 / 523, 400 keys 519 / 526, 900 keys 592 / 580; 1024 wide: 250 / 272, 288 / 276,
  // 355 / 324; 128 blocks: 400 keys 572 / 626 and 346 / 381, 900 keys 639 / 653 and 421 / 408; 8 blocks: 400 keys 483 / 434.
  // (Blocks of dead row groups count here: the merge and the finishing launch carry their rows too.  2560 wide, 300 keys, 8
  // sequences of 2 rows beside one of 8, us per step of 4 layers: 208, by the living alone 212.)
  return c->att_bucket <= 4 * blocks;
}

// Whether `rows` packed activation rows of width K (both planes, plus n_parts partial sums of squares per row) stay in
// LDS for the one-tile-per-block kernel of an [N, K] projection (otherwise the LDS-tiled kernel takes them).
bool mfma_rows_fit(const dmtd_ctx* c, int rows, int N, int K, int n_parts) {
  if (rows > kMfmaRows) return false;
  const size_t lds_rows = (size_t)rows * ((size_t)4 * K + (size_t)n_parts * 4);
  return lds_rows <= ((N + 15) / 16 <= c->num_cus ? (size_t)120 * 1024 : (size_t)DMTD_FIT_SMALL_KB * 1024);
}

// More than kTiledRows rows: the wide GEMM, one block per CU.  Whole rounds of the CUs compute a tile per block; the tiles left
// over are split along K so that their blocks fill a round too, if that saves more than their raw sums and the finishing launch
// cost.  The residual projections go through the finishing kernel whole (their few tiles are nearly always split, and it
// owns their epilogue).
struct WidePlan { double us; int n_full, ksplit; };
template <int EPI, int BM, int BN>
WidePlan plan_wide(const dmtd_config& cf, int num_cus, int rows, int nt, int KS) {
  typedef GwTile<BM, BN> T;
  const int tiles = (rows + BM - 1) / BM * nt, slots = num_cus;
  // a k-step of 32 takes 0.8 us with 128 rows; with 256 it takes 1.3, and 1.45 in long runs, where the card lowers its clock (also where
  // it is summed by itself); a block's start and end take about 4 us.  Fitted to 300 launches of five widths from 200 to 2048 rows of an
  // earlier form of the loops, in which the chosen tile was 0.4 % slower than the better one on average (with one figure of 1.25 0.7 %).  The loops
  // have since become 2 to 4 % faster, by different amounts; of 360 launches of these the chosen tile is 0.6 % slower on average and up to 16 % (us,
  // tiles of 128 / 256: 2560 wide, gate/up with 200 rows 53 / 61, chosen 256; down with 701 rows 75 / 80, chosen 256; QKV with 2048 rows 114 / 98, chosen
  // 128, whose chains of 4 k-steps are also the nearer sums).  The figures stand, since another choice is another order of the sums;
  // a raw tile's bytes are written and read by blocks all over the chip at about 3.5 TB/s in all; the finishing launch itself 5 us.
  // Against 256 weight rows a step of 192 takes 0.93 times as long (1.31 to 1.4; 0.75 with 128 rows).
  auto step_us = [&](int ks) {
    const double whole = BM == 128 ? 0.8 : (EPI == EPI_STORE || 2 * KS >= 40 * ks ? 1.45 : 1.3);
    return BN == GW_BN ? whole : 0.93 * whole;
  };
  const int part_tiles = (int)std::min<size_t>(gemm_part_floats(cf) / T::PART, 1 << 20);
  const int whole = EPI == EPI_RESID ? 0 : tiles / slots * slots, left = tiles - whole;
  auto round_us = [&](int ks) { return (left * ks + slots - 1) / slots * (2.0 * KS / ks * step_us(ks) + 4.0); };
  auto parts_us = [&](int ks) { return left * ks * (T::PART * 4) / 3.5e6 + 5.0; };
  WidePlan p{round_us(1) + (EPI == EPI_RESID ? parts_us(1) : 0.0), EPI == EPI_RESID ? 0 : tiles, 1};
  if (EPI == EPI_RESID && left > part_tiles) p.us = 1e30;            // the raw sums do not fit
  if (EPI != EPI_LOGITS)
    for (int ks = 2; ks <= kGemmMaxSplit && ks * 4 <= KS && left > 0 && (long)left * ks <= part_tiles; ++ks) {      // at least 8 steps per part
      const double us = round_us(ks) + parts_us(ks);
      if (us < p.us * 0.97) p = WidePlan{us, whole, ks};
    }
  p.us += whole / slots * (2.0 * KS * step_us(1) + 4.0);
  return p;
}

template <int EPI, bool NORM, int BM, int BN>
hipError_t launch_wide_tiles(dmtd_ctx* c, const MfmaArgs& g, int nt, const WidePlan& p) {
  typedef GwTile<BM, BN> T;
  const int mt = (g.M + BM - 1) / BM, n_tail = mt * nt - p.n_full;
  if (BN != GW_BN && n_tail > 0) return hipErrorInvalidValue;      // tiles of another width are whole (choose_wide)
  auto kern = gemm_wide_mfma_kernel<EPI, NORM, BM, BN>;
  static bool big_lds = false;
  if (!big_lds) {
    hipError_t ae = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)T::LDS);
    if (ae != hipSuccess) return ae;
    big_lds = true;
  }
  hipLaunchKernelGGL(kern, dim3(p.n_full + n_tail * p.ksplit), dim3(64 * GW_WAVES), T::LDS, c->stream, g.W, g.W2, g.xb, g.xb_lo,
                     g.M, g.N, g.K, p.n_full, n_tail, p.ksplit, mt, nt, g);
  if constexpr (EPI != EPI_LOGITS && EPI != EPI_NLL && BN == GW_BN) {
    if (n_tail > 0)
      hipLaunchKernelGGL((gemm_wide_finish_kernel<EPI, NORM, BM>), dim3(n_tail, BM / 16), dim3(256), 0, c->stream, (const float*)g.part,
                         g.M, g.N, p.n_full, n_tail, p.ksplit, mt, nt, g);
  }
  return hipGetLastError();
}

// How a launch of `rows` rows of an [N, K] projection is laid out: rows of a launch, and the tile (rows bm, weight rows bn, nt of them along
// the outputs) with its plan
struct WideChoice { int nt, pass, bm, bn; WidePlan p; };
template <int EPI> int wide_col_tiles(int N, int bn) { const int out = EPI == EPI_SWIGLU ? bn / 2 : bn; return (N + out - 1) / out; }
template <int EPI>
WideChoice choose_wide(const dmtd_config& cf, int num_cus, int rows, int N, int K) {
  WideChoice w{};
  w.nt = wide_col_tiles<EPI>(N, GW_BN);
  w.bn = GW_BN;
  const int part_tiles = (int)std::min<size_t>(gemm_part_floats(cf) / GwTile<256, GW_BN>::PART, 1 << 20);      // at least nt
  w.pass = rows;
  if (EPI == EPI_RESID && (long)(rows + 255) / 256 * w.nt > part_tiles) w.pass = part_tiles / w.nt * 256;
  const WidePlan p256 = plan_wide<EPI, 256, GW_BN>(cf, num_cus, w.pass, w.nt, K / 64), p128 = plan_wide<EPI, 128, GW_BN>(cf, num_cus, w.pass, w.nt, K / 64);
  w.bm = p128.us < p256.us ? 128 : 256;
  w.p = w.bm == 128 ? p128 : p256;
  // 192 weight rows where all tiles of 256 are whole, of the same height: a sum is then the same chain over all of K either way.  (Where tiles of 256
  // are split, their sums in parts are nearer to 64 bits: see gemm_wide.hpp.)  In one round of the chip they are always the faster ones, of 62
  // launches by 6 to 18 % (tiles of 256 / 192, us: gate/up 1024 wide, 144 / 192 45.0 / 38.2, 160 / 215 45.1 / 39.7, 192 / 256 44.4 / 39.9; 2048 wide,
  // 192 / 256 91.8 / 83.0; QKV in tiles of 128 rows 1024 wide, 96 / 128 26.1 / 22.7, 2560 wide, 112 / 154 54.0 / 46.3, 160 / 220 59.7 / 55.3, 192 /
  // 256 65.8 / 61.0); in more rounds where they fill more than 7/8 of them.
  if constexpr (EPI == EPI_STORE || EPI == EPI_SWIGLU) {
    const WideChoice base = w;
    auto narrow = [&](auto bm_c) {
      constexpr int BM = decltype(bm_c)::value, BN = 192;
      if (base.bm != BM || base.p.ksplit > 1) return;
      const int nt = wide_col_tiles<EPI>(N, BN), tiles = (rows + BM - 1) / BM * nt, rounds = (tiles + num_cus - 1) / num_cus;
      const WidePlan p = plan_wide<EPI, BM, BN>(cf, num_cus, rows, nt, K / 64);
      if (p.ksplit == 1 && (rounds == 1 || tiles * 8L > rounds * (long)num_cus * 7) && p.us < w.p.us) w = WideChoice{nt, rows, BM, BN, p};
    };
    narrow(std::integral_constant<int, 256>());
    if constexpr (EPI == EPI_STORE) narrow(std::integral_constant<int, 128>());
  }
  return w;
}

template <int EPI, bool NORM>
hipError_t launch_wide(dmtd_ctx* c, const MfmaArgs& a, int rows) {
  WideChoice w = choose_wide<EPI>(c->cfg, c->num_cus, rows, a.N, a.K);
  const int pass = w.pass;
  for (int m0 = 0; m0 < rows; m0 += pass) {
    MfmaArgs g = a;
    g.M = std::min(pass, rows - m0);
    if (g.M < pass) w = choose_wide<EPI>(c->cfg, c->num_cus, g.M, a.N, a.K);
    g.xb = a.xb + (size_t)m0 * a.ldxb;             // m0 is a multiple of 256: whole row groups of the blocked layout
    g.xb_lo = a.xb_lo + (size_t)m0 * a.ldxb;
    if (a.ssp) g.ssp = a.ssp + m0;
    if (a.y) g.y = a.y + (size_t)m0 * a.ldy;
    if (a.yb) { g.yb = a.yb + (size_t)m0 * a.ldyb; g.yb_lo = a.yb_lo + (size_t)m0 * a.ldyb; }
    if (a.ssp_next) g.ssp_next = a.ssp_next + m0;
    if (a.amax) g.amax = a.amax + m0;
    g.part = c->gemm_part;
    hipError_t e = hipErrorInvalidValue;
    if (w.bn == GW_BN) e = w.bm == 128 ? launch_wide_tiles<EPI, NORM, 128, GW_BN>(c, g, w.nt, w.p) : launch_wide_tiles<EPI, NORM, 256, GW_BN>(c, g, w.nt, w.p);
    if constexpr (EPI == EPI_STORE || EPI == EPI_SWIGLU)
      if (w.bn == 192 && w.bm == 256) e = launch_wide_tiles<EPI, NORM, 256, 192>(c, g, w.nt, w.p);
    if constexpr (EPI == EPI_STORE)
      if (w.bn == 192 && w.bm == 128) e = launch_wide_tiles<EPI, NORM, 128, 192>(c, g, w.nt, w.p);
    if (e != hipSuccess) return e;
  }
  if (EPI == EPI_RESID) c->resid_parts = w.nt;
  return hipSuccess;
}

template <int EPI, bool NORM, int PF = kMfmaPF, int ROLL_NW = 0>
hipError_t launch_mfma(dmtd_ctx* c, MfmaArgs a, int rows, const MergeSrc& merge = MergeSrc{} /* po: the rows are still the attention's partial results */) {
  a.blocked = a.blocked || blocked_rows(c, rows);
  if (a.blocked) return launch_wide<EPI, NORM>(c, a, rows);
  if (EPI == EPI_RESID) c->resid_parts = (a.N + 15) / 16;      // one per 16 outputs; launches with a finishing kernel: see there
  const int KS = a.K / 64;
  constexpr int MATS = EPI == EPI_SWIGLU ? 2 : 1;
  const int nw_max = EPI == EPI_SWIGLU ? 5 : 8;
  int nw = 2;
  while (nw < nw_max && (KS + nw - 1) / nw > PF) nw = (EPI == EPI_SWIGLU && nw == 4) ? 5 : nw * 2;
  // ROLL_NW: a fixed number of waves per matrix, each keeping a rolling window of PF k-steps in flight
  if (ROLL_NW > 0) nw = ROLL_NW;
  const dim3 grid((a.N + 15) / 16);
  // The one-tile-per-block kernel keeps all rows (both planes) in LDS: comfortably (two blocks per CU) in general,
  // up to most of a CU's LDS when the launch has no more blocks than the chip has CUs anyway.  Rows that do not
  // fit, and more than 16 rows (batched steps), go through the LDS-tiled kernel in passes of up to kGemmRows rows.
  // Two more that the tiled kernel takes, unsplit, although the rows would fit: an LM head with tile streams in abundance (4B
  // shape, in the step, 1 / 5 rows: 127 / 150 us here, 121 there; 1024 wide, 12 rows: 123 / 57), and gate/up with many tiles
  // from 50 KiB of rows on (2560 wide, 5 rows: 20.5 / 19.4; 896 wide, 304 tiles, 8 rows: 6.7 / 8.5, hence the tile count).
  // An LM head with up to 4 rows stays here where the tiled kernel's blocks leave a fifth of their rounds of the chip empty and the
  // rows are long enough for this kernel's waves (us per step of one layer, 3 rows, here / there: 2048 wide, 70000 entries, 71 %
  // 93 / 100, 100352, 77 % 113 / 124, 80000, 81 % 99 / 102, 92000, 94 % 107 / 109, 128256, 98 % 131 / 132; 2560 wide 120 / 125,
  // 143 / 149, 127 / 127, 137 / 133, 165 / 161; 896 wide, 70000: 59 / 57).
  const int out_tiles = (a.N + 15) / 16;
  const int lm_blocks = (out_tiles + 2 * gemm_waves(1, EPI_LOGITS) - 1) / (2 * gemm_waves(1, EPI_LOGITS));
  const int lm_slots = (lm_blocks + c->num_cus - 1) / c->num_cus * c->num_cus;
  const bool lm_stays = rows <= 4 && a.K >= 1024 && lm_blocks * 5L < lm_slots * 4L;
  const bool prefers_tiled = EPI == EPI_LOGITS ? out_tiles >= 16 * c->num_cus && !lm_stays
                                               : (EPI == EPI_SWIGLU && out_tiles >= 2 * c->num_cus && (size_t)rows * 4 * a.K >= (size_t)50 * 1024);
  const bool fits = a.ldxb == a.K && !prefers_tiled && mfma_rows_fit(c, rows, a.N, a.K, NORM ? a.n_parts : 0);
  // one launch of the tiled kernel; with 64 and more rows its ring of activation slices is dynamic LDS beyond the default limit
#define DMTD_LAUNCH_GEMM(CG_, SPLIT_, GRID_) DMTD_LAUNCH_GEMM_W(CG_, SPLIT_, GRID_, gemm_waves(CG_, EPI))
#define DMTD_LAUNCH_GEMM_W(CG_, SPLIT_, GRID_, WAVES_)                                                                         \
  do {                                                                                                                         \
    auto kern = gemm_mfma_kernel<EPI, NORM, CG_, SPLIT_, WAVES_>;                                                              \
    constexpr size_t dyn = gemm_dyn_lds(CG_);                                                                                  \
    static bool big_lds = false;                                                                                               \
    if (dyn > 0 && !big_lds) {                                                                                                 \
      hipError_t ae = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);            \
      if (ae != hipSuccess) return ae;                                                                                         \
      big_lds = true;                                                                                                          \
    }                                                                                                                          \
    hipLaunchKernelGGL(kern, GRID_, dim3(64 * (WAVES_)), dyn, c->stream, g.W, g.W2, g.xb, g.xb_lo, g.M, g.N, g.K, \
                       g.ldxb, g.ksplit, g);                                                                                   \
  } while (0)
  if (!fits) {
    const int n_tiles = (a.N + 15) / 16;
    // An LM head with 17 to 32 rows: two blocks share a CU, of 8 waves or of kLmWaves; those that take fewer rounds of the chip for their waves, where
    // one round takes them all (us, 8 / 10 waves, 32 rows: 2560 wide, 140000 entries 142 / 132, 151936, 1.16 and 0.93 rounds, 148 / 140, 163840 155 / 148;
    // 1024 wide 68 / 58, 70 / 62, 76 / 66; 24 rows, 151936 entries: 768 wide 48.4 / 47.5, 640 43.2 / 43.1, 512 37.1 / 35.4, but 384 30.4 / 31.1; up to
    // 131072 entries are one round either way).  In two rounds against three, or three against four, only at widths of whole 1024s, which blocks of
    // 8 waves read at a lower rate (24 rows, 300000 / 400000 entries: 768 wide 90.7 / 95.7, 123.7 / 123.4, 1024 126 / 115, 165 / 148, 1536 167 / 174,
    // 228 / 226, 2048 219 / 220, 293 / 283, 2560 274 / 285, 375 / 369, 4096 433 / 423, 590 / 556).  The wider ones walk K in whole rounds of their pipeline.
    const auto lm_cost = [&](int waves) { return (n_tiles + 4 * waves * c->num_cus - 1) / (4 * waves * c->num_cus) * waves; };
    const bool lm_wide = KS % gemm_pf(2, EPI_LOGITS) == 0 && a.K >= 512 && (lm_cost(kLmWaves) == kLmWaves || a.K % 1024 == 0) && lm_cost(kLmWaves) < lm_cost(8);
    for (int m0 = 0; m0 < rows; m0 += kGemmRows) {
      MfmaArgs g = a;
      g.M = rows - m0 < kGemmRows ? rows - m0 : kGemmRows;
      g.xb = a.xb + (size_t)m0 * a.ldxb;
      g.xb_lo = a.xb_lo + (size_t)m0 * a.ldxb;
      if (a.ssp) g.ssp = a.ssp + m0;
      if (a.y) g.y = a.y + (size_t)m0 * a.ldy;
      if (a.yb) { g.yb = a.yb + (size_t)m0 * a.ldyb; g.yb_lo = a.yb_lo + (size_t)m0 * a.ldyb; }
      if (a.ssp_next) g.ssp_next = a.ssp_next + m0;
      if (a.amax) g.amax = a.amax + m0;
      const int cg = g.M <= 16 ? 1 : (g.M <= 32 ? 2 : (g.M <= 64 ? 4 : 8));
      const int gw = gemm_waves(cg, EPI);                  // a wave owns 2 tiles (SwiGLU: the gate and up tile of one)
      const dim3 ggrid(EPI == EPI_SWIGLU ? (n_tiles + gw - 1) / gw : (n_tiles + 2 * gw - 1) / (2 * gw));
      // K is split so that the launch has about one block per CU and no more (a partly filled second wave of blocks costs more than
      // it brings; measured at 4B shapes, 128 rows: QKV 288 blocks 32.4 us, 240 blocks 24.4 us; gate/up 152 blocks 50.0 us,
      // 228 blocks 42.4 us, 304 blocks 57.3 us; down 160 / 240 / 320 blocks 31.6 / 27.0 / 38.1 us); the LM head has
      // blocks enough without splitting
      const int KS = a.K / 64;
      int ksplit = 1;
      if constexpr (EPI != EPI_LOGITS) {
        ksplit = c->num_cus / (int)ggrid.x;
        if (ksplit < 1) ksplit = 1;
        if (EPI == EPI_STORE && ksplit > ATT_KSMAX) ksplit = ATT_KSMAX;      // what the attention launch can sum in its prologue
        if (EPI == EPI_RESID && ksplit > KS / 8) ksplit = KS / 8 > 0 ? KS / 8 : 1;
        if (ksplit > kGemmMaxSplit) ksplit = kGemmMaxSplit;
        if (ksplit > KS / 3) ksplit = KS / 3 > 0 ? KS / 3 : 1;
        // gate/up with up to 16 rows: its 1216 tile streams do without a split, and without the finishing launch (4B shapes,
        // 8 rows: 20.3 against 24.2 us); with 32 and more rows the 8-wave blocks are too few unsplit (36 against 24 us)
        if (EPI == EPI_SWIGLU && cg == 1) ksplit = 1;
      }
      if (ksplit > 1) {
        if constexpr (EPI != EPI_LOGITS) {
          g.ksplit = ksplit;
          g.ldp = (EPI == EPI_SWIGLU ? 2 : 1) * a.N;
          g.part = c->gemm_part;
          const dim3 sgrid(ggrid.x, ksplit);
          if (cg == 1) DMTD_LAUNCH_GEMM(1, true, sgrid);
          else if (cg == 2) DMTD_LAUNCH_GEMM(2, true, sgrid);
          else if (cg == 4) DMTD_LAUNCH_GEMM(4, true, sgrid);
          else DMTD_LAUNCH_GEMM(8, true, sgrid);
          if (EPI == EPI_STORE && NORM && c->fold_qkv && rows <= kGemmRows && ksplit <= ATT_KSMAX && c->batch > 0 &&
              attention_single_range(c, rows / c->batch)) {
            // the attention launch that follows sums the splits and applies the norm scale while it prepares its rows; only in
            // its one-range shape, where a vector is prepared once (with key ranges every range's block would repeat the sums:
            // C5 measured 2 % slower, C4 2 % faster)
            c->qkv_pending = QkvSrc{nullptr, 0, g.part, ksplit, g.M, g.ldp, g.ssp, g.n_parts, g.ssp_ld, 1.0f / (float)g.K, g.eps};
          } else {
            hipLaunchKernelGGL((gemm_finish_kernel<EPI, NORM>), dim3((a.N / 4 + 255) / 256, g.M), dim3(256), 0, c->stream,
                               (const float*)g.part, (const float*)g.y, (const bf16_t*)g.g_next, g.ksplit, g.M, g.N, g.ldp, g.ldy, g);
            if (EPI == EPI_RESID) c->resid_parts = (a.N / 4 + 255) / 256;
          }
        }
      } else {
        // Gate/up whose blocks of 4 waves are a quarter to a half of the CUs: blocks of 2 (us, 16 rows, blocks of 4 waves / 2, at 65, 96 and 128 blocks of 4:
        // 1024 wide 9.3 / 8.4, 9.8 / 8.8, 10.2 / 9.4; 1536 12.7 / 10.6, 13.7 / 11.3, 13.7 / 12.2; 2048 15.7 / 13.8, 16.0 / 14.1, 16.9 / 15.4; 2560 19.2 / 17.4,
        // 20.7 / 17.5, 21.2 / 18.4; 4096 28.3 / 25.4, 29.9 / 25.1, 31.7 / 27.1; with 8 rows of 2048 to 4096 wide 11 to 19 % faster, with 4 to 7 where they come
        // this way 8 to 30 %).  Outside: 1536 wide, 560 tiles, 140 blocks 14.0 / 13.8 / 14.2 (8 / 12 / 16 rows) against 14.0 / 15.9 / 16.8; 2560 wide, 608
        // 19.6 / 20.4 / 21.0 against 22.4 / 23.8 / 25.0: each block draws the activations once more; 1024 wide, 16 rows, 48 blocks 6.0 / 6.2.
        const bool gu_narrow = EPI == EPI_SWIGLU && cg == 1 && 4 * (int)ggrid.x > c->num_cus && 2 * (int)ggrid.x <= c->num_cus;
        if (gu_narrow) {
          if constexpr (EPI == EPI_SWIGLU) DMTD_LAUNCH_GEMM_W(1, false, dim3((n_tiles + 1) / 2), 2);
        } else if (cg == 1) DMTD_LAUNCH_GEMM(1, false, ggrid);
        else if (EPI == EPI_LOGITS && cg == 2 && lm_wide) {
          if constexpr (EPI == EPI_LOGITS) DMTD_LAUNCH_GEMM_W(2, false, dim3((n_tiles + 2 * kLmWaves - 1) / (2 * kLmWaves)), kLmWaves);
        } else if (cg == 2) DMTD_LAUNCH_GEMM(2, false, ggrid);
        else if (cg == 4) DMTD_LAUNCH_GEMM(4, false, ggrid);
        else DMTD_LAUNCH_GEMM(8, false, ggrid);
      }
    }
    return hipGetLastError();
  }
  for (int m0 = 0; m0 < rows; m0 += kMfmaRows) {
    MfmaArgs g = a;
    g.M = rows - m0 < kMfmaRows ? rows - m0 : kMfmaRows;
    g.xb = a.xb + (size_t)m0 * a.ldxb;
    g.xb_lo = a.xb_lo + (size_t)m0 * a.ldxb;
    if (a.ssp) g.ssp = a.ssp + m0;
    if (a.y) g.y = a.y + (size_t)m0 * a.ldy;
    if (a.yb) { g.yb = a.yb + (size_t)m0 * a.ldyb; g.yb_lo = a.yb_lo + (size_t)m0 * a.ldyb; }
    if (a.ssp_next) g.ssp_next = a.ssp_next + m0;
    if (a.amax) g.amax = a.amax + m0;
    const size_t lds = (size_t)2 * g.M * a.K * 2 + (NORM ? (size_t)g.M * a.n_parts * 4 : 0);   // the rows, both planes; partial sums of squares
#define DMTD_LAUNCH_MFMA_MR(NWT_, MR_, MG_)                                                                               \
    do {                                                                                                                  \
      auto kern = gemv_mfma_kernel<EPI, NORM, PF, NWT_, (ROLL_NW > 0), MR_>;                                             \
      static bool big_lds = false;                                                                                        \
      if (lds > 48 * 1024 && !big_lds) {                                                                                  \
        hipError_t ae = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 120 * 1024);   \
        if (ae != hipSuccess) return ae;                                                                                  \
        big_lds = true;                                                                                                   \
      }                                                                                                                   \
      hipLaunchKernelGGL(kern, grid, dim3(64 * NWT_), lds, c->stream, g.W, g.W2, g.xb, g.xb_lo, (const float*)g.ssp, g.M, g.N, g.K, g.n_parts, g.ssp_ld, g, MG_); \
    } while (0)
#define DMTD_LAUNCH_MFMA(NWT_) DMTD_LAUNCH_MFMA_MR(NWT_, 0, MergeArg<0>{})
    if constexpr (EPI == EPI_RESID && ROLL_NW == DMTD_O_NW) {
      if (merge.po && merge.ns <= kMergeFew) { DMTD_LAUNCH_MFMA_MR(ROLL_NW, kMergeFew, MergeArg<kMergeFew>{merge}); continue; }
      if (merge.po) { DMTD_LAUNCH_MFMA_MR(ROLL_NW, kMergeRanges, MergeArg<kMergeRanges>{merge}); continue; }
    }
    if constexpr (ROLL_NW > 0) DMTD_LAUNCH_MFMA(ROLL_NW * MATS);
    else if (nw == 2) DMTD_LAUNCH_MFMA(2 * MATS);
    else if (nw == 4) DMTD_LAUNCH_MFMA(4 * MATS);
    else if (nw == 5) {
      if constexpr (EPI == EPI_SWIGLU) DMTD_LAUNCH_MFMA(10);
    } else {
      if constexpr (EPI != EPI_SWIGLU) DMTD_LAUNCH_MFMA(8);
    }
#undef DMTD_LAUNCH_MFMA
#undef DMTD_LAUNCH_MFMA_MR
  }
  return hipGetLastError();
}

hipError_t launch_lmhead(dmtd_ctx* c, MfmaArgs a, int rows) {
  if constexpr (DMTD_LM_NW > 0) return launch_mfma<EPI_LOGITS, true, DMTD_LM_PF, DMTD_LM_NW>(c, a, rows);
  else return launch_mfma<EPI_LOGITS, true>(c, a, rows);
}
hipError_t launch_qkv(dmtd_ctx* c, MfmaArgs a, int rows) {
  if constexpr (DMTD_Q_NW > 0) return launch_mfma<EPI_STORE, true, DMTD_Q_PF, DMTD_Q_NW>(c, a, rows);
  else return launch_mfma<EPI_STORE, true, kMfmaPFQkv>(c, a, rows);
}
hipError_t launch_down(dmtd_ctx* c, MfmaArgs a, int rows) {
  if constexpr (DMTD_DN_NW > 0) return launch_mfma<EPI_RESID, false, DMTD_DN_PF, DMTD_DN_NW>(c, a, rows);
  else return launch_mfma<EPI_RESID, false>(c, a, rows);
}
hipError_t launch_oproj(dmtd_ctx* c, MfmaArgs a, int rows) {
  const MergeSrc merge = c->merge_pending;
  c->merge_pending = MergeSrc{};
  if constexpr (DMTD_O_NW > 0) return launch_mfma<EPI_RESID, false, DMTD_O_PF, DMTD_O_NW>(c, a, rows, merge);
  else return launch_mfma<EPI_RESID, false>(c, a, rows);
}
hipError_t launch_gateup(dmtd_ctx* c, MfmaArgs a, int rows) {
  if constexpr (DMTD_GU_NW > 0) return launch_mfma<EPI_SWIGLU, true, DMTD_GU_PF, DMTD_GU_NW>(c, a, rows);
  else return launch_mfma<EPI_SWIGLU, true>(c, a, rows);
}

// ------------------------------------------------------------------------- attention

// a3 + a4: QK-RMSNorm, RoPE, KV append and split-K attention in one launch over static key ranges, then the merge.
// The ranges follow from the context bucket (c->att_bucket, 256 or a multiple of 512 that covers the context), so a
// captured step stays valid until the sequence grows into the next bucket.
template <int HD, int QVT>
void launch_attention_t(dmtd_ctx* c, int l, const float* qkv, float* attn, int sel, int offset, int r, int append) {
  const dmtd_config& cf = c->cfg;
  const int B = c->batch, nqkv = (cf.n_q_heads + 2 * cf.n_kv_heads) * HD, qd = cf.n_q_heads * HD;
  const int gq = cf.n_q_heads / cf.n_kv_heads, rpb = QVT / gq, n_rg = (r + rpb - 1) / rpb;
  constexpr int KPI = AttKeysPerIter<HD>::value;
  float* kc = (float*)(c->ws + c->o.kv + (size_t)l * c->o.kv_layer_stride);
  float* vc = (float*)(c->ws + c->o.kv + (size_t)l * c->o.kv_layer_stride + c->o.kv_v_off);
  const LayerW& w = c->layers[l];
  // keys per range: one block iteration while that keeps the ranges within the partials buffer and puts no
  // more than about four blocks on every CU; longer ranges (several iterations) for long contexts or big batches
  const int bucket = c->att_bucket;
  const long per_split_blocks = cf.n_kv_heads * row_groups(c, r, rpb);
  int want_splits = (int)((4L * c->num_cus + per_split_blocks - 1) / per_split_blocks);
  if (want_splits > ATT_MAX_SPLITS) want_splits = ATT_MAX_SPLITS;
  if (want_splits < 1) want_splits = 1;
  int kps = ((bucket + want_splits - 1) / want_splits + KPI - 1) / KPI * KPI;
  // short contexts: one range of at most two block iterations instead of the merge launch (4.4 us; an iteration takes about 2)
  const bool one = bucket <= 2 * KPI;
  if (one) kps = bucket;
  const int ns = (bucket + kps - 1) / kps;
  float* po = c->part_o;
  float* pml = c->part_ml;
  const DevState* st = dev_state(c);
  const auto split_kern = c->fmap ? attn_split_kernel<HD, QVT, true> : attn_split_kernel<HD, QVT, false>;
  hipLaunchKernelGGL(split_kern, dim3(ns * n_rg, cf.n_kv_heads, B), dim3(256), 0, c->stream, qkv, nqkv,
                     w.q_norm, w.k_norm, (const float2*)(c->ws + c->o.rope_tab), kc, vc, po, pml, cf.n_q_heads, cf.n_kv_heads,
                     cf.max_seq_len, cf.rms_eps, kps, ns, c->part_rows * gq, st, sel, offset, r, append, c->fmap, one ? attn : (float*)nullptr, qd);
  if (one) return;
  const auto merge_kern = c->fmap ? attn_merge_kernel<HD, float, true> : attn_merge_kernel<HD, float, false>;
  hipLaunchKernelGGL(merge_kern, dim3(r, cf.n_q_heads, B), dim3(256), 0, c->stream, po, pml, attn, (float*)nullptr, qd,
                     cf.n_q_heads, cf.n_kv_heads, kps, ns, c->part_rows * gq, st, sel, offset, r, c->fmap, blocked_rows(c, B * r));
}

// Key ranges of a launch with r rows per sequence that is not in one range: keys per range (whole iterations of 64 keys) and ranges
struct AttRanges { int kps, ns; };
AttRanges attention_ranges(const dmtd_ctx* c, int r) {
  const dmtd_config& cf = c->cfg;
  const int gq = cf.n_q_heads / cf.n_kv_heads;
  const long per_split_blocks = cf.n_kv_heads * row_groups(c, r, 16 / gq);
  int want_splits = (int)((4L * c->num_cus + per_split_blocks - 1) / per_split_blocks);
  if (want_splits > ATT_MAX_SPLITS) want_splits = ATT_MAX_SPLITS;
  if (want_splits < 1) want_splits = 1;
  AttRanges a;
  a.kps = ((c->att_bucket + want_splits - 1) / want_splits + 63) / 64 * 64;
  a.ns = (c->att_bucket + a.kps - 1) / a.kps;
  return a;
}
// Few partial results: the O projection's blocks merge them on the way in (it has to be the one-tile-per-block kernel)
bool oproj_merges(const dmtd_ctx* c, int r, const AttRanges& ar) {
  const int qd = c->cfg.n_q_heads * c->cfg.head_dim, rows = c->batch * r;
  return DMTD_O_NW > 0 && ar.ns <= kMergeRanges && (size_t)rows * qd * ar.ns * 4 <= kMergeBytes && mfma_rows_fit(c, rows, c->cfg.hidden, qd, 0);
}
MergeSrc merge_source(dmtd_ctx* c, int r, const AttRanges& ar, int sel, int offset) {
  const int gq = c->cfg.n_q_heads / c->cfg.n_kv_heads;
  return MergeSrc{c->part_o, c->part_ml, dev_state(c), c->fmap, ar.kps, ar.ns, c->part_rows * gq, ATT_MAX_SPLITS, c->cfg.n_kv_heads, gq, c->cfg.head_dim, sel, offset, r};
}

// The matrix-core kernel (bf16 caches): one pass over K and V serves up to 16 query vectors per KV head.
// Two launch shapes.  (1) ONE key range per (row group, KV head, sequence), 8 waves per block, the output written
// by the kernel itself (no partials, no merge launch): for batches whose (KV head, sequence) pairs fill the chip
// without splitting.  (2) Key ranges over 4-wave blocks plus the merge, by a launch of its own or, where
// the partial results are few, by the O projection's blocks (kMergeBytes): everything else.
template <typename OT, int HD>
hipError_t launch_attention_mfma_t(dmtd_ctx* c, int l, const float* qkv, OT* attn, OT* attn_lo, int sel, int offset, int r, int append) {
  const dmtd_config& cf = c->cfg;
  const int B = c->batch, nqkv = (cf.n_q_heads + 2 * cf.n_kv_heads) * HD, qd = cf.n_q_heads * HD;
  const int gq = cf.n_q_heads / cf.n_kv_heads, rpb = 16 / gq, n_rg = (r + rpb - 1) / rpb;
  const int qv_max = (r < rpb ? r : rpb) * gq;             // query vectors of the fullest block
  bf16_t* kc = (bf16_t*)(c->ws + c->o.kv + (size_t)l * c->o.kv_layer_stride);
  bf16_t* vc = (bf16_t*)(c->ws + c->o.kv + (size_t)l * c->o.kv_layer_stride + c->o.kv_v_off);
  const LayerW& w = c->layers[l];
  float* po = c->part_o;
  float* pml = c->part_ml;
  const DevState* st = dev_state(c);
  QkvSrc qs = c->qkv_pending;           // the QKV projection's unfinished partial sums, if it left them to this launch
  c->qkv_pending = QkvSrc{};
  qs.qkv = qkv; qs.ldq = nqkv;
  if (attention_single_range(c, r)) {
    constexpr int NW = 8;
    const int kps = (c->att_bucket + 16 * NW - 1) / (16 * NW) * (16 * NW);
    const size_t lds = (size_t)NW * qv_max * HD * 4;
    const auto kern = c->fmap ? attn_split_mfma_kernel<HD, NW, true, true> : attn_split_mfma_kernel<HD, NW, true, false>;
    static bool big_lds[2] = {false, false};
    if (lds > 32 * 1024 && !big_lds[c->fmap != nullptr]) {
      hipError_t ae = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, NW * 16 * HD * 4);
      if (ae != hipSuccess) return ae;
      big_lds[c->fmap != nullptr] = true;
    }
    hipLaunchKernelGGL(kern, dim3(n_rg, cf.n_kv_heads, B), dim3(64 * NW), lds, c->stream,
                       kc, vc, cf.n_q_heads, cf.n_kv_heads, cf.max_seq_len, kps, r, c->fmap, st, sel, offset, 1, w.q_norm,
                       w.k_norm, (const float2*)(c->ws + c->o.rope_tab), po, pml, cf.rms_eps, c->part_rows * gq, append,
                       (bf16_t*)attn, (bf16_t*)attn_lo, qd, blocked_rows(c, B * r), qs);
    return hipGetLastError();
  }
  const AttRanges ar = attention_ranges(c, r);
  const int kps = ar.kps, ns = ar.ns;
  const auto split_kern = c->fmap ? attn_split_mfma_kernel<HD, 4, false, true> : attn_split_mfma_kernel<HD, 4, false, false>;
  hipLaunchKernelGGL(split_kern, dim3(ns * n_rg, cf.n_kv_heads, B), dim3(256), (size_t)4 * qv_max * HD * 4, c->stream,
                     kc, vc, cf.n_q_heads, cf.n_kv_heads, cf.max_seq_len, kps, r, c->fmap, st, sel, offset, ns, w.q_norm,
                     w.k_norm, (const float2*)(c->ws + c->o.rope_tab), po, pml, cf.rms_eps, c->part_rows * gq, append,
                     (bf16_t*)nullptr, (bf16_t*)nullptr, 0, 0, qs);
  if (c->fold_merge && oproj_merges(c, r, ar)) {
    c->merge_pending = merge_source(c, r, ar, sel, offset);
    return hipGetLastError();
  }
  const auto merge_kern = c->fmap ? attn_merge_kernel<HD, OT, true> : attn_merge_kernel<HD, OT, false>;
  hipLaunchKernelGGL(merge_kern, dim3(r, cf.n_q_heads, B), dim3(256), 0, c->stream, po, pml, attn, attn_lo, qd,
                     cf.n_q_heads, cf.n_kv_heads, kps, ns, c->part_rows * gq, st, sel, offset, r, c->fmap, blocked_rows(c, B * r));
  return hipGetLastError();
}

// Passes whose keys and values are in the cache already (append = 2: more than kMaxRows rows per sequence), with so many rows
// that launch_attention sends them here.
template <int HD>
hipError_t launch_attention_prefill(dmtd_ctx* c, int l, const float* qkv, bf16_t* attn, bf16_t* attn_lo, int sel, int offset, int r) {
  const dmtd_config& cf = c->cfg;
  const int nqkv = (cf.n_q_heads + 2 * cf.n_kv_heads) * HD, rpb = AP_QV / (cf.n_q_heads / cf.n_kv_heads);
  const bf16_t* kc = (const bf16_t*)(c->ws + c->o.kv + (size_t)l * c->o.kv_layer_stride);
  const bf16_t* vc = (const bf16_t*)(c->ws + c->o.kv + (size_t)l * c->o.kv_layer_stride + c->o.kv_v_off);
  // KV heads fastest: with 8 of them a compute die's blocks share one head's keys and values in its L2
  const dim3 grid(cf.n_kv_heads, c->batch, (r + rpb - 1) / rpb);
  // Blocks of later rows have more keys.  Two blocks share a CU, so up to 2 num_cus of them are all resident from the start and nothing
  // evens out what a CU got: the first round of the CUs goes from the longest down, the second from the shortest up, and a CU's
  // two come to about the same (2048 rows behind 0 / 6k keys, all from the longest down 108 / 510 us, so 97 / 500, long and short in
  // turn 123 / 538).  More blocks than that start as others end, longest first.
  const int per_z = (int)(grid.x * grid.y);
  const int n_down = (long)per_z * grid.z <= 2L * c->num_cus ? std::min((int)grid.z, (c->num_cus + per_z - 1) / per_z) : (int)grid.z;
  auto launch = [&](auto kg_c) -> hipError_t {
    constexpr int KG = decltype(kg_c)::value;
    auto kern = attn_prefill_mfma_kernel<HD, KG>;
    static bool big_lds = false;
    if (!big_lds) {
      hipError_t ae = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)attn_prefill_lds(HD, KG));
      if (ae != hipSuccess) return ae;
      big_lds = true;
    }
    hipLaunchKernelGGL(kern, grid, dim3(256 * KG), attn_prefill_lds(HD, KG), c->stream, qkv, nqkv, kc, vc,
                       cf.n_q_heads, cf.n_kv_heads, cf.max_seq_len, r, (const DevState*)dev_state(c), sel, offset, (const bf16_t*)c->layers[l].q_norm,
                       (const float2*)(c->ws + c->o.rope_tab), cf.rms_eps, attn, attn_lo, cf.n_q_heads * HD, blocked_rows(c, c->batch * r), n_down);
    return hipGetLastError();
  };
  return (long)grid.x * grid.y * grid.z <= c->num_cus ? launch(std::integral_constant<int, 2>()) : launch(std::integral_constant<int, 1>());
}

// Kernel choice.  bf16 caches: the matrix-core kernel (measured faster than the vector kernel even for
// one row and 4 query heads per KV head: 11.7 vs 13.2 us at 1k context, 99 vs 119 us at 8 x 16k).
// fp32 caches: the vector kernel; share_kv: all rows of a sequence go through one block so that K and V
// are read once (long contexts), else rows are spread over blocks (K/V re-reads hit in L2).
template <typename CT, typename OT>
hipError_t launch_attention(dmtd_ctx* c, int l, const float* qkv, OT* attn, OT* attn_lo, int sel, int offset, int r, int append = 1) {
  const dmtd_config& cf = c->cfg;
  const int gq = cf.n_q_heads / cf.n_kv_heads;
  if (r > kMaxRows && append != 2) return hipErrorInvalidValue;    // more rows than an attention block keeps in LDS: their keys must be in the cache
  if constexpr (std::is_same<CT, bf16_t>::value) {
    // Blocks of 16 query vectors put at most two on a CU: the decode kernel (its 8 waves share a tile's keys, where the prefill
    // kernel's few blocks of 128 vectors walk the key tiles one after the other).  Layers of 4B shapes, whole pass, us, prefill
    // kernel / decode kernel: 64 positions 476 / 443, 128: 632 / 584, 256: 869 / 852, 400: 1189 / 1215, 8 x 24: 994 / 990, 8 x 64:
    // 1224 / 1270, 32 x 64: 3493 / 3725; the last 32 and 128 positions behind 8192: the prompt 18367 / 17398 and 18652 / 17965.
    const long blocks = (long)cf.n_kv_heads * c->batch * ((r + 16 / gq - 1) / (16 / gq));
    // the prefill kernel addresses a head's rows with 32 bits
    if (append == 2 && blocks > 2 * c->num_cus && (long)cf.max_seq_len * cf.head_dim < (1L << 31)) {
      if (cf.head_dim == 128) return launch_attention_prefill<128>(c, l, qkv, attn, attn_lo, sel, offset, r);
      return launch_attention_prefill<64>(c, l, qkv, attn, attn_lo, sel, offset, r);
    }
    if (cf.head_dim == 128) return launch_attention_mfma_t<OT, 128>(c, l, qkv, attn, attn_lo, sel, offset, r, append);
    return launch_attention_mfma_t<OT, 64>(c, l, qkv, attn, attn_lo, sel, offset, r, append);
  } else {
    const int want = c->share_kv ? r * gq : gq;
    const int qvt = want <= 4 ? 4 : (want <= 8 ? 8 : 16);
    if (cf.head_dim == 128) {
      if (qvt == 4) launch_attention_t<128, 4>(c, l, qkv, attn, sel, offset, r, append);
      else if (qvt == 8) launch_attention_t<128, 8>(c, l, qkv, attn, sel, offset, r, append);
      else launch_attention_t<128, 16>(c, l, qkv, attn, sel, offset, r, append);
    } else {
      if (qvt == 4) launch_attention_t<64, 4>(c, l, qkv, attn, sel, offset, r, append);
      else if (qvt == 8) launch_attention_t<64, 8>(c, l, qkv, attn, sel, offset, r, append);
      else launch_attention_t<64, 16>(c, l, qkv, attn, sel, offset, r, append);
    }
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------- the steps of a pass

// a1: rows <- embeddings of the tokens at the rows' positions (next reader: the norm of layer next_layer)
hipError_t embed_rows(dmtd_ctx* c, Rows& R, int sel, int offset, int r, int next_layer) {
  const dmtd_config& cf = c->cfg;
  const int rows = c->batch * r;
  if (c->packed) {
    // a prefill pass has few blocks of 16 rows: its columns in four parts; a step's late rows may come from the front layers too, in one
    const int parts = blocked_rows(c, rows) && sel == POS_EXPLICIT ? 4 : 1;
    if (blocked_rows(c, rows))
      hipLaunchKernelGGL(embed_pack_blocked_kernel, dim3((rows + 15) / 16, parts), dim3(256), 0, c->stream, (const bf16_t*)c->embed, dev_tokens(c),
                         cf.max_seq_len, dev_state(c), sel, offset, r, cf.hidden, R.h, (const bf16_t*)norm_gain_for_layer(c, next_layer),
                         R.xb, R.xb_lo, R.ssp, c->ssp_ld, c->fmap, rows);
    else
      hipLaunchKernelGGL(embed_pack_kernel, dim3(rows), dim3(256), 0, c->stream, (const bf16_t*)c->embed, dev_tokens(c),
                         cf.max_seq_len, dev_state(c), sel, offset, r, cf.hidden, R.h, (const bf16_t*)norm_gain_for_layer(c, next_layer),
                         R.xb, R.xb_lo, R.ssp, c->fmap);
    R.n_parts = parts;
  } else {
    hipLaunchKernelGGL(embed_kernel<float>, dim3(rows), dim3(256), 0, c->stream, (const float*)c->embed, dev_tokens(c),
                       cf.max_seq_len, dev_state(c), sel, offset, r, cf.hidden, R.h, c->fmap);
  }
  return hipGetLastError();
}

// literal Eq. 4 during prefill: rows += their embeddings, before layer next_layer
hipError_t add_embed_rows(dmtd_ctx* c, Rows& R, int sel, int offset, int r, int next_layer) {
  const dmtd_config& cf = c->cfg;
  const int rows = c->batch * r;
  if (c->packed) {
    hipLaunchKernelGGL(add_embed_pack_kernel, dim3(rows), dim3(256), 0, c->stream, R.h, (const bf16_t*)c->embed, dev_tokens(c),
                       cf.max_seq_len, dev_state(c), sel, offset, r, cf.hidden, (const bf16_t*)norm_gain_for_layer(c, next_layer),
                       R.xb, R.xb_lo, R.ssp, blocked_rows(c, rows));
    R.n_parts = 1;
  } else {
    hipLaunchKernelGGL(add_embed_rows_kernel<float>, dim3(rows), dim3(256), 0, c->stream, R.h, (const float*)c->embed,
                       dev_tokens(c), cf.max_seq_len, dev_state(c), sel, offset, r, cf.hidden);
  }
  return hipGetLastError();
}

// a8: only each sequence's newest row continues (Sec. 2.2); under the literal Eq. 4 reading its embedding is added
// last_pos (prefill of prompts of different lengths): sequence b's row is the one at explicit position last_pos[b]
hipError_t take_last_rows(dmtd_ctx* c, const Rows& src, Rows& dst, int r, int add_embed, int sel, int offset, int next_layer,
                          const int* last_pos = nullptr) {
  const dmtd_config& cf = c->cfg;
  if (c->packed) {
    const int late_blocked = blocked_rows(c, c->late_batch > 0 ? c->late_batch : c->batch);      // the late rows are one per sequence of the whole batch
    hipLaunchKernelGGL(take_last_pack_kernel, dim3(c->batch), dim3(256), 0, c->stream, src.h, dst.h, r, cf.hidden, add_embed,
                       (const bf16_t*)c->embed, dev_tokens(c), cf.max_seq_len, dev_state(c), sel, offset,
                       (const bf16_t*)norm_gain_for_layer(c, next_layer), dst.xb, dst.xb_lo, dst.ssp, (const float*)nullptr, last_pos, c->fmap, late_blocked);
    dst.n_parts = 1;
  } else {
    hipLaunchKernelGGL(take_last_rows_kernel<float>, dim3(c->batch), dim3(256), 0, c->stream, src.h, dst.h, r, cf.hidden,
                       add_embed, (const float*)c->embed, dev_tokens(c), cf.max_seq_len, dev_state(c), sel, offset, (const float*)nullptr, last_pos, c->fmap);
  }
  return hipGetLastError();
}

// a3 as a launch of its own, for passes with more rows per sequence than an attention block keeps in LDS (prefill, the
// whole-sequence forward): the rows' keys (QK-RMSNorm + RoPE) and values go to the cache before the attention launch
template <typename CT>
hipError_t launch_kv_append(dmtd_ctx* c, int l, const float* qkv, int sel, int offset, int r) {
  const dmtd_config& cf = c->cfg;
  const int nqkv = (cf.n_q_heads + 2 * cf.n_kv_heads) * cf.head_dim;
  CT* kc = (CT*)(c->ws + c->o.kv + (size_t)l * c->o.kv_layer_stride);
  CT* vc = (CT*)(c->ws + c->o.kv + (size_t)l * c->o.kv_layer_stride + c->o.kv_v_off);
  const dim3 grid(c->batch * r, cf.n_kv_heads);
  if (cf.head_dim == 128)
    hipLaunchKernelGGL((kv_append_kernel<CT, 128>), grid, dim3(64), 0, c->stream, qkv, nqkv, c->layers[l].k_norm, (const float2*)(c->ws + c->o.rope_tab),
                       kc, vc, cf.n_q_heads, cf.n_kv_heads, cf.max_seq_len, cf.rms_eps, (const DevState*)dev_state(c), sel, offset, r);
  else
    hipLaunchKernelGGL((kv_append_kernel<CT, 64>), grid, dim3(64), 0, c->stream, qkv, nqkv, c->layers[l].k_norm, (const float2*)(c->ws + c->o.rope_tab),
                       kc, vc, cf.n_q_heads, cf.n_kv_heads, cf.max_seq_len, cf.rms_eps, (const DevState*)dev_state(c), sel, offset, r);
  return hipGetLastError();
}

// a2..a7: one transformer block over r rows per sequence at positions base + offset + i
hipError_t run_layer(dmtd_ctx* c, int l, Rows& R, int r, int sel, int offset) {
  const dmtd_config& cf = c->cfg;
  const int rows = c->batch * r, d = cf.hidden, hd = cf.head_dim, ff = cf.intermediate;
  const int nqkv = (cf.n_q_heads + 2 * cf.n_kv_heads) * hd, qd = cf.n_q_heads * hd;
  float* qkv = (float*)(c->ws + c->o.qkv);
  const LayerW& w = c->layers[l];
  hipError_t e;
  if (c->packed) {
    const LayerSw& s = c->sw[l];
    const size_t rows_cap = row_capacity(cf, c->wide_rows);
    bf16_t* ab = (bf16_t*)(c->ws + c->o.attn);      // attention output, high parts; low parts behind them
    bf16_t* ab_lo = ab + rows_cap * qd;
    bf16_t* ub = (bf16_t*)(c->ws + c->o.mlp);       // SwiGLU output, likewise
    bf16_t* ub_lo = ub + rows_cap * ff;
    MfmaArgs a{};
    // a2: RMSNorm + fused QKV projection
    a.W = s.qkv; a.xb = R.xb; a.xb_lo = R.xb_lo; a.ldxb = d; a.N = nqkv; a.K = d; a.ssp = R.ssp; a.n_parts = R.n_parts; a.ssp_ld = c->ssp_ld;
    a.eps = cf.rms_eps; a.y = qkv; a.ldy = nqkv;
    const bool wide = r > kMaxRows;      // more rows per sequence than an attention block keeps in LDS: the append is a launch of its own
    c->fold_qkv = !wide;
    e = launch_qkv(c, a, rows);
    c->fold_qkv = false;
    if (e != hipSuccess) { c->qkv_pending = QkvSrc{}; return e; }
    // a3 + a4: QK-RMSNorm + RoPE + KV append + split-K attention, then the merge (output packed for the O projection)
    if (wide && (e = launch_kv_append<bf16_t>(c, l, qkv, sel, offset, r)) != hipSuccess) return e;
    c->fold_merge = true;
    e = launch_attention<bf16_t, bf16_t>(c, l, qkv, ab, ab_lo, sel, offset, r, wide ? 2 : 1);
    c->fold_merge = false;
    if (e != hipSuccess) { c->merge_pending = MergeSrc{}; return e; }
    // a5: O projection + residual; emits the MLP norm's input
    a = MfmaArgs{};
    a.W = s.o; a.xb = ab; a.xb_lo = ab_lo; a.ldxb = qd; a.N = d; a.K = qd; a.y = R.h; a.ldy = d; a.yb = R.xb; a.yb_lo = R.xb_lo; a.ldyb = d;
    a.g_next = (const bf16_t*)w.mlp_norm; a.ssp_next = R.ssp; a.ssp_ld = c->ssp_ld;
    if ((e = launch_oproj(c, a, rows)) != hipSuccess) return e;
    R.n_parts = c->resid_parts;
    // a6: RMSNorm + gate/up + SwiGLU
    a = MfmaArgs{};
    a.W = s.gate; a.W2 = s.up; a.xb = R.xb; a.xb_lo = R.xb_lo; a.ldxb = d; a.N = ff; a.K = d; a.ssp = R.ssp; a.n_parts = R.n_parts;
    a.ssp_ld = c->ssp_ld; a.eps = cf.rms_eps; a.yb = ub; a.yb_lo = ub_lo; a.ldyb = ff;
    if ((e = launch_gateup(c, a, rows)) != hipSuccess) return e;
    // a7: down projection + residual; emits the next layer's (or the final) norm input
    a = MfmaArgs{};
    a.W = s.down; a.xb = ub; a.xb_lo = ub_lo; a.ldxb = ff; a.N = d; a.K = ff; a.y = R.h; a.ldy = d; a.yb = R.xb; a.yb_lo = R.xb_lo; a.ldyb = d;
    a.g_next = (const bf16_t*)norm_gain_for_layer(c, l + 1); a.ssp_next = R.ssp; a.ssp_ld = c->ssp_ld;
    if ((e = launch_down(c, a, rows)) != hipSuccess) return e;
    R.n_parts = c->resid_parts;
    return hipSuccess;
  }
  float* attn = (float*)(c->ws + c->o.attn);
  float* mlp = (float*)(c->ws + c->o.mlp);
  GemvArgs a{};
  a.eps = cf.rms_eps;
  // a2: RMSNorm + fused QKV projection (q, k, v are contiguous in the blob)
  a.W = w.q; a.gain = w.attn_norm; a.x = R.h; a.ldx = d; a.y = qkv; a.ldy = nqkv; a.N = nqkv; a.K = d;
  if ((e = gemv_rows<EPI_STORE, true>(c, a, rows)) != hipSuccess) return e;
  // a3 + a4: QK-RMSNorm + RoPE + KV append + split-K attention, then the merge
  if (r > kMaxRows && (e = launch_kv_append<float>(c, l, qkv, sel, offset, r)) != hipSuccess) return e;
  if ((e = launch_attention<float, float>(c, l, qkv, attn, (float*)nullptr, sel, offset, r, r > kMaxRows ? 2 : 1)) != hipSuccess) return e;
  // a5: O projection + residual
  a = GemvArgs{};
  a.W = w.o; a.x = attn; a.ldx = qd; a.y = R.h; a.ldy = d; a.N = d; a.K = qd;
  if ((e = gemv_rows<EPI_RESID, false>(c, a, rows)) != hipSuccess) return e;
  // a6: RMSNorm + gate/up + SwiGLU
  a = GemvArgs{};
  a.eps = cf.rms_eps;
  a.W = w.gate; a.W2 = w.up; a.gain = w.mlp_norm; a.x = R.h; a.ldx = d; a.y = mlp; a.ldy = ff; a.N = ff; a.K = d;
  if ((e = gemv_rows<EPI_SWIGLU, true>(c, a, rows)) != hipSuccess) return e;
  // a7: down projection + residual
  a = GemvArgs{};
  a.W = w.down; a.x = mlp; a.ldx = ff; a.y = R.h; a.ldy = d; a.N = d; a.K = ff;
  return gemv_rows<EPI_RESID, false>(c, a, rows);
}

// a9, first part: final RMSNorm + LM head (Eq. 5) of n_rows rows into logits [n_rows, vocab], selection keys into amax
hipError_t head_logits(dmtd_ctx* c, const Rows& R, int n_rows, float* logits, unsigned long long* amax, int amax_ld, int blocked = 0) {
  const dmtd_config& cf = c->cfg;
  if (c->packed) {
    MfmaArgs a{};
    a.W = c->lm_head_sw; a.xb = R.xb; a.xb_lo = R.xb_lo; a.ldxb = cf.hidden; a.N = cf.vocab; a.K = cf.hidden; a.ssp = R.ssp; a.n_parts = R.n_parts;
    a.ssp_ld = c->ssp_ld; a.eps = cf.rms_eps; a.y = logits; a.ldy = cf.vocab;
    a.amax = amax; a.amax_ld = amax_ld;
    a.blocked = blocked;         // rows of a larger pass (else the row count decides)
    return launch_lmhead(c, a, n_rows);
  }
  GemvArgs a{};
  a.eps = cf.rms_eps;
  a.W = c->lm_head; a.gain = c->final_norm; a.x = R.h; a.ldx = cf.hidden;
  a.y = logits; a.ldy = cf.vocab; a.N = cf.vocab; a.K = cf.hidden;
  a.amax = amax; a.amax_ld = amax_ld;
  return gemv_rows<EPI_LOGITS, true>(c, a, n_rows);
}

// a9: final RMSNorm + LM head + greedy selection for one row per sequence; then the step's bookkeeping
hipError_t run_head(dmtd_ctx* c, const Rows& R, int full, int write_tokens, int n_rows) {
  const dmtd_config& cf = c->cfg;
  unsigned long long* amax = c->amax;
  hipError_t e = head_logits(c, R, n_rows, (float*)(c->ws + c->o.logits), amax, cf.max_batch);
  if (e != hipSuccess) return e;
  if (c->sampling && write_tokens) {
    const float* z = (const float*)(c->ws + c->o.logits);
    const SampleCfg* sc = (const SampleCfg*)(c->ws + c->o.state + kStateSampleOff);
    const int slices = (cf.vocab + SAMPLE_SLICE - 1) / SAMPLE_SLICE;
    const SampleScratch ss{sample_count(c), (SampleCand*)(c->ws + c->o.sample_list), (unsigned long long*)(c->ws + c->o.sample_best), slices, sample_cap(cf)};
    hipLaunchKernelGGL(sample_scan_kernel, dim3(slices, n_rows), dim3(256), 0, c->stream, z, cf.vocab, sc, (const DevState*)dev_state(c),
                       (const unsigned long long*)amax, AMAX_CELLS, cf.max_batch, ss);
    hipLaunchKernelGGL(sample_pick_kernel, dim3(n_rows), dim3(1024), 0, c->stream, z, cf.vocab, sc, (const DevState*)dev_state(c), amax, AMAX_CELLS,
                       cf.max_batch, ss);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(finish_step_kernel, dim3(1), dim3(n_rows >= 16 ? 1024 : 64 * n_rows), 0, c->stream, dev_state(c), amax, AMAX_CELLS, cf.max_batch,
                     dev_tokens(c), (int*)(c->ws + c->o.emitted), cf.max_seq_len, n_rows, full, write_tokens, c->full_mask);
  return hipGetLastError();
}

Rows front_rows(dmtd_ctx* c) {
  bf16_t* xb = (bf16_t*)(c->ws + c->o.xb);
  return Rows{(float*)(c->ws + c->o.h), xb, xb + (size_t)row_capacity(c->cfg, c->wide_rows) * c->cfg.hidden, (float*)(c->ws + c->o.ssp), 1};
}
Rows late_rows(dmtd_ctx* c) {
  bf16_t* xb = (bf16_t*)(c->ws + c->o.xb_late);
  return Rows{(float*)(c->ws + c->o.h_late), xb, xb + late_row_capacity(c->cfg) * c->cfg.hidden, (float*)(c->ws + c->o.ssp_late), 1};
}

// One decode step (Sec. 2.2).  Full: embed the pending rows and the newest row, run the front
// layers on all of them, keep the newest row, run the late layers on it.  Late: embed the
// newest token and run the late layers only (Eq. 4, m = 0).
// ExDy row moves (rows_op_kernel): with or without the packed input of the norm of layer next_layer
hipError_t rows_op(dmtd_ctx* c, int mode, int n_rows, float* dst, const float* src_a, const float* src_b, int r, int c0, int rc,
                   int next_layer, bf16_t* xb, bf16_t* xb_lo, float* ssp) {
  const dmtd_config& cf = c->cfg;
  if (c->packed)
    hipLaunchKernelGGL(rows_op_kernel<true>, dim3(n_rows), dim3(256), 0, c->stream, mode, dst, src_a, src_b, cf.hidden, kMaxTau, r, c0, rc,
                       dev_state(c), (const bf16_t*)norm_gain_for_layer(c, next_layer), xb, xb_lo, ssp, blocked_rows(c, n_rows));
  else
    hipLaunchKernelGGL(rows_op_kernel<false>, dim3(n_rows), dim3(256), 0, c->stream, mode, dst, src_a, src_b, cf.hidden, kMaxTau, r, c0, rc,
                       dev_state(c), (const bf16_t*)nullptr, (bf16_t*)nullptr, (bf16_t*)nullptr, (float*)nullptr, 0);
  return hipGetLastError();
}

// One decode step (Sec. 2.2).  Full: embed the pending rows and the newest row, run the front
// layers on all of them, keep the newest row, run the late layers on it.  Late: embed the
// newest token and run the late layers only (Eq. 4, m = 0).
// ExDy variant (n_early = E > 0): every step first runs its own token through the E encoding layers; a late
// step stores that output for the refill and jumps to the late layers; a full step gathers the stored outputs
// of the pending tokens and the newest token's, runs the thinking layers E .. F-1 on them, and goes on as before.
hipError_t enqueue_step(dmtd_ctx* c, bool full, int r, int n_late) {
  const dmtd_config& cf = c->cfg;
  const int F = cf.n_layers - n_late, E = c->sched.n_early;
  Rows front = front_rows(c), late = late_rows(c);
  float* pend = (float*)(c->ws + c->o.pend_enc);
  hipError_t e;
  if (E > 0) {
    if ((e = embed_rows(c, late, POS_NTOK, 0, 1, 0)) != hipSuccess) return e;
    for (int l = 0; l < E; ++l)
      if ((e = run_layer(c, l, late, 1, POS_NTOK, 0)) != hipSuccess) return e;
  }
  if (full) {
    // the pending rows are causal among themselves, so groups of rows may pass the front
    // layers one after another (each group streams those layers' weights once)
    int c0 = 0, rc = 0;
    if (F > E) {
      for (; c0 < r; c0 += rc) {
        rc = r - c0 < kMaxRows ? r - c0 : kMaxRows;
        if (E > 0) {
          if ((e = rows_op(c, ROWS_GATHER, c->batch * rc, front.h, pend, late.h, r, c0, rc, E, front.xb, front.xb_lo, front.ssp)) != hipSuccess) return e;
          front.n_parts = 1;
        } else {
          if ((e = embed_rows(c, front, POS_NFRONT, c0, rc, 0)) != hipSuccess) return e;
        }
        for (int l = E; l < F; ++l)
          if ((e = run_layer(c, l, front, rc, POS_NFRONT, c0)) != hipSuccess) return e;
      }
      if (E > 0) {
        // the newest row continues; the literal Eq. 4 reading adds its encoding output (still in the late row buffer)
        if (c->packed)
          hipLaunchKernelGGL(take_last_pack_kernel, dim3(c->batch), dim3(256), 0, c->stream, front.h, late.h, rc, cf.hidden, 0,
                             (const bf16_t*)c->embed, dev_tokens(c), cf.max_seq_len, dev_state(c), (int)POS_NFRONT, c0 - rc,
                             (const bf16_t*)norm_gain_for_layer(c, F), late.xb, late.xb_lo, late.ssp,
                             cf.full_pos_add_embed ? (const float*)late.h : (const float*)nullptr, (const int*)nullptr, (const int*)nullptr,
                             blocked_rows(c, c->batch));
        else
          hipLaunchKernelGGL(take_last_rows_kernel<float>, dim3(c->batch), dim3(256), 0, c->stream, front.h, late.h, rc, cf.hidden,
                             0, (const float*)c->embed, dev_tokens(c), cf.max_seq_len, dev_state(c), (int)POS_NFRONT, c0 - rc,
                             cf.full_pos_add_embed ? (const float*)late.h : (const float*)nullptr, (const int*)nullptr, (const int*)nullptr);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        late.n_parts = 1;
      } else {
        if ((e = take_last_rows(c, front, late, rc, cf.full_pos_add_embed ? 1 : 0, POS_NFRONT, c0 - rc, F)) != hipSuccess) return e;
      }
    } else if (E > 0 && cf.full_pos_add_embed) {
      // no thinking layers: h_think = h_enc, and the literal reading feeds their sum
      if ((e = rows_op(c, ROWS_ADD, c->batch, late.h, late.h, late.h, 1, 0, 1, F, late.xb, late.xb_lo, late.ssp)) != hipSuccess) return e;
      late.n_parts = 1;
    } else if (E == 0) {
      // n_late = all layers: the newest token's embedding enters the late layers directly
      if ((e = embed_rows(c, late, POS_NTOK, 0, 1, F)) != hipSuccess) return e;
      if (cf.full_pos_add_embed && (e = add_embed_rows(c, late, POS_NTOK, 0, 1, F)) != hipSuccess) return e;
    }
  } else {
    if (E > 0) {
      // keep the encoding output for the refill; the row itself jumps to the late layers
      if (F > E) {
        if ((e = rows_op(c, ROWS_STASH, c->batch, pend, late.h, nullptr, 1, 0, 1, F, late.xb, late.xb_lo, late.ssp)) != hipSuccess) return e;
        late.n_parts = 1;
      }
    } else {
      if ((e = embed_rows(c, late, POS_NTOK, 0, 1, F)) != hipSuccess) return e;
    }
  }
  for (int l = F; l < cf.n_layers; ++l)
    if ((e = run_layer(c, l, late, 1, POS_NTOK, 0)) != hipSuccess) return e;
  return run_head(c, late, full ? 1 : 0, 1, c->batch);
}

// One decode step of a batch whose sequences are at different points of their cycles (Sec. 2.2, per sequence).  The
// sequences that start a new cycle pass the front layers with their pending rows - in one front pass or a few,
// over those sequences only (full_list: their slots, sorted by row count; groups: see front_groups) - and every
// sequence's newest token then shares ONE pass through the late layers and the LM head: the late layers read the front
// output for the former and the raw embedding for the others (Eq. 4).
hipError_t enqueue_step_mixed(dmtd_ctx* c, const std::vector<std::pair<int, int>>& groups /* (rows, sequences) */,
                              const std::vector<int>& full_rows /* of the sequences in full_list */, int n_late, const int* full_list,
                              const unsigned char* full_mask) {
  const dmtd_config& cf = c->cfg;
  const int F = cf.n_layers - n_late, B = c->batch;
  Rows front = front_rows(c), late = late_rows(c);
  hipError_t e;
  if ((e = embed_rows(c, late, POS_NTOK, 0, 1, F)) != hipSuccess) return e;
  int first = 0;
  for (const auto& grp : groups) {
    const int r = grp.first, n = grp.second;
    c->batch = n;
    c->late_batch = B;
    c->fmap = full_list + first;
    c->live = full_rows.data() + first;
    e = embed_rows(c, front, POS_NFRONT, 0, r, 0);
    for (int l = 0; l < F && e == hipSuccess; ++l) e = run_layer(c, l, front, r, POS_NFRONT, 0);
    if (e == hipSuccess) e = take_last_rows(c, front, late, r, cf.full_pos_add_embed ? 1 : 0, POS_NFRONT, 0, F);
    c->batch = B;
    c->late_batch = 0;
    c->fmap = nullptr;
    c->live = nullptr;
    if (e != hipSuccess) return e;
    first += n;
  }
  for (int l = F; l < cf.n_layers; ++l)
    if ((e = run_layer(c, l, late, 1, POS_NTOK, 0)) != hipSuccess) return e;
  c->full_mask = full_mask;
  e = run_head(c, late, 0, 1, B);
  c->full_mask = nullptr;
  return e;
}

// What a front pass with that many rows costs.  bf16, us per layer: the attention and the launches 25, the layer's weights, and little
// per row, dead or alive, as long as the projections stay in the same kernel: beyond 64 and beyond 128 rows the tiled one takes longer steps.
// (Projections alone, us with 1 / 16 / 64 / 72 / 128 / 136 rows: 2560 wide 42 / 54 / 81 / 98 / 113 / 163, 1536 29 / 37 / 62 / 75 / 84 / 121, 1024
// 18 / 27 / 50 / 59 / 70 / 102, 896 20 / 26 / 54 / 68 / 80 / 108, 512 wide with one KV head 17 / 19 / 43 / 52 / 57 / 84.  With one price for every width
// and row, 70 rows a pass, 8 sequences of 2 rows beside one of 8 went together in narrow models too; us per step of 6 layers, a pass per row count /
// together: 896 wide, 300 keys 162 / 171, 8k keys 191 / 202, 512 wide 132 / 138.)
// fp32, in rows: rows up to 1024 wide go through gemv_direct_kernel, whose launches cost more than another group of 4 rows; wider ones
// take 4 rows per weight stream.  us per step, a pass priced at 8 / 24 rows: 16 sequences in cycles of 1 to 8, 64 wide 125 / 112, 256 wide 138 / 124,
// 512 167 / 155, 1024 321 / 321, 1536 697 / 740, 2048 745 / 797; cycles of 1, 2, 4 and 6, 1024 wide 180 / 173, 1536 305 / 315.
double front_pass_cost(const dmtd_config& cf, int rows) {
  if (cf.dtype == DMTD_DTYPE_F32) return (cf.hidden <= 1024 ? 24.0 : 8.0) + rows;
  const double weight_us = (double)swizzled_layer_elems(cf) * 2 / 6.0e6;
  return 25.0 + weight_us + 0.5 * rows + (rows > 64 ? 10.0 : 0.0) + (rows > 128 && rows <= kTiledRows ? 25.0 : 0.0);
}

// The front passes of such a step: the sequences that start a cycle, sorted by row count, cut into runs; a run passes the front
// layers together, with room for its largest row count per sequence (live_rows).  The cut with the least cost is taken.
// 2560 wide, 5 sequences with cycles of 1 to 4 tokens, 24 steps: a pass per row count 19.0 ms for the whole request, its prefill included,
// one pass per step 16.3 ms.
std::vector<std::pair<int, int>> front_groups(const dmtd_config& cf, const std::vector<int>& rows /* ascending */) {
  std::vector<std::pair<int, int>> counts, groups;      // (rows, sequences): the distinct row counts; the passes
  for (int r : rows) {
    if (counts.empty() || counts.back().first != r) counts.emplace_back(r, 0);
    counts.back().second += 1;
  }
  const int n = (int)counts.size();
  std::vector<double> cost(n + 1, 0.0);   // cost[i]: the first i counts
  std::vector<int> from(n + 1, 0);
  for (int i = 1; i <= n; ++i) {
    int seqs = 0;
    for (int j = i - 1; j >= 0; --j) {
      seqs += counts[j].second;
      const double v = cost[j] + front_pass_cost(cf, seqs * counts[i - 1].first);
      if (j == i - 1 || v < cost[i]) { cost[i] = v; from[i] = j; }
    }
  }
  for (int i = n; i > 0; i = from[i]) {
    int seqs = 0;
    for (int j = from[i]; j < i; ++j) seqs += counts[j].second;
    groups.emplace_back(counts[i - 1].first, seqs);
  }
  std::reverse(groups.begin(), groups.end());
  return groups;
}

// K/V bytes one layer's attention reads for the whole batch at context length ctx
bool kv_is_large(const dmtd_ctx* c, int ctx) {
  const size_t bytes = (size_t)c->batch * ctx * c->cfg.n_kv_heads * c->cfg.head_dim * 2 * c->elem;
  return bytes > ((size_t)48 << 20);
}

void choose_attention(dmtd_ctx* c, int ctx) {
  c->att_bucket = ctx <= 256 ? 256 : (ctx + 511) / 512 * 512;      // 256: contexts short enough for one range per block at small batches
  c->share_kv = kv_is_large(c, ctx);
}

int run_step(dmtd_ctx* c, const Step& s, int n_late) {
  choose_attention(c, s.pos + 1);
  if (!c->cfg.use_graphs) {
    HIP_TRY(c, enqueue_step(c, s.full, s.rows, n_late));
    return DMTD_OK;
  }
  // everything a captured step bakes in: grids and row counts follow from the batch, the attention launch shape from the context bucket
  const auto key = std::make_tuple(s.full ? 1 : 0, s.rows, n_late * 4096 + c->sched.n_early + (c->sampling ? (1 << 30) : 0), c->att_bucket * 2 + (c->share_kv ? 1 : 0), c->batch);
  auto it = c->graphs.find(key);
  if (it == c->graphs.end()) {
    hipGraph_t graph = nullptr;
    HIP_TRY(c, hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal));
    hipError_t e = enqueue_step(c, s.full, s.rows, n_late);
    hipError_t e2 = hipStreamEndCapture(c->stream, &graph);
    if (e != hipSuccess || e2 != hipSuccess) {
      if (graph) (void)hipGraphDestroy(graph);
      c->err = std::string("graph capture failed: ") + hipGetErrorString(e != hipSuccess ? e : e2);
      return DMTD_EHIP;
    }
    hipGraphExec_t exec = nullptr;
    hipError_t e3 = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e3 != hipSuccess) { c->err = std::string("hipGraphInstantiate: ") + hipGetErrorString(e3); return DMTD_EHIP; }
    it = c->graphs.emplace(key, exec).first;
  }
  HIP_TRY(c, hipGraphLaunch(it->second, c->stream));
  return DMTD_OK;
}

// Several consecutive steps of one call as ONE graph (dmtd_decode): the steps of a cycle - a full step and the late-only
// steps behind it - or, at tau = 1, up to kStepsPerGraph full steps.  Between two graph launches the GPU idles for ~8 us
// (end of one graph to the first kernel of the next), three times per C3 cycle with a graph per step.  The steps of a
// group share their attention launch shape (context bucket, KV sharing), otherwise the group ends early.
constexpr int kStepsPerGraph = 4;
int run_steps_grouped(dmtd_ctx* c, const std::vector<Step>& steps, int tau, int n_late) {
  const int n = (int)steps.size();
  int i = 0;
  while (i < n) {
    choose_attention(c, steps[i].pos + 1);
    const int bucket = c->att_bucket;
    const bool share = c->share_kv;
    int j = i + 1;
    const int limit = tau > 1 ? tau : kStepsPerGraph;
    while (j < n && j - i < limit && !(tau > 1 && steps[j].full)) {
      choose_attention(c, steps[j].pos + 1);
      if (c->att_bucket != bucket || c->share_kv != share) break;
      ++j;
    }
    if (!c->cfg.use_graphs || j - i == 1) {
      const int rc = run_step(c, steps[i], n_late);
      if (rc != DMTD_OK) return rc;
      i += 1;
      continue;
    }
    std::vector<int> key = {c->batch, n_late, c->sched.n_early, c->sampling ? 1 : 0, bucket, share ? 1 : 0};
    for (int k = i; k < j; ++k) { key.push_back(steps[k].full ? 1 : 0); key.push_back(steps[k].rows); }
    auto it = c->group_graphs.find(key);
    if (it == c->group_graphs.end()) {
      hipGraph_t graph = nullptr;
      HIP_TRY(c, hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal));
      hipError_t e = hipSuccess;
      for (int k = i; k < j && e == hipSuccess; ++k) {
        choose_attention(c, steps[k].pos + 1);
        e = enqueue_step(c, steps[k].full, steps[k].rows, n_late);
      }
      hipError_t e2 = hipStreamEndCapture(c->stream, &graph);
      if (e != hipSuccess || e2 != hipSuccess) {
        if (graph) (void)hipGraphDestroy(graph);
        c->err = std::string("graph capture failed: ") + hipGetErrorString(e != hipSuccess ? e : e2);
        return DMTD_EHIP;
      }
      hipGraphExec_t exec = nullptr;
      hipError_t e3 = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
      (void)hipGraphDestroy(graph);
      if (e3 != hipSuccess) { c->err = std::string("hipGraphInstantiate: ") + hipGetErrorString(e3); return DMTD_EHIP; }
      it = c->group_graphs.emplace(key, exec).first;
    }
    HIP_TRY(c, hipGraphLaunch(it->second, c->stream));
    i = j;
  }
  return DMTD_OK;
}

struct PartRowsGuard {     // restores the partials' row layout on every way out of a prefill-type pass
  dmtd_ctx* c; int saved;
  ~PartRowsGuard() { c->part_rows = saved; }
};

// Prefill (Sec. 2.2): all prompt positions through all layers, in chunks of rows
hipError_t enqueue_prefill(dmtd_ctx* c, int P, int n_late, bool ragged) {
  const dmtd_config& cf = c->cfg;
  Rows front = front_rows(c), late = late_rows(c);
  const int add_at = cf.full_pos_add_embed ? cf.n_layers - n_late : -1;
  hipError_t e;
  hipLaunchKernelGGL(set_state_kernel, dim3(1), dim3(64), 0, c->stream, dev_state(c), P - 1, P - 1, cf.max_batch, sample_count(c));
  int r_last = 0, p_last = 0;
  const int chunk = pass_positions(cf, c->wide_rows, c->batch);
  PartRowsGuard guard{c, c->part_rows};
  c->part_rows = step_positions(c->batch);   // the attention partials of a pass (see attention_single_range)
  for (int p0 = 0; p0 < P; p0 += chunk) {
    const int r = P - p0 < chunk ? P - p0 : chunk;
    choose_attention(c, p0 + r);
    if ((e = embed_rows(c, front, POS_EXPLICIT, p0, r, 0)) != hipSuccess) return e;
    const int E = c->sched.n_early;
    for (int l = 0; l < cf.n_layers; ++l) {
      if (add_at >= 0 && E > 0 && l == E) {
        // literal Eq. 4, ExDy variant: the encoding output is what full positions get added at the late boundary
        if ((e = hipMemcpyAsync(c->ws + c->o.enc_tmp, front.h, (size_t)c->batch * r * cf.hidden * 4, hipMemcpyDeviceToDevice, c->stream)) != hipSuccess) return e;
      }
      if (l == add_at) {
        if (E > 0) {
          if ((e = rows_op(c, ROWS_ADD, c->batch * r, front.h, front.h, (const float*)(c->ws + c->o.enc_tmp), 1, 0, 1, l, front.xb, front.xb_lo, front.ssp)) != hipSuccess) return e;
          front.n_parts = 1;
        } else if ((e = add_embed_rows(c, front, POS_EXPLICIT, p0, r, l)) != hipSuccess) return e;
      }
      if ((e = run_layer(c, l, front, r, POS_EXPLICIT, p0)) != hipSuccess) return e;
    }
    r_last = r; p_last = p0;
    // prompts of different lengths: a sequence whose last prompt position lies in this chunk hands that row to the LM head
    if (ragged && (e = take_last_rows(c, front, late, r, 0, POS_EXPLICIT, p0, cf.n_layers,
                                      (const int*)(c->ws + c->o.state + kStateDeltaOff) + 2 * cf.max_batch)) != hipSuccess) return e;
  }
  if (!ragged && (e = take_last_rows(c, front, late, r_last, 0, POS_EXPLICIT, p_last, cf.n_layers)) != hipSuccess) return e;
  return run_head(c, late, 1, 1, c->batch);   // state goes from P-1 to n_tok = n_front = P
}

// One chunk of the whole-sequence masked forward (Sec. 2.1, Eqs. 1-5): positions p0 .. p0+r-1 of every sequence pass the
// encoding and thinking layers, Eq. 4 picks each position's input to the decoding layers by its mask bit, the
// decoding layers and the LM head follow for every row, and a row kernel takes the Eq. 6 summands and the argmax.
// Earlier chunks are seen through the KV caches, exactly as later decode steps would see them.
hipError_t enqueue_masked_chunk(dmtd_ctx* c, Rows& R, int p0, int r, int n_late) {
  const dmtd_config& cf = c->cfg;
  const int F = cf.n_layers - n_late, E = c->sched.n_early, rows = c->batch * r;
  R = front_rows(c);
  float* enc = (float*)(c->ws + c->o.enc_tmp);
  hipError_t e;
  choose_attention(c, p0 + r);
  if ((e = embed_rows(c, R, POS_EXPLICIT, p0, r, 0)) != hipSuccess) return e;
  for (int l = 0; l <= F; ++l) {
    if (E > 0 && l == E &&
        (e = hipMemcpyAsync(enc, R.h, (size_t)rows * cf.hidden * 4, hipMemcpyDeviceToDevice, c->stream)) != hipSuccess) return e;
    if (l < F && (e = run_layer(c, l, R, r, POS_EXPLICIT, p0)) != hipSuccess) return e;
  }
  const int* mask = (const int*)(c->ws + c->o.mask);
  if (c->packed) {
    hipLaunchKernelGGL((mask_combine_kernel<bf16_t, true>), dim3(rows), dim3(256), 0, c->stream, R.h, E > 0 ? (const float*)enc : (const float*)nullptr,
                       (const bf16_t*)c->embed, dev_tokens(c), cf.max_seq_len, mask, p0, r, cf.hidden, cf.full_pos_add_embed,
                       (const bf16_t*)norm_gain_for_layer(c, F), R.xb, R.xb_lo, R.ssp, blocked_rows(c, rows));
    R.n_parts = 1;
  } else {
    hipLaunchKernelGGL((mask_combine_kernel<float, false>), dim3(rows), dim3(256), 0, c->stream, R.h, E > 0 ? (const float*)enc : (const float*)nullptr,
                       (const float*)c->embed, dev_tokens(c), cf.max_seq_len, mask, p0, r, cf.hidden, cf.full_pos_add_embed,
                       (const bf16_t*)nullptr, (bf16_t*)nullptr, (bf16_t*)nullptr, (float*)nullptr, 0);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  for (int l = F; l < cf.n_layers; ++l)
    if ((e = run_layer(c, l, R, r, POS_EXPLICIT, p0)) != hipSuccess) return e;
  return hipSuccess;
}

// The LM head and the Eq. 6 summands of rows [m0, m0 + n_rows) of the chunk that enqueue_masked_chunk left in the row buffers
hipError_t enqueue_masked_head(dmtd_ctx* c, const Rows& R, int m0 /* a multiple of 16 */, int n_rows, int p0, int r, int n) {
  const dmtd_config& cf = c->cfg;
  Rows H = R;
  H.h += (size_t)m0 * cf.hidden;
  if (c->packed) { H.xb += (size_t)m0 * cf.hidden; H.xb_lo += (size_t)m0 * cf.hidden; H.ssp += m0; }
  float* logits = (float*)(c->ws + c->o.logits_rows);
  const hipError_t e = head_logits(c, H, n_rows, logits, (unsigned long long*)(c->ws + c->o.amax_rows), head_row_capacity(cf, c->wide_rows), blocked_rows(c, c->batch * r));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(nll_rows_kernel, dim3(n_rows), dim3(1024), 0, c->stream, (const float*)logits, cf.vocab, (const int*)dev_tokens(c), cf.max_seq_len,
                     m0, p0, r, n, (float*)(c->ws + c->o.nll), (int*)(c->ws + c->o.best));
  return hipGetLastError();
}

// The same for all rows of a chunk that went through the wide GEMM, without their logits: the LM head's tiles leave per row what the loss and
// the greedy choice need (EPI_NLL).  Against 512 rows of logits at a time and a launch
// that reads them again (2046 rows, 2560 wide, 152k entries): four times 781 + 67 us before, 2741 + 12 now: no logits written, the weights read once, and
// 4752 tiles in 19 rounds of the chip where 1188 took 5.
// The results live in the layers' scratch, like the logits do; false: they do not fit (a vocabulary of a few entries).
bool masked_nll_fits(const dmtd_config& cf, int wide_rows, int rows) {
  const size_t nt = (size_t)(cf.vocab + GW_BN - 1) / GW_BN, ld = ((size_t)rows + 15) / 16 * 16;
  return cf.dtype == DMTD_DTYPE_BF16 && rows > kTiledRows && ld * (nt * GwTile<128, GW_BN>::WN * sizeof(float2) + 16) <= (size_t)head_row_capacity(cf, wide_rows) * cf.vocab * 4;
}
hipError_t enqueue_masked_nll(dmtd_ctx* c, const Rows& R, int rows, int p0, int r, int n) {
  const dmtd_config& cf = c->cfg;
  const WideChoice w = choose_wide<EPI_LOGITS>(cf, c->num_cus, rows, cf.vocab, cf.hidden);      // the same tiles, all whole
  const int ld = (rows + 15) / 16 * 16, n_parts = w.nt * (w.bm == 128 ? GwTile<128, GW_BN>::WN : GwTile<256, GW_BN>::WN);
  char* base = c->ws + c->o.logits_rows;
  float2* part = (float2*)base;
  unsigned long long* keys = (unsigned long long*)(part + (size_t)n_parts * ld);
  float* zt = (float*)(keys + ld);
  int* target = (int*)(zt + ld);
  hipLaunchKernelGGL(nll_targets_kernel, dim3((rows + 255) / 256), dim3(256), 0, c->stream, (const int*)dev_tokens(c), cf.max_seq_len, rows, p0, r, n, target, keys);
  MfmaArgs a{};
  a.W = c->lm_head_sw; a.xb = R.xb; a.xb_lo = R.xb_lo; a.ldxb = cf.hidden; a.M = rows; a.N = cf.vocab; a.K = cf.hidden; a.ssp = R.ssp; a.n_parts = R.n_parts;
  a.ssp_ld = c->ssp_ld; a.eps = cf.rms_eps; a.blocked = 1;
  a.part = (float*)part; a.ldp = ld; a.amax = keys; a.ssp_next = zt; a.g_next = (const bf16_t*)target;
  const hipError_t e = w.bm == 128 ? launch_wide_tiles<EPI_NLL, true, 128, GW_BN>(c, a, w.nt, w.p) : launch_wide_tiles<EPI_NLL, true, 256, GW_BN>(c, a, w.nt, w.p);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(nll_merge_kernel, dim3((rows + 7) / 8), dim3(256), 0, c->stream, (const float2*)part, n_parts, ld, (const int*)target, (const float*)zt,
                     (const unsigned long long*)keys, cf.max_seq_len, rows, p0, r, (float*)(c->ws + c->o.nll), (int*)(c->ws + c->o.best));
  return hipGetLastError();
}

// One launch of one kernel kind on layer l, for dmtd_time_kernel.  Outputs go to scratch
// buffers only (never the late rows, the caches, the token history or the scheduler state).
hipError_t time_one(dmtd_ctx* c, int kind, int l, int rows) {
  const dmtd_config& cf = c->cfg;
  const int d = cf.hidden, hd = cf.head_dim, ff = cf.intermediate;
  const int nqkv = (cf.n_q_heads + 2 * cf.n_kv_heads) * hd, qd = cf.n_q_heads * hd;
  Rows R = front_rows(c);
  float* qkv = (float*)(c->ws + c->o.qkv);
  const LayerW& w = c->layers[l];
  if (kind >= DMTD_K_READ_QKV && kind <= DMTD_K_READ_DOWN) {
    // nothing but a read of the bytes the projection of that kind streams for layer l (the stored weight image)
    const LayerSw& s = c->sw[l];
    const bf16_t *p0 = nullptr, *p1 = nullptr;
    size_t n0 = 0, n1 = 0;                       // 16-byte units
    switch (kind) {
      case DMTD_K_READ_QKV:    p0 = s.qkv;  n0 = swizzled_elems(nqkv, d) / 8; break;
      case DMTD_K_READ_OPROJ:  p0 = s.o;    n0 = swizzled_elems(d, qd) / 8; break;
      case DMTD_K_READ_GATEUP: p0 = s.gate; n0 = swizzled_elems(ff, d) / 8; p1 = s.up; n1 = n0; break;
      default:                 p0 = s.down; n0 = swizzled_elems(d, ff) / 8; break;
    }
    hipLaunchKernelGGL(read_only_kernel, dim3(2048), dim3(256), 0, c->stream, (const u32x4*)p0, n0, (const u32x4*)(p1 ? p1 : p0), n1,
                       (u32x4*)qkv);
    return hipGetLastError();
  }
  if (kind == DMTD_K_ATTN) {
    // attention for `rows` query rows per sequence ending at the newest cached position
    const int last = c->sched.n_tok - 1;
    const int r = rows <= last + 1 ? rows : 1;
    // the cache append is switched off: the launch scores the rows' new keys from the scratch q/k/v, writes nothing
    choose_attention(c, last + 1);
    if (c->packed) {
      c->fold_merge = true;      // as in a step: no merge launch where the O projection merges
      const hipError_t e = launch_attention<bf16_t, bf16_t>(c, l, qkv, (bf16_t*)(c->ws + c->o.attn), (bf16_t*)(c->ws + c->o.attn) + (size_t)row_capacity(cf, c->wide_rows) * cf.n_q_heads * cf.head_dim, (int)POS_EXPLICIT, last - r + 1, r, 0);
      c->fold_merge = false;
      c->merge_pending = MergeSrc{};
      return e;
    }
    return launch_attention<float, float>(c, l, qkv, (float*)(c->ws + c->o.attn), (float*)nullptr, (int)POS_EXPLICIT, last - r + 1, r, 0);
  }
  if (kind == DMTD_K_LMHEAD) {
    R.n_parts = 1;
    return run_head(c, R, 0, 0, rows);     // the real LM-head kernel; keys cleared, no token or state side effects
  }
  if (c->packed) {
    const LayerSw& s = c->sw[l];
    const size_t rows_cap = row_capacity(cf, c->wide_rows);
    bf16_t* ab = (bf16_t*)(c->ws + c->o.attn);
    bf16_t* ab_lo = ab + rows_cap * qd;
    bf16_t* ub = (bf16_t*)(c->ws + c->o.mlp);
    bf16_t* ub_lo = ub + rows_cap * ff;
    MfmaArgs a{};
    a.ssp_ld = c->ssp_ld; a.eps = cf.rms_eps;
    switch (kind) {
      case DMTD_K_QKV:
        a.W = s.qkv; a.xb = R.xb; a.xb_lo = R.xb_lo; a.ldxb = d; a.N = nqkv; a.K = d; a.ssp = R.ssp; a.n_parts = 1; a.y = qkv; a.ldy = nqkv;
        return launch_qkv(c, a, rows);
      case DMTD_K_OPROJ:
        a.W = s.o; a.xb = ab; a.xb_lo = ab_lo; a.ldxb = qd; a.N = d; a.K = qd; a.y = R.h; a.ldy = d; a.yb = R.xb; a.yb_lo = R.xb_lo; a.ldyb = d;
        a.g_next = (const bf16_t*)w.mlp_norm; a.ssp_next = R.ssp;
        if (const int r = rows / c->batch, last = c->sched.n_tok - 1; r * c->batch == rows && r <= kMaxRows && r <= last + 1) {
          choose_attention(c, last + 1);
          if (const AttRanges ar = attention_ranges(c, r); !attention_single_range(c, r) && oproj_merges(c, r, ar))
            c->merge_pending = merge_source(c, r, ar, (int)POS_EXPLICIT, last - r + 1);
        }
        return launch_oproj(c, a, rows);
      case DMTD_K_GATEUP:
        a.W = s.gate; a.W2 = s.up; a.xb = R.xb; a.xb_lo = R.xb_lo; a.ldxb = d; a.N = ff; a.K = d; a.ssp = R.ssp; a.n_parts = c->resid_parts;
        a.yb = ub; a.yb_lo = ub_lo; a.ldyb = ff;
        return launch_gateup(c, a, rows);
      default:
        a.W = s.down; a.xb = ub; a.xb_lo = ub_lo; a.ldxb = ff; a.N = d; a.K = ff; a.y = R.h; a.ldy = d; a.yb = R.xb; a.yb_lo = R.xb_lo; a.ldyb = d;
        a.g_next = (const bf16_t*)norm_gain_for_layer(c, l + 1); a.ssp_next = R.ssp;
        return launch_down(c, a, rows);
    }
  }
  float* attn = (float*)(c->ws + c->o.attn);
  float* mlp = (float*)(c->ws + c->o.mlp);
  GemvArgs a{};
  a.eps = cf.rms_eps;
  switch (kind) {
    case DMTD_K_QKV:
      a.W = w.q; a.gain = w.attn_norm; a.x = R.h; a.ldx = d; a.y = qkv; a.ldy = nqkv; a.N = nqkv; a.K = d;
      return gemv_rows<EPI_STORE, true>(c, a, rows);
    case DMTD_K_OPROJ:
      a.W = w.o; a.x = attn; a.ldx = qd; a.y = R.h; a.ldy = d; a.N = d; a.K = qd;
      return gemv_rows<EPI_RESID, false>(c, a, rows);
    case DMTD_K_GATEUP:
      a.W = w.gate; a.W2 = w.up; a.gain = w.mlp_norm; a.x = R.h; a.ldx = d; a.y = mlp; a.ldy = ff; a.N = ff; a.K = d;
      return gemv_rows<EPI_SWIGLU, true>(c, a, rows);
    default:
      a.W = w.down; a.x = mlp; a.ldx = ff; a.y = R.h; a.ldy = d; a.N = d; a.K = ff;
      return gemv_rows<EPI_RESID, false>(c, a, rows);
  }
}

void destroy_graphs(dmtd_ctx* c) {
  for (auto& kv : c->graphs) (void)hipGraphExecDestroy(kv.second);
  c->graphs.clear();
  for (auto& kv : c->group_graphs) (void)hipGraphExecDestroy(kv.second);
  c->group_graphs.clear();
  for (auto& kv : c->mixed_graphs) (void)hipGraphExecDestroy(kv.second);
  c->mixed_graphs.clear();
}

}  // namespace

// ============================================================================ C ABI

extern "C" {

size_t dmtd_workspace_bytes(const dmtd_config* cfg) {
  std::string why;
  if (!valid_config(cfg, why)) return 0;
  return layout(*cfg).total;
}

int dmtd_create(const dmtd_config* cfg, const void* weights_dev, size_t weights_bytes, void* workspace_dev,
                size_t workspace_bytes, dmtd_ctx** out) {
  std::string why;
  if (!out) { g_create_error = "null out pointer"; return DMTD_EINVAL; }
  *out = nullptr;
  if (!valid_config(cfg, why)) { g_create_error = why; return DMTD_EINVAL; }
  const size_t elem = cfg->dtype == DMTD_DTYPE_F32 ? 4 : 2;
  int wide = kWideRows;
  Ws lay = layout(*cfg);
  if (!cfg->dry_run) {
    if (!weights_dev || !workspace_dev) { g_create_error = "null device pointer"; return DMTD_EINVAL; }
    if (((uintptr_t)weights_dev & 15) || ((uintptr_t)workspace_dev & 255)) {
      g_create_error = "weights must be 16-byte aligned and the workspace 256-byte aligned"; return DMTD_EINVAL;
    }
    if (weights_bytes != weight_elems(*cfg) * elem) {
      g_create_error = "weight blob size does not match the configuration"; return DMTD_EINVAL;
    }
    // a workspace with no room for full passes gets shorter ones, down to kPassRows rows
    while (workspace_bytes < lay.total && wide > kPassRows) lay = layout(*cfg, wide /= 2);
    if (workspace_bytes < lay.total) { g_create_error = "workspace too small"; return DMTD_ECAPACITY; }
  }
  dmtd_ctx* c = new dmtd_ctx();
  c->cfg = *cfg;
  c->elem = (int)elem;
  c->o = lay;
  c->stream = (hipStream_t)cfg->stream;
  c->sched.n_layers = cfg->n_layers;
  c->sched.max_seq_len = cfg->max_seq_len;
  c->packed = cfg->dtype == DMTD_DTYPE_BF16;
  c->wide_rows = wide;
  c->ssp_ld = row_capacity(*cfg, wide);
  if (const char* ev = std::getenv("DMTD_TEST_FAIL_STEP")) c->test_fail_step = std::atoi(ev);
  c->plan_buf.reserve(kMaxTau + 1);
  c->sched.trace.reserve((size_t)12 * cfg->max_seq_len + 64);        // at most 3 records of 4 per step: later steps never reallocate
  if (!cfg->dry_run) {
    c->wbase = (const char*)weights_dev;
    c->ws = (char*)workspace_dev;
    c->part_o = (float*)(c->ws + lay.part_o);
    c->part_ml = (float*)(c->ws + lay.part_ml);
    c->amax = (unsigned long long*)(c->ws + lay.amax);
    c->gemm_part = c->packed ? (float*)(c->ws + lay.gemm_part) : nullptr;
    c->part_rows = kMaxRows;
    {
      hipError_t se = static_scratch_for_current_device(&c->static_scratch);
      if (se != hipSuccess) { g_create_error = std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(se); delete c; return DMTD_EHIP; }
    }
    // carve the blob
    const size_t d = cfg->hidden, qd = (size_t)cfg->n_q_heads * cfg->head_dim, kd = (size_t)cfg->n_kv_heads * cfg->head_dim;
    const size_t ff = cfg->intermediate, hd = cfg->head_dim;
    size_t off = 0;
    auto take = [&](size_t n) { const void* p = c->wbase + off * elem; off += n; return p; };
    c->embed = take((size_t)cfg->vocab * d);
    c->layers.resize(cfg->n_layers);
    for (LayerW& w : c->layers) {
      w.attn_norm = take(d); w.q = take(qd * d); w.k = take(kd * d); w.v = take(kd * d);
      w.q_norm = take(hd); w.k_norm = take(hd); w.o = take(d * qd); w.mlp_norm = take(d);
      w.gate = take(ff * d); w.up = take(ff * d); w.down = take(d * ff);
    }
    c->final_norm = take(d);
    c->lm_head = cfg->tied_embeddings ? c->embed : take((size_t)cfg->vocab * d);

    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
      g_create_error = "no HIP device"; delete c; return DMTD_EHIP;
    }
    c->num_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    // rotary frequency table theta^(-2i/hd) in double; counters and state cleared
    std::vector<double> inv(hd / 2);
    for (size_t i = 0; i < hd / 2; ++i) inv[i] = std::pow((double)cfg->rope_theta, -2.0 * (double)i / (double)hd);
    hipError_t e = hipMemcpyAsync(c->ws + lay.inv_freq, inv.data(), inv.size() * 8, hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) {
      hipLaunchKernelGGL(rope_table_kernel, dim3(1024), dim3(256), 0, c->stream, (const double*)(c->ws + lay.inv_freq),
                         (float2*)(c->ws + lay.rope_tab), cfg->max_seq_len, (int)(hd / 2));
      e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemsetAsync(c->ws + lay.amax, 0, (size_t)AMAX_CELLS * cfg->max_batch * 8, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(c->ws + lay.state, 0, kStateDeltaOff + 12 * (size_t)cfg->max_batch, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(c->ws + lay.kv, 0, lay.kv_layer_stride * cfg->n_layers, c->stream);
    if (e == hipSuccess && c->packed) {
      // one-time repack of every matrix into MFMA operand order (q, k, v are contiguous: one fused matrix)
      bf16_t* dst = (bf16_t*)(c->ws + lay.wsw);
      auto swz = [&](const void* src, size_t N, size_t K) {
        const bf16_t* out = dst;
        hipLaunchKernelGGL(swizzle_weights_kernel, dim3(2048), dim3(256), 0, c->stream, (const bf16_t*)src, dst, (int)N, (int)K);
        dst += swizzled_elems(N, K);
        return out;
      };
      const size_t nqkv = qd + 2 * kd;
      c->sw.resize(cfg->n_layers);
      for (int l = 0; l < cfg->n_layers; ++l) {
        const LayerW& w = c->layers[l];
        LayerSw& s = c->sw[l];
        s.qkv = swz(w.q, nqkv, d); s.o = swz(w.o, d, qd); s.gate = swz(w.gate, ff, d); s.up = swz(w.up, ff, d);
        s.down = swz(w.down, d, ff);
      }
      c->lm_head_sw = swz(c->lm_head, cfg->vocab, d);
      e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) { g_create_error = std::string("workspace setup: ") + hipGetErrorString(e); delete c; return DMTD_EHIP; }
  }
  *out = c;
  return DMTD_OK;
}

static int prefill_impl(dmtd_ctx* c, const int32_t* tokens, int32_t batch, int32_t prompt_len, const int32_t* lengths, int32_t n_late,
                        int32_t* first_tokens) {
  if (!c) return DMTD_EINVAL;
  const dmtd_config& cf = c->cfg;
  if (!tokens) { c->err = "null tokens"; return DMTD_EINVAL; }
  if (batch < 1 || batch > cf.max_batch) { c->err = "batch outside [1, max_batch]"; return DMTD_EINVAL; }
  if (prompt_len < 1) { c->err = "prompt_len must be >= 1"; return DMTD_EINVAL; }
  if (cf.full_pos_add_embed && (n_late < 1 || n_late > cf.n_layers)) { c->err = "the literal Eq. 4 reading needs n_late at prefill"; return DMTD_EINVAL; }
  if (cf.full_pos_add_embed && c->sched.n_early + n_late > cf.n_layers) { c->err = "n_early + n_late exceeds the number of layers"; return DMTD_EINVAL; }
  if (c->sched.n_tok != 0) { c->err = "already prefilled; call dmtd_reset first"; return DMTD_ESTATE; }
  if (prompt_len >= cf.max_seq_len) { c->err = "prompt does not leave room for a generated token"; return DMTD_ECAPACITY; }
  bool ragged = false;
  if (lengths) {
    int longest = 0;
    for (int b = 0; b < batch; ++b) {
      if (lengths[b] < 1 || lengths[b] > prompt_len) { c->err = "prompt length outside [1, prompt_len]"; return DMTD_EINVAL; }
      if (lengths[b] > longest) longest = lengths[b];
      ragged = ragged || lengths[b] != prompt_len;
    }
    if (longest != prompt_len) { c->err = "prompt_len must be the longest prompt's length"; return DMTD_EINVAL; }
  }
  for (int b = 0; b < batch; ++b) {
    const int len = lengths ? lengths[b] : prompt_len;
    for (int i = 0; i < len; ++i) {
      const int32_t t = tokens[(size_t)b * prompt_len + i];
      if (t < 0 || t >= cf.vocab) { c->err = "token id outside the vocabulary"; return DMTD_EINVAL; }
    }
  }
  c->batch = batch;
  if (!cf.dry_run) {
    int* dtok = (int*)(c->ws + c->o.tokens);
    // padding behind a shorter prompt is replaced by token 0: those rows run (their results are never read) and must index the table safely
    std::vector<int32_t> tk(tokens, tokens + (size_t)batch * prompt_len);
    std::vector<int32_t> meta(3 * (size_t)cf.max_batch, 0);       // (delta, front)[max_batch], last_prompt_pos[max_batch]
    for (int b = 0; b < batch; ++b) {
      const int len = lengths ? lengths[b] : prompt_len;
      for (int i = len; i < prompt_len; ++i) tk[(size_t)b * prompt_len + i] = 0;
      meta[2 * b] = len - prompt_len;                            // the front positions are set by the prefill itself
      meta[2 * cf.max_batch + b] = len - 1;
    }
    HIP_TRY(c, hipMemcpyAsync(c->ws + c->o.state + kStateDeltaOff, meta.data(), meta.size() * 4, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpy2DAsync(dtok, (size_t)cf.max_seq_len * 4, tk.data(), (size_t)prompt_len * 4, (size_t)prompt_len * 4, batch,
                                hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, enqueue_prefill(c, prompt_len, n_late, ragged));
    std::vector<int32_t> first(batch);
    HIP_TRY(c, hipMemcpyAsync(first.data(), c->ws + c->o.emitted, (size_t)batch * 4, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    if (first_tokens) std::memcpy(first_tokens, first.data(), (size_t)batch * 4);
  } else if (first_tokens) {
    for (int b = 0; b < batch; ++b) first_tokens[b] = -1;
  }
  c->sched.note_prefill(prompt_len, cf.full_pos_add_embed ? n_late : 0);
  return DMTD_OK;
}

int dmtd_prefill(dmtd_ctx* c, const int32_t* tokens, int32_t batch, int32_t prompt_len, int32_t n_late, int32_t* first_tokens) {
  return prefill_impl(c, tokens, batch, prompt_len, nullptr, n_late, first_tokens);
}

int dmtd_prefill_ragged(dmtd_ctx* c, const int32_t* tokens, int32_t batch, int32_t prompt_len, const int32_t* lengths, int32_t n_late,
                        int32_t* first_tokens) {
  if (c && !lengths) { c->err = "null lengths"; return DMTD_EINVAL; }
  return prefill_impl(c, tokens, batch, prompt_len, lengths, n_late, first_tokens);
}

// Decode steps of one call: plan (host only), enqueue everything on the stream, one copy of the emitted tokens and one
// synchronisation at the end.  cycles: false = stop when the current cycle is complete (dmtd_decode_cycle); true = go on
// with further cycles until n_steps steps have run (dmtd_decode).
static int decode_steps(dmtd_ctx* c, int32_t tau, int32_t n_late, int32_t n_steps, bool cycles, const int32_t* forced_inputs,
                        int32_t n_forced, int32_t* out_tokens, int32_t out_stride, int32_t* n_emitted) {
  if (!c) return DMTD_EINVAL;
  const dmtd_config& cf = c->cfg;
  if (n_emitted) *n_emitted = 0;
  if (!out_tokens || !n_emitted) { c->err = "null output pointer"; return DMTD_EINVAL; }
  if (tau > kMaxTau) { c->err = "tau above the supported maximum (64)"; return DMTD_EINVAL; }
  if (forced_inputs && n_forced < 1) { c->err = "forced_inputs given with n_forced < 1"; return DMTD_EINVAL; }
  if (cycles && (n_steps < 1 || n_steps > kMaxTau)) { c->err = "n_steps must be in [1, 64]"; return DMTD_EINVAL; }
  if (c->diverged) { c->err = "the sequences are at different points of their cycles: use dmtd_decode_per_seq"; return DMTD_ESTATE; }
  const int f_stride = forced_inputs ? n_forced : 0;
  std::vector<Step> steps;
  int err = 0;
  std::string why;
  if (!cycles) {
    if (!c->sched.plan(tau, n_late, n_steps, kMaxTau, steps, err, why)) {
      c->err = why;
      return err == 1 ? DMTD_EINVAL : (err == 2 ? DMTD_ESTATE : DMTD_ECAPACITY);
    }
  } else {
    // cycle after cycle on a copy of the host state (the plan of a cycle depends on where the one before it ended);
    // nothing runs unless every cycle can be planned
    Sched ahead = c->sched;
    ahead.trace.clear();
    std::vector<Step> one;
    while ((int)steps.size() < n_steps) {
      if (!ahead.plan(tau, n_late, n_steps - (int)steps.size(), kMaxTau, one, err, why)) {
        c->err = why;
        return err == 1 ? DMTD_EINVAL : (err == 2 ? DMTD_ESTATE : DMTD_ECAPACITY);
      }
      ahead.commit(one, n_late);
      ahead.trace.clear();
      steps.insert(steps.end(), one.begin(), one.end());
    }
  }
  const int n = (int)steps.size();
  if (out_stride < n) { c->err = "out_stride smaller than the number of steps"; return DMTD_ECAPACITY; }
  const int B = c->batch;
  const int nf = f_stride < n ? f_stride : n;   // forced inputs beyond the steps run are ignored
  for (int b = 0; b < B && forced_inputs; ++b)
    for (int i = 0; i < nf; ++i) {
      const int32_t t = forced_inputs[(size_t)b * f_stride + i];
      if (t < 0 || t >= cf.vocab) { c->err = "forced token id outside the vocabulary"; return DMTD_EINVAL; }
    }
  if (!cf.dry_run) {
    int* fdev = (int*)(c->ws + c->o.forced);
    std::vector<int32_t> fhost((size_t)B * (nf > 0 ? nf : 1));
    if (nf > 0) {
      for (int b = 0; b < B; ++b)
        for (int i = 0; i < nf; ++i) fhost[(size_t)b * nf + i] = forced_inputs[(size_t)b * f_stride + i];
      HIP_TRY(c, hipMemcpyAsync(fdev, fhost.data(), (size_t)B * nf * 4, hipMemcpyHostToDevice, c->stream));
    }
    hipLaunchKernelGGL(begin_call_kernel, dim3(1), dim3(256), 0, c->stream, (DevState*)(c->ws + c->o.state),
                       (int*)(c->ws + c->o.tokens), cf.max_seq_len, fdev, nf, nf, cf.vocab, B, sample_count(c));
    HIP_TRY(c, hipGetLastError());
    int rc = DMTD_OK;
    if (c->test_fail_step >= 0) {
      // failure injected from the host (DMTD_TEST_FAIL_STEP at create): the steps before it run, then the call fails the
      // way a refused launch would; every kernel that was enqueued completes normally
      for (int i = 0; i < n && i < c->test_fail_step && rc == DMTD_OK; ++i) rc = run_step(c, steps[i], n_late);
      if (rc == DMTD_OK) { c->err = "injected launch failure (DMTD_TEST_FAIL_STEP)"; rc = DMTD_EHIP; }
      c->test_fail_step = -1;
    } else if (cycles) rc = run_steps_grouped(c, steps, tau, n_late);
    else
      for (const Step& s : steps)
        if ((rc = run_step(c, s, n_late)) != DMTD_OK) break;
    {
      if (rc != DMTD_OK) {
        // device state may be ahead of the host's; resynchronise it to the host's unchanged view
        (void)hipStreamSynchronize(c->stream);
        hipLaunchKernelGGL(set_state_kernel, dim3(1), dim3(64), 0, c->stream, (DevState*)(c->ws + c->o.state),
                           c->sched.n_tok, c->sched.n_front, cf.max_batch, sample_count(c));
        (void)hipStreamSynchronize(c->stream);
        return rc;
      }
    }
    std::vector<int32_t> em((size_t)n * B);
    HIP_TRY(c, hipMemcpyAsync(em.data(), c->ws + c->o.emitted, em.size() * 4, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    for (int b = 0; b < B; ++b)
      for (int i = 0; i < n; ++i) out_tokens[(size_t)b * out_stride + i] = em[(size_t)i * B + b];
  } else {
    for (int b = 0; b < B; ++b)
      for (int i = 0; i < n; ++i) out_tokens[(size_t)b * out_stride + i] = -1;
  }
  c->sched.commit(steps, n_late);
  *n_emitted = n;
  return DMTD_OK;
}

int dmtd_decode_cycle(dmtd_ctx* c, int32_t tau, int32_t n_late, int32_t max_new, const int32_t* forced_inputs,
                      int32_t n_forced, int32_t* out_tokens, int32_t out_stride, int32_t* n_emitted) {
  return decode_steps(c, tau, n_late, max_new, false, forced_inputs, n_forced, out_tokens, out_stride, n_emitted);
}

int dmtd_decode(dmtd_ctx* c, int32_t tau, int32_t n_late, int32_t n_steps, const int32_t* forced_inputs,
                int32_t n_forced, int32_t* out_tokens, int32_t out_stride, int32_t* n_emitted) {
  return decode_steps(c, tau, n_late, n_steps, true, forced_inputs, n_forced, out_tokens, out_stride, n_emitted);
}

int dmtd_decode_cycle_noalloc(dmtd_ctx* c, int32_t tau, int32_t n_late, int32_t max_new, const int32_t* forced_dev,
                              int32_t n_forced, int32_t* out_tokens_dev, int32_t out_stride, int32_t* n_emitted) {
  if (!c) return DMTD_EINVAL;
  const dmtd_config& cf = c->cfg;
  if (n_emitted) *n_emitted = 0;
  if (!n_emitted || (!out_tokens_dev && !cf.dry_run)) { c->err = "null output pointer"; return DMTD_EINVAL; }
  if (tau > kMaxTau) { c->err = "tau above the supported maximum (64)"; return DMTD_EINVAL; }
  if (forced_dev && n_forced < 1) { c->err = "forced inputs given with n_forced < 1"; return DMTD_EINVAL; }
  if (c->diverged) { c->err = "the sequences are at different points of their cycles: use dmtd_decode_per_seq"; return DMTD_ESTATE; }
  std::vector<Step>& steps = c->plan_buf;       // capacity reserved at create: planning allocates nothing
  int err = 0;
  std::string why;
  if (!c->sched.plan(tau, n_late, max_new, kMaxTau, steps, err, why)) {
    c->err = why;
    return err == 1 ? DMTD_EINVAL : (err == 2 ? DMTD_ESTATE : DMTD_ECAPACITY);
  }
  const int n = (int)steps.size();
  if (out_stride < n) { c->err = "out_stride smaller than the number of steps"; return DMTD_ECAPACITY; }
  if (!cf.dry_run) {
    const int B = c->batch, gq = cf.n_q_heads / cf.n_kv_heads;
    const int nf = forced_dev ? (n_forced < n ? n_forced : n) : 0;
    // what the steps' kernels need beyond the workspace's state: sized for this call, carved from the library's array
    int max_rows = 1;
    bool tiled = false;
    const int d = cf.hidden, qd = cf.n_q_heads * cf.head_dim, ff = cf.intermediate, nqkv = qd + 2 * cf.n_kv_heads * cf.head_dim;
    const int tiles_d = (d + 15) / 16;
    for (const Step& s : steps) {
      if (s.rows > max_rows) max_rows = s.rows;
      const int rows = B * (s.rows < kMaxRows ? s.rows : kMaxRows);
      if (c->packed)
        for (int rr : {rows, B})
          tiled = tiled || !mfma_rows_fit(c, rr, nqkv, d, tiles_d) || !mfma_rows_fit(c, rr, d, qd, 0) || !mfma_rows_fit(c, rr, ff, d, tiles_d) ||
                  !mfma_rows_fit(c, rr, d, ff, 0) || !mfma_rows_fit(c, rr, cf.vocab, d, tiles_d);
    }
    if (max_rows > kMaxRows) max_rows = kMaxRows;
    const size_t qv_stride = (size_t)max_rows * gq;
    const size_t amax_b = align_up((size_t)AMAX_CELLS * cf.max_batch * 8, 256);
    const size_t pml_b = align_up((size_t)B * cf.n_kv_heads * ATT_MAX_SPLITS * qv_stride * 2 * 4, 256);
    const size_t po_b = align_up((size_t)B * cf.n_kv_heads * ATT_MAX_SPLITS * qv_stride * cf.head_dim * 4, 256);
    size_t gp_b = 0;
    if (tiled) {
      size_t widest = 2 * (size_t)ff > (size_t)nqkv ? 2 * (size_t)ff : (size_t)nqkv;
      if ((size_t)d > widest) widest = d;
      const size_t rows_max = (size_t)B * max_rows < (size_t)kGemmRows ? (size_t)B * max_rows : (size_t)kGemmRows;
      gp_b = align_up((size_t)kGemmMaxSplit * rows_max * widest * 4, 256);
    }
    if (amax_b + pml_b + po_b + gp_b > kStaticScratchBytes) {
      c->err = "dmtd_decode_cycle_noalloc: this call's partial results (" + std::to_string((amax_b + pml_b + po_b + gp_b) >> 10) +
               " KiB for batch " + std::to_string(B) + " with " + std::to_string(max_rows) + " rows per sequence) exceed the library's " +
               std::to_string(kStaticScratchBytes >> 20) + " MiB scratch; use dmtd_decode_cycle";
      return DMTD_ECAPACITY;
    }
    // the steps run eagerly on the context's stream with their scratch in the library's array
    struct Saved { float *po, *pml, *gp; unsigned long long* amax; int rows; } saved{c->part_o, c->part_ml, c->gemm_part, c->amax, c->part_rows};
    char* base = c->static_scratch;
    c->amax = (unsigned long long*)base;
    c->part_ml = (float*)(base + amax_b);
    c->part_o = (float*)(base + amax_b + pml_b);
    c->gemm_part = (float*)(base + amax_b + pml_b + po_b);
    c->part_rows = max_rows;
    // the array keeps the last call's contents: the selection-key cells must start at zero (a fill kernel, so that a
    // caller may capture this call into a graph)
    hipLaunchKernelGGL(zero_u64_kernel, dim3(4), dim3(256), 0, c->stream, c->amax, AMAX_CELLS * cf.max_batch);
    hipLaunchKernelGGL(begin_call_kernel, dim3(1), dim3(256), 0, c->stream, (DevState*)(c->ws + c->o.state),
                       (int*)(c->ws + c->o.tokens), cf.max_seq_len, forced_dev, nf, n_forced, cf.vocab, B, sample_count(c));
    hipError_t e = hipGetLastError();
    for (int i = 0; i < n && e == hipSuccess; ++i) {
      choose_attention(c, steps[i].pos + 1);
      e = enqueue_step(c, steps[i].full, steps[i].rows, n_late);
    }
    if (e == hipSuccess) {
      hipLaunchKernelGGL(emitted_to_rows_kernel, dim3(1), dim3(256), 0, c->stream, (const int*)(c->ws + c->o.emitted), out_tokens_dev, n, B, out_stride);
      e = hipGetLastError();
    }
    c->part_o = saved.po; c->part_ml = saved.pml; c->gemm_part = saved.gp; c->amax = saved.amax; c->part_rows = saved.rows;
    if (e != hipSuccess) {
      c->err = std::string("dmtd_decode_cycle_noalloc: ") + hipGetErrorString(e);
      return DMTD_EHIP;
    }
  }
  c->sched.commit(steps, n_late);
  *n_emitted = n;
  return DMTD_OK;
}

int dmtd_decode_per_seq(dmtd_ctx* c, const int32_t* tau, int32_t n_late, int32_t n_steps, const int32_t* forced_inputs,
                        int32_t n_forced, int32_t* out_tokens, int32_t out_stride, int32_t* n_emitted) {
  if (!c) return DMTD_EINVAL;
  const dmtd_config& cf = c->cfg;
  if (n_emitted) *n_emitted = 0;
  if (!out_tokens || !n_emitted || !tau) { c->err = "null pointer"; return DMTD_EINVAL; }
  if (c->sched.n_tok == 0) { c->err = "decode before prefill"; return DMTD_ESTATE; }
  if (n_steps < 1 || n_steps > kMaxTau) { c->err = "n_steps must be in [1, 64]"; return DMTD_EINVAL; }
  if (n_late < 1 || n_late > cf.n_layers) { c->err = "n_late must be in [1, n_layers]"; return DMTD_EINVAL; }
  if (c->sched.n_early != 0) { c->err = "per-sequence cycle lengths are not available in the ExDy variant"; return DMTD_ESTATE; }
  if (forced_inputs && n_forced < 1) { c->err = "forced_inputs given with n_forced < 1"; return DMTD_EINVAL; }
  if (out_stride < n_steps) { c->err = "out_stride smaller than the number of steps"; return DMTD_ECAPACITY; }
  const int B = c->batch, n = n_steps;
  for (int b = 0; b < B; ++b)
    if (tau[b] < 1 || tau[b] > kMaxTau) { c->err = "every sequence's tau must be in [1, 64]"; return DMTD_EINVAL; }
  if (c->sched.n_tok + n > cf.max_seq_len) { c->err = "sequence would exceed max_seq_len"; return DMTD_ECAPACITY; }
  // plan on copies of the per-sequence state: rows[i][b] = 0 for a late-only step of sequence b, else its row count
  std::vector<int> phase = c->diverged ? c->seq_phase : std::vector<int>(B, c->sched.phase);
  std::vector<int> front = c->diverged ? c->seq_front : std::vector<int>(B, c->sched.n_front);
  if (c->sched.n_late_in_use != 0 && c->sched.n_late_in_use != n_late)
    for (int b = 0; b < B; ++b)
      if (front[b] != c->sched.n_tok) { c->err = "n_late changed while tokens await refill"; return DMTD_ESTATE; }
  std::vector<std::vector<int>> rows(n, std::vector<int>(B, 0));
  int t = c->sched.n_tok;
  for (int i = 0; i < n; ++i, ++t)
    for (int b = 0; b < B; ++b) {
      if (phase[b] >= tau[b]) {
        rows[i][b] = t - front[b] + 1;
        if (rows[i][b] > kMaxRows) { c->err = "more pending refill rows than the workspace holds"; return DMTD_ECAPACITY; }
        front[b] = t + 1; phase[b] = 1;
      } else {
        phase[b] += 1;
      }
    }
  const int f_stride = forced_inputs ? n_forced : 0;
  const int nf = f_stride < n ? f_stride : n;
  for (int b = 0; b < B && forced_inputs; ++b)
    for (int i = 0; i < nf; ++i) {
      const int32_t tk = forced_inputs[(size_t)b * f_stride + i];
      if (tk < 0 || tk >= cf.vocab) { c->err = "forced token id outside the vocabulary"; return DMTD_EINVAL; }
    }
  if (!cf.dry_run) {
    int* fdev = (int*)(c->ws + c->o.forced);
    std::vector<int32_t> fhost((size_t)B * (nf > 0 ? nf : 1));
    if (nf > 0) {
      for (int b = 0; b < B; ++b)
        for (int i = 0; i < nf; ++i) fhost[(size_t)b * nf + i] = forced_inputs[(size_t)b * f_stride + i];
      HIP_TRY(c, hipMemcpyAsync(fdev, fhost.data(), (size_t)B * nf * 4, hipMemcpyHostToDevice, c->stream));
    }
    hipLaunchKernelGGL(begin_call_kernel, dim3(1), dim3(256), 0, c->stream, (DevState*)(c->ws + c->o.state),
                       (int*)(c->ws + c->o.tokens), cf.max_seq_len, fdev, nf, nf, cf.vocab, B, sample_count(c));
    HIP_TRY(c, hipGetLastError());
    std::vector<std::vector<char>> uploads;           // host images of new patterns: alive until the call's synchronisation
    int rc = DMTD_OK;
    for (int i = 0; i < n && rc == DMTD_OK; ++i) {
      const int pos = c->sched.n_tok + i;
      bool same = true;
      for (int b = 1; b < B; ++b) same = same && rows[i][b] == rows[i][0];
      if (same) {       // all sequences at the same point of their cycles: the ordinary step (and its graph)
        rc = run_step(c, Step{rows[i][0] > 0, rows[i][0] > 0 ? rows[i][0] : 1, pos}, n_late);
        continue;
      }
      choose_attention(c, pos + 1);
      // the sequences that start a cycle, sorted by row count
      std::vector<int> order;
      for (int b = 0; b < B; ++b) if (rows[i][b] > 0) order.push_back(b);
      std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return rows[i][x] < rows[i][y]; });
      std::vector<int> order_rows;
      for (int b : order) order_rows.push_back(rows[i][b]);
      // the pattern's device image: the list (ints) and the mask (bytes); cached patterns keep their slot for good (graphs
      // refer to it), the last slot serves patterns beyond the table, without a graph
      auto it = c->pattern_ids.find(rows[i]);
      int slot;
      const bool cached = it != c->pattern_ids.end() || (int)c->pattern_ids.size() < kMaxPatterns - 1;
      if (it != c->pattern_ids.end()) slot = it->second;
      else {
        slot = cached ? (int)c->pattern_ids.size() : kMaxPatterns - 1;
        uploads.emplace_back(kPatternStride(cf.max_batch), 0);
        std::vector<char>& img = uploads.back();
        for (size_t k = 0; k < order.size(); ++k) std::memcpy(img.data() + 4 * k, &order[k], 4);
        for (int b = 0; b < B; ++b) img[(size_t)4 * cf.max_batch + b] = rows[i][b] > 0 ? 1 : 0;
        hipError_t ce = hipMemcpyAsync(c->ws + c->o.patterns + (size_t)slot * kPatternStride(cf.max_batch), img.data(), img.size(),
                                       hipMemcpyHostToDevice, c->stream);
        if (ce != hipSuccess) { c->err = std::string("pattern upload: ") + hipGetErrorString(ce); rc = DMTD_EHIP; break; }
        if (cached) c->pattern_ids.emplace(rows[i], slot);
      }
      const char* img_dev = c->ws + c->o.patterns + (size_t)slot * kPatternStride(cf.max_batch);
      const int* list_dev = (const int*)img_dev;
      const unsigned char* mask_dev = (const unsigned char*)img_dev + (size_t)4 * cf.max_batch;
      if (!cf.use_graphs || !cached) {
        hipError_t e = enqueue_step_mixed(c, front_groups(cf, order_rows), order_rows, n_late, list_dev, mask_dev);
        if (e != hipSuccess) { c->err = std::string("mixed step: ") + hipGetErrorString(e); rc = DMTD_EHIP; }
        continue;
      }
      const std::vector<int> key = {slot, n_late, c->sampling ? 1 : 0, c->att_bucket, c->share_kv ? 1 : 0, B};
      auto git = c->mixed_graphs.find(key);
      if (git == c->mixed_graphs.end()) {
        hipGraph_t graph = nullptr;
        hipError_t e0 = hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal);
        if (e0 != hipSuccess) { c->err = std::string("hipStreamBeginCapture: ") + hipGetErrorString(e0); rc = DMTD_EHIP; break; }
        hipError_t e = enqueue_step_mixed(c, front_groups(cf, order_rows), order_rows, n_late, list_dev, mask_dev);
        hipError_t e2 = hipStreamEndCapture(c->stream, &graph);
        if (e != hipSuccess || e2 != hipSuccess) {
          if (graph) (void)hipGraphDestroy(graph);
          c->err = std::string("graph capture failed: ") + hipGetErrorString(e != hipSuccess ? e : e2);
          rc = DMTD_EHIP; break;
        }
        hipGraphExec_t exec = nullptr;
        hipError_t e3 = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e3 != hipSuccess) { c->err = std::string("hipGraphInstantiate: ") + hipGetErrorString(e3); rc = DMTD_EHIP; break; }
        git = c->mixed_graphs.emplace(key, exec).first;
      }
      hipError_t le = hipGraphLaunch(git->second, c->stream);
      if (le != hipSuccess) { c->err = std::string("hipGraphLaunch: ") + hipGetErrorString(le); rc = DMTD_EHIP; }
    }
    if (rc != DMTD_OK) {
      // back to the host's unchanged view: counters, and every sequence's front position
      (void)hipStreamSynchronize(c->stream);
      hipLaunchKernelGGL(set_state_kernel, dim3(1), dim3(64), 0, c->stream, (DevState*)(c->ws + c->o.state), c->sched.n_tok, c->sched.n_front, cf.max_batch, sample_count(c));
      if (c->diverged) {
        int* tmp = (int*)(c->ws + c->o.forced);
        (void)hipMemcpyAsync(tmp, c->seq_front.data(), (size_t)B * 4, hipMemcpyHostToDevice, c->stream);
        hipLaunchKernelGGL(set_fronts_kernel, dim3(1), dim3(64), 0, c->stream, (DevState*)(c->ws + c->o.state), (const int*)tmp, B);
      }
      (void)hipStreamSynchronize(c->stream);
      return rc;
    }
    std::vector<int32_t> em((size_t)n * B);
    HIP_TRY(c, hipMemcpyAsync(em.data(), c->ws + c->o.emitted, em.size() * 4, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    for (int b = 0; b < B; ++b)
      for (int i = 0; i < n; ++i) out_tokens[(size_t)b * out_stride + i] = em[(size_t)i * B + b];
  } else {
    for (int b = 0; b < B; ++b)
      for (int i = 0; i < n; ++i) out_tokens[(size_t)b * out_stride + i] = -1;
  }
  // commit: the counters and the trace follow sequence 0; the per-sequence state is kept while the sequences differ
  const int F = cf.n_layers - n_late;
  for (int i = 0; i < n; ++i) {
    Sched& sc = c->sched;
    sc.pass_no += 1;
    if (rows[i][0] > 0) {
      if (F > 0) sc.record(0, sc.n_tok - (rows[i][0] - 1), rows[i][0]);
      sc.record(1, sc.n_tok, 1);
      sc.gen_layer_visits += cf.n_layers;
      sc.refill_layer_visits += (int64_t)(rows[i][0] - 1) * F;
      sc.n_full_steps += 1;
    } else {
      sc.record(1, sc.n_tok, 1);
      sc.gen_layer_visits += n_late;
    }
    sc.n_tok += 1;
    sc.n_emitted += 1;
  }
  c->sched.n_late_in_use = n_late;
  c->sched.n_front = front[0];
  c->sched.phase = phase[0];
  c->seq_phase = phase;
  c->seq_front = front;
  c->diverged = false;
  for (int b = 1; b < B; ++b) c->diverged = c->diverged || phase[b] != phase[0] || front[b] != front[0];
  *n_emitted = n;
  return DMTD_OK;
}

int dmtd_get_seq_state(const dmtd_ctx* c, int32_t b, int32_t* n_front, int32_t* phase) {
  if (!c) return DMTD_EINVAL;
  if (b < 0 || b >= c->batch) return DMTD_EINVAL;
  if (n_front) *n_front = c->diverged ? c->seq_front[b] : c->sched.n_front;
  if (phase) *phase = c->diverged ? c->seq_phase[b] : c->sched.phase;
  return DMTD_OK;
}

int dmtd_logits(dmtd_ctx* c, float* out, size_t out_elems) {
  if (!c) return DMTD_EINVAL;
  if (!out) { c->err = "null output pointer"; return DMTD_EINVAL; }
  if (c->sched.n_tok == 0 || c->cfg.dry_run) { c->err = "no logits before prefill"; return DMTD_ESTATE; }
  const size_t need = (size_t)c->batch * c->cfg.vocab;
  if (out_elems < need) { c->err = "logits buffer too small"; return DMTD_ECAPACITY; }
  HIP_TRY(c, hipMemcpyAsync(out, c->ws + c->o.logits, need * 4, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return DMTD_OK;
}

int dmtd_get_state(const dmtd_ctx* c, int32_t* n_tok, int32_t* n_front, int32_t* phase, int64_t* counters) {
  if (!c) return DMTD_EINVAL;
  if (n_tok) *n_tok = c->sched.n_tok;
  if (n_front) *n_front = c->sched.n_front;
  if (phase) *phase = c->sched.phase;
  if (counters) {
    counters[0] = c->sched.gen_layer_visits;
    counters[1] = c->sched.refill_layer_visits;
    counters[2] = c->sched.n_emitted;
    counters[3] = c->sched.n_full_steps;
  }
  return DMTD_OK;
}

int dmtd_get_trace(const dmtd_ctx* c, int32_t* buf, int32_t cap_records, int32_t* n_records) {
  if (!c || !n_records) return DMTD_EINVAL;
  const int total = (int)(c->sched.trace.size() / 4);
  *n_records = total;
  if (buf && cap_records > 0) {
    const int n = total < cap_records ? total : cap_records;
    std::memcpy(buf, c->sched.trace.data(), (size_t)n * 16);
  }
  return DMTD_OK;
}

int dmtd_read_kv(dmtd_ctx* c, int32_t layer, int32_t b, int32_t n_pos, float* out, size_t out_elems) {
  if (!c) return DMTD_EINVAL;
  const dmtd_config& cf = c->cfg;
  if (!out || layer < 0 || layer >= cf.n_layers || b < 0 || b >= cf.max_batch || n_pos < 1 || n_pos > cf.max_seq_len) {
    c->err = "bad argument to dmtd_read_kv"; return DMTD_EINVAL;
  }
  if (cf.dry_run) { c->err = "no device state in a dry run"; return DMTD_ESTATE; }
  const size_t half = (size_t)cf.n_kv_heads * n_pos * cf.head_dim;
  if (out_elems < 2 * half) { c->err = "KV buffer too small"; return DMTD_ECAPACITY; }
  // each (b, g) owns a contiguous run of positions in the cache: copy the raw rows and widen on the host
  const size_t elem = c->elem, run = (size_t)n_pos * cf.head_dim;
  std::vector<char> raw(2 * half * elem);
  const char* kc = c->ws + c->o.kv + (size_t)layer * c->o.kv_layer_stride;
  const char* vc = kc + c->o.kv_v_off;
  for (int which = 0; which < 2; ++which)
    for (int g = 0; g < cf.n_kv_heads; ++g) {
      const char* src = (which ? vc : kc) + (((size_t)b * cf.n_kv_heads + g) * cf.max_seq_len) * cf.head_dim * elem;
      HIP_TRY(c, hipMemcpyAsync(raw.data() + ((size_t)which * cf.n_kv_heads + g) * run * elem, src, run * elem,
                                hipMemcpyDeviceToHost, c->stream));
    }
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  if (elem == 4) {
    std::memcpy(out, raw.data(), 2 * half * 4);
  } else {
    const uint16_t* r16 = (const uint16_t*)raw.data();
    for (size_t i = 0; i < 2 * half; ++i) {
      const uint32_t u = (uint32_t)r16[i] << 16;
      std::memcpy(out + i, &u, 4);
    }
  }
  return DMTD_OK;
}

int dmtd_time_kernel(dmtd_ctx* c, int32_t kind, int32_t rows, int32_t reps, float* avg_us) {
  if (!c) return DMTD_EINVAL;
  // attention: rows per sequence (at most 16); projections: total activation rows, at most what a decode step may carry
  const int rows_max = kind == DMTD_K_ATTN ? kMaxRows : step_row_capacity(c->cfg.max_batch);
  if (!avg_us || kind < 0 || kind > DMTD_K_READ_DOWN || rows < 1 || rows > rows_max || reps < 1) {
    c->err = "bad argument to dmtd_time_kernel"; return DMTD_EINVAL;
  }
  if (kind >= DMTD_K_READ_QKV && !c->packed) { c->err = "the read-only kinds need a bf16 model (they read its stored weight image)"; return DMTD_EINVAL; }
  if (c->cfg.dry_run || c->sched.n_tok == 0) { c->err = "dmtd_time_kernel needs a prefilled context"; return DMTD_ESTATE; }
  if (kind == DMTD_K_LMHEAD && rows > c->batch) { c->err = "the LM head carries one row per sequence"; return DMTD_EINVAL; }
  hipEvent_t e0, e1;
  HIP_TRY(c, hipEventCreate(&e0));
  HIP_TRY(c, hipEventCreate(&e1));
  // rows is per sequence for attention, total activation rows for the projections
  const int saved_batch = c->batch;
  long launches = 0;
  hipError_t e = hipSuccess;
  // what a step launches before the kernel leaves something that kernel reads: the attention's partial results, and the partial sums
  // of squares of the O projection (their number depends on its route)
  if (c->packed && (kind == DMTD_K_OPROJ || kind == DMTD_K_GATEUP) && rows % c->batch == 0 && rows / c->batch <= kMaxRows)
    e = time_one(c, DMTD_K_ATTN, 0, rows / c->batch);
  if (c->packed && kind == DMTD_K_GATEUP && e == hipSuccess) e = time_one(c, DMTD_K_OPROJ, 0, rows);
  for (int pass = 0; pass < 2 && e == hipSuccess; ++pass) {   // pass 0 warms up (one repetition)
    const int n = pass == 0 ? 1 : reps;
    if (pass == 1) e = hipEventRecord(e0, c->stream);
    for (int i = 0; i < n && e == hipSuccess; ++i) {
      if (kind == DMTD_K_LMHEAD) {
        e = time_one(c, kind, 0, rows);
        if (pass == 1) launches += 1;
      } else {
        for (int l = 0; l < c->cfg.n_layers && e == hipSuccess; ++l) {
          e = time_one(c, kind, l, rows);
          if (pass == 1) launches += 1;
        }
      }
    }
    if (pass == 1 && e == hipSuccess) e = hipEventRecord(e1, c->stream);
  }
  c->batch = saved_batch;
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  float ms = 0.f;
  if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (e != hipSuccess) { c->err = std::string("dmtd_time_kernel: ") + hipGetErrorString(e); return DMTD_EHIP; }
  *avg_us = ms * 1000.0f / (float)launches;
  return DMTD_OK;
}

namespace {
// What a launch of the wide GEMM would be, for the queries below; false: not one it takes
bool wide_choice(const dmtd_config* cfg, int32_t kind, int32_t rows, int32_t num_cus, WideChoice& w) {
  std::string why;
  if (!valid_config(cfg, why) || cfg->dtype != DMTD_DTYPE_BF16 || rows <= kTiledRows || num_cus < 1) return false;
  const int d = cfg->hidden, qd = cfg->n_q_heads * cfg->head_dim, nqkv = qd + 2 * cfg->n_kv_heads * cfg->head_dim, ff = cfg->intermediate;
  switch (kind) {
    case DMTD_K_QKV:    w = choose_wide<EPI_STORE>(*cfg, num_cus, rows, nqkv, d); break;
    case DMTD_K_OPROJ:  w = choose_wide<EPI_RESID>(*cfg, num_cus, rows, d, qd); break;
    case DMTD_K_GATEUP: w = choose_wide<EPI_SWIGLU>(*cfg, num_cus, rows, ff, d); break;
    case DMTD_K_DOWN:   w = choose_wide<EPI_RESID>(*cfg, num_cus, rows, d, ff); break;
    case DMTD_K_LMHEAD: w = choose_wide<EPI_LOGITS>(*cfg, num_cus, rows, cfg->vocab, d); break;
    default: return false;
  }
  return true;
}
}  // namespace

int dmtd_wide_plan(const dmtd_config* cfg, int32_t kind, int32_t rows, int32_t num_cus, int32_t plan[5]) {
  WideChoice w{};
  if (!plan || !wide_choice(cfg, kind, rows, num_cus, w)) return DMTD_EINVAL;
  plan[0] = w.pass;
  plan[1] = w.bm;
  plan[2] = w.p.n_full;
  plan[3] = (w.pass + w.bm - 1) / w.bm * w.nt - w.p.n_full;
  plan[4] = w.p.ksplit;
  return DMTD_OK;
}

int dmtd_wide_tile_width(const dmtd_config* cfg, int32_t kind, int32_t rows, int32_t num_cus) {
  WideChoice w{};
  return wide_choice(cfg, kind, rows, num_cus, w) ? w.bn : DMTD_EINVAL;
}

int dmtd_front_plan(const dmtd_config* cfg, const int32_t* rows, int32_t n, int32_t* plan, int32_t* n_passes) {
  std::string why;
  if (!rows || !plan || !n_passes || !valid_config(cfg, why) || n < 1 || n > cfg->max_batch) return DMTD_EINVAL;
  std::vector<int> sorted(rows, rows + n);
  std::sort(sorted.begin(), sorted.end());
  if (sorted.front() < 1 || sorted.back() > kMaxRows) return DMTD_EINVAL;
  const std::vector<std::pair<int, int>> groups = front_groups(*cfg, sorted);
  for (size_t i = 0; i < groups.size(); ++i) { plan[2 * i] = groups[i].first; plan[2 * i + 1] = groups[i].second; }
  *n_passes = (int32_t)groups.size();
  return DMTD_OK;
}

int dmtd_score_plan(const dmtd_config* cfg, int32_t batch, int32_t n, int32_t plan[2]) {
  std::string why;
  if (!plan || !valid_config(cfg, why) || batch < 1 || batch > cfg->max_batch || n < 1 || n > cfg->max_seq_len) return DMTD_EINVAL;
  plan[0] = std::min(n, pass_positions(*cfg, kWideRows, batch));
  plan[1] = masked_nll_fits(*cfg, kWideRows, batch * plan[0]) ? 1 : 0;
  return DMTD_OK;
}

int dmtd_masked_forward(dmtd_ctx* c, const int32_t* tokens, int32_t batch, int32_t n, const uint8_t* mask, int32_t n_late,
                        float* nll, int32_t* best, float* logits, size_t logits_elems, float* loss) {
  if (!c) return DMTD_EINVAL;
  const dmtd_config& cf = c->cfg;
  if (!tokens || !mask) { c->err = "null tokens or mask"; return DMTD_EINVAL; }
  if (batch < 1 || batch > cf.max_batch) { c->err = "batch outside [1, max_batch]"; return DMTD_EINVAL; }
  if (n < 1) { c->err = "sequence length must be >= 1"; return DMTD_EINVAL; }
  if (n_late < 1 || n_late > cf.n_layers) { c->err = "n_late must be in [1, n_layers]"; return DMTD_EINVAL; }
  if (c->sched.n_early + n_late > cf.n_layers) { c->err = "n_early + n_late exceeds the number of layers"; return DMTD_EINVAL; }
  if (c->sched.n_tok != 0) { c->err = "the masked forward needs an empty context; call dmtd_reset first"; return DMTD_ESTATE; }
  if (n > cf.max_seq_len) { c->err = "sequence longer than max_seq_len"; return DMTD_ECAPACITY; }
  if (logits && logits_elems < (size_t)batch * n * cf.vocab) { c->err = "logits buffer too small"; return DMTD_ECAPACITY; }
  for (size_t i = 0; i < (size_t)batch * n; ++i)
    if (tokens[i] < 0 || tokens[i] >= cf.vocab) { c->err = "token id outside the vocabulary"; return DMTD_EINVAL; }
  if (cf.dry_run) { c->err = "no device work in a dry run"; return DMTD_ESTATE; }
  const int saved_batch = c->batch;
  c->batch = batch;
  std::vector<int32_t> m32(n);
  for (int i = 0; i < n; ++i) m32[i] = mask[i] ? 1 : 0;
  int rc = DMTD_OK;
  hipError_t e = hipMemcpy2DAsync(c->ws + c->o.tokens, (size_t)cf.max_seq_len * 4, tokens, (size_t)n * 4, (size_t)n * 4, batch,
                                  hipMemcpyHostToDevice, c->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(c->ws + c->o.mask, m32.data(), (size_t)n * 4, hipMemcpyHostToDevice, c->stream);
  const int chunk = pass_positions(cf, c->wide_rows, batch);
  PartRowsGuard guard{c, c->part_rows};
  c->part_rows = step_positions(batch);
  for (int p0 = 0; p0 < n && e == hipSuccess; p0 += chunk) {
    const int r = n - p0 < chunk ? n - p0 : chunk;
    Rows R = front_rows(c);
    e = enqueue_masked_chunk(c, R, p0, r, n_late);
    const int rows = batch * r, head = head_row_capacity(cf, c->wide_rows);
    if (!logits && masked_nll_fits(cf, c->wide_rows, rows)) {
      if (e == hipSuccess) e = enqueue_masked_nll(c, R, rows, p0, r, n);
      continue;
    }
    for (int m0 = 0; m0 < rows && e == hipSuccess; m0 += head) {
      const int m1 = std::min(rows, m0 + head);
      e = enqueue_masked_head(c, R, m0, m1 - m0, p0, r, n);
      if (!logits || e != hipSuccess) continue;
      // the block's rows of sequence b follow each other: one copy per sequence, before the next block reuses the buffer
      for (int b = m0 / r; b <= (m1 - 1) / r && e == hipSuccess; ++b) {
        const int i0 = std::max(m0, b * r), i1 = std::min(m1, (b + 1) * r);
        e = hipMemcpyAsync(logits + ((size_t)b * n + p0 + (i0 - b * r)) * cf.vocab, c->ws + c->o.logits_rows + (size_t)(i0 - m0) * cf.vocab * 4,
                           (size_t)(i1 - i0) * cf.vocab * 4, hipMemcpyDeviceToHost, c->stream);
      }
      if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    }
  }
  std::vector<float> nll_h((size_t)batch * n), loss_h(batch);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(mean_nll_kernel, dim3(batch), dim3(256), 0, c->stream, (const float*)(c->ws + c->o.nll), cf.max_seq_len, n,
                       (float*)(c->ws + c->o.loss));
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(loss_h.data(), c->ws + c->o.loss, (size_t)batch * 4, hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipMemcpy2DAsync(nll_h.data(), (size_t)n * 4, c->ws + c->o.nll, (size_t)cf.max_seq_len * 4, (size_t)n * 4, batch,
                                            hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess && best) e = hipMemcpy2DAsync(best, (size_t)n * 4, c->ws + c->o.best, (size_t)cf.max_seq_len * 4, (size_t)n * 4, batch,
                                                    hipMemcpyDeviceToHost, c->stream);
  // the caches served as scratch: back to the empty state on the device as on the host
  if (e == hipSuccess) {
    hipLaunchKernelGGL(set_state_kernel, dim3(1), dim3(64), 0, c->stream, dev_state(c), 0, 0, cf.max_batch, sample_count(c));
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  c->batch = saved_batch;
  if (e != hipSuccess) { c->err = std::string("dmtd_masked_forward: ") + hipGetErrorString(e); (void)hipStreamSynchronize(c->stream); return DMTD_EHIP; }
  if (nll) std::memcpy(nll, nll_h.data(), nll_h.size() * 4);
  if (loss) std::memcpy(loss, loss_h.data(), (size_t)batch * 4);
  return rc;
}

int dmtd_set_sampling(dmtd_ctx* c, float temperature, int32_t top_k, uint64_t seed) {
  if (!c) return DMTD_EINVAL;
  if (!(temperature == temperature) || temperature > 1e30f) { c->err = "temperature must be a finite number"; return DMTD_EINVAL; }
  if (top_k < 0) { c->err = "top_k must be >= 0"; return DMTD_EINVAL; }
  const bool on = temperature > 0.f && top_k != 1;      // top_k = 1 is the greedy choice whatever the temperature
  if (on && !c->cfg.dry_run) {
    SampleCfg sc{1.0f / temperature, top_k, (unsigned int)(seed & 0xFFFFFFFFull), (unsigned int)(seed >> 32)};
    HIP_TRY(c, hipMemcpyAsync(c->ws + c->o.state + kStateSampleOff, &sc, sizeof sc, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));        // sc is a stack object
  }
  c->sampling = on;
  return DMTD_OK;
}

int dmtd_set_n_early(dmtd_ctx* c, int32_t n_early) {
  if (!c) return DMTD_EINVAL;
  if (n_early < 0 || n_early >= c->cfg.n_layers) { c->err = "n_early must be in [0, n_layers - 1]"; return DMTD_EINVAL; }
  if (c->sched.n_tok != c->sched.n_front || c->diverged) { c->err = "n_early changed while tokens await refill"; return DMTD_ESTATE; }
  if (c->sched.n_tok != 0 && c->cfg.full_pos_add_embed && n_early != c->sched.n_early) {
    c->err = "under the literal Eq. 4 reading n_early is fixed at prefill"; return DMTD_ESTATE;
  }
  c->sched.n_early = n_early;
  return DMTD_OK;
}

int dmtd_reset(dmtd_ctx* c) {
  if (!c) return DMTD_EINVAL;
  if (!c->cfg.dry_run) {
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    hipLaunchKernelGGL(set_state_kernel, dim3(1), dim3(64), 0, c->stream, (DevState*)(c->ws + c->o.state), 0, 0, c->cfg.max_batch, sample_count(c));
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipMemsetAsync(c->ws + c->o.state + kStateDeltaOff, 0, 12 * (size_t)c->cfg.max_batch, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
  }
  c->sched.reset();
  c->batch = 0;
  c->diverged = false;
  c->seq_phase.clear();
  c->seq_front.clear();
  return DMTD_OK;
}

void dmtd_destroy(dmtd_ctx* c) {
  if (!c) return;
  if (!c->cfg.dry_run) {
    (void)hipStreamSynchronize(c->stream);
    destroy_graphs(c);
  }
  delete c;
}

const char* dmtd_last_error(const dmtd_ctx* c) { return c ? c->err.c_str() : g_create_error.c_str(); }

}  // extern "C"
