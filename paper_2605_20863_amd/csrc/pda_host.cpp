// Host side of the C interface in include/pda.h: argument validation (pure
// host code, no HIP call), the launch plan, the per-(device, stream)
// workspace and the kernel launches of a decode step, a KV append and a
// prefill.

#include "pda.h"
#include "pda_internal.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
#include <map>
#include <memory>
#include <mutex>
#include <numeric>
#include <string>
#include <tuple>
#include <utility>
#include <vector>

static_assert(pda::kScratchBytes == PDA_NOALLOC_SCRATCH_BYTES, "fixed scratch size differs from the header's");

namespace {

thread_local std::string g_error;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_error = buf;
  return code;
}

int fail_hip(hipError_t e, const char* what) {
  return fail(PDA_EHIP, "%s: %s", what, hipGetErrorString(e));
}

constexpr int kDefaultWavesPerCu = 8;   // upper bound used by pda_query_plan
constexpr int kDefaultMinShare = 8;     // blocks: below this a wave's fixed costs dominate
// Static split by default: with chunk switches that drain a wave's load
// pipeline, handing out chunks dynamically measured slower on every step
// shape tried (the last chunk's tail outweighs the balance it buys).
constexpr int kDefaultChunksPerWave = 1;
constexpr int64_t kChunkMinBytes = 512 << 10;  // of K and V: a chunk outlasts its start-up costs
constexpr int64_t kAlign = 256;

int64_t align_up(int64_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct PtrAlign {
  const void* p;
  uintptr_t align;
  const char* name;
};

// Null pointers pass (the callers check which ones are required).
int check_alignment(std::initializer_list<PtrAlign> ptrs) {
  for (const PtrAlign& x : ptrs)
    if (reinterpret_cast<uintptr_t>(x.p) % x.align)
      return fail(PDA_EINVAL, "%s is not %d-byte aligned", x.name, (int)x.align);
  return PDA_OK;
}

struct Plan {
  int requested;  // the pda_variant the options asked for
  int Q;          // query tokens per sequence
  pda::Variant variant;
  pda::KvType kv;
  int G;
  int len_cap;
  int waves_per_cu;  // 0 = decide from occupancy at launch
  int min_share;
  int chunks_per_wave;
  int chunk_min;
};

// Validate everything that does not need a device. Returns PDA_OK or an error.
int validate(const pda_problem* pr, const pda_options* op, float softmax_scale, Plan* plan) {
  if (!pr) return fail(PDA_EINVAL, "problem is NULL");
  if (pr->num_seqs < 0) return fail(PDA_EINVAL, "num_seqs = %d < 0", pr->num_seqs);
  if (pr->num_q_heads < 1 || pr->num_kv_heads < 1)
    return fail(PDA_EINVAL, "num_q_heads = %d and num_kv_heads = %d must be >= 1", pr->num_q_heads,
                pr->num_kv_heads);
  if (pr->num_q_heads % pr->num_kv_heads)
    return fail(PDA_EINVAL, "num_q_heads = %d is not a multiple of num_kv_heads = %d", pr->num_q_heads,
                pr->num_kv_heads);
  const int G = pr->num_q_heads / pr->num_kv_heads;
  if (G > pda::kMaxGroup)
    return fail(PDA_EUNSUPPORTED, "GQA group of %d query heads per KV head (max %d)", G, pda::kMaxGroup);
  if (pr->head_dim != 64 && pr->head_dim != 128)
    return fail(PDA_EUNSUPPORTED, "head_dim = %d (supported: 64, 128)", pr->head_dim);
  if (pr->block_size != pda::kBlockSize)
    return fail(PDA_EUNSUPPORTED, "block_size = %d (supported: 16)", pr->block_size);
  if (pr->max_blocks_per_seq < 1) return fail(PDA_EINVAL, "max_blocks_per_seq = %d < 1", pr->max_blocks_per_seq);
  if (pr->num_blocks < 1) return fail(PDA_EINVAL, "num_blocks = %lld < 1", (long long)pr->num_blocks);
  const int64_t table_tokens = (int64_t)pr->max_blocks_per_seq * pda::kBlockSize;
  if (table_tokens > INT32_MAX) return fail(PDA_EINVAL, "max_blocks_per_seq * 16 overflows int32");
  if ((int64_t)pr->num_seqs * ((int64_t)pr->max_blocks_per_seq + pda::kUnitCostPlain) * pr->num_kv_heads > INT32_MAX)
    return fail(PDA_EINVAL, "num_seqs * (max_blocks_per_seq + %d) * num_kv_heads overflows int32", pda::kUnitCostPlain);
  if ((int64_t)pr->num_seqs * pr->num_q_heads > INT32_MAX) return fail(PDA_EINVAL, "num_seqs * num_q_heads too large");
  if (pr->max_seq_len < 0) return fail(PDA_EINVAL, "max_seq_len = %d < 0", pr->max_seq_len);
  if (pr->max_seq_len > table_tokens)
    return fail(PDA_EINVAL, "max_seq_len = %d exceeds max_blocks_per_seq * 16 = %lld", pr->max_seq_len,
                (long long)table_tokens);
  // every cache byte offset must fit int64 (and the tile index p * Hkv + kvh)
  const int64_t tile = (int64_t)pda::kBlockSize * pr->head_dim * 4;
  if (pr->num_blocks > INT64_MAX / pr->num_kv_heads / tile) return fail(PDA_EINVAL, "num_blocks too large");

  const int qd = pr->q_dtype, kd = pr->kv_dtype;
  if (qd != PDA_DTYPE_F32 && qd != PDA_DTYPE_BF16)
    return fail(qd == PDA_DTYPE_FP8_E4M3 ? PDA_EUNSUPPORTED : PDA_EINVAL, "q_dtype = %d (supported: F32, BF16)", qd);
  if (kd != PDA_DTYPE_F32 && kd != PDA_DTYPE_BF16 && kd != PDA_DTYPE_FP8_E4M3)
    return fail(PDA_EINVAL, "kv_dtype = %d is not a pda_dtype", kd);
  if (kd == PDA_DTYPE_F32 && qd != PDA_DTYPE_F32)
    return fail(PDA_EUNSUPPORTED, "an f32 KV cache needs f32 q");
  if (kd != PDA_DTYPE_F32 && qd != PDA_DTYPE_BF16)
    return fail(PDA_EUNSUPPORTED, "a bf16 or fp8 KV cache needs bf16 q");
  if (pr->out_dtype != qd && pr->out_dtype != PDA_DTYPE_F32)
    return fail(PDA_EINVAL, "out_dtype = %d (must be q_dtype or F32)", pr->out_dtype);
  if (!std::isfinite(softmax_scale)) return fail(PDA_EINVAL, "softmax_scale is not finite");
  if (pr->q_tokens < 0) return fail(PDA_EINVAL, "q_tokens = %d < 0", pr->q_tokens);
  const int Q = pr->q_tokens > 1 ? pr->q_tokens : 1;
  if ((int64_t)pr->num_seqs * Q * pr->num_q_heads > INT32_MAX)
    return fail(PDA_EINVAL, "num_seqs * q_tokens * num_q_heads too large");

  int variant = op ? op->variant : PDA_VARIANT_AUTO;
  if (variant != PDA_VARIANT_AUTO && variant != PDA_VARIANT_VECTOR && variant != PDA_VARIANT_MFMA)
    return fail(PDA_EINVAL, "options.variant = %d is not a pda_variant", variant);
  if (Q > 1) {  // several query tokens: MFMA columns are (token, head) pairs
    if (kd == PDA_DTYPE_F32 || variant == PDA_VARIANT_VECTOR)
      return fail(PDA_EUNSUPPORTED, "q_tokens > 1 runs on the MFMA kernel: it needs a bf16 or fp8 KV cache");
    if (Q * G > pda::kWideColumns)
      return fail(PDA_EUNSUPPORTED, "q_tokens * (num_q_heads / num_kv_heads) = %d exceeds %d", Q * G,
                  pda::kWideColumns);
    variant = PDA_VARIANT_MFMA;
  }
  if (variant == PDA_VARIANT_AUTO)
    variant = (kd != PDA_DTYPE_F32 && G >= 4) ? PDA_VARIANT_MFMA : PDA_VARIANT_VECTOR;
  if (variant == PDA_VARIANT_MFMA && kd == PDA_DTYPE_F32)
    return fail(PDA_EUNSUPPORTED, "the MFMA kernel needs a bf16 or fp8 KV cache");
  if (variant == PDA_VARIANT_VECTOR && G > pda::kMaxGroupVector)
    return fail(PDA_EUNSUPPORTED, "the vector kernel handles at most %d query heads per KV head (got %d)",
                pda::kMaxGroupVector, G);
  if (op && (op->waves_per_cu < 0 || op->waves_per_cu > 64))
    return fail(PDA_EINVAL, "options.waves_per_cu = %d (0..64)", op->waves_per_cu);
  if (op && op->min_blocks_per_wave < 0)
    return fail(PDA_EINVAL, "options.min_blocks_per_wave = %d < 0", op->min_blocks_per_wave);
  if (op && (op->chunks_per_wave < 0 || op->chunks_per_wave > 64))
    return fail(PDA_EINVAL, "options.chunks_per_wave = %d (0..64)", op->chunks_per_wave);
  if (op && op->min_blocks_per_chunk < 0)
    return fail(PDA_EINVAL, "options.min_blocks_per_chunk = %d < 0", op->min_blocks_per_chunk);

  plan->requested = op ? op->variant : PDA_VARIANT_AUTO;
  plan->variant = variant == PDA_VARIANT_MFMA ? pda::Variant::Mfma : pda::Variant::Vector;
  plan->kv = kd == PDA_DTYPE_F32 ? pda::KvType::F32 : (kd == PDA_DTYPE_BF16 ? pda::KvType::BF16 : pda::KvType::FP8);
  plan->G = G;
  plan->Q = Q;
  plan->len_cap = pr->max_seq_len > 0 ? pr->max_seq_len : (int)table_tokens;
  plan->waves_per_cu = op ? op->waves_per_cu : 0;
  plan->min_share = (op && op->min_blocks_per_wave > 0) ? op->min_blocks_per_wave : kDefaultMinShare;
  plan->chunks_per_wave = (op && op->chunks_per_wave > 0) ? op->chunks_per_wave : kDefaultChunksPerWave;
  const int esz = kd == PDA_DTYPE_F32 ? 4 : (kd == PDA_DTYPE_BF16 ? 2 : 1);
  const int64_t block_head_bytes = 2LL * pda::kBlockSize * pr->head_dim * esz;
  plan->chunk_min = (op && op->min_blocks_per_chunk > 0) ? op->min_blocks_per_chunk
                                                         : (int)(kChunkMinBytes / block_head_bytes);
  return PDA_OK;
}

// Shared-prefix mode: groups of group_size consecutive sequences; each
// group's shared blocks become nsub work entries of M members (M * G <= 32
// query columns), ahead of one entry per sequence for the rest of it.
struct Groups {
  bool on = false;
  int group_size = 1, M = 1, nsub = 0, num_groups = 0;
  int64_t n_prefix = 0;
  const int32_t* shared_blocks = nullptr;
};

int validate_groups(const pda_problem* pr, int32_t group_size, const int32_t* shared_blocks, Plan* plan,
                    Groups* gr) {
  if (group_size < 1) return fail(PDA_EINVAL, "group_size = %d < 1", group_size);
  if (pr->num_seqs % group_size)
    return fail(PDA_EINVAL, "num_seqs = %d is not a multiple of group_size = %d", pr->num_seqs, group_size);
  if (plan->kv == pda::KvType::F32)
    return fail(PDA_EUNSUPPORTED, "shared-prefix decode runs on the MFMA kernel: it needs a bf16 or fp8 KV cache");
  if (plan->requested == PDA_VARIANT_VECTOR)
    return fail(PDA_EUNSUPPORTED, "shared-prefix decode runs on the MFMA kernel, not the vector kernel");
  if (pr->num_seqs > 0 && !shared_blocks) return fail(PDA_EINVAL, "shared_blocks is NULL");
  if (plan->Q > 1) return fail(PDA_EUNSUPPORTED, "shared-prefix decode takes one query token per sequence");
  plan->variant = pda::Variant::Mfma;
  gr->on = true;
  gr->group_size = group_size;
  const int per = pda::kWideColumns / plan->G;  // members whose heads fill two MFMA N-tiles
  gr->M = group_size < per ? group_size : (per > 0 ? per : 1);
  gr->nsub = (group_size + gr->M - 1) / gr->M;
  gr->num_groups = pr->num_seqs / group_size;
  gr->n_prefix = (int64_t)gr->num_groups * gr->nsub;
  gr->shared_blocks = shared_blocks;
  if ((gr->n_prefix + pr->num_seqs) * pr->num_kv_heads *
          ((int64_t)pr->max_blocks_per_seq + pda::kUnitCostShared) > INT32_MAX)
    return fail(PDA_EINVAL, "(entries) * num_kv_heads * (max_blocks_per_seq + %d) overflows int32",
                pda::kUnitCostShared);
  return PDA_OK;
}

struct Layout {
  int64_t hdr, sg, cum, m, l, acc, total;
};

// header | sg[num_groups] | cum[entries] | m, l [slots, Gp] | acc [slots, Gp, D]
Layout workspace_layout(const pda_problem* pr, const Plan& plan, const Groups& gr, int chunks_max) {
  Layout w;
  const int64_t entries = gr.n_prefix + pr->num_seqs;
  const int64_t gp = gr.on ? (int64_t)gr.M * plan.G : (int64_t)plan.Q * plan.G;
  const int64_t slots = pda::partial_slots(entries, pr->num_kv_heads, chunks_max);
  w.hdr = 0;
  w.sg = align_up(pda::kHdrWords * 4);
  w.cum = w.sg + align_up((int64_t)gr.num_groups * 4);
  w.m = w.cum + align_up(entries * 4);
  w.l = w.m + align_up(slots * gp * 4);
  w.acc = w.l + align_up(slots * gp * 4);
  w.total = w.acc + align_up(slots * gp * pr->head_dim * 4);
  return w;
}

// ------------------------------------------------------------- device state

struct DeviceInfo {
  bool ok = false;
  int cus = 0;
  std::string arch;
};

struct Workspace {
  std::mutex mu;
  void* ptr = nullptr;  // `bytes` usable bytes; the short decode's arrival counts lie right before
  int64_t bytes = 0;
  uint32_t epoch = 0;  // of the last short decode made outside capture
  // the capture whose graph clears the captured calls' counts already (0: none)
  unsigned long long cleared_in = 0;
  // The combine kernel zeroes the chunk counter after each decode kernel; if a
  // combine launch failed, the next call zeroes it first.
  bool rearm = false;
  // A graph captured on the stream holds `ptr`: growth then keeps the old
  // allocation (in `retired`) so that replays stay valid.
  bool captured = false;
  std::vector<void*> retired;
};

// The no-allocation entry point's per-device state: the device address of
// that device's copy of the fixed scratch array (looked up on the first call
// with the device current) and the counter re-arm flag. A fixed table, so
// that the entry point allocates nothing, not even host memory for its state.
constexpr int kMaxDevices = 64;
struct FixedScratch {
  std::mutex mu;
  void* ptr = nullptr;
  bool rearm = false;
};
FixedScratch g_fixed[kMaxDevices];

std::mutex g_mu;
std::map<int, DeviceInfo> g_devices;
std::map<std::pair<int, hipStream_t>, std::unique_ptr<Workspace>> g_workspaces;
std::map<std::tuple<int, int, int, int, int>, int> g_occupancy;

// *out stays valid: entries are never erased.
int device_info(int dev, const DeviceInfo** out) {
  std::lock_guard<std::mutex> lk(g_mu);
  auto it = g_devices.find(dev);
  if (it != g_devices.end()) {
    *out = &it->second;
    return PDA_OK;
  }
  DeviceInfo d;
  hipDeviceProp_t prop;
  hipError_t e = hipGetDeviceProperties(&prop, dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDeviceProperties");
  d.cus = prop.multiProcessorCount;
  d.arch = prop.gcnArchName;
  d.ok = d.arch.rfind("gfx950", 0) == 0;
  *out = &(g_devices[dev] = d);
  return PDA_OK;
}

int occupancy(int dev, pda::Variant v, pda::KvType kv, int D, int G, bool wide, int* wgs) {
  const int gb = v == pda::Variant::Mfma ? (wide ? pda::kWideColumns : 16) : (G <= 1 ? 1 : G <= 2 ? 2 : G <= 4 ? 4 : 8);
  auto key = std::make_tuple(dev, (int)v, (int)kv, D, gb);
  {
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_occupancy.find(key);
    if (it != g_occupancy.end()) {
      *wgs = it->second;
      return PDA_OK;
    }
  }
  int n = 0;
  hipError_t e = pda::decode_occupancy(v, kv, D, G, wide, &n);
  if (e != hipSuccess) return fail_hip(e, "hipOccupancyMaxActiveBlocksPerMultiprocessor");
  if (n < 1) n = 1;
  std::lock_guard<std::mutex> lk(g_mu);
  g_occupancy[key] = n;
  *wgs = n;
  return PDA_OK;
}

Workspace* workspace_for(int dev, hipStream_t s) {
  std::lock_guard<std::mutex> lk(g_mu);
  auto& slot = g_workspaces[std::make_pair(dev, s)];
  if (!slot) slot.reset(new Workspace);
  return slot.get();
}

// True while `s` records into a HIP graph: allocation, frees, waits and
// memsets must then stay out of the call.
bool capturing(hipStream_t s) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(s, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone;
}

// Identifies the capture that `s` records into (0 if it cannot be told).
unsigned long long capture_id(hipStream_t s) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  unsigned long long id = 0;
  return hipStreamGetCaptureInfo(s, &cs, &id) == hipSuccess ? id : 0;
}

hipError_t free_workspace(void* ptr) { return hipFree(static_cast<char*>(ptr) - pda::kShortCountBytes); }

// Grow ws (caller holds ws->mu) to at least `bytes`; growth waits for `s`.
int ensure_workspace(Workspace* ws, int64_t bytes, hipStream_t s) {
  const bool cap = capturing(s);
  if (cap) ws->captured = true;
  if (ws->bytes >= bytes) return PDA_OK;
  if (cap)
    return fail(PDA_EINVAL,
                "the stream's workspace must grow to %lld bytes, which cannot be recorded into a graph: make one "
                "call of this size (or larger) on the stream before capturing it",
                (long long)bytes);
  hipError_t e;
  if (ws->ptr) {
    if (ws->captured) {
      ws->retired.push_back(ws->ptr);
    } else {
      if ((e = hipStreamSynchronize(s)) != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
      if ((e = free_workspace(ws->ptr)) != hipSuccess) return fail_hip(e, "hipFree");
    }
    ws->ptr = nullptr;
    ws->bytes = 0;
  }
  const int64_t want = bytes + bytes / 4;  // headroom so small growth does not reallocate
  void* p = nullptr;
  if ((e = hipMalloc(&p, (size_t)(pda::kShortCountBytes + want))) != hipSuccess) {
    return fail(PDA_ENOMEM, "hipMalloc(%lld) of the workspace: %s", (long long)want, hipGetErrorString(e));
  }
  ws->ptr = static_cast<char*>(p) + pda::kShortCountBytes;
  ws->bytes = want;
  ws->rearm = false;
  ws->cleared_in = 0;
  if ((e = hipMemsetAsync(p, 0, pda::kShortCountBytes + pda::kHdrWords * 4, s)) != hipSuccess)
    return fail_hip(e, "hipMemsetAsync");
  return PDA_OK;
}

}  // namespace

extern "C" {

int pda_version(void) { return PDA_VERSION; }

const char* pda_last_error(void) { return g_error.c_str(); }

}  // extern "C"

namespace {

int query_plan(const pda_problem* problem, const pda_options* options, float softmax_scale,
               int32_t num_compute_units, const int32_t* group_size, pda_plan_info* info) {
  g_error.clear();
  if (!info) return fail(PDA_EINVAL, "info is NULL");
  if (num_compute_units < 1) return fail(PDA_EINVAL, "num_compute_units = %d < 1", num_compute_units);
  Plan plan;
  int rc = validate(problem, options, softmax_scale, &plan);
  if (rc != PDA_OK) return rc;
  Groups gr;
  static const int32_t kAny = 0;  // shared_blocks is not read by a plan query
  if (group_size && (rc = validate_groups(problem, *group_size, &kAny, &plan, &gr)) != PDA_OK) return rc;
  const int wpc = plan.waves_per_cu > 0 ? plan.waves_per_cu : kDefaultWavesPerCu;
  if ((int64_t)num_compute_units * wpc * plan.chunks_per_wave > INT32_MAX)
    return fail(PDA_EINVAL, "num_compute_units = %d is too large", num_compute_units);
  info->variant = plan.variant == pda::Variant::Mfma ? PDA_VARIANT_MFMA : PDA_VARIANT_VECTOR;
  info->waves = num_compute_units * wpc;
  info->group_size = plan.G;
  info->chunks_max = info->waves * plan.chunks_per_wave;
  info->workspace_bytes = workspace_layout(problem, plan, gr, info->chunks_max).total;
  return PDA_OK;
}

// Parts per unit of the short decode kernel, or 0 for the stream-K kernels.
// The host knows the units and the bound on the lengths, not the lengths. The
// line lies where the stream-K kernels, which share the whole batch's blocks
// evenly, were not yet ahead on lognormal lengths (sigma 0.5, the bound at the
// longest; us per call, stream-K against short, bf16, 28 / 4 heads): 4 units of
// 64 tokens 17.1 against 4.2, of 12,000 38.4 / 17.5; 32 units of 1,000 tokens
// 20.3 / 9.1, of 12,000 54.7 / 47.6; 64 units of 1,000 21.3 / 10.4, of 3,000
// 32.0 / 26.5, of 12,000 84.5 / 87.2; 128 units of 300 19.5 / 13.1, of 1,000
// 25.9 / 28.1, of 3,000 47.4 / 71.2. The first bound is on units times length
// (half of it for the two-tile body and for f32 caches, whose steps take about
// twice as long per token), the second on the work in flight, which grows with
// units and length. With at most kShortParts parts, few units leave compute units
// idle and a wave with many steps, and are ahead all the same, as far as the first
// bound goes (every length the same, stream-K / short): 1 unit of 16,384 tokens
// 39.2 / 17.0, of 98,304 157.9 / 50.5, of 393,216 216 / 175 (f32 246 / 192; 4 query
// tokens 226 / 174); 2 units of 196,608 130 / 96, 4 of 98,304 85 / 57.
// With more units, parts are a whole number, and cus / units between two of them
// makes a wave's steps more than the first bound says: the third bound is on the
// steps that a wave of the longest length runs one after the other. One sequence
// of the longest length beside others of a sixteenth: 96 units (2 parts) of 3,184
// tokens, 13 steps, 23.5 / 27.4 (fp8 20.8 / 19.0); 80 (3 parts) of 4,576, 12 steps,
// 24.1 / 26.4; f32, 96 of 2,048, 16 steps, 26.4 / 29.8; 64 units of 6,144, 12 steps,
// 27.1 / 26.6; 128 of 1,792, 7 steps, 20.6 / 17.4; 4 query tokens, 96 units of
// 2,048, 8 steps, 24.4 / 21.6.
int short_parts(const pda_problem* pr, const Plan& plan, const Groups& gr, const pda_options* op, int cus,
                int chunks_max) {
  // f32 caches and the MFMA body; options that ask for a split mean the stream's
  if (gr.on || (plan.variant == pda::Variant::Vector && plan.kv != pda::KvType::F32)) return 0;
  if (op && (op->waves_per_cu || op->min_blocks_per_wave || op->chunks_per_wave || op->min_blocks_per_chunk)) return 0;
  const int64_t units = (int64_t)pr->num_seqs * pr->num_kv_heads;
  const bool wide = plan.Q * plan.G > 16, slow = wide || plan.kv == pda::KvType::F32;
  if (units > pda::kShortUnits || units * plan.len_cap > (slow ? 3 << 16 : 3 << 17) ||
      units * units * plan.len_cap > 7 << 22)
    return 0;
  // one workgroup per compute unit (more gained nothing), a group of steps each at least
  const int64_t step = plan.kv == pda::KvType::F32 ? 16 : 32;
  const int64_t groups = (plan.len_cap + step * pda::kShortGroup - 1) / (step * pda::kShortGroup);
  const int64_t most = wide ? pda::kShortParts / 2 : pda::kShortParts;
  int64_t parts = cus / units;
  if (parts > most) parts = most;
  if (parts > groups) parts = groups;
  if (parts < 1) parts = 1;
  const int64_t steps = (groups + parts - 1) / parts;
  const int64_t steps_max = wide ? 8 : plan.kv == pda::KvType::F32 ? 13 : plan.kv == pda::KvType::FP8 ? 16 : parts > 3 ? 12 : 9;
  if (parts < most && steps > steps_max) return 0;
  return units * parts <= units + chunks_max ? (int)parts : 0;  // the layout's partial slots
}

// fixed_scratch: take the workspace from the device's fixed scratch array
// (pda_paged_decode_attention_noalloc) instead of the stream's allocation.
int run(const void* q, const void* k_cache, const void* v_cache, const int32_t* block_table,
        const int32_t* seq_lens, const float* kv_scales, void* out, float softmax_scale,
        const int32_t* group_size, const int32_t* shared_blocks, const pda_problem* problem,
        const pda_options* options, hipStream_t stream, bool fixed_scratch = false) {
  g_error.clear();
  Plan plan;
  int rc = validate(problem, options, softmax_scale, &plan);
  if (rc != PDA_OK) return rc;
  Groups gr;
  if (group_size && (rc = validate_groups(problem, *group_size, shared_blocks, &plan, &gr)) != PDA_OK) return rc;
  if (problem->num_seqs == 0) return PDA_OK;
  if (!q || !k_cache || !v_cache || !block_table || !seq_lens || !out)
    return fail(PDA_EINVAL, "a required pointer (q, k_cache, v_cache, block_table, seq_lens, out) is NULL");
  if (problem->kv_dtype == PDA_DTYPE_FP8_E4M3 && !kv_scales)
    return fail(PDA_EINVAL, "an fp8 KV cache needs kv_scales");
  if ((rc = check_alignment({{q, 16, "q"}, {k_cache, 16, "k_cache"}, {v_cache, 16, "v_cache"}, {out, 16, "out"},
                             {block_table, 4, "block_table"}, {seq_lens, 4, "seq_lens"},
                             {kv_scales, 4, "kv_scales"}})) != PDA_OK)
    return rc;

  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  const DeviceInfo* di = nullptr;
  if ((rc = device_info(dev, &di)) != PDA_OK) return rc;
  if (!di->ok) return fail(PDA_EUNSUPPORTED, "device %d is %s; this library is built for gfx950", dev, di->arch.c_str());

  int wpc = plan.waves_per_cu;
  if (wpc == 0) {
    const bool wide = (gr.on ? gr.M * plan.G : plan.Q * plan.G) > 16;
    if ((rc = occupancy(dev, plan.variant, plan.kv, problem->head_dim, plan.G, wide, &wpc)) != PDA_OK) return rc;
    if (wpc > kDefaultWavesPerCu) wpc = kDefaultWavesPerCu;
  }
  const int waves = di->cus * wpc;
  const int chunks_max = waves * plan.chunks_per_wave;
  const Layout lay = workspace_layout(problem, plan, gr, chunks_max);

  std::unique_lock<std::mutex> lk;
  char* base = nullptr;
  bool* rearm = nullptr;
  Workspace* ws = nullptr;  // the stream's; null with the fixed scratch
  if (fixed_scratch) {
    if (dev < 0 || dev >= kMaxDevices) return fail(PDA_EUNSUPPORTED, "device %d: at most %d devices", dev, kMaxDevices);
    if (lay.total > pda::kScratchBytes)
      return fail(PDA_EINVAL,
                  "this call needs %lld bytes of workspace; the no-allocation entry point's fixed scratch holds %lld "
                  "(fewer sequences, KV heads or waves per call, or pda_paged_decode_attention)",
                  (long long)lay.total, (long long)pda::kScratchBytes);
    FixedScratch* fs = &g_fixed[dev];
    lk = std::unique_lock<std::mutex>(fs->mu);
    if (!fs->ptr) {  // first call on this device (current here): its copy of the array
      void* p = nullptr;
      if ((e = pda::scratch_address(&p)) != hipSuccess) return fail_hip(e, "hipGetSymbolAddress(scratch)");
      fs->ptr = p;
    }
    base = static_cast<char*>(fs->ptr) + pda::kShortCountBytes;
    rearm = &fs->rearm;
  } else {
    ws = workspace_for(dev, stream);
    lk = std::unique_lock<std::mutex>(ws->mu);
    if ((rc = ensure_workspace(ws, lay.total, stream)) != PDA_OK) return rc;
    base = static_cast<char*>(ws->ptr);
    rearm = &ws->rearm;
  }
  if (*rearm) {
    if (capturing(stream))
      return fail(PDA_EINVAL, "the workspace needs a reset after a failed launch: make one call outside capture");
    if ((e = hipMemsetAsync(base + pda::kHdrNext * 4, 0, 4, stream)) != hipSuccess)
      return fail_hip(e, "hipMemsetAsync");
    *rearm = false;
  }

  pda::DecodeArgs a;
  a.q = q;
  a.k_cache = k_cache;
  a.v_cache = v_cache;
  a.block_table = block_table;
  a.seq_lens = seq_lens;
  a.kv_scales = kv_scales;
  a.out = out;
  a.scale_log2 = softmax_scale * 1.4426950408889634f;
  a.mfma_scale_log2 = std::fabs(softmax_scale) * 1.4426950408889634f;
  a.neg_scale = softmax_scale < 0.f;
  a.B = problem->num_seqs;
  a.Hq = problem->num_q_heads;
  a.Hkv = problem->num_kv_heads;
  a.G = plan.G;
  a.D = problem->head_dim;
  a.max_blocks = problem->max_blocks_per_seq;
  a.num_blocks = problem->num_blocks;
  a.len_cap = plan.len_cap;
  a.min_share = plan.min_share;
  a.chunk_min = plan.chunk_min;
  a.chunks_max = chunks_max;
  a.waves = waves;
  // Workgroups of 4 (or 2) independent waves when every CU gets whole groups:
  // fewer, larger workgroups dispatch faster than one-wave groups.
  a.waves_per_group = wpc % 4 == 0 ? 4 : (wpc % 2 == 0 ? 2 : 1);
  a.out_bf16 = problem->out_dtype == PDA_DTYPE_BF16;
  a.E = (int32_t)(gr.n_prefix + problem->num_seqs);
  a.shared = gr.on ? 1 : 0;
  a.group_size = gr.group_size;
  a.M = gr.M;
  a.nsub = gr.nsub;
  a.n_prefix = (int32_t)gr.n_prefix;
  a.Gp = gr.on ? gr.M * plan.G : plan.Q * plan.G;
  a.Qn = plan.Q;
  a.shared_blocks = gr.shared_blocks;
  a.sg = reinterpret_cast<int32_t*>(base + lay.sg);
  a.hdr = reinterpret_cast<int32_t*>(base + lay.hdr);
  a.share = a.hdr + pda::kHdrShare;
  a.cum = reinterpret_cast<int32_t*>(base + lay.cum);
  a.ws_m = reinterpret_cast<float*>(base + lay.m);
  a.ws_l = reinterpret_cast<float*>(base + lay.l);
  a.ws_acc = reinterpret_cast<float*>(base + lay.acc);
  a.short_parts = short_parts(problem, plan, gr, options, di->cus, chunks_max);
  a.short_epoch = 0;
  // Arrival counts that no earlier call's can spoil: counted from this call's
  // epoch; in a capture, whose every replay has the same arguments, from zero,
  // which the first such call recorded into the graph writes (2 us per replay);
  // on the fixed scratch from zero at every call, which any stream may make.
  a.short_clear = 0;
  if (a.short_parts > 0) {
    if (!ws) {
      a.short_clear = 1;
    } else if (capturing(stream)) {
      const unsigned long long id = capture_id(stream);
      a.short_clear = id == 0 || id != ws->cleared_in;
      ws->cleared_in = id;
    } else {
      if (++ws->epoch == 0) {  // after 2^32 calls: start again
        if ((e = hipMemsetAsync(base - pda::kShortCountBytes, 0, pda::kShortCountBytes, stream)) != hipSuccess)
          return fail_hip(e, "hipMemsetAsync");
        ws->epoch = 1;
      }
      a.short_epoch = ws->epoch;
    }
  }
  if (gr.on && (e = pda::launch_prefix(a, gr.num_groups, stream)) != hipSuccess)
    return fail_hip(e, "prefix kernel launch");
  if ((e = pda::launch_decode(a, plan.variant, plan.kv, stream)) != hipSuccess)
    return fail_hip(e, "decode kernel launch");
  if ((e = pda::launch_combine(a, stream)) != hipSuccess) {
    *rearm = true;
    return fail_hip(e, "combine kernel launch");
  }
  return PDA_OK;
}

int append_run(const void* k_new, const void* v_new, void* k_cache, void* v_cache, float* kv_scales,
               const int32_t* block_table, const int32_t* positions, const pda_append_problem* pr,
               hipStream_t stream) {
  g_error.clear();
  if (!pr) return fail(PDA_EINVAL, "problem is NULL");
  if (pr->num_seqs < 0) return fail(PDA_EINVAL, "num_seqs = %d < 0", pr->num_seqs);
  if (pr->num_kv_heads < 1) return fail(PDA_EINVAL, "num_kv_heads = %d < 1", pr->num_kv_heads);
  if (pr->head_dim != 64 && pr->head_dim != 128)
    return fail(PDA_EUNSUPPORTED, "head_dim = %d (supported: 64, 128)", pr->head_dim);
  if (pr->block_size != pda::kBlockSize)
    return fail(PDA_EUNSUPPORTED, "block_size = %d (supported: 16)", pr->block_size);
  if (pr->max_blocks_per_seq < 1) return fail(PDA_EINVAL, "max_blocks_per_seq = %d < 1", pr->max_blocks_per_seq);
  if ((int64_t)pr->max_blocks_per_seq * pda::kBlockSize > INT32_MAX)
    return fail(PDA_EINVAL, "max_blocks_per_seq * 16 overflows int32");
  if ((int64_t)pr->num_seqs * pr->num_kv_heads > INT32_MAX) return fail(PDA_EINVAL, "num_seqs * num_kv_heads too large");
  if (pr->num_blocks < 1) return fail(PDA_EINVAL, "num_blocks = %lld < 1", (long long)pr->num_blocks);
  const int64_t tile = (int64_t)pda::kBlockSize * pr->head_dim * 4;
  if (pr->num_blocks > INT64_MAX / pr->num_kv_heads / tile) return fail(PDA_EINVAL, "num_blocks too large");
  if (pr->new_dtype != PDA_DTYPE_F32 && pr->new_dtype != PDA_DTYPE_BF16)
    return fail(PDA_EINVAL, "new_dtype = %d (supported: F32, BF16)", pr->new_dtype);
  const int kd = pr->kv_dtype;
  if (kd != PDA_DTYPE_F32 && kd != PDA_DTYPE_BF16 && kd != PDA_DTYPE_FP8_E4M3)
    return fail(PDA_EINVAL, "kv_dtype = %d is not a pda_dtype", kd);
  if (pr->num_seqs == 0) return PDA_OK;
  if (!k_new || !v_new || !k_cache || !v_cache || !block_table || !positions)
    return fail(PDA_EINVAL, "a required pointer (k_new, v_new, k_cache, v_cache, block_table, positions) is NULL");
  if (kd == PDA_DTYPE_FP8_E4M3 && !kv_scales) return fail(PDA_EINVAL, "an fp8 KV cache needs kv_scales");

  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  const DeviceInfo* di = nullptr;
  int rc;
  if ((rc = device_info(dev, &di)) != PDA_OK) return rc;
  if (!di->ok) return fail(PDA_EUNSUPPORTED, "device %d is %s; this library is built for gfx950", dev, di->arch.c_str());
  Workspace* ws = workspace_for(dev, stream);
  std::lock_guard<std::mutex> lk(ws->mu);
  if ((rc = ensure_workspace(ws, align_up(pda::kHdrWords * 4), stream)) != PDA_OK) return rc;

  pda::AppendArgs a;
  a.k_new = k_new;
  a.v_new = v_new;
  a.k_cache = k_cache;
  a.v_cache = v_cache;
  a.kv_scales = kv_scales;
  a.block_table = block_table;
  a.positions = positions;
  a.B = pr->num_seqs;
  a.Hkv = pr->num_kv_heads;
  a.D = pr->head_dim;
  a.max_blocks = pr->max_blocks_per_seq;
  a.num_blocks = pr->num_blocks;
  a.new_bf16 = pr->new_dtype == PDA_DTYPE_BF16;
  a.status = static_cast<int32_t*>(ws->ptr) + pda::kHdrStatus;
  const pda::KvType kv = kd == PDA_DTYPE_F32 ? pda::KvType::F32
                         : kd == PDA_DTYPE_BF16 ? pda::KvType::BF16 : pda::KvType::FP8;
  if ((e = pda::launch_append(a, kv, stream)) != hipSuccess) return fail_hip(e, "append kernel launch");
  return PDA_OK;
}

// Largest prefill image in bytes: PDA_PREFILL_IMAGE_MAX_MB (MiB, read on each
// call; 0 always stages through registers), 8 GiB by default.
int64_t prefill_image_cap() {
  const char* v = std::getenv("PDA_PREFILL_IMAGE_MAX_MB");
  if (!v || !*v) return 8ll << 30;
  char* end = nullptr;
  const long long mb = std::strtoll(v, &end, 10);
  if (end == v || mb < 0) return 8ll << 30;
  return mb > (INT64_MAX >> 20) ? INT64_MAX : (int64_t)mb << 20;
}

// Query tiles per sequence (the call's average) from which a prefill writes
// the image: PDA_PREFILL_IMAGE_MIN_TILES (read on each call; 0 writes it
// whenever it fits), by default where both ways take the same time.
int64_t prefill_image_tiles(bool fp8, int len_cap) {
  const int by_default = len_cap > pda::kPfImageKeys ? (fp8 ? pda::kPfImageTilesFp8 : pda::kPfImageTilesBf16)
                                                     : (fp8 ? pda::kPfImageTilesShortFp8 : pda::kPfImageTilesShortBf16);
  const char* v = std::getenv("PDA_PREFILL_IMAGE_MIN_TILES");
  if (!v || !*v) return by_default;
  char* end = nullptr;
  const long long n = std::strtoll(v, &end, 10);
  return end == v || n < 0 || n > INT32_MAX ? by_default : (int64_t)n;
}

int prefill_run(const void* q, const int32_t* q_offsets, const void* k_cache, const void* v_cache,
                const int32_t* block_table, const int32_t* seq_lens, const float* kv_scales, void* out,
                float softmax_scale, const pda_prefill_problem* pr, hipStream_t stream) {
  g_error.clear();
  if (!pr) return fail(PDA_EINVAL, "problem is NULL");
  if (pr->num_seqs < 0) return fail(PDA_EINVAL, "num_seqs = %d < 0", pr->num_seqs);
  if (pr->num_tokens < 0) return fail(PDA_EINVAL, "num_tokens = %d < 0", pr->num_tokens);
  if (pr->num_q_heads < 1 || pr->num_kv_heads < 1)
    return fail(PDA_EINVAL, "num_q_heads = %d and num_kv_heads = %d must be >= 1", pr->num_q_heads,
                pr->num_kv_heads);
  if (pr->num_q_heads % pr->num_kv_heads)
    return fail(PDA_EINVAL, "num_q_heads = %d is not a multiple of num_kv_heads = %d", pr->num_q_heads,
                pr->num_kv_heads);
  const int G = pr->num_q_heads / pr->num_kv_heads;
  if (G > pda::kMaxGroup)
    return fail(PDA_EUNSUPPORTED, "GQA group of %d query heads per KV head (max %d)", G, pda::kMaxGroup);
  if (pr->head_dim != 64 && pr->head_dim != 128)
    return fail(PDA_EUNSUPPORTED, "head_dim = %d (supported: 64, 128)", pr->head_dim);
  if (pr->block_size != pda::kBlockSize)
    return fail(PDA_EUNSUPPORTED, "block_size = %d (supported: 16)", pr->block_size);
  if (pr->max_blocks_per_seq < 1) return fail(PDA_EINVAL, "max_blocks_per_seq = %d < 1", pr->max_blocks_per_seq);
  if (pr->num_blocks < 1) return fail(PDA_EINVAL, "num_blocks = %lld < 1", (long long)pr->num_blocks);
  const int64_t table_tokens = (int64_t)pr->max_blocks_per_seq * pda::kBlockSize;
  if (table_tokens > INT32_MAX) return fail(PDA_EINVAL, "max_blocks_per_seq * 16 overflows int32");
  if ((int64_t)pr->num_seqs * pr->max_blocks_per_seq > INT32_MAX)
    return fail(PDA_EINVAL, "num_seqs * max_blocks_per_seq overflows int32");
  if ((int64_t)pr->num_tokens * pr->num_q_heads > INT32_MAX)
    return fail(PDA_EINVAL, "num_tokens * num_q_heads overflows int32");
  if (pr->max_seq_len < 0) return fail(PDA_EINVAL, "max_seq_len = %d < 0", pr->max_seq_len);
  if (pr->max_seq_len > table_tokens)
    return fail(PDA_EINVAL, "max_seq_len = %d exceeds max_blocks_per_seq * 16 = %lld", pr->max_seq_len,
                (long long)table_tokens);
  const int64_t tile = (int64_t)pda::kBlockSize * pr->head_dim * 4;
  if (pr->num_blocks > INT64_MAX / pr->num_kv_heads / tile) return fail(PDA_EINVAL, "num_blocks too large");
  if (pr->q_dtype != PDA_DTYPE_BF16)
    return fail(pr->q_dtype == PDA_DTYPE_F32 ? PDA_EUNSUPPORTED : PDA_EINVAL, "q_dtype = %d (supported: BF16)",
                pr->q_dtype);
  const int kd = pr->kv_dtype;
  if (kd == PDA_DTYPE_F32) return fail(PDA_EUNSUPPORTED, "prefill runs on the matrix cores: it needs a bf16 or fp8 cache");
  if (kd != PDA_DTYPE_BF16 && kd != PDA_DTYPE_FP8_E4M3) return fail(PDA_EINVAL, "kv_dtype = %d is not a pda_dtype", kd);
  if (pr->out_dtype != PDA_DTYPE_BF16 && pr->out_dtype != PDA_DTYPE_F32)
    return fail(PDA_EINVAL, "out_dtype = %d (must be BF16 or F32)", pr->out_dtype);
  if (!std::isfinite(softmax_scale)) return fail(PDA_EINVAL, "softmax_scale is not finite");
  const int TQ = pda::kPfColumns / G;
  // every sequence's tiles: sum of ceil(n_b / TQ) <= (T + B (TQ - 1)) / TQ
  const int64_t items_max = ((int64_t)pr->num_tokens + (int64_t)pr->num_seqs * (TQ - 1)) / TQ;
  // the attention grid names a claimed unit (item, KV head) as 8 * index + queue in an int32
  if (items_max * pr->num_kv_heads > INT32_MAX / 8)
    return fail(PDA_EINVAL, "too many work units (%lld tiles x %d KV heads) for the unit queues", (long long)items_max,
                pr->num_kv_heads);
  if (pr->num_seqs == 0 || pr->num_tokens == 0) return PDA_OK;
  if (!q || !q_offsets || !k_cache || !v_cache || !block_table || !seq_lens || !out)
    return fail(PDA_EINVAL, "a required pointer (q, q_offsets, k_cache, v_cache, block_table, seq_lens, out) is NULL");
  if (kd == PDA_DTYPE_FP8_E4M3 && !kv_scales) return fail(PDA_EINVAL, "an fp8 KV cache needs kv_scales");
  {
    const int rc = check_alignment({{q, 16, "q"}, {k_cache, 16, "k_cache"}, {v_cache, 16, "v_cache"},
                                    {out, 16, "out"}, {q_offsets, 4, "q_offsets"}, {block_table, 4, "block_table"},
                                    {seq_lens, 4, "seq_lens"}, {kv_scales, 4, "kv_scales"}});
    if (rc != PDA_OK) return rc;
  }

  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  const DeviceInfo* di = nullptr;
  int rc;
  if ((rc = device_info(dev, &di)) != PDA_OK) return rc;
  if (!di->ok) return fail(PDA_EUNSUPPORTED, "device %d is %s; this library is built for gfx950", dev, di->arch.c_str());
  Workspace* ws = workspace_for(dev, stream);
  std::lock_guard<std::mutex> lk(ws->mu);
  const int len_cap = pr->max_seq_len > 0 ? pr->max_seq_len : (int)table_tokens;
  // Workspace: header, work items, and as room and caps allow the split plan's
  // partials and the image. A capture that cannot grow the workspace, or a
  // failed allocation, goes without the image (the staging kernel's results
  // are the same), then without the split.
  const int64_t items_off = align_up(pda::kHdrWords * 4);
  // A KV head's partial slots: a tile split into items of at least the grid's
  // even share has at most twice its pairs over that share of them, so a call
  // has at most 2 * wgs / Hkv, and never more than every tile cut to the
  // fewest pairs. No split where the longest cache has no room for one.
  const int64_t most_cut = ((int64_t)len_cap / 32 + 1 + pda::kPfSplitPairs - 1) / pda::kPfSplitPairs;
  int64_t slots = 2 * (((int64_t)di->cus + pr->num_kv_heads - 1) / pr->num_kv_heads) + 2;
  if (slots > items_max * most_cut) slots = items_max * most_cut;
  if (items_max * pr->num_kv_heads > (int64_t)pda::kPfSplitUnits * di->cus || items_max > pda::kPfSplitTiles ||
      pr->num_seqs > pda::kPfSplitSeqs || most_cut < 2)
    slots = 0;
  // Image: V in fp16; for an fp8 cache K in bf16 too.
  const int64_t img_half = pr->num_blocks * pr->num_kv_heads * (int64_t)pda::kBlockSize * pr->head_dim * 2;
  const int64_t img_bytes = kd == PDA_DTYPE_FP8_E4M3 ? 2 * img_half : img_half;
  const bool cap = capturing(stream);
  // The image pays where several tiles read what it converts once; an fp8
  // cache's takes twice the work. Measured (image / converting in the kernel, us
  // per call, bf16; fp8), n query tiles of each of B sequences of L cached tokens:
  //   28 / 4 heads,  8 x 4,096: n = 2  72 /  72;  84 /  74   n = 5 141 / 159; 161 / 168
  //                             n = 8 151 / 165; 166 / 174
  //                 32 x 2,048: n = 2 103 /  99; 121 / 103   n = 5 225 / 229; 254 / 243
  //                             n = 8 294 / 303; 322 / 319
  //   32 / 8 heads, 32 x 2,048: n = 2 207 / 183; 250 / 189   n = 5 403 / 398; 450 / 405
  //                             n = 8 544 / 559; 588 / 595   n = 16 897 / 963; 944 / 1,025
  //                 64 x   600: n = 5 273 / 261; 300 / 275   n = 9 380 / 374; 411 / 394
  // (short sequences' images cost the same per key and are read for fewer pairs).
  //
  // The average says too little where a batch mixes long prompts with one-token
  // rows or empty slots. With fewer tiles per sequence on average, but many in
  // all and room for long sequences, the call is mixed: the plan decides
  // sequence by sequence. That is a
  // second attention launch, 3 us if its list is empty and 10 to 25 with a few
  // short items, for about 10% of the prompts' time: from 100 tiles on. One
  // prompt of 8,192 beside 31 rows of one key each, converting / mixed: 28 / 4
  // heads bf16 546 / 483, fp8 577 / 514; beside 31 rows over 256 keys 547 / 507,
  // 579 / 527; over 2,048 582 / 542, 620 / 574. One of 2,048 (57 tiles) beside 31
  // rows: 94 / 98. Rows of up to kPfMixedKeys keys go with the image (31 of one
  // key 489 / 483), no longer ones (127 of 100 keys 540 there, 506 from the cache).
  const int64_t tiles_min = prefill_image_tiles(kd == PDA_DTYPE_FP8_E4M3, len_cap), tiles_all = pr->num_tokens / TQ;
  const bool mixed = tiles_all < tiles_min * pr->num_seqs;
  bool use_img = img_bytes <= prefill_image_cap() && (!mixed || (tiles_all >= pda::kPfMixedTiles && tiles_all >= 2 * tiles_min && len_cap > pda::kPfImageKeys));
  struct PrefillLayout {
    int64_t list_max, parts, splits, ml, acc, img, total;
  };
  auto layout = [&](int64_t n, bool image) {
    PrefillLayout w;
    w.list_max = items_max + n;  // a split adds at most its slots
    const int64_t lists = image && mixed ? 2 : 1, cols = n * pr->num_kv_heads * pda::kPfColumns;
    w.parts = items_off + lists * w.list_max * 16;
    w.splits = align_up(w.parts + lists * w.list_max * 16);
    w.ml = align_up(w.splits + n / 2 * 16);
    w.acc = align_up(w.ml + cols * 8);
    w.total = n ? w.acc + cols * pr->head_dim * 4 : w.parts;
    w.img = align_up(w.total);
    if (image) w.total = w.img + img_bytes;
    return w;
  };
  if (cap && ws->bytes < layout(slots, false).total) slots = 0;
  if (use_img && cap && ws->bytes < layout(slots, true).total) use_img = false;
  PrefillLayout lay;
  for (;;) {
    lay = layout(slots, use_img);
    rc = ensure_workspace(ws, lay.total, stream);
    if (rc != PDA_ENOMEM || !(use_img || slots)) break;
    if (use_img) use_img = false;
    else slots = 0;
    g_error.clear();
  }
  if (rc != PDA_OK) return rc;
  char* base = static_cast<char*>(ws->ptr);

  pda::PrefillArgs a;
  a.q = q;
  a.q_offsets = q_offsets;
  a.k_cache = k_cache;
  a.v_cache = v_cache;
  a.block_table = block_table;
  a.seq_lens = seq_lens;
  a.kv_scales = kv_scales;
  a.out = out;
  a.scale_log2 = std::fabs(softmax_scale) * 1.4426950408889634f;
  a.neg_scale = softmax_scale < 0.f;
  a.B = pr->num_seqs;
  a.T = pr->num_tokens;
  a.Hq = pr->num_q_heads;
  a.Hkv = pr->num_kv_heads;
  a.G = G;
  a.D = pr->head_dim;
  a.TQ = TQ;
  a.max_blocks = pr->max_blocks_per_seq;
  a.num_blocks = pr->num_blocks;
  a.len_cap = len_cap;
  int shift = 0;
  while ((a.len_cap >> shift) >= pda::kPfBuckets) ++shift;
  a.len_shift = shift;
  a.items_max = (int32_t)items_max;
  a.out_bf16 = pr->out_dtype == PDA_DTYPE_BF16;
  a.cus = di->cus;
  a.nq = std::gcd(a.Hkv, 8);
  a.hdr = reinterpret_cast<int32_t*>(base);
  a.items = reinterpret_cast<int4*>(base + items_off);
  a.slots = (int32_t)slots;
  a.list_max = (int32_t)lay.list_max;
  a.img_tiles = use_img && mixed ? (int32_t)tiles_min : 0;
  a.wgs = a.img_shift = 0;  // the launcher's
  a.parts = reinterpret_cast<int4*>(base + lay.parts);
  a.splits = reinterpret_cast<int4*>(base + lay.splits);
  a.part_ml = reinterpret_cast<float2*>(base + lay.ml);
  a.part_acc = reinterpret_cast<float*>(base + lay.acc);
  a.v_img = use_img ? base + lay.img : nullptr;
  a.k_img = use_img && kd == PDA_DTYPE_FP8_E4M3 ? base + lay.img + img_half : nullptr;
  const pda::KvType kv = kd == PDA_DTYPE_BF16 ? pda::KvType::BF16 : pda::KvType::FP8;
  if ((e = pda::launch_prefill(a, kv, stream)) != hipSuccess) return fail_hip(e, "prefill kernel launch");
  return PDA_OK;
}

}  // namespace

extern "C" {

int pda_query_plan(const pda_problem* problem, const pda_options* options, float softmax_scale,
                   int32_t num_compute_units, pda_plan_info* info) {
  return query_plan(problem, options, softmax_scale, num_compute_units, nullptr, info);
}

int pda_query_plan_shared_prefix(const pda_problem* problem, const pda_options* options, float softmax_scale,
                                 int32_t group_size, int32_t num_compute_units, pda_plan_info* info) {
  return query_plan(problem, options, softmax_scale, num_compute_units, &group_size, info);
}

int pda_paged_decode_attention(const void* q, const void* k_cache, const void* v_cache,
                               const int32_t* block_table, const int32_t* seq_lens, const float* kv_scales,
                               void* out, float softmax_scale, const pda_problem* problem,
                               const pda_options* options, hipStream_t stream) {
  return run(q, k_cache, v_cache, block_table, seq_lens, kv_scales, out, softmax_scale, nullptr, nullptr,
             problem, options, stream);
}

int pda_paged_decode_attention_noalloc(const void* q, const void* k_cache, const void* v_cache,
                                       const int32_t* block_table, const int32_t* seq_lens, const float* kv_scales,
                                       void* out, float softmax_scale, const pda_problem* problem,
                                       const pda_options* options, hipStream_t stream) {
  return run(q, k_cache, v_cache, block_table, seq_lens, kv_scales, out, softmax_scale, nullptr, nullptr,
             problem, options, stream, /*fixed_scratch=*/true);
}

int pda_paged_kv_append(const void* k_new, const void* v_new, void* k_cache, void* v_cache, float* kv_scales,
                        const int32_t* block_table, const int32_t* positions, const pda_append_problem* problem,
                        hipStream_t stream) {
  return append_run(k_new, v_new, k_cache, v_cache, kv_scales, block_table, positions, problem, stream);
}

int pda_paged_decode_attention_shared_prefix(const void* q, const void* k_cache, const void* v_cache,
                                             const int32_t* block_table, const int32_t* seq_lens,
                                             const float* kv_scales, void* out, float softmax_scale,
                                             int32_t group_size, const int32_t* shared_blocks,
                                             const pda_problem* problem, const pda_options* options,
                                             hipStream_t stream) {
  return run(q, k_cache, v_cache, block_table, seq_lens, kv_scales, out, softmax_scale, &group_size,
             shared_blocks, problem, options, stream);
}

int pda_paged_prefill_attention(const void* q, const int32_t* q_offsets, const void* k_cache, const void* v_cache,
                                const int32_t* block_table, const int32_t* seq_lens, const float* kv_scales,
                                void* out, float softmax_scale, const pda_prefill_problem* problem,
                                hipStream_t stream) {
  return prefill_run(q, q_offsets, k_cache, v_cache, block_table, seq_lens, kv_scales, out, softmax_scale, problem,
                     stream);
}

int pda_read_device_status(hipStream_t stream) {
  g_error.clear();
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  Workspace* ws = workspace_for(dev, stream);
  std::lock_guard<std::mutex> lk(ws->mu);
  if ((e = hipStreamSynchronize(stream)) != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
  // the current workspace and any a captured graph still writes to
  int32_t all = 0;
  std::vector<void*> headers = ws->retired;
  if (ws->ptr) headers.push_back(ws->ptr);
  for (void* p : headers) {
    for (int half : {0, pda::kHdrStaged}) {
      int32_t word = 0;
      int32_t* hdr = static_cast<int32_t*>(p) + half + pda::kHdrStatus;
      if ((e = hipMemcpy(&word, hdr, 4, hipMemcpyDeviceToHost)) != hipSuccess) return fail_hip(e, "hipMemcpy");
      if (word && (e = hipMemset(hdr, 0, 4)) != hipSuccess) return fail_hip(e, "hipMemset");
      all |= word;
    }
  }
  // the device's fixed scratch, once the no-allocation entry point has used it
  if (dev >= 0 && dev < kMaxDevices) {
    FixedScratch* fs = &g_fixed[dev];
    std::lock_guard<std::mutex> fl(fs->mu);
    if (fs->ptr) {
      int32_t word = 0;
      int32_t* hdr = reinterpret_cast<int32_t*>(static_cast<char*>(fs->ptr) + pda::kShortCountBytes) + pda::kHdrStatus;
      if ((e = hipMemcpy(&word, hdr, 4, hipMemcpyDeviceToHost)) != hipSuccess) return fail_hip(e, "hipMemcpy");
      if (word && (e = hipMemset(hdr, 0, 4)) != hipSuccess) return fail_hip(e, "hipMemset");
      all |= word;
    }
  }
  return all;
}

int pda_release_workspaces(void) {
  g_error.clear();
  std::lock_guard<std::mutex> lk(g_mu);
  int rc = PDA_OK;
  int cur = 0;
  const bool have_dev = hipGetDevice(&cur) == hipSuccess;
  for (auto& kv : g_workspaces) {
    Workspace* ws = kv.second.get();
    std::lock_guard<std::mutex> wl(ws->mu);
    if (!ws->ptr && ws->retired.empty()) continue;
    hipError_t e = hipSetDevice(kv.first.first);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e == hipSuccess && ws->ptr) e = free_workspace(ws->ptr);
    for (void* p : ws->retired)
      if (e == hipSuccess) e = free_workspace(p);
    if (e != hipSuccess) rc = fail_hip(e, "releasing a workspace");
    ws->ptr = nullptr;
    ws->bytes = 0;
    ws->retired.clear();
  }
  g_workspaces.clear();
  if (have_dev) (void)hipSetDevice(cur);
  return rc;
}

}  // extern "C"
