// Host side of the C ABI declared in include/vc_jointattn.h: argument
// validation, workspace layout, device check and kernel launches. Nothing
// here allocates, frees or synchronises.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <initializer_list>
#include <limits>
#include <mutex>

#include "common.hpp"
#include "vc_jointattn.h"

namespace {

constexpr int kMaxDevices = 64;

struct DeviceInfo {
  std::once_flag once;
  bool is_gfx950 = false;
  int cus = 0;  // compute units
};
DeviceInfo g_devices[kMaxDevices];

vc_status check_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return VC_ERR_DEVICE;
  DeviceInfo& di = g_devices[dev];
  std::call_once(di.once, [&] {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) == hipSuccess) {
      di.is_gfx950 = strncmp(prop.gcnArchName, "gfx950", 6) == 0;
      di.cus = prop.multiProcessorCount;
    }
  });
  return di.is_gfx950 ? VC_OK : VC_ERR_DEVICE;
}

// Workspace of vc_jointattn_fwd_noalloc: a file-scope device array (each device holds its
// own copy from the library's first use on it until the process ends). In host code
// `scratch` names a host-side stand-in, not device memory: kernels and copies take the
// device address looked up below, never the array's name.
static __device__ __align__(256) char scratch[VC_JOINTATTN_NOALLOC_SCRATCH_BYTES];

struct ScratchAddr {
  std::once_flag once;
  void* ptr = nullptr;
};
ScratchAddr g_scratch[kMaxDevices];

// Device address of this device's copy of `scratch`, looked up once per device with that
// device current (the caller has checked it with check_device); NULL if the lookup failed.
void* scratch_ptr() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  ScratchAddr& sa = g_scratch[dev];
  std::call_once(sa.once, [&] {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) == hipSuccess) sa.ptr = p;
  });
  return sa.ptr;
}

// Compute units of the current device (after check_device succeeded).
int device_cus() {
  int dev = 0;
  (void)hipGetDevice(&dev);
  return g_devices[dev].cus;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool aligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }

// Validates a descriptor; on success fills N.
vc_status check_desc(const vc_jointattn_desc* d, int64_t* n_out) {
  if (!d) return VC_ERR_NULL;
  if (d->head_dim != 64 && d->head_dim != 128) return VC_ERR_HEAD_DIM;
  if (d->batch < 1 || d->heads < 1 || d->text_slot < 0 || d->frames < 1 || d->grid_h < 1 || d->grid_w < 1)
    return VC_ERR_SHAPE;
  if (d->heads > 65535 || d->batch > 65535) return VC_ERR_SHAPE;
  if (!(d->softmax_scale <= 0.0f || isfinite(d->softmax_scale))) return VC_ERR_SHAPE;
  if (d->deterministic != 0 && d->deterministic != 1) return VC_ERR_SHAPE;
  const int64_t video = (int64_t)d->frames * d->grid_h * d->grid_w;
  const int64_t n = (int64_t)d->text_slot + video;
  if (video <= 0 || n > (int64_t)1 << 30) return VC_ERR_SHAPE;
  // Element counts of a [B, N, H, D] tensor must stay well inside 64-bit byte offsets.
  const int64_t elems = (int64_t)d->batch * n * d->heads * d->head_dim;
  if (elems <= 0 || elems > ((int64_t)1 << 40)) return VC_ERR_SHAPE;
  *n_out = n;
  return VC_OK;
}

float scale_of(const vc_jointattn_desc* d) {
  return d->softmax_scale > 0.0f ? d->softmax_scale : 1.0f / sqrtf((float)d->head_dim);
}
// The joint and spatial backward start their score accumulators from -LSE / c, which must stay
// finite down to the smallest positive c (LSE is about ln N more than the largest c s). Where c
// is under 1e-30, one factor of the scores is taken times `down` and c divided by it: a
// power of two, so every probability keeps its value. (bf16 scores reach 1e38, so that even
// c = 1e-38 gives logits of order 1.)
struct ProbScale {
  float c, down;
};
ProbScale prob_scale_of(const vc_jointattn_desc* d) {
  ProbScale p{scale_of(d), 1.0f};
  for (; p.c < 1e-30f && p.down > 1e-18f; p.c *= 2.0f) p.down *= 0.5f;
  return p;
}

int ntiles(int64_t n) { return (int)((n + vcja::kTileTok - 1) / vcja::kTileTok); }

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Size of one [B, N, H, D] tensor in token-major tiles: what the workspaces are still sized by,
// from versions that kept such copies (callers' sizes and the no-allocation forward's limit
// stay as they were).
size_t tiles_bytes(const vc_jointattn_desc* d, int64_t n) {
  return align256((size_t)d->batch * d->heads * ntiles(n) * vcja::tile_elems(d->head_dim) * sizeof(__bf16));
}

// Per-row fp32 array [B, H, Npad].
size_t rows_bytes(const vc_jointattn_desc* d, int64_t n) {
  return align256((size_t)d->batch * d->heads * (size_t)ntiles(n) * vcja::kTileTok * sizeof(float));
}

// Joint attention: split of the last, partial round of a kernel's dispatch. With W items
// (256-row blocks x heads x samples) on `cus` compute units, the R = W mod cus items of the
// last round (all of them when W < cus) can each be split into C workgroups over runs of
// `span` tiles along the other token axis, whose fp32 partials are merged afterwards. With
// `over` the tiles' worth of time a split workgroup spends on its partials and `merge` that
// of the merge launch, the round takes ceil(R C / cus) (span + over) + merge tiles instead
// of ntile: the C of least time is taken, if it saves at least a tenth. Measured (tile =
// 64 tokens; forward, dQ: about 2 us a tile, dK/dV 3.4 us, 8 to 13 us to write a
// workgroup's partials, 6 to 15 us a merge): see kSplit*. `max_wgs` bounds R C (workspace). At
// head_dim 64 a tile takes about half of that and the same costs hold back splits that would
// pay rather than take any that do not: at 25 shapes of 12 to 1,056 items no split lost (forward,
// both backwards, us unsplit / split: 16 x 2,000 tokens 40 / 33, 105 / 79; 4 x 1,500 31 / 23, 76 /
// 36; 5 x 20,000 680 / 614, 1906 / 1799), and costs 1.5 to 3 times as high lose such ones.
struct SplitCost {
  int over, merge;
};
constexpr SplitCost kSplitFwd{3, 5}, kSplitDkdv{5, 6}, kSplitDq{3, 5};
constexpr int kTailMinWgs = 256;  // split workgroups the least accepted workspace has room for
constexpr int kTailMaxWgs = 512;  // ... and the largest queried one
constexpr int kPlanCus = 256;     // compute units the queries (which touch no device) assume
constexpr int kRowsPerItem = 256;
struct TailPlan {
  int items, chunks, span;
};
TailPlan tail_plan(int64_t work_items, int ntile, int cus, SplitCost cost, int64_t max_wgs) {
  const TailPlan none{0, 1, 0};
  if (cus < 2) return none;
  const int r = (int)(work_items % cus);
  if (r == 0) return none;
  TailPlan best = none;
  int64_t least = (int64_t)ntile * 9 / 10;
  for (int c = 2; c <= std::min(ntile, 64) && (int64_t)r * c <= max_wgs; ++c) {
    const int span = (ntile + c - 1) / c, chunks = (ntile + span - 1) / span;
    const int64_t rounds = ((int64_t)r * chunks + cus - 1) / cus;
    const int64_t t = rounds * (span + cost.over) + cost.merge;
    if (t < least) {
      least = t;
      best = TailPlan{r, chunks, span};
    }
  }
  return best;
}
// Items of the joint kernels (256-row blocks x heads x samples).
int64_t joint_items(const vc_jointattn_desc* d, int64_t n) {
  return ((n + kRowsPerItem - 1) / kRowsPerItem) * d->heads * d->batch;
}
// Split workgroups that the queried workspaces have room for: the least accepted number, or
// what the largest plan of these kernels takes.
int64_t queried_wgs(const vc_jointattn_desc* d, int64_t n, std::initializer_list<SplitCost> costs) {
  int64_t wgs = std::min<int64_t>(kTailMinWgs, joint_items(d, n));
  for (const SplitCost& c : costs) {
    const TailPlan t = tail_plan(joint_items(d, n), ntiles(n), kPlanCus, c, kTailMaxWgs);
    wgs = std::max<int64_t>(wgs, (int64_t)t.items * t.chunks);
  }
  return wgs;
}
// fp32 partials of the split tail: dK and dV of `wgs` workgroups of 256 keys (the dQ pass
// reuses the region for its single tensor). The least accepted region: kTailMinWgs of them,
// or one per item where there are fewer; the plans take what the caller's workspace holds.
constexpr size_t tail_wg_bytes(int head_dim) { return (size_t)2 * kRowsPerItem * head_dim * sizeof(float); }
size_t tail_part_bytes(const vc_jointattn_desc* d, int64_t n) {
  const int64_t wgs = std::min<int64_t>(kTailMinWgs, joint_items(d, n));
  return align256(wgs * tail_wg_bytes(d->head_dim));
}

// Fused backward: the key blocks [0, fused_dq_blocks) add their dQ share with atomics in
// the key-stationary pass; the dQ pass covers the others. Per key block, the atomics (an
// fp32 dQ tile per query tile) cost about what the dQ pass's recomputation of S and dP
// costs at head_dim 128, so the backward's time is nearly flat in the fraction between 1/2
// and 7/8 there. Measured, us at 0, 50, 65, 80, 100%: 24 heads x 20,000 tokens 13558, 13706, 13293,
// 13812, 15629; 64 x 9,856 9001, 9224, 9018, 8942, 9879; 24 x 5,000 914, 947, 921, 945, 1040. At
// head_dim 64 fusing every key block is fastest on clips of some thousand tokens (32 x 8,320 1938,
// 1989, 1920, 1885, 1802; 48 x 4,000 692, 736, 707, 681, 663) and within 5% of the best beyond
// (24 x 20,000 8144, 8471, 8380, 8023, 8401); the dQ pass then only converts the accumulator.
constexpr int kFusedDqPercent128 = 65;
constexpr int kFusedDqPercent64 = 100;
// The fused pass runs only while a sample's N*H*D elements number less than 2^32; larger inputs
// take the separate passes. (Its addresses no longer need that bound: a uniform 64-bit base and
// lane offsets of a few rows. It stays because no larger sample has been run or timed through
// the atomics.)
bool dq_offsets_fit(const vc_jointattn_desc* d, int64_t n) {
  return n * d->heads * d->head_dim < ((int64_t)1 << 32);
}
int fused_dq_blocks(const vc_jointattn_desc* d, int64_t n) {
  if (!dq_offsets_fit(d, n)) return 0;
  const int nblk = (int)((n + vcja::kDkdvKeys - 1) / vcja::kDkdvKeys);
  const int pct = d->head_dim == 128 ? kFusedDqPercent128 : kFusedDqPercent64;
  return (int)(((int64_t)nblk * pct + 50) / 100);
}
// Every key block carries its dQ share: no dQ pass over key tiles.
bool all_keys_fused(const vc_jointattn_desc* d, int64_t n) {
  return (int64_t)fused_dq_blocks(d, n) * vcja::kDkdvKeys >= n;
}

// Small problems at head_dim 128 form all of dQ in the key-stationary pass too when the whole
// backward is one call: the dQ pass over 35% of the keys is mostly its launch, prologue and
// last round there, and the atomics are few. From a few rounds of workgroups on, that pass is
// cheap and the atomics of long samples are not. Measured, backward in us at 65% / 100%, (heads x
// samples) x tokens: 384 x 512 294 / 266, 768 x 512 620 / 526, 384 x 768 574 / 530, 192 x 1,024
// 416 / 418, 1536 x 1,024 3350 / 3128; 24 x 1,280 134 / 113, 72 x 1,280 290 / 263, 48 x 1,792
// 318 / 307, 24 x 2,048 199 / 189, 48 x 2,048 396 / 385 and 381 / 386, 72 x 1,536 345 / 327; 3 x
// 1,000 57 / 38, 4 x 4,000 149 / 141, 1 x 12,000 273 / 265, 1 x 14,000 363 / 344. Not so: 96 x
// 1,280 304 / 314, 192 x 1,280 611 / 616, 96 x 2,048 687 / 722, 1 x 16,384 444 / 460, 16 x 4,096
// 401 / 448, 24 x 2,525 257 / 272, 24 x 5,000 921 / 1040.
bool fuse_every_key(const vc_jointattn_desc* d, int64_t n) {
  const int64_t items = joint_items(d, n);
  return dq_offsets_fit(d, n) && (all_keys_fused(d, n) || n <= 1024 || (n <= 2048 && items <= 448) ||
                                  (n <= 14336 && items <= 64));
}

// Spatial backward (deterministic = 0): every key block adds its dQ share with atomics in the
// key-stationary pass, or the separate passes run. The atomics, one per element and key block of
// a query's frame at the memory side, set the length of the fused pass; a dQ pass of its own
// pays for its launch, prologue and last round, so small problems fuse, and so do frames of
// up to 160 tokens, which leave much of a dQ workgroup's 256 rows empty. With a key mask the dQ
// pass tests every key of every tile against the mask and its frame's bounds, and loses. At
// head_dim 64 the two are within 3% of each other and all fuse. Measured, D = 128, backward in
// us, fused / separate (video rows x heads x samples in thousands): 1382 9889 / 8406, 530 2415 /
// 2100, 322 2218 / 1940, 196 532 / 453 and 308 / 274, 173 1320 / 1165, 122 350 / 322, 92 217 / 201
// and 751 / 671; 71 212 / 220, 52 76 / 79, 22 260 / 284, 12 162 / 181. Frames of 48 tokens 319 /
// 423 and 210 / 244, of 100 519 / 549 and 285 / 311, of 120 321 / 363, of 128 175 / 172 and 419 /
// 433, of 144 192 / 190 and 372 / 404, of 192 463 / 447, of 240 212 / 200. Masked: 1382 9919 /
// 11019, 794 3696 / 4184, 614 1820 / 2051, 122 266 / 278, 92 (frames of 60) 192 / 235. D = 64: 1382
// 5660 / 5522, 307 481 / 487, 262 362 / 373, 74 247 / 252.
constexpr int64_t kSpatialFusedRows = 80 * 1024;
constexpr int kSpatialFusedFrame = 160;
bool spatial_fused(const vc_jointattn_desc* d, int64_t n, bool key_mask) {
  return dq_offsets_fit(d, n) &&
         (d->head_dim == 64 || key_mask || (int64_t)d->grid_h * d->grid_w <= kSpatialFusedFrame ||
          (n - d->text_slot) * d->heads * d->batch < kSpatialFusedRows);
}

// Forward workspace: one tensor's tiles (unused) | split-tail partials (unnormalised O, base, sum
// per row).
constexpr size_t fwd_wg_bytes(int head_dim) { return (size_t)kRowsPerItem * (head_dim + 2) * sizeof(float); }
size_t fwd_tail_bytes(const vc_jointattn_desc* d, int64_t n) {
  const int64_t wgs = std::min<int64_t>(kTailMinWgs, joint_items(d, n));
  return align256(wgs * fwd_wg_bytes(d->head_dim));
}
size_t fwd_ws_bytes(const vc_jointattn_desc* d, int64_t n) { return tiles_bytes(d, n) + fwd_tail_bytes(d, n); }
// Split workgroups that a workspace of `have` bytes holds after its first `used` bytes.
int64_t tail_wgs(size_t have, size_t used, size_t wg_bytes) {
  return have <= used ? 0 : std::min<int64_t>(kTailMaxWgs, (int64_t)((have - used) / wg_bytes));
}

// Plans of the three joint kernels in a workspace of `have` bytes. With the queried size or
// more, on any number of compute units, a plan does not depend on `have` (no more split
// workgroups are taken than the queried size holds), so results do not either; and where the
// no-allocation forward accepts the problem, its scratch array and a workspace give one plan.
TailPlan fwd_plan(const vc_jointattn_desc* d, int64_t n, int cus, size_t have) {
  if (fwd_ws_bytes(d, n) <= VC_JOINTATTN_NOALLOC_SCRATCH_BYTES)
    have = std::min<size_t>(have, VC_JOINTATTN_NOALLOC_SCRATCH_BYTES);
  return tail_plan(joint_items(d, n), ntiles(n), cus, kSplitFwd,
                   std::min(queried_wgs(d, n, {kSplitFwd}), tail_wgs(have, tiles_bytes(d, n), fwd_wg_bytes(d->head_dim))));
}

// Backward workspace: -D | -LSE/c | fp32 dQ accumulator (in the place of three sets of token
// tiles, >= 4 bytes per element of dq) | tail partials.
struct BwdWorkspace {
  float* dd;
  float* nls;
  float* dq_acc;
};

size_t bwd_ws_bytes(const vc_jointattn_desc* d, int64_t n) {
  return 2 * rows_bytes(d, n) + 3 * tiles_bytes(d, n) + tail_part_bytes(d, n);
}
size_t bwd_ws_query_bytes(const vc_jointattn_desc* d, int64_t n) {
  return bwd_ws_bytes(d, n) - tail_part_bytes(d, n) +
         align256(queried_wgs(d, n, {kSplitDkdv, kSplitDq}) * tail_wg_bytes(d->head_dim));
}
// `skip` key tiles are not visited by the dQ pass (their share of dQ is fused).
TailPlan bwd_plan(const vc_jointattn_desc* d, int64_t n, int cus, SplitCost cost, int skip, size_t have) {
  return tail_plan(joint_items(d, n), ntiles(n) - skip, cus, cost,
                   std::min(queried_wgs(d, n, {kSplitDkdv, kSplitDq}),
                            tail_wgs(have, bwd_ws_bytes(d, n) - tail_part_bytes(d, n), tail_wg_bytes(d->head_dim))));
}
float* tail_part_of(const vc_jointattn_desc* d, int64_t n, void* ws) {
  return reinterpret_cast<float*>(static_cast<char*>(ws) + 2 * rows_bytes(d, n) + 3 * tiles_bytes(d, n));
}

BwdWorkspace split_bwd_ws(const vc_jointattn_desc* d, int64_t n, void* ws) {
  char* p = static_cast<char*>(ws);
  const size_t rb = rows_bytes(d, n);
  return BwdWorkspace{reinterpret_cast<float*>(p), reinterpret_cast<float*>(p + rb),
                      reinterpret_cast<float*>(p + 2 * rb)};
}

// Spatial branch: split of the text key blocks' video query tiles into chunks of about one
// frame (at least kMinTextSpan tiles), so that no dK/dV workgroup visits every video tile.
constexpr int kMinTextSpan = 8;
constexpr int kMaxTextChunks = 64;
struct TextSplit {
  int blocks, chunks, span;
};
TextSplit text_split(const vc_jointattn_desc* d, int64_t n) {
  const int T = d->text_slot;
  const int blocks = (T + vcja::kDkdvKeys - 1) / vcja::kDkdvKeys;
  const int nvq = ntiles(n) - T / vcja::kTileTok;  // tiles holding video queries
  const int L = d->grid_h * d->grid_w;
  const int span = std::max((L + vcja::kTileTok - 1) / vcja::kTileTok + 1, kMinTextSpan);
  const int chunks = blocks ? std::min(kMaxTextChunks, (nvq + span - 1) / span) : 1;
  if (chunks < 2) return TextSplit{blocks, 1, nvq};
  return TextSplit{blocks, chunks, (nvq + chunks - 1) / chunks};
}
// fp32 partial dK and dV of the split text blocks.
size_t text_part_bytes(const vc_jointattn_desc* d, int64_t n) {
  const TextSplit t = text_split(d, n);
  if (t.chunks < 2) return 0;
  return align256((size_t)2 * t.chunks * d->batch * d->heads * t.blocks * vcja::kDkdvKeys * d->head_dim *
                  sizeof(float));
}
size_t spatial_bwd_ws_bytes(const vc_jointattn_desc* d, int64_t n) {
  return bwd_ws_bytes(d, n) + text_part_bytes(d, n);
}

vc_status check_ws(void* ws, size_t have, size_t need) {
  if (!ws) return VC_ERR_WORKSPACE;
  if ((reinterpret_cast<uintptr_t>(ws) & 255u) != 0) return VC_ERR_ALIGN;
  if (have < need) return VC_ERR_WORKSPACE;
  return VC_OK;
}

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

// Temporal branch arguments common to the forward and the backward.
vcja::TemporalArgs temporal_args(const vc_jointattn_desc* d, int64_t n) {
  vcja::TemporalArgs a{};
  a.B = d->batch;
  a.H = d->heads;
  a.N = (int)n;
  a.T = d->text_slot;
  a.F = d->frames;
  a.L = d->grid_h * d->grid_w;
  a.G = d->frames <= vcja::kMaxTemporalFramesShort ? 32 / d->frames : 1;
  a.npad = ntiles(n) * vcja::kTileTok;
  a.scale = d->softmax_scale > 0.0f ? d->softmax_scale : 1.0f / sqrtf((float)d->head_dim);
  a.scale_log2 = a.scale * vcja::kLog2e;
  return a;
}
inline const __bf16* bf(const void* p) { return static_cast<const __bf16*>(p); }

}  // namespace

extern "C" {

int vc_jointattn_abi_version(void) { return VC_JOINTATTN_ABI_VERSION; }

const char* vc_status_string(int status) {
  switch (status) {
    case VC_OK: return "ok";
    case VC_ERR_NULL: return "a required pointer is NULL";
    case VC_ERR_SHAPE: return "a size is out of range";
    case VC_ERR_HEAD_DIM: return "head_dim must be 64 or 128";
    case VC_ERR_ALIGN: return "a pointer is not sufficiently aligned";
    case VC_ERR_WORKSPACE: return "workspace missing or too small";
    case VC_ERR_DEVICE: return "no current HIP device, or it is not gfx950";
    case VC_ERR_HIP: return "a HIP kernel launch failed";
    case VC_ERR_UNSUPPORTED: return "requested mode is not available";
    case VC_ERR_ALIAS: return "an output is the same buffer as another output";
    case VC_ERR_SCRATCH:
      return "the problem needs more workspace than the no-allocation entry point's fixed scratch array holds";
    default: return "unknown status";
  }
}

int64_t vc_jointattn_tokens(const vc_jointattn_desc* desc) {
  int64_t n = 0;
  const vc_status st = check_desc(desc, &n);
  return st == VC_OK ? n : (int64_t)st;
}

size_t vc_jointattn_fwd_workspace_bytes(const vc_jointattn_desc* desc) {
  int64_t n = 0;
  if (check_desc(desc, &n) != VC_OK) return 0;
  return tiles_bytes(desc, n) + align256(queried_wgs(desc, n, {kSplitFwd}) * fwd_wg_bytes(desc->head_dim));
}

size_t vc_jointattn_bwd_workspace_bytes(const vc_jointattn_desc* desc) {
  int64_t n = 0;
  if (check_desc(desc, &n) != VC_OK) return 0;
  return bwd_ws_query_bytes(desc, n);
}

int64_t vc_jointattn_fused_dq_keys(const vc_jointattn_desc* desc) {
  int64_t n = 0;
  const vc_status st = check_desc(desc, &n);
  if (st != VC_OK) return (int64_t)st;
  return std::min<int64_t>(n, (int64_t)fused_dq_blocks(desc, n) * vcja::kDkdvKeys);
}

size_t vc_spatialattn_bwd_workspace_bytes(const vc_jointattn_desc* desc) {
  int64_t n = 0;
  if (check_desc(desc, &n) != VC_OK) return 0;
  return bwd_ws_query_bytes(desc, n) + text_part_bytes(desc, n);
}

}  // extern "C"

namespace {

vc_status prepare_impl(const vc_jointattn_desc* desc, const void* q, const void* k, const void* o, const float* lse,
                       const void* dout, void* workspace, size_t workspace_bytes, void* stream, bool zero_acc = false);

// Joint attention (frame_len 0) or the spatial branch (frame_len = tokens per frame).
vc_status fwd_impl(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v,
                   const int32_t* text_len, const uint8_t* key_mask, void* o, float* lse, void* workspace,
                   size_t workspace_bytes, void* stream, bool spatial) {
  int64_t n = 0;
  vc_status st = check_desc(desc, &n);
  if (st != VC_OK) return st;
  if (!q || !k || !v || !o || !lse) return VC_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(lse) || !aligned4(text_len))
    return VC_ERR_ALIGN;
  if ((st = check_ws(workspace, workspace_bytes, fwd_ws_bytes(desc, n))) != VC_OK) return st;
  if ((st = check_device()) != VC_OK) return st;
  vcja::FwdArgs a{};
  a.q = bf(q);
  a.k = bf(k);
  a.v = bf(v);
  a.text_len = text_len;
  a.key_mask = key_mask;
  a.o = static_cast<__bf16*>(o);
  a.lse = lse;
  a.B = desc->batch;
  a.H = desc->heads;
  a.N = (int)n;
  a.T = desc->text_slot;
  a.ntile = ntiles(n);
  a.frame_len = spatial ? desc->grid_h * desc->grid_w : 0;
  a.scale_log2 = scale_of(desc) * vcja::kLog2e;
  const TailPlan tp = spatial ? TailPlan{0, 1, 0} : fwd_plan(desc, n, device_cus(), workspace_bytes);
  a.tail_part = reinterpret_cast<float*>(static_cast<char*>(workspace) + tiles_bytes(desc, n));
  a.tail_blocks = tp.items;
  a.tail_chunks = tp.chunks;
  a.tail_span = tp.span;
  return vcja::launch_fwd(a, desc->head_dim, as_stream(stream)) == hipSuccess ? VC_OK : VC_ERR_HIP;
}

}  // namespace

extern "C" {

vc_status vc_jointattn_fwd(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v,
                           const int32_t* text_len, const uint8_t* key_mask, void* o, float* lse, void* workspace,
                           size_t workspace_bytes, void* stream) {
  return fwd_impl(desc, q, k, v, text_len, key_mask, o, lse, workspace, workspace_bytes, stream, false);
}

vc_status vc_jointattn_fwd_noalloc(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v,
                                   const int32_t* text_len, const uint8_t* key_mask, void* o, float* lse,
                                   void* stream) {
  int64_t n = 0;
  vc_status st = check_desc(desc, &n);
  if (st != VC_OK) return st;
  if (fwd_ws_bytes(desc, n) > VC_JOINTATTN_NOALLOC_SCRATCH_BYTES) return VC_ERR_SCRATCH;
  if ((st = check_device()) != VC_OK) return st;
  void* ws = scratch_ptr();
  if (!ws) return VC_ERR_HIP;
  return fwd_impl(desc, q, k, v, text_len, key_mask, o, lse, ws, VC_JOINTATTN_NOALLOC_SCRATCH_BYTES, stream,
                  false);
}

vc_status vc_spatialattn_fwd(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v,
                             const int32_t* text_len, const uint8_t* key_mask, void* o, float* lse, void* workspace,
                             size_t workspace_bytes, void* stream) {
  return fwd_impl(desc, q, k, v, text_len, key_mask, o, lse, workspace, workspace_bytes, stream, true);
}

vc_status vc_jointattn_bwd_prepare(const vc_jointattn_desc* desc, const void* q, const void* k, const void* o,
                                   const float* lse, const void* dout, void* workspace, size_t workspace_bytes,
                                   void* stream) {
  int64_t n = 0;
  const vc_status st = check_desc(desc, &n);
  if (st != VC_OK) return st;
  return prepare_impl(desc, q, k, o, lse, dout, workspace, workspace_bytes, stream);
}

}  // extern "C"

namespace {

// Backward stage 1; with zero_acc it also clears the fused pass's dQ accumulator.
vc_status prepare_impl(const vc_jointattn_desc* desc, const void* q, const void* k, const void* o, const float* lse,
                       const void* dout, void* workspace, size_t workspace_bytes, void* stream, bool zero_acc) {
  int64_t n = 0;
  vc_status st = check_desc(desc, &n);
  if (st != VC_OK) return st;
  if (!q || !k || !o || !lse || !dout) return VC_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(o) || !aligned16(lse) || !aligned16(dout)) return VC_ERR_ALIGN;
  if ((st = check_ws(workspace, workspace_bytes, bwd_ws_bytes(desc, n))) != VC_OK) return st;
  if ((st = check_device()) != VC_OK) return st;
  const BwdWorkspace w = split_bwd_ws(desc, n, workspace);
  const int B = desc->batch, H = desc->heads, D = desc->head_dim, N = (int)n;
  hipStream_t s = as_stream(stream);
  if (vcja::launch_bwd_prepare(bf(o), lse, bf(dout), w.dd, w.nls, B, H, N, ntiles(n) * vcja::kTileTok, D, prob_scale_of(desc).c,
                               zero_acc ? w.dq_acc : nullptr, s) != hipSuccess)
    return VC_ERR_HIP;
  return VC_OK;
}

vc_status dkdv_impl(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v, const void* dout,
                    const int32_t* text_len, const uint8_t* key_mask, void* dk, void* dv, void* workspace,
                    size_t workspace_bytes, void* stream, bool spatial, bool fused = false,
                    bool staged = false, bool zero_acc = true, bool every_key = false) {
  int64_t n = 0;
  vc_status st = check_desc(desc, &n);
  if (st != VC_OK) return st;
  if (!q || !k || !v || !dout || !dk || !dv) return VC_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(dout) || !aligned16(dk) || !aligned16(dv) ||
      !aligned4(text_len))
    return VC_ERR_ALIGN;
  if ((st = check_ws(workspace, workspace_bytes, spatial ? spatial_bwd_ws_bytes(desc, n) : bwd_ws_bytes(desc, n))) !=
      VC_OK)
    return st;
  if ((st = check_device()) != VC_OK) return st;
  // The separate stage 2 belongs to the deterministic backward; with the flag off it stays refused,
  // as stage 3 would then look for an accumulator that it does not fill.
  if (staged && !desc->deterministic) return VC_ERR_UNSUPPORTED;
  const BwdWorkspace w = split_bwd_ws(desc, n, workspace);
  vcja::DkdvArgs a{};
  const TextSplit ts = spatial ? text_split(desc, n) : TextSplit{0, 1, 0};
  a.text_part = reinterpret_cast<float*>(static_cast<char*>(workspace) + bwd_ws_bytes(desc, n));
  a.text_blocks = ts.blocks;
  a.text_chunks = ts.chunks;
  a.text_span = ts.span;
  const TailPlan tp = spatial ? TailPlan{0, 1, 0} : bwd_plan(desc, n, device_cus(), kSplitDkdv, 0, workspace_bytes);
  a.tail_part = tail_part_of(desc, n, workspace);
  a.tail_blocks = tp.items;
  a.tail_chunks = tp.chunks;
  a.tail_span = tp.span;
  a.q = bf(q);
  a.k = bf(k);
  a.v = bf(v);
  a.dout = bf(dout);
  a.nls = w.nls;
  a.dd = w.dd;
  a.text_len = text_len;
  a.key_mask = key_mask;
  a.dk = static_cast<__bf16*>(dk);
  a.dv = static_cast<__bf16*>(dv);
  a.dq_acc = fused ? w.dq_acc : nullptr;
  a.zero_acc = zero_acc;
  a.dq_blocks = !fused ? 0 : spatial || every_key ? std::numeric_limits<int>::max() : fused_dq_blocks(desc, n);
  a.B = desc->batch;
  a.H = desc->heads;
  a.N = (int)n;
  a.T = desc->text_slot;
  a.ntile = ntiles(n);
  a.frame_len = spatial ? desc->grid_h * desc->grid_w : 0;
  a.scale = scale_of(desc);
  const ProbScale ps = prob_scale_of(desc);
  a.scale_log2 = ps.c * vcja::kLog2e;
  a.score_down = ps.down;
  return vcja::launch_bwd_dkdv(a, desc->head_dim, as_stream(stream)) == hipSuccess ? VC_OK : VC_ERR_HIP;
}

vc_status dq_impl(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v, const void* dout,
                  const int32_t* text_len, const uint8_t* key_mask, void* dq, void* workspace,
                  size_t workspace_bytes, void* stream, bool spatial, bool fused = false, bool every_key = false) {
  int64_t n = 0;
  vc_status st = check_desc(desc, &n);
  if (st != VC_OK) return st;
  if (!q || !k || !v || !dout || !dq) return VC_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(dout) || !aligned16(dq) || !aligned4(text_len))
    return VC_ERR_ALIGN;
  if ((st = check_ws(workspace, workspace_bytes, bwd_ws_bytes(desc, n))) != VC_OK) return st;
  if ((st = check_device()) != VC_OK) return st;
  const BwdWorkspace w = split_bwd_ws(desc, n, workspace);
  vcja::DqArgs a{};
  // Completing a fused backward: the key tiles of the blocks that did not add their dQ
  // share, plus the accumulator the others filled; when every block added its share, the
  // accumulator alone, scaled and rounded.
  if (fused) {
    if (spatial || every_key || all_keys_fused(desc, n)) {  // spatial: text rows are not queries, their dq is zero
      const size_t tok = (size_t)desc->heads * desc->head_dim;
      return vcja::launch_dq_from_acc(w.dq_acc, static_cast<__bf16*>(dq), desc->batch, n * tok,
                                      spatial ? desc->text_slot * tok : 0, scale_of(desc),
                                      as_stream(stream)) == hipSuccess
                 ? VC_OK
                 : VC_ERR_HIP;
    }
    a.kt_min = fused_dq_blocks(desc, n) * (vcja::kDkdvKeys / vcja::kTileTok);
    a.dq_acc = w.dq_acc;
  }
  a.q = bf(q);
  a.k = bf(k);
  a.v = bf(v);
  a.dout = bf(dout);
  a.nls = w.nls;
  a.dd = w.dd;
  a.text_len = text_len;
  a.key_mask = key_mask;
  a.dq = static_cast<__bf16*>(dq);
  const TailPlan tp = spatial ? TailPlan{0, 1, 0} : bwd_plan(desc, n, device_cus(), kSplitDq, a.kt_min, workspace_bytes);
  a.tail_part = tail_part_of(desc, n, workspace);
  a.tail_blocks = tp.items;
  a.tail_chunks = tp.chunks;
  a.tail_span = tp.span;
  a.B = desc->batch;
  a.H = desc->heads;
  a.N = (int)n;
  a.T = desc->text_slot;
  a.ntile = ntiles(n);
  a.frame_len = spatial ? desc->grid_h * desc->grid_w : 0;
  a.scale = scale_of(desc);
  a.scale_log2 = a.scale * vcja::kLog2e;
  a.nls_log2 = prob_scale_of(desc).c * vcja::kLog2e;
  return vcja::launch_bwd_dq(a, desc->head_dim, as_stream(stream)) == hipSuccess ? VC_OK : VC_ERR_HIP;
}

vc_status bwd_impl(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v, const void* o,
                   const float* lse, const void* dout, const int32_t* text_len, const uint8_t* key_mask, void* dq,
                   void* dk, void* dv, void* workspace, size_t workspace_bytes, void* stream, bool spatial) {
  int64_t n = 0;
  vc_status st = check_desc(desc, &n);
  if (st != VC_OK) return st;
  if (!q || !k || !v || !o || !lse || !dout || !dq || !dk || !dv) return VC_ERR_NULL;
  if (spatial && (st = check_ws(workspace, workspace_bytes, spatial_bwd_ws_bytes(desc, n))) != VC_OK) return st;
  // dQ fused into the key-stationary kernel (atomics) unless the caller asks for bitwise
  // reproducible results: joint attention for its leading key blocks (the dQ pass covers
  // the others), the spatial branch, where it fuses, for every key block;
  // neither for samples of 2^32 elements or more.
  if (!desc->deterministic && (spatial ? spatial_fused(desc, n, key_mask != nullptr) : fused_dq_blocks(desc, n) > 0)) {
    if ((st = prepare_impl(desc, q, k, o, lse, dout, workspace, workspace_bytes, stream, true)) != VC_OK ||
        (st = dkdv_impl(desc, q, k, v, dout, text_len, key_mask, dk, dv, workspace, workspace_bytes, stream,
                        spatial, true, false, false, fuse_every_key(desc, n))) != VC_OK)
      return st;
    return dq_impl(desc, q, k, v, dout, text_len, key_mask, dq, workspace, workspace_bytes, stream, spatial, true,
                   fuse_every_key(desc, n));
  }
  if ((st = prepare_impl(desc, q, k, o, lse, dout, workspace, workspace_bytes, stream)) != VC_OK)
    return st;
  if ((st = dkdv_impl(desc, q, k, v, dout, text_len, key_mask, dk, dv, workspace, workspace_bytes, stream,
                      spatial)) != VC_OK)
    return st;
  return dq_impl(desc, q, k, v, dout, text_len, key_mask, dq, workspace, workspace_bytes, stream, spatial);
}

}  // namespace

extern "C" {

vc_status vc_jointattn_bwd_dkdv(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v,
                                const void* dout, const int32_t* text_len, const uint8_t* key_mask, void* dk,
                                void* dv, void* workspace, size_t workspace_bytes, void* stream) {
  return dkdv_impl(desc, q, k, v, dout, text_len, key_mask, dk, dv, workspace, workspace_bytes, stream, false,
                   false, true);
}

vc_status vc_jointattn_bwd_dq(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v,
                              const void* dout, const int32_t* text_len, const uint8_t* key_mask, void* dq,
                              void* workspace, size_t workspace_bytes, void* stream) {
  return dq_impl(desc, q, k, v, dout, text_len, key_mask, dq, workspace, workspace_bytes, stream, false,
                 desc && !desc->deterministic);
}

vc_status vc_jointattn_bwd_fused(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v,
                                 const void* dout, const int32_t* text_len, const uint8_t* key_mask, void* dk,
                                 void* dv, void* workspace, size_t workspace_bytes, void* stream) {
  return dkdv_impl(desc, q, k, v, dout, text_len, key_mask, dk, dv, workspace, workspace_bytes, stream, false, true);
}

vc_status vc_jointattn_bwd(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v, const void* o,
                           const float* lse, const void* dout, const int32_t* text_len, const uint8_t* key_mask,
                           void* dq, void* dk, void* dv, void* workspace, size_t workspace_bytes, void* stream) {
  return bwd_impl(desc, q, k, v, o, lse, dout, text_len, key_mask, dq, dk, dv, workspace, workspace_bytes, stream,
                  false);
}

vc_status vc_spatialattn_bwd(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v,
                             const void* o, const float* lse, const void* dout, const int32_t* text_len,
                             const uint8_t* key_mask, void* dq, void* dk, void* dv, void* workspace,
                             size_t workspace_bytes, void* stream) {
  return bwd_impl(desc, q, k, v, o, lse, dout, text_len, key_mask, dq, dk, dv, workspace, workspace_bytes, stream,
                  true);
}

}  // extern "C"

namespace {

// Temporal forward; with `out`, also the branch sum out = o_joint + o_spatial + o.
vc_status temporal_fwd_impl(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v,
                            const uint8_t* key_mask, const void* o_joint, const void* o_spatial, void* o, float* lse,
                            void* out, void* stream) {
  int64_t n = 0;
  vc_status st = check_desc(desc, &n);
  if (st != VC_OK) return st;
  if (desc->frames > vcja::kMaxTemporalFramesLong) return VC_ERR_SHAPE;
  if (!q || !k || !v || !o || !lse) return VC_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(lse) || !aligned16(o_joint) ||
      !aligned16(o_spatial) || !aligned16(out))
    return VC_ERR_ALIGN;
  if (out && out == o) return VC_ERR_ALIAS;
  if ((st = check_device()) != VC_OK) return st;
  vcja::TemporalArgs a = temporal_args(desc, n);
  a.q = bf(q);
  a.k = bf(k);
  a.v = bf(v);
  a.key_mask = key_mask;
  a.o = static_cast<__bf16*>(o);
  a.lse = lse;
  a.sum_a = bf(o_joint);
  a.sum_b = bf(o_spatial);
  a.sum_out = static_cast<__bf16*>(out);
  hipStream_t s = as_stream(stream);
  const hipError_t e = desc->frames > vcja::kMaxTemporalFramesShort
                          ? vcja::launch_temporal_long_fwd(a, desc->head_dim, device_cus(), s)
                          : vcja::launch_temporal_fwd(a, desc->head_dim, s);
  return e == hipSuccess ? VC_OK : VC_ERR_HIP;
}

}  // namespace

extern "C" {

vc_status vc_temporalattn_fwd(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v,
                              const uint8_t* key_mask, void* o, float* lse, void* stream) {
  return temporal_fwd_impl(desc, q, k, v, key_mask, nullptr, nullptr, o, lse, nullptr, stream);
}

vc_status vc_temporalattn_fwd_sum(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v,
                                  const uint8_t* key_mask, const void* o_joint, const void* o_spatial, void* o,
                                  float* lse, void* out, void* stream) {
  if (!out) return VC_ERR_NULL;
  return temporal_fwd_impl(desc, q, k, v, key_mask, o_joint, o_spatial, o, lse, out, stream);
}

vc_status vc_branchsum(const vc_jointattn_desc* desc, const void* o_joint, const void* o_spatial,
                       const void* o_temporal, void* out, void* stream) {
  int64_t n = 0;
  vc_status st = check_desc(desc, &n);
  if (st != VC_OK) return st;
  if (!out || (!o_joint && !o_spatial && !o_temporal)) return VC_ERR_NULL;
  if (!aligned16(o_joint) || !aligned16(o_spatial) || !aligned16(o_temporal) || !aligned16(out)) return VC_ERR_ALIGN;
  if ((st = check_device()) != VC_OK) return st;
  const int rows = (int)n;
  return vcja::launch_branch_sum(bf(o_joint), bf(o_spatial), bf(o_temporal), static_cast<__bf16*>(out),
                                 desc->batch, rows, rows, desc->heads * desc->head_dim, as_stream(stream)) == hipSuccess
             ? VC_OK
             : VC_ERR_HIP;
}

size_t vc_temporalattn_bwd_workspace_bytes(const vc_jointattn_desc* desc) {
  int64_t n = 0;
  if (check_desc(desc, &n) != VC_OK) return 0;
  return 2 * rows_bytes(desc, n);
}

vc_status vc_temporalattn_bwd(const vc_jointattn_desc* desc, const void* q, const void* k, const void* v,
                              const void* o, const float* lse, const void* dout, const uint8_t* key_mask, void* dq,
                              void* dk, void* dv, void* /*workspace*/, size_t /*workspace_bytes*/,
                              void* stream) {
  int64_t n = 0;
  vc_status st = check_desc(desc, &n);
  if (st != VC_OK) return st;
  if (desc->frames > vcja::kMaxTemporalFramesLong) return VC_ERR_SHAPE;
  if (!q || !k || !v || !o || !lse || !dout || !dq || !dk || !dv) return VC_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(lse) || !aligned16(dout) ||
      !aligned16(dq) || !aligned16(dk) || !aligned16(dv))
    return VC_ERR_ALIGN;
  const bool long_clip = desc->frames > vcja::kMaxTemporalFramesShort;
  if ((st = check_device()) != VC_OK) return st;
  vcja::TemporalArgs a = temporal_args(desc, n);
  a.q = bf(q);
  a.k = bf(k);
  a.v = bf(v);
  a.dout = bf(dout);
  a.key_mask = key_mask;
  a.o = static_cast<__bf16*>(dq);
  a.dk = static_cast<__bf16*>(dk);
  a.dv = static_cast<__bf16*>(dv);
  hipStream_t s = as_stream(stream);
  // -D and LSE*log2(e) are formed inside the kernels from o and lse: no workspace.
  a.lse = const_cast<float*>(lse);
  a.o_in = bf(o);
  if (long_clip)
    return vcja::launch_temporal_long_bwd(a, desc->head_dim, device_cus(), s) == hipSuccess ? VC_OK : VC_ERR_HIP;
  return vcja::launch_temporal_bwd(a, desc->head_dim, s) == hipSuccess ? VC_OK : VC_ERR_HIP;
}

}  // extern "C"
