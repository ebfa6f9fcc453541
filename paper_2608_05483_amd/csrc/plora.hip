// plora.hip -- host side and C ABI of the gfx950 batched heterogeneous-
// adapter LoRA apply (declared in include/plora.h).
//
// What runs where:
//   plora_segment  one work group.  Up to 1024 tokens: one thread per token
//                  ranks its (adapter id, token index) key by counting the
//                  keys before it in LDS.  Larger batches: LSD radix sort of
//                  packed keys in LDS with ballot-based stable ranking per
//                  wavefront.  Both then write the segment and tile lists.
//   plora_shrink   one work group per work item: one tile (up to
//   plora_expand   PLORA_TILE_TOKENS tokens of one adapter, section VI-B's
//   plora_apply    per-adapter batch B_i split into tiles) and one slice of
//                  h_in or of the y columns: the kernels of plora_small.h for
//                  batches of up to kFusedTokens tokens, those of plora_dev.h
//                  above.
#include "plora_small.h"

#include <mutex>

namespace plora_impl {
namespace {
// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline int ceil_log2(int64_t v) {
  int b = 0;
  while ((int64_t(1) << b) < v) ++b;
  return b;
}

// Every rank from 0 (a no-op adapter) to max_rank is applied.
inline bool usable_rank(int r, int max_rank) { return r >= 0 && r <= max_rank; }

// Compute units of the current device, queried once per device.
int cu_count() {
  static std::atomic<int> cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 256;
  if (dev < 64) {
    const int c = cache[dev].load();
    if (c > 0) return c;
  }
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      n <= 0)
    n = 256;
  if (dev < 64) cache[dev].store(n);
  return n;
}

// Apply work groups that one compute unit holds at once, as its LDS allows:
// the dynamic section for this h_in and max_rank with slack for the
// allocation granularity; at most kWGPerCU.  At max_rank 128 (82 KB dynamic) that is one.
int wg_per_cu(int32_t h_in, int32_t max_rank) {
  const size_t per = smem_bytes(h_in, max_rank) + 1024;
  return std::max(1, std::min<int>(kWGPerCU, (int)(kMaxLds / per)));
}

// Resident apply work groups of the device at this h_in and max_rank.
int slots_for_device(int32_t h_in, int32_t max_rank) {
  return std::max(8, cu_count() * wg_per_cu(h_in, max_rank));
}

// One work group per item: the most items make_plan can produce for any tile
// count up to tile_cap with at most s_max slices per tile (see there).
unsigned grid_for(const ApplyArgs& g, int s_max) {
  const int64_t cap8 = (g.tile_cap + 7) & ~7;
  if (s_max <= 1) return (unsigned)std::max<int64_t>(8, cap8);
  // fit = round(kPlanItems slots / n8) >= 2 needs n8 <= 2/3 kPlanItems slots,
  // so n8 fit <= 4/3 kPlanItems slots
  const int64_t spread = ((int64_t)kPlanItems * g.slots * 4 / 3 + 8 + 7) & ~7;
  return (unsigned)std::max<int64_t>(8, std::min(cap8 * s_max, std::max(cap8, spread)));
}

// Most h_in slices per tile: slices of at least 512 rows, at most 8.
int ks_max_for(int h_in) { return std::max(1, std::min(8, h_in / 512)); }

// plora_apply runs as one launch for batches of up to kFusedTokens tokens.
bool fused_for(int32_t T) { return T <= kFusedTokens; }

// Most slices of a tile (h_in and the columns alike): slices of at least 512
// rows and columns, at most 8.
int slice_limit(int32_t h_in, int32_t h_out) {
  return std::min(ks_max_for(h_in), std::max(1, h_out / kMinSlice));
}

// Workspace sections, each 256-byte aligned: the epochs of the exchange's
// tile slots (64-bit, kXSlots of them) and the counters; the readiness words
// of the one-launch two-part form (kReadyTiles); the exchange regions of the
// one-launch form (kSlotWords 64-bit words for each of the first
// min(cap8, kXSlots) tile slots); then the partial sums of v of the
// two-part forms and plora_shrink (fp32 [ks_max][T][max_rank]).  The epochs,
// the readiness words and each slot's region sit at the same offsets for
// every batch size, rank and slice count, which their tags rely on (no
// other section ever writes there); only the last section's place and size
// follow the shapes.
struct WsLayout {
  size_t xep, counters, ready, xw, vpart, total;
};

// Workspace bytes of the multi-work-group segmentation (batches above 1024
// tokens over 2048 to 8191 adapters: a table of (ceil(T / 1024) + 1) x
// (N + 2) int32, the groups' counts and the keys' first positions); 0 where
// plora_segment takes a one-work-group kernel (fewer adapters: the counting
// sort of kCountKeys keys; more: the radix sort).
size_t segment_scratch_bytes(int32_t T, int32_t N) {
  if (T <= 1024 || N < 0 || N + 1 <= kCountKeys || N + 1 > 8192) return 0;
  const size_t groups = ((size_t)T + 1023) / 1024;
  return (((groups + 1) * (size_t)(N + 2) * sizeof(int32_t)) + 255) & ~(size_t)255;
}

constexpr int kCounters = 2;   // workspace counters after the epochs (see ApplyArgs)
// Readiness words of the one-launch two-part form (one per tile slot); a
// batch whose tile capacity exceeds it takes two launches.
constexpr int32_t kReadyTiles = 4096;

constexpr size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// n adapter stacks (the projections of plora_apply_multi; n = 1 otherwise)
// sharing the batch: n cap8 tile slots, and the largest partial-sum section.
WsLayout ws_layout(int32_t T, const plora_adapters* ad, int n = 1) {
  WsLayout l{0, 0, 0, 0, 0, 0};
  if (!ad || T <= 0 || n < 1) return l;
  size_t nvp = 0;
  for (int p = 0; p < n; ++p) {
    if (ad[p].h_in <= 0 || ad[p].max_rank <= 0) return l;
    nvp = std::max(nvp, (size_t)ks_max_for(ad[p].h_in) * T * ad[p].max_rank * sizeof(float));
  }
  // the last section also serves plora_segment_apply's segmentation, which
  // runs before the partial sums are written
  nvp = std::max(nvp, segment_scratch_bytes(T, ad->n_adapters));
  const int32_t tcap = plora_tile_capacity(T, ad->n_adapters);
  const size_t slots = (size_t)std::min(kXSlots, std::max(8, n * ((tcap + 7) & ~7)));
  l.xep = 0;
  l.counters = (size_t)kXSlots * sizeof(uint64_t);
  l.ready = align256(l.counters + kCounters * sizeof(uint64_t));
  l.xw = align256(l.ready + kReadyTiles * sizeof(uint64_t));
  l.vpart = align256(l.xw + slots * kSlotWords * sizeof(uint64_t));
  l.total = align256(l.vpart + nvp);
  return l;
}

size_t workspace_bytes(int32_t T, const plora_adapters* ad) { return ws_layout(T, ad).total; }

plora_status check_adapters_host(const plora_adapters* ad) {
  if (!ad) return PLORA_ERR_INVALID_ARG;
  if (ad->n_adapters < 0 || ad->h_in <= 0 || ad->h_out <= 0 || ad->max_rank < 0 ||
      ad->a_len < 0 || ad->b_len < 0 || ad->a_pool_len < 0 || ad->b_pool_len < 0)
    return PLORA_ERR_INVALID_ARG;
  if ((ad->h_in & 7) || (ad->h_out & 7)) return PLORA_ERR_UNSUPPORTED;
  // adapter blocks are read through 32-bit byte offsets
  if ((int64_t)std::max(ad->h_in, ad->h_out) * std::max(ad->max_rank, 0) * 2 >= (INT64_C(1) << 31))
    return PLORA_ERR_UNSUPPORTED;
  if (ad->max_rank == 0 || (ad->max_rank & 7) || ad->max_rank > PLORA_MAX_RANK)
    return PLORA_ERR_UNSUPPORTED;
  if (smem_bytes(ad->h_in, ad->max_rank) > kMaxLds) return PLORA_ERR_UNSUPPORTED;
  if (ad->n_adapters > 0 &&
      ((!ad->A && !ad->A_pool) || (!ad->B && !ad->B_pool) || !ad->a_off || !ad->b_off ||
       !ad->ranks || !ad->scales))
    return PLORA_ERR_INVALID_ARG;
  if (!aligned16(ad->A) || !aligned16(ad->B) || !aligned16(ad->a_off) ||
      !aligned16(ad->b_off) || !aligned16(ad->ranks) || !aligned16(ad->scales) ||
      !aligned16(ad->A_pool) || !aligned16(ad->B_pool))
    return PLORA_ERR_UNSUPPORTED;
  return PLORA_OK;
}

// Host mirror of adapter_block: whether offset o names an n-element block
// inside the device stack (o >= 0) or the pool (o < 0).
bool block_ok(const uint16_t* dev, int64_t dev_len, const uint16_t* pool, int64_t pool_len,
              int64_t o, int64_t n) {
  const bool in_pool = o < 0;
  const int64_t e = in_pool ? -1 - o : o;
  return (in_pool ? pool : dev) && (e & 7) == 0 && e + n <= (in_pool ? pool_len : dev_len);
}

plora_status check_segments_host(const plora_segments* seg, int32_t N) {
  if (!seg) return PLORA_ERR_INVALID_ARG;
  if (seg->T < 0) return PLORA_ERR_INVALID_ARG;
  if (seg->T > PLORA_MAX_TOKENS) return PLORA_ERR_UNSUPPORTED;
  if (seg->cap != std::min(seg->T, N) || seg->tile_cap != plora_tile_capacity(seg->T, N))
    return PLORA_ERR_INVALID_ARG;
  if (seg->T == 0) return PLORA_OK;
  if (!seg->perm || !seg->seg_ptr || !seg->seg_id || !seg->meta || !seg->tiles)
    return PLORA_ERR_INVALID_ARG;
  if (!aligned16(seg->tiles) || !aligned16(seg->perm)) return PLORA_ERR_UNSUPPORTED;
  return PLORA_OK;
}

// The status of a call reports its own launch: an error left pending by
// earlier HIP calls of the caller is cleared before launching.
void clear_stale_error() { (void)hipGetLastError(); }

std::atomic<int32_t> g_last_hip_error{0};
std::atomic<int32_t> g_exchange_polls{kSpinLimit};

plora_status launch_status() {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return PLORA_OK;
  g_last_hip_error.store((int32_t)e);
  return PLORA_ERR_HIP;
}

plora_status prepare(const plora_adapters* ad, const plora_segments* seg, void* ws,
                     size_t ws_bytes, ApplyArgs& g, bool needs_ws) {
  plora_status st = check_adapters_host(ad);
  if (st != PLORA_OK) return st;
  st = check_segments_host(seg, ad->n_adapters);
  if (st != PLORA_OK) return st;
  memset(&g, 0, sizeof g);
  g.A = ad->A; g.B = ad->B; g.a_len = ad->a_len; g.b_len = ad->b_len;
  g.A_pool = ad->A_pool; g.B_pool = ad->B_pool;
  g.a_pool_len = ad->a_pool_len; g.b_pool_len = ad->b_pool_len;
  g.a_off = ad->a_off; g.b_off = ad->b_off; g.ranks = ad->ranks; g.scales = ad->scales;
  g.perm = seg->perm;
  g.tiles = reinterpret_cast<const int4*>(seg->tiles);
  g.meta = seg->meta;
  g.T = seg->T; g.N = ad->n_adapters; g.h_in = ad->h_in; g.h_out = ad->h_out;
  g.max_rank = ad->max_rank; g.tile_cap = seg->tile_cap;
  g.js_max = std::max(1, ad->h_out / kMinSlice);
  g.slots = slots_for_device(ad->h_in, ad->max_rank);
  g.polls = g_exchange_polls.load();
  g.ks_max = ks_max_for(ad->h_in);
  g.count_skips = 1;
  if (needs_ws && seg->T > 0) {
    const WsLayout l = ws_layout(seg->T, ad);
    if (!ws) return PLORA_ERR_INVALID_ARG;
    if (!aligned16(ws)) return PLORA_ERR_UNSUPPORTED;
    if (ws_bytes < l.total) return PLORA_ERR_WORKSPACE_TOO_SMALL;
    char* base = reinterpret_cast<char*>(ws);
    g.vpart = reinterpret_cast<float*>(base + l.vpart);
    g.xw = reinterpret_cast<uint64_t*>(base + l.xw);
    g.xep = reinterpret_cast<uint64_t*>(base + l.xep);
    g.counters = reinterpret_cast<unsigned long long*>(base + l.counters);
    g.ready = reinterpret_cast<uint64_t*>(base + l.ready);
  } else if (ws && aligned16(ws) && ws_bytes >= ws_layout(1, ad).xw) {
    // a call that needs no workspace still counts into one it is given
    g.counters = reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(ws) +
                                                       ws_layout(1, ad).counters);
  }
  return PLORA_OK;
}

// How a small batch's launch is split, from its tile slots (all projections'
// of them): every slot in S slices that exchange partial v, as many as give
// kSmallTarget work groups of kST threads, three of which a compute unit
// holds (7B-shaped decode steps of 64 tokens at rank 16: 121 us for 768, 130
// for 640, 148 for 1024).  A slice of at least kDeepBytes of A_i streams
// longer than its chain of latencies: its kernels keep twice the chunks in
// flight, two work groups per compute unit, and it is better not split
// further (256 tokens at rank 64: 182 us per step, 192 split in three).  With
// one slice (h_in, or the narrowest output of the launch, below 1024) a work
// group computes its tile's v whole.  The kernels stage a slice's x in LDS, so h_in above kSXW
// sets the fewest slices; slices longer than that (h_in above 8 kSXW) are deep,
// since max_rank is at least 8, and the deep kernels go on window by window.
// (The slots are at most kXSlots: a batch this small has at most 256 tiles, and
// plora_apply_multi sees to its sum.)
constexpr int kSmallTarget = 768, kDeepTarget = 512;
constexpr int64_t kDeepBytes = 128 * 1024;

struct SmallPlan {
  int S, J;        // h_in slices, column slices (as many where S > 1)
  int gl, slots;   // slots per group of the numbering (log2), slots of the launch
  int deep;
};

SmallPlan small_plan(int cap, int32_t h_in, int32_t h_out, int32_t max_rank) {
  SmallPlan p;
  p.gl = cap <= 1 ? 0 : cap <= 2 ? 1 : cap <= 4 ? 2 : 3;
  p.slots = (cap + (1 << p.gl) - 1) >> p.gl << p.gl;
  const int s_min = std::min<int>(kMaxSlices, (h_in + kSXW - 1) / kSXW);
  auto slices = [&](int target) {
    return std::max(s_min, std::min(slice_limit(h_in, h_out), (target + p.slots / 2) / p.slots));
  };
  p.S = std::max(1, slices(kSmallTarget));
  p.deep = (int64_t)h_in * max_rank * 2 / p.S > kDeepBytes;
  if (p.deep) p.S = std::max(1, slices(kDeepTarget));
  // Fewer slices, by at most half, where that gives whole ones: rows that are
  // whole batches of every thread at ranks that are powers of two, and a power
  // of two of column octets, so that no thread of the expand is idle (100
  // tokens, h = 4096: 7 slices of 640 columns leave 48 of 128 octets' threads
  // idle).  us a call, whole and uneven slices, formerly: 100 tokens at rank 8
  // 10.3 (4), 12.2 (7), 11.0; at 16 12.1, 13.6, 14.9; at 32 15.7, 18.0, 17.5;
  // 256 tokens at rank 16 16.7 (2), 18.8 (3), 18.0.  Low ranks only: longer
  // slices of mixed ranks wait for the longest (256 tokens of ranks 8 to 32, a
  // step of four layers 352 in 2 and 341 in 3; 100 tokens of ranks 8 to 64, two
  // layers 127 and 124), and other ranks have no whole batches (256 tokens of
  // ranks 4 to 40 22.4 and 21.3).  Not where the slices are the most there may
  // be: those batches have too few work groups as it is.
  if (max_rank <= (p.S > 5 ? 32 : 16) && (max_rank & (max_rank - 1)) == 0 && !p.deep &&
      p.S < slice_limit(h_in, h_out)) {
    for (int q = p.S; q >= std::max(2, std::max(s_min, (p.S + 1) / 2)); --q) {
      const int oct = h_out / (8 * q);
      if (h_in % (256 * q) == 0 && h_out % (64 * q) == 0 && (oct & (oct - 1)) == 0) {
        p.S = q;
        break;
      }
    }
  }
  // one slice of h_in: the work groups of a tile's column slices each compute
  // v whole (5 tokens, 792 -> 4512, rank 64: 12.5 us, 21.5 undivided)
  p.J = p.S > 1 ? p.S : std::max(1, std::min(h_out / kMinSlice, kSmallTarget / p.slots));
  return p;
}

// plora_segment_apply runs as one launch for batches of up to kSegApplyMax
// tokens whose tiles can be split: at most 256 slots, so small_plan then takes
// two slices or more, and its kernels always exchange (words (key << tbits) | t with key <= N + 1
// and tbits 6 up to 64 tokens, 8 above; tokens without an adapter read
// adapter 0's metadata, so N >= 1).
bool segment_apply_one_launch(int32_t T, const plora_adapters* ad) {
  const int32_t n_limit = T <= 64 ? (1 << 26) - 1 : (1 << 24) - 1;
  return T <= kSegApplyMax && ad->n_adapters > 0 && ad->n_adapters < n_limit &&
         slice_limit(ad->h_in, ad->h_out) > 1;
}

typedef void (*ItemLauncher)(const ApplyArgs&, unsigned, size_t, hipStream_t);

plora_status launch_items(ItemLauncher launch, const ApplyArgs& g, int s_max,
                          hipStream_t stream) {
  const size_t lds = smem_bytes(g.h_in, g.max_rank);
  const unsigned grid = grid_for(g, s_max);
  clear_stale_error();
  launch(g, grid, lds, stream);
  return launch_status();
}

// ---------------------------------------------------------------------------
// the allocation-free entry point's scratch
// ---------------------------------------------------------------------------

// Largest batch plora_segment_apply_noalloc takes, and the workspace such a
// batch needs at most: the exchange regions of min(kXSlots, cap8) tile
// slots (cap8 <= kNoAllocTokens) and the partial sums of v for up to 8
// slices of h_in at rank 128, after the epochs, counters and readiness words.
constexpr int32_t kNoAllocTokens = 256;
constexpr size_t kScratchBytes =
    align256(align256(align256(align256((size_t)(kXSlots + kCounters) * sizeof(uint64_t)) +
                               (size_t)kReadyTiles * sizeof(uint64_t)) +
                      (size_t)std::min(kXSlots, kNoAllocTokens) * kSlotWords * sizeof(uint64_t)) +
             (size_t)8 * kNoAllocTokens * PLORA_MAX_RANK * sizeof(float));

// The device address of `scratch` on the current device, looked up once per
// device with that device current (each device holds its own copy of the
// array at its own address); null if the lookup fails.
void* scratch_for_device();

}  // namespace
}  // namespace plora_impl

// The workspace of plora_segment_apply_noalloc: one per device, zero from
// the module's load, then carrying the exchange's epochs from call to call as
// any workspace does.  Host code never uses this name as an address (it is a
// host-side stand-in); it takes the pointer scratch_for_device() returns.
static __device__ __align__(256) unsigned char scratch[plora_impl::kScratchBytes];

namespace plora_impl {
namespace {

std::mutex g_scratch_mu;
void* g_scratch_ptr[64];

void* scratch_for_device() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    (void)hipGetLastError();
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

}  // namespace
}  // namespace plora_impl

using namespace plora_impl;

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------

extern "C" {

int32_t plora_tile_capacity(int32_t T, int32_t n_adapters) {
  if (T <= 0) return 0;
  const int32_t cap = std::min(T, std::max(n_adapters, 0));
  return std::min(T, cap + T / tile_tokens(T));
}

size_t plora_workspace_bytes(int32_t T, const plora_adapters* ad) {
  return workspace_bytes(T, ad);
}

plora_status plora_workspace_init(void* ws, size_t ws_bytes, hipStream_t stream) {
  if (ws_bytes == 0) return PLORA_OK;
  if (!ws) return PLORA_ERR_INVALID_ARG;
  if (!aligned16(ws) || (ws_bytes & 15)) return PLORA_ERR_UNSUPPORTED;
  const size_t n16 = ws_bytes / 16;
  const unsigned blocks = (unsigned)std::min<size_t>((n16 + 255) / 256, 4096);
  clear_stale_error();
  launch_zero(reinterpret_cast<uint4*>(ws), n16, blocks, stream);
  return launch_status();
}

size_t plora_segment_workspace_bytes(int32_t T, int32_t n_adapters) {
  return segment_scratch_bytes(T, n_adapters);
}

plora_status plora_segment(const int32_t* idx, const plora_segments* seg, int32_t n_adapters,
                           void* ws, size_t ws_bytes, hipStream_t stream) {
  if (!seg || n_adapters < 0) return PLORA_ERR_INVALID_ARG;
  plora_status st = check_segments_host(seg, n_adapters);
  if (st != PLORA_OK) return st;
  const int32_t T = seg->T;
  if (T == 0) return PLORA_OK;
  if (!idx) return PLORA_ERR_INVALID_ARG;
  const int tbits = ceil_log2(T);
  const int key_bits = n_adapters > 0 ? 32 - __builtin_clz((unsigned)n_adapters) : 0;
  if (tbits + key_bits > 32) return PLORA_ERR_UNSUPPORTED;
  clear_stale_error();
  int4* tiles = reinterpret_cast<int4*>(seg->tiles);
  const size_t scratch = segment_scratch_bytes(T, n_adapters);
  if (scratch > 0 && ws && aligned16(ws) && ws_bytes >= scratch) {
    launch_segment_groups(idx, T, n_adapters, seg->cap, seg->tile_cap, seg->perm, seg->seg_ptr,
                          seg->seg_id, seg->meta, tiles, reinterpret_cast<int32_t*>(ws), stream);
  } else {
    launch_segment(idx, T, n_adapters, seg->cap, seg->tile_cap, tbits, key_bits, seg->perm,
                   seg->seg_ptr, seg->seg_id, seg->meta, tiles, stream);
  }
  return launch_status();
}

plora_status plora_shrink(const uint16_t* x, int64_t ldx, const plora_adapters* ad,
                          const plora_segments* seg, float* v, int64_t ldv, void* ws,
                          size_t ws_bytes, hipStream_t stream) {
  ApplyArgs g;
  plora_status st = prepare(ad, seg, ws, ws_bytes, g, true);
  if (st != PLORA_OK) return st;
  if (seg->T == 0) return PLORA_OK;
  if (!x || !v) return PLORA_ERR_INVALID_ARG;
  if (ldx < ad->h_in || ldv < ad->max_rank) return PLORA_ERR_INVALID_ARG;
  if ((ldx & 7) || (ldv & 3) || !aligned16(x) || !aligned16(v)) return PLORA_ERR_UNSUPPORTED;
  g.x = x; g.ldx = ldx; g.v = v; g.ldv = ldv;
  if (fused_for(seg->T)) {
    const SmallPlan p = small_plan(g.tile_cap, g.h_in, g.h_out, g.max_rank);
    clear_stale_error();
    launch_small_shrink(SmallArgs{g, p.S, p.J, p.gl, p.deep}, (unsigned)(p.slots * p.S), stream);
    return launch_status();
  }
  st = launch_items(launch_shrink_part, g, g.ks_max, stream);
  if (st != PLORA_OK) return st;
  clear_stale_error();
  launch_gather_v(g, (unsigned)g.tile_cap, stream);
  return launch_status();
}

plora_status plora_expand(const float* v, int64_t ldv, const plora_adapters* ad,
                          const plora_segments* seg, uint16_t* y, int64_t ldy, void* ws,
                          size_t ws_bytes, hipStream_t stream) {
  ApplyArgs g;
  plora_status st = prepare(ad, seg, ws, ws_bytes, g, false);
  if (st != PLORA_OK) return st;
  if (seg->T == 0) return PLORA_OK;
  if (!v || !y) return PLORA_ERR_INVALID_ARG;
  if (ldy < ad->h_out || ldv < ad->max_rank) return PLORA_ERR_INVALID_ARG;
  if ((ldy & 7) || (ldv & 3) || !aligned16(y) || !aligned16(v)) return PLORA_ERR_UNSUPPORTED;
  g.v = const_cast<float*>(v); g.ldv = ldv; g.y = y; g.ldy = ldy;
  if (fused_for(seg->T)) {
    const SmallPlan p = small_plan(g.tile_cap, g.h_in, g.h_out, g.max_rank);
    clear_stale_error();
    launch_small_expand(SmallArgs{g, p.S, p.J, p.gl, p.deep}, (unsigned)(p.slots * p.J), stream);
    return launch_status();
  }
  return launch_items(launch_expand_v, g, g.js_max, stream);
}

plora_status plora_apply(const uint16_t* x, int64_t ldx, const plora_adapters* ad,
                         const plora_segments* seg, uint16_t* y, int64_t ldy, void* ws,
                         size_t ws_bytes, hipStream_t stream) {
  ApplyArgs g;
  plora_status st = prepare(ad, seg, ws, ws_bytes, g, true);
  if (st != PLORA_OK) return st;
  if (seg->T == 0) return PLORA_OK;
  if (!x || !y) return PLORA_ERR_INVALID_ARG;
  if (ldx < ad->h_in || ldy < ad->h_out) return PLORA_ERR_INVALID_ARG;
  if ((ldx & 7) || (ldy & 7) || !aligned16(x) || !aligned16(y)) return PLORA_ERR_UNSUPPORTED;
  g.x = x; g.ldx = ldx; g.y = y; g.ldy = ldy;
  if (fused_for(seg->T)) {
    const SmallPlan p = small_plan(g.tile_cap, g.h_in, g.h_out, g.max_rank);
    clear_stale_error();
    launch_small_apply(SmallArgs{g, p.S, p.J, p.gl, p.deep}, (unsigned)(p.slots * p.J), stream);
    return launch_status();
  }
  if (g.tile_cap <= kReadyTiles) {
    clear_stale_error();
    launch_parts(g, grid_for(g, g.ks_max), grid_for(g, g.js_max),
                 smem_bytes(g.h_in, g.max_rank), stream);
    return launch_status();
  }
  ApplyArgs gs = g;
  gs.count_skips = 0;                 // the expand launch counts the call's skips
  st = launch_items(launch_shrink_part, gs, g.ks_max, stream);
  if (st != PLORA_OK) return st;
  return launch_items(launch_expand_parts, g, g.js_max, stream);
}

plora_status plora_segment_apply_noalloc(const int32_t* idx, const uint16_t* x, int64_t ldx,
                                         const plora_adapters* ad, const plora_segments* seg,
                                         uint16_t* y, int64_t ldy, hipStream_t stream) {
  if (!ad || !seg) return PLORA_ERR_INVALID_ARG;
  plora_status st = check_adapters_host(ad);
  if (st != PLORA_OK) return st;
  st = check_segments_host(seg, ad->n_adapters);
  if (st != PLORA_OK) return st;
  if (seg->T > kNoAllocTokens) return PLORA_ERR_UNSUPPORTED;
  if (seg->T == 0) return PLORA_OK;
  if (!idx || !x || !y) return PLORA_ERR_INVALID_ARG;
  if (ldx < ad->h_in || ldy < ad->h_out) return PLORA_ERR_INVALID_ARG;
  if ((ldx & 7) || (ldy & 7) || !aligned16(x) || !aligned16(y)) return PLORA_ERR_UNSUPPORTED;
  if (ws_layout(seg->T, ad).total > kScratchBytes) return PLORA_ERR_UNSUPPORTED;
  void* ws = scratch_for_device();
  if (!ws) {
    g_last_hip_error.store((int32_t)hipErrorInvalidSymbol);
    return PLORA_ERR_HIP;
  }
  return plora_segment_apply(idx, x, ldx, ad, seg, y, ldy, ws, kScratchBytes, stream);
}

int32_t plora_segment_apply_launches(int32_t T, const plora_adapters* ad) {
  if (T <= 0 || !ad || check_adapters_host(ad) != PLORA_OK) return 0;
  if (segment_apply_one_launch(T, ad)) return 1;
  return fused_for(T) || plora_tile_capacity(T, ad->n_adapters) <= kReadyTiles ? 2 : 3;
}

plora_status plora_segment_apply(const int32_t* idx, const uint16_t* x, int64_t ldx,
                                 const plora_adapters* ad, const plora_segments* seg,
                                 uint16_t* y, int64_t ldy, void* ws, size_t ws_bytes,
                                 hipStream_t stream) {
  ApplyArgs g;
  plora_status st = prepare(ad, seg, ws, ws_bytes, g, true);
  if (st != PLORA_OK) return st;
  const int32_t T = seg->T;
  if (T == 0) return PLORA_OK;
  if (!idx || !x || !y) return PLORA_ERR_INVALID_ARG;
  if (ldx < ad->h_in || ldy < ad->h_out) return PLORA_ERR_INVALID_ARG;
  if ((ldx & 7) || (ldy & 7) || !aligned16(x) || !aligned16(y)) return PLORA_ERR_UNSUPPORTED;
  if (!segment_apply_one_launch(T, ad)) {
    // the segmentation's scratch is the partial-sum section, free until the
    // apply that follows on the same stream
    const WsLayout l = ws_layout(T, ad);
    st = plora_segment(idx, seg, ad->n_adapters, reinterpret_cast<char*>(ws) + l.vpart,
                       ws_bytes - l.vpart, stream);
    if (st != PLORA_OK) return st;
    return plora_apply(x, ldx, ad, seg, y, ldy, ws, ws_bytes, stream);
  }
  g.x = x; g.ldx = ldx; g.y = y; g.ldy = ldy;
  const SegOut so{seg->perm, seg->seg_ptr, seg->seg_id, seg->meta,
                  reinterpret_cast<int4*>(seg->tiles), seg->cap, seg->tile_cap};
  const SmallPlan p = small_plan(g.tile_cap, g.h_in, g.h_out, g.max_rank);
  clear_stale_error();
  launch_small_segment_apply(SmallArgs{g, p.S, p.J, p.gl, p.deep}, idx, so, (unsigned)(p.slots * p.J + (T <= kDecodeTokens && !p.deep ? 1 : 0)),
                             stream);
  return launch_status();
}

size_t plora_workspace_bytes_multi(int32_t T, const plora_adapters* ads, int32_t n_proj) {
  if (!ads || n_proj < 1 || n_proj > PLORA_MAX_PROJECTIONS) return 0;
  return ws_layout(T, ads, n_proj).total;
}

plora_status plora_apply_multi(const uint16_t* x, int64_t ldx, const plora_adapters* ads,
                               int32_t n_proj, const plora_segments* seg,
                               uint16_t* const* ys, const int64_t* ldys, void* ws,
                               size_t ws_bytes, hipStream_t stream) {
  if (!ads || !ys || !ldys || n_proj < 1) return PLORA_ERR_INVALID_ARG;
  if (n_proj > PLORA_MAX_PROJECTIONS) return PLORA_ERR_UNSUPPORTED;
  for (int p = 0; p < n_proj; ++p) {
    const plora_status st = check_adapters_host(&ads[p]);
    if (st != PLORA_OK) return st;
    if (ads[p].n_adapters != ads[0].n_adapters || ads[p].h_in != ads[0].h_in)
      return PLORA_ERR_INVALID_ARG;
  }
  plora_status st = check_segments_host(seg, ads[0].n_adapters);
  if (st != PLORA_OK) return st;
  if (seg->T == 0) return PLORA_OK;
  if (!x || ldx < ads[0].h_in) return PLORA_ERR_INVALID_ARG;
  if ((ldx & 7) || !aligned16(x)) return PLORA_ERR_UNSUPPORTED;
  int max_rank = 0;
  for (int p = 0; p < n_proj; ++p) {
    if (!ys[p] || ldys[p] < ads[p].h_out) return PLORA_ERR_INVALID_ARG;
    if ((ldys[p] & 7) || !aligned16(ys[p])) return PLORA_ERR_UNSUPPORTED;
    max_rank = std::max(max_rank, ads[p].max_rank);
  }
  if (smem_bytes(ads[0].h_in, max_rank) > kMaxLds) return PLORA_ERR_UNSUPPORTED;
  const WsLayout l = ws_layout(seg->T, ads, n_proj);
  if (!ws) return PLORA_ERR_INVALID_ARG;
  if (!aligned16(ws)) return PLORA_ERR_UNSUPPORTED;
  if (ws_bytes < l.total) return PLORA_ERR_WORKSPACE_TOO_SMALL;
  const int cap = seg->tile_cap <= 8 ? seg->tile_cap : (seg->tile_cap + 7) & ~7;
  if (!fused_for(seg->T) || n_proj * cap > kXSlots) {
    // one projection after another (the launch overheads are small next to
    // batches this large)
    for (int p = 0; p < n_proj; ++p) {
      st = plora_apply(x, ldx, &ads[p], seg, ys[p], ldys[p], ws, ws_bytes, stream);
      if (st != PLORA_OK) return st;
    }
    return PLORA_OK;
  }
  // (the narrowest projection's columns limit the slices of all.  One launch
  // even where that leaves one slice: 7168 -> 7168, 896, 896 at rank 128, two
  // layers, 1 and 40 tokens 166 and 236 us, one projection after another 311
  // and 375 on the former kernels)
  int min_out = ads[0].h_out;
  for (int p = 1; p < n_proj; ++p) min_out = std::min(min_out, ads[p].h_out);
  const SmallPlan sp = small_plan(n_proj * cap, ads[0].h_in, min_out, max_rank);
  MultiArgs m;
  memset(&m, 0, sizeof m);
  st = prepare(&ads[0], seg, ws, ws_bytes, m.g, true);
  if (st != PLORA_OK) return st;
  char* base = reinterpret_cast<char*>(ws);
  m.g.vpart = reinterpret_cast<float*>(base + l.vpart);
  m.g.x = x;
  m.g.ldx = ldx;
  m.n_proj = n_proj;
  m.cap = cap;
  for (int p = 0; p < n_proj; ++p) {
    ProjArgs& q = m.proj[p];
    q.A = ads[p].A; q.B = ads[p].B; q.a_len = ads[p].a_len; q.b_len = ads[p].b_len;
    q.A_pool = ads[p].A_pool; q.B_pool = ads[p].B_pool;
    q.a_pool_len = ads[p].a_pool_len; q.b_pool_len = ads[p].b_pool_len;
    q.a_off = ads[p].a_off; q.b_off = ads[p].b_off; q.ranks = ads[p].ranks;
    q.scales = ads[p].scales; q.y = ys[p]; q.ldy = ldys[p]; q.h_out = ads[p].h_out;
    q.max_rank = ads[p].max_rank;
  }
  clear_stale_error();
  launch_small_multi(m, sp.S, sp.J, sp.gl, sp.deep, (unsigned)(sp.slots * sp.J), stream);
  return launch_status();
}

plora_status plora_check_adapters(const plora_adapters* ad, int32_t* bad_index,
                                  hipStream_t stream) {
  plora_status st = check_adapters_host(ad);
  if (st != PLORA_OK) return st;
  const int N = ad->n_adapters;
  if (bad_index) *bad_index = -1;
  if (N == 0) return PLORA_OK;
  int32_t* ranks = new int32_t[N];
  int64_t* ao = new int64_t[N];
  int64_t* bo = new int64_t[N];
  plora_status res = PLORA_OK;
  if (hipMemcpyAsync(ranks, ad->ranks, sizeof(int32_t) * N, hipMemcpyDeviceToHost, stream) !=
          hipSuccess ||
      hipMemcpyAsync(ao, ad->a_off, sizeof(int64_t) * N, hipMemcpyDeviceToHost, stream) !=
          hipSuccess ||
      hipMemcpyAsync(bo, ad->b_off, sizeof(int64_t) * N, hipMemcpyDeviceToHost, stream) !=
          hipSuccess ||
      hipStreamSynchronize(stream) != hipSuccess) {
    res = PLORA_ERR_HIP;
  } else {
    for (int i = 0; i < N; ++i) {
      const int r = ranks[i];
      bool ok = usable_rank(r, ad->max_rank);
      if (ok && r > 0) {
        ok = block_ok(ad->A, ad->a_len, ad->A_pool, ad->a_pool_len, ao[i],
                      (int64_t)ad->h_in * r) &&
             block_ok(ad->B, ad->b_len, ad->B_pool, ad->b_pool_len, bo[i],
                      (int64_t)ad->h_out * r);
      }
      if (!ok) {
        if (bad_index) *bad_index = i;
        res = PLORA_ERR_INVALID_ARG;
        break;
      }
    }
  }
  delete[] ranks;
  delete[] ao;
  delete[] bo;
  return res;
}

const char* plora_status_string(plora_status status) {
  switch (status) {
    case PLORA_OK: return "PLORA_OK";
    case PLORA_ERR_INVALID_ARG: return "PLORA_ERR_INVALID_ARG";
    case PLORA_ERR_UNSUPPORTED: return "PLORA_ERR_UNSUPPORTED";
    case PLORA_ERR_WORKSPACE_TOO_SMALL: return "PLORA_ERR_WORKSPACE_TOO_SMALL";
    case PLORA_ERR_HIP: return "PLORA_ERR_HIP";
  }
  return "PLORA_ERR_UNKNOWN";
}

plora_status plora_pool_device_pointer(const void* host, const void** device) {
  if (!host || !device) return PLORA_ERR_INVALID_ARG;
  *device = nullptr;
  void* d = nullptr;
  if (hipHostGetDevicePointer(&d, const_cast<void*>(host), 0) != hipSuccess || !d) {
    (void)hipGetLastError();
    return PLORA_ERR_UNSUPPORTED;
  }
  *device = d;
  return PLORA_OK;
}

plora_status plora_workspace_counters(const void* ws, size_t ws_bytes, int64_t* counts,
                                      hipStream_t stream) {
  if (!ws || !counts) return PLORA_ERR_INVALID_ARG;
  const size_t off = (size_t)kXSlots * sizeof(uint64_t);
  if (!aligned16(ws)) return PLORA_ERR_UNSUPPORTED;
  if (ws_bytes < off + kCounters * sizeof(uint64_t)) return PLORA_ERR_WORKSPACE_TOO_SMALL;
  uint64_t host[kCounters];
  if (hipMemcpyAsync(host, reinterpret_cast<const char*>(ws) + off, sizeof host,
                     hipMemcpyDeviceToHost, stream) != hipSuccess ||
      hipStreamSynchronize(stream) != hipSuccess) {
    g_last_hip_error.store((int32_t)hipGetLastError());
    return PLORA_ERR_HIP;
  }
  for (int i = 0; i < kCounters; ++i) counts[i] = (int64_t)host[i];
  return PLORA_OK;
}

int32_t plora_debug_last_hip_error(void) { return g_last_hip_error.load(); }

void plora_debug_set_exchange_polls(int32_t polls) {
  g_exchange_polls.store(polls < 0 ? kSpinLimit : polls);
}

}  // extern "C"
