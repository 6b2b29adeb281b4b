// Host side of the C ABI declared in include/ckv.h: argument checks,
// workspace carving, kernel launches.  No device memory is allocated here.
#include "../../include/ckv.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "ckv_books.h"
#include "ckv_kernels.h"
#include "ckv_layer_kernel.h"
#include "ckv_unit_kernel.h"

using namespace ckv;

constexpr int kManyEntries = 1 << 20;   // `excess` of a layer about which the host knows nothing
constexpr int kSide = 2;   // streams of the context's own for deferred bookkeeping

// Scratch of ckv_probe_noalloc: device memory the library owns from the moment it is loaded, so that the
// call never needs a caller's workspace or an allocation.  In host code `scratch` is only a handle: the
// array's address on a device comes from hipGetSymbolAddress, once per device (scratch_setup), and that
// pointer is what kernels and fills get.  One array per GPU, shared by every context on it.
constexpr size_t kScratchBytes = (size_t)128 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
constexpr int kMaxDevices = 64;

struct ckv_ctx {
  ckv_layout lay;
  ckv_lrfu_params par;
  ckv_buffers buf;
  Dev dev;
  int units = 0;
  int units_per_layer = 0;
  long long budget_total = 0;   // of all units, as last set by the host (a re-allocation keeps every sequence's total)
  int next_layer = 0;
  int n_cu = 256;
  float* seedmi = nullptr;      // workspace of the prompt replay
  float* seedrw = nullptr;
  int device = 0;               // the HIP device the context was created on
  size_t finish_lds = 0, layer_lds = 0;
  // fused path (unit_kernel)
  int path_mode = 0;            // 0 auto, 1 units split among workgroups, 2 fused kernel, 3 / 4 fused with 4 / 2 wavefronts per unit
  struct Fused {                // one variant of the fused kernel
    bool ok = false;
    int waves = 0;              // wavefronts per workgroup (= per unit)
    int grid = 0;
    int lds_main = 0;           // bytes of the logits / values tile
    size_t lds = 0;             // dynamic LDS per workgroup
  } fused[2];                   // [0]: 4 wavefronts, 2 workgroups per CU; [1]: 2 wavefronts, 4 workgroups per CU
  std::vector<uint8_t> prompt_loaded;
  std::vector<int32_t> prompt_len;   // per layer: length of a prompt loaded whole and untouched since, else -1
  // Deferred bookkeeping of single-layer steps (CKV_DEFER_BOOKKEEPING): finish_kernel runs on
  // one of the `side` streams (layer l on side[l % kSide], so that the bookkeeping of consecutive layers, which
  // share nothing, can overlap), ordered by events against the caller's stream.  books: the layers whose
  // bookkeeping has been queued there and nothing on the caller's side has waited for yet.
  // The bookkeeping of several consecutive layers (book_group) goes out as one launch (a fork from the caller's
  // stream costs about as much as a small kernel, and more units per launch fill the chip better): after a
  // deferred step, layers [group_first, group_first + group_count) have been scanned on group_stream and wait
  // for theirs; the group goes out when it is full, with the last layer, and before anything else looks.
  hipStream_t side[kSide] = {};
  hipEvent_t ev_out = nullptr;
  std::vector<hipEvent_t> ev_book;
  PendingBooks books;
  // Shared pools: budgets (or a prompt) have changed what units should own (dirty); once an eviction over all
  // layers has been issued since, the segments are dealt out again when the next step begins (due).
  bool dirty = false, due = false;
  // Layers whose budgets have changed since their last eviction: their units may have to give up many entries at once, which
  // a step then leaves to evict_kernel behind it.
  std::vector<uint8_t> many;
  // Per layer: entries above its budget that a unit may hold, as far as the host has seen (a replayed graph may have added more).
  std::vector<int> excess;
  int group_first = 0, group_count = 0, group_launches = 0;
  uint32_t group_flags = 0;
  hipStream_t group_stream = nullptr;
  std::string err;
  // scan timing
  bool profile = false;
  std::vector<hipEvent_t> ev;      // pairs
  size_t ev_used = 0;
  double scan_ms = 0.0;
  int scan_launches = 0;
};

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

int fail(ckv_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg;
  return code;
}

int hip_fail(ckv_ctx* c, hipError_t e, const char* what) {
  std::string m = std::string(what) + ": " + hipGetErrorString(e);
  return fail(c, CKV_EHIP, m);
}

#define CKV_HIP(ctx, call)                                   \
  do {                                                       \
    hipError_t e_ = (call);                                  \
    if (e_ != hipSuccess) return hip_fail((ctx), e_, #call); \
  } while (0)

bool layout_ok(const ckv_layout* l, std::string* why) {
  if (!l) { *why = "layout is NULL"; return false; }
  if (l->head_dim != kDim) { *why = "head_dim must be 128"; return false; }
  if (l->n_layers < 1 || l->n_layers > kMaxLayers) { *why = "n_layers must be in [1, 256]"; return false; }
  if (l->batch < 1) { *why = "batch must be >= 1"; return false; }
  if (l->n_kv_heads < 1 || l->n_kv_heads > kMaxKvHeads) { *why = "n_kv_heads must be in [1, 32]"; return false; }
  if (l->n_q_heads < l->n_kv_heads || l->n_q_heads % l->n_kv_heads != 0) { *why = "n_q_heads must be a multiple of n_kv_heads"; return false; }
  if (l->n_q_heads / l->n_kv_heads > kMaxGroup) { *why = "at most 8 query heads per KV head"; return false; }
  if (l->cap < kBlk || l->cap % kBlk != 0 || l->cap > kMaxChunks * kChunk) { *why = "cap must be a multiple of 32 in [32, 32768]"; return false; }
  if (l->out_dtype != CKV_F32 && l->out_dtype != CKV_BF16) { *why = "out_dtype must be CKV_F32 or CKV_BF16"; return false; }
  long long units = (long long)l->n_layers * l->batch * l->n_kv_heads;
  if (units * l->cap > (1ll << 40) || units > (1ll << 24)) { *why = "geometry too large"; return false; }
  const long long segs = (l->cap + kSeg - 1) / kSeg;
  if (l->headroom < 0 || l->headroom >= l->cap) { *why = "headroom must be in [0, cap)"; return false; }
  if (l->pool_slots <= 0 || l->pool_slots % kSeg != 0 || l->pool_slots > (1ll << 40)) { *why = "pool_slots must be a positive multiple of 256"; return false; }
  if (l->headroom == 0 && l->pool_slots < units * segs * kSeg) { *why = "pool_slots too small: with headroom 0 every unit owns ceil(cap / 256) segments"; return false; }
  return true;
}

bool params_ok(const ckv_layout* l, const ckv_lrfu_params* p, std::string* why) {
  if (!p) { *why = "params is NULL"; return false; }
  if (!(p->lambda >= 0.0f && p->lambda <= 1.0f)) { *why = "lambda must be in [0, 1]"; return false; }
  if (!(p->top_p > 0.0f)) { *why = "top_p must be > 0"; return false; }
  if (!(p->softmax_scale > 0.0f) || !std::isfinite(p->softmax_scale)) { *why = "softmax_scale must be positive"; return false; }
  if (p->reward_mode != CKV_REWARD_TOPP_HIT && p->reward_mode != CKV_REWARD_ATTN_WEIGHTED) { *why = "unknown reward_mode"; return false; }
  if (p->t0 < 0) { *why = "t0 must be >= 0"; return false; }
  if (p->budget_min < 1 || p->budget_min > p->budget_max || p->budget_max >= l->cap) { *why = "need 1 <= budget_min <= budget_max < cap"; return false; }
  return true;
}

// lambda^delta as float, flushed to zero below FLT_MIN; the table ends at its
// first zero entry (one entry for lambda = 1, capped at 2^20 + 1 entries).
std::vector<float> make_decay_table(float lambda) {
  std::vector<float> tab;
  tab.push_back(1.0f);
  const double lam = (double)lambda;
  if (lam == 1.0) return tab;
  for (int delta = 1; delta <= (1 << 20); ++delta) {
    float v = (float)std::pow(lam, (double)delta);
    if (v < FLT_MIN) v = 0.0f;
    tab.push_back(v);
    if (v == 0.0f) break;
  }
  return tab;
}

struct Carve {
  size_t n, budget, t_unit, nev, window, sc, tab, partial, ml, logits, btotal, order, layer_ts, arrive, msum, tbl, owned, spare, seedmi, seedrw, total;
};

Carve carve(const ckv_layout* l, size_t tab_len) {
  Carve c{};
  const size_t U = (size_t)l->n_layers * l->batch * l->n_kv_heads;
  const size_t G = (size_t)(l->n_q_heads / l->n_kv_heads);
  const size_t mc = (size_t)(l->cap + kChunk - 1) / kChunk;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
  c.n = take(U * 4);
  c.budget = take(U * 4);
  c.t_unit = take(U * 4);
  c.nev = take(U * 4);
  c.arrive = take(U * 4);
  c.window = take(U * 8);
  c.sc = take(SC_COUNT * 4);
  c.tab = take(tab_len * 4);
  c.partial = take(U * (mc + 1) * G * kDim * 4);
  c.ml = take(U * (mc + 1) * G * 2 * 4);
  c.logits = take(U * G * (size_t)l->cap * 4);
  c.btotal = take((size_t)l->batch * 8);
  c.order = take(U * 4);
  c.layer_ts = take((size_t)l->n_layers * 4);
  c.msum = take(U * kMaxGroup * 2 * 4);
  c.tbl = take(U * mc * 4);
  c.owned = take(U * 4);
  c.spare = take((size_t)(l->pool_slots / kSeg) * 4);
  // prompt replay (ckv_seed_prompt), one layer at a time: softmax maximum and 1 / sum per query column of a
  // batch; and, for contexts whose logits are too small to lend the replay room for several groups of queries, the
  // weights (then hits) of one group's 16 queries
  const size_t UL = (size_t)l->batch * l->n_kv_heads;
  c.seedmi = take((size_t)kSeedTiles * UL * kSeedCols * 2 * 4);
  c.seedrw = take(UL * (size_t)l->cap * kSeedCols * 4);
  c.total = off;
  return c;
}

int check_budgets(ckv_ctx* c, const ckv_layout* l, const ckv_lrfu_params* p, const int32_t* budgets) {
  if (!budgets) return fail(c, CKV_EINVAL, "budgets is NULL");
  const size_t U = (size_t)l->n_layers * l->batch * l->n_kv_heads;
  for (size_t u = 0; u < U; ++u)
    if (budgets[u] < p->budget_min || budgets[u] > p->budget_max)
      return fail(c, CKV_EINVAL, "a budget lies outside [budget_min, budget_max]");
  return CKV_OK;
}

// The variant of the fused kernel the current path mode selects (nullptr: none fits, or units are split).
const ckv_ctx::Fused* fused_variant(const ckv_ctx* c) {
  if (c->path_mode == 1) return nullptr;
  const ckv_ctx::Fused* f = c->path_mode == 3 ? &c->fused[0] : c->path_mode == 4 ? &c->fused[1]
                            : c->fused[0].ok ? &c->fused[0] : &c->fused[1];
  return f->ok ? f : nullptr;
}

// A pair of timing events from the context's pool (ckv_profile_enable).
int profile_events(ckv_ctx* c, hipEvent_t* e0, hipEvent_t* e1) {
  if (c->ev_used + 2 > c->ev.size()) {
    for (int i = 0; i < 2; ++i) {
      hipEvent_t e;
      CKV_HIP(c, hipEventCreate(&e));
      c->ev.push_back(e);
    }
  }
  *e0 = c->ev[c->ev_used];
  *e1 = c->ev[c->ev_used + 1];
  c->ev_used += 2;
  return CKV_OK;
}

// Side streams outlive the context that created them: making and destroying two cost 100 us per context (183 + 59 us for
// creating and closing a small one, 135 + 5 without), which a server that makes one per batch of sequences pays each time.  Idle ones wait here, at most kIdleStreams per device; more are
// destroyed.  A stream is handed back after everything on it has completed.
constexpr size_t kIdleStreams = 16;
std::mutex g_streams_mutex;
std::vector<hipStream_t> g_streams[kMaxDevices];

hipError_t take_stream(int devid, hipStream_t* out) {
  if (devid >= 0 && devid < kMaxDevices) {
    std::lock_guard<std::mutex> lock(g_streams_mutex);
    if (!g_streams[devid].empty()) {
      *out = g_streams[devid].back();
      g_streams[devid].pop_back();
      return hipSuccess;
    }
  }
  return hipStreamCreateWithFlags(out, hipStreamNonBlocking);
}

void give_stream(int devid, hipStream_t s) {
  const bool idle = hipStreamSynchronize(s) == hipSuccess;
  if (idle && devid >= 0 && devid < kMaxDevices) {
    std::lock_guard<std::mutex> lock(g_streams_mutex);
    if (g_streams[devid].size() < kIdleStreams) {
      try {
        g_streams[devid].push_back(s);
        return;
      } catch (const std::bad_alloc&) {
      }
    }
  }
  (void)hipStreamDestroy(s);
}

// Eviction of `count` units from `begin` on: select, then move.  A unit's keys sit in the registers of one workgroup:
// 1024 threads, or 256 where four entries per thread are enough for every unit, or 32 are and there is more than a unit per
// compute unit, which has room for one wide workgroup (window policy, two evicted each, 1024 / 256 threads: 256 units of 7500
// entries 31.7 / 35.1 us, 384 units of 2000 27.1 / 21.3, 512 units of 2000 28.3 / 22.1, 768 units of 7500 84.0 / 74.7).
// The moves have a kernel of their own where a unit may have more to move than its workgroup moves in two rounds: `excess` counts
// what the host has seen (window policy, 64 units of 9000 entries, 1024 threads each, 2 / 40 / 150 evicted, one kernel 35.4 / 39.3 / 48.5 us,
// two 40.3 / 41.5 / 45.1; half of the entries evicted by score, 64 of 9000 267 / 92 us, 256 of 7500 439 / 365, 1024 of 2048 416 / 395.  With 256
// threads the two are level up to about 150 evicted: 512 of 2000, window policy, 40 each 31.6 / 36.0, by score 150 each 96 / 97, half 184 / 175);
// and for up to four units per compute unit, beyond which a unit's own workgroup is as fast (window policy, 40 evicted each, one kernel / two, the moves
// in a launch per 1024 units: 4096 units of 1000 103 / 150, 8192 of 500 160 / 242; half by score, 2048 of 1000 411 / 372, 8192 of 500 821 / 826).
// Never for more than kMoveUnits, whatever the chip: that kernel keeps a place in LDS for each unit's first move and would leave out those beyond.  A
// replayed graph may find more than was seen when it was captured; it then takes longer and does the same.  (With the second kernel in
// every captured eviction: 512 units of 300 entries, a captured attention-only step with a window eviction, 36 us, without 34.)
int launch_evict(ckv_ctx* c, hipStream_t s, int begin, int count, int n_sink, int after_step = 0) {
  const int cap = c->lay.cap;
  const bool small = cap <= 4 * kThreads || (cap <= 32 * kThreads && count > c->n_cu);
  const int threads = small ? kThreads : kWideThreads, per_round = 4 * threads / 64;
  bool moves = after_step != 0;
  for (int l = begin / c->units_per_layer; l < (begin + count) / c->units_per_layer; ++l) {
    moves = moves || c->excess[l] > 2 * per_round;
    c->excess[l] = 0;
  }
  moves = moves && count <= std::min(4 * c->n_cu, kMoveUnits);
  auto select = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)count), dim3((unsigned)threads), 0, s, c->dev, begin, n_sink, after_step, moves ? 1 : 0);
  };
  const int per = (cap + threads - 1) / threads;
  if (small) {
    if (per <= 4) select(evict_kernel<kThreads, 4>);
    else if (per <= 8) select(evict_kernel<kThreads, 8>);
    else if (per <= 16) select(evict_kernel<kThreads, 16>);
    else select(evict_kernel<kThreads, 32>);
  } else {
    if (per <= 4) select(evict_kernel<kWideThreads, 4>);
    else if (per <= 8) select(evict_kernel<kWideThreads, 8>);
    else if (per <= 16) select(evict_kernel<kWideThreads, 16>);
    else select(evict_kernel<kWideThreads, 32>);
  }
  CKV_HIP(c, hipGetLastError());
  if (!moves) return CKV_OK;
  // two workgroups per compute unit, or as many as have four moves per wavefront if every unit moves half of what it may hold
  const long long most = ((long long)count * (cap / 2) + 15) / 16;
  const int groups = std::max(8, (int)std::min<long long>(2ll * c->n_cu, (most + 7) / 8 * 8) & ~7);
  hipLaunchKernelGGL(evict_move_kernel, dim3((unsigned)groups), dim3(kThreads), 0, s, c->dev, begin, count);
  CKV_HIP(c, hipGetLastError());
  return CKV_OK;
}

// Whether a step after a change of budgets leaves evictions of several entries per unit to the kernels behind it.  Those
// use more threads per unit; the step's own kernel deals units out as workgroups come free.  Re-allocation and the two steps behind it beyond two
// ordinary steps, us, in the step's kernel / left, units of 1024 entries on average and G = 4: all layers 128 units 117 / 27, 512 177 / 85, 1024
// 284 / 142, 1280 315 / 240, 2048 425 / 325, 6144 745 / 645; one call per layer of 1024 424 / 200, of 1280 590 / 350, of 2048 670 / 475; deferred bookkeeping of
// several layers of 128 per launch, 4 layers 126 / 53, 8 188 / 85, 16 242 / 137.  Of 2048 on average and G = 5: all layers 512 units 395 / 150, 2048 816 / 590, 6144
// 1220 .. 1770 / 1075; one call per layer of 2048 1235 / 850; deferred, 8 layers 336 / 170, 16 460 / 290.  The lines date from moves that
// had a few workgroups per unit, where the unit with the most decided (2048 units 790 / 938, 6144 units 1705 / 2474): since moves are dealt out over the whole chip,
// leaving them is the faster at all of these sizes, and what lies above the lines could follow.
bool leave_many_pays(const ckv_ctx* c, int count, bool deferred) {
  if (deferred) return count * std::min(book_group(c->n_cu, c->units_per_layer), c->lay.n_layers) <= 3 * c->n_cu;
  return count <= 5 * c->n_cu;
}

// The bookkeeping of `count` units from `begin` on in a kernel of its own, behind their scan (deferred or not).  Workgroups of 256 threads where no unit can
// hold more than eight entries per thread, else 1024.
int launch_finish(ckv_ctx* c, hipStream_t s, int begin, int count, uint32_t flags) {
  if (c->lay.cap <= 8 * kThreads)
    hipLaunchKernelGGL(finish_kernel<kThreads>, dim3((unsigned)count), dim3(kThreads), c->finish_lds, s, c->dev, begin, flags);
  else
    hipLaunchKernelGGL(finish_kernel<kWideThreads>, dim3((unsigned)count), dim3(kWideThreads), c->finish_lds, s, c->dev, begin, flags);
  CKV_HIP(c, hipGetLastError());
  return CKV_OK;
}

// Entries that a unit's budget allows, on average.
long long mean_budget(const ckv_ctx* c) { return c->budget_total / c->units; }

// A step of `count` units from `begin` on (or its scan, or attention alone: `mode`).
int launch_layer_step(ckv_ctx* c, hipStream_t s, int begin, int count, const uint16_t* q, const uint16_t* k_new, const uint16_t* v_new, void* out,
                      uint32_t flags, int mode, int advance) {
  const int upl = c->units_per_layer, cap = c->lay.cap;
  auto go = [&](auto one_block, auto entries) {
    constexpr bool kOne = decltype(one_block)::value;
    constexpr int kRmax = decltype(entries)::value;
    const int pieces = step_pieces(cap, kOne);
    const LayerCall call{q, k_new, v_new, out, begin, flags, mode, begin / upl, count / upl, advance, looks_early((long long)count * pieces, kOne, c->n_cu)};
    hipLaunchKernelGGL((layer_step_kernel<kOne, kRmax>), dim3((unsigned)count, (unsigned)pieces), dim3(kLayerThreads),
                       kRmax ? c->layer_lds : (size_t)kLayerScanLds, s, c->dev, call);
  };
  auto by_length = [&](auto one_block) {
    if (mode != kWholeStep) go(one_block, std::integral_constant<int, 0>{});
    else if (cap <= 4 * kLayerThreads) go(one_block, std::integral_constant<int, 4>{});
    else go(one_block, std::integral_constant<int, 12>{});
  };
  if (one_block_each(mean_budget(c), count, c->n_cu)) by_length(std::true_type{});
  else by_length(std::false_type{});
  CKV_HIP(c, hipGetLastError());
  return CKV_OK;
}

// Queue the bookkeeping of the layers scanned since the last group went out.
int flush_group(ckv_ctx* c) {
  if (c->group_count == 0) return CKV_OK;
  const int first = c->group_first, count = c->group_count;
  c->group_count = 0;
  const int upl = c->lay.batch * c->lay.n_kv_heads;
  CKV_HIP(c, hipEventRecord(c->ev_out, c->group_stream));
  hipStream_t side = c->side[c->group_launches++ % kSide];
  CKV_HIP(c, hipStreamWaitEvent(side, c->ev_out, 0));
  if (int rc = launch_finish(c, side, first * upl, count * upl, c->group_flags)) return rc;
  if (c->group_flags & kLeaveMany)
    if (int rc = launch_evict(c, side, first * upl, count * upl, -1, 1)) return rc;
  CKV_HIP(c, hipEventRecord(c->ev_book[first], side));
  c->books.record(first, count);
  return CKV_OK;
}

// Order `s` after the deferred bookkeeping still in flight on the side streams (all layers, or one).
int join_side(ckv_ctx* c, hipStream_t s, int layer = -1) {
  if (c->group_count && (layer < 0 || (layer >= c->group_first && layer < c->group_first + c->group_count)))
    if (int rc = flush_group(c)) return rc;
  return c->books.join(layer, [&](int first) -> int {
    CKV_HIP(c, hipStreamWaitEvent(s, c->ev_book[first], 0));
    return CKV_OK;
  });
}

// Deal the pool segments out again (shared pools only); units [x_begin, x_begin + x_count) get room for
// x_entries entries whatever their budgets say.
int launch_rebalance(ckv_ctx* c, hipStream_t s, int x_begin = 0, int x_count = 0, int x_entries = 0, const int32_t* x_len = nullptr) {
  if (c->lay.headroom == 0) return CKV_OK;
  hipLaunchKernelGGL(rebalance_kernel, dim3(1), dim3(kBalanceThreads), 0, s, c->dev, (int)c->lay.headroom, x_begin, x_count, x_entries, x_len);
  CKV_HIP(c, hipGetLastError());
  return CKV_OK;
}

// After an eviction that covered the last layer: the segments the shrunken units gave up can go to the others.
// Not yet, though: the slots behind a unit's entries hold the record of what it has just evicted, which a
// caller may still want to read, and with deferred bookkeeping the evictions have not even run.  The segments
// move when the next step begins.
int rebalance_after_eviction(ckv_ctx* c) {
  if (c->lay.headroom > 0 && c->dirty) c->due = true;
  return CKV_OK;
}

// Before a step begins: what a deferred eviction left to do.
int rebalance_if_due(ckv_ctx* c, hipStream_t s) {
  if (!c->due) return CKV_OK;
  if (int rc = join_side(c, s)) return rc;
  c->dirty = c->due = false;
  return launch_rebalance(c, s);
}

// (Re)build the fused kernel's schedule (units by descending budget) from the budgets in device memory.
int launch_schedule(ckv_ctx* c, hipStream_t s) {
  hipLaunchKernelGGL(schedule_kernel, dim3(1), dim3(1024), 0, s, c->dev);
  CKV_HIP(c, hipGetLastError());
  return CKV_OK;
}

// Answer-probe classes of `count` units from `begin` on.  Workgroups of 256 threads for the classes where 32 entries per
// thread are enough and there are units to fill the chip with them.
int launch_probe(ckv_ctx* c, const Dev& d, int begin, int count, const uint16_t* q, uint8_t* classes, hipStream_t s) {
  const int spans = (d.cap + kProbeSpan - 1) / kProbeSpan;
  hipLaunchKernelGGL(probe_scan_kernel, dim3((unsigned)count, (unsigned)((spans + 3) / 4)), dim3(kThreads), 0, s, d, begin, q);
  CKV_HIP(c, hipGetLastError());
  if (d.cap <= 32 * kThreads && count >= 4 * c->n_cu)
    hipLaunchKernelGGL(probe_kernel<kThreads>, dim3((unsigned)count), dim3(kThreads), 0, s, d, begin, classes);
  else
    hipLaunchKernelGGL(probe_kernel<kWideThreads>, dim3((unsigned)count), dim3(kWideThreads), 0, s, d, begin, classes);
  CKV_HIP(c, hipGetLastError());
  return CKV_OK;
}

// Wavefronts that share a unit's blocks in the replay's passes over the keys: a multiple of four (a workgroup's), at
// most one per block.  Three workgroups fit on a compute unit; of the splits that the partials have room for, the one
// that leaves the least of the chip idle (places in the last round, and the unit's blocks not dividing evenly),
// the coarsest of equals.
// Room: a group of 16 queries takes 32 G floats per wavefront and unit, the decode partials hold 128 G per chunk of 256
// entries, unit and layer: four wavefronts per chunk and layer for one group (a batch has at most one per two layers).
int seed_spans(const ckv_ctx* c, int entries, int count) {
  const long long blocks = (entries + kBlk - 1) / kBlk, places = 3ll * c->n_cu;
  const long long most = std::min<long long>((blocks + 3) / 4 * 4, (long long)std::min(kSegBlocks, 4 * c->lay.n_layers) * c->dev.max_chunks);
  int best = 4;
  double best_eff = 0.0;
  for (long long S = 4; S <= most; S += 4) {
    const long long per = (blocks + S - 1) / S, wgs = (long long)count * S / 4, rounds = (wgs + places - 1) / places;
    const double eff = (double)(blocks * count) / (double)(rounds * places * 4 * per);
    if (eff > 1.02 * best_eff) {
      best_eff = eff;
      best = (int)S;
    }
    if (rounds > 4) break;
  }
  return best;
}

int upload_budgets(ckv_ctx* c, const int32_t* budgets, hipStream_t s) {
  const ckv_layout& l = c->lay;
  std::vector<long long> tot(l.batch, 0);
  for (int i = 0; i < l.n_layers; ++i)
    for (int b = 0; b < l.batch; ++b)
      for (int h = 0; h < l.n_kv_heads; ++h) tot[b] += budgets[((size_t)i * l.batch + b) * l.n_kv_heads + h];
  c->budget_total = 0;
  for (long long t : tot) c->budget_total += t;
  CKV_HIP(c, hipMemcpyAsync(c->dev.budget, budgets, (size_t)c->units * 4, hipMemcpyHostToDevice, s));
  CKV_HIP(c, hipMemcpyAsync(c->dev.btotal, tot.data(), (size_t)l.batch * 8, hipMemcpyHostToDevice, s));
  if (int rc = launch_schedule(c, s)) return rc;
  CKV_HIP(c, hipStreamSynchronize(s));
  return CKV_OK;
}

int fill32(ckv_ctx* c, void* p, uint32_t v, size_t count, hipStream_t s) {
  if (count == 0) return CKV_OK;
  size_t blocks = (count + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (uint32_t*)p, v, count);
  CKV_HIP(c, hipGetLastError());
  return CKV_OK;
}

// Dynamic LDS that a kernel may be launched with on a device: raised when a context needs more than any before it.
std::mutex g_lds_mutex;
std::map<std::pair<int, const void*>, size_t> g_lds;

bool allow_lds(int devid, const void* fn, size_t bytes) {
  try {
    std::lock_guard<std::mutex> lock(g_lds_mutex);
    size_t& have = g_lds[{devid, fn}];
    if (bytes <= have) return true;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return false;
    have = bytes;
    return true;
  } catch (const std::bad_alloc&) {
    return false;
  }
}

// Address of the library's static scratch on each device.
std::mutex g_scratch_mutex;
unsigned char* g_scratch_ptr[kMaxDevices] = {};

int scratch_setup(int devid) {
  if (devid < 0 || devid >= kMaxDevices) return CKV_EINVAL;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[devid]) return CKV_OK;
  unsigned char* p = nullptr;
  if (hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return CKV_EHIP;
  g_scratch_ptr[devid] = p;
  return CKV_OK;
}

int layer_range(ckv_ctx* c, int32_t layer, int* begin, int* count) {
  if (layer == -1) {
    *begin = 0;
    *count = c->units;
  } else if (layer >= 0 && layer < c->lay.n_layers) {
    *begin = layer * c->units_per_layer;
    *count = c->units_per_layer;
  } else {
    return fail(c, CKV_EINVAL, "layer out of range");
  }
  return CKV_OK;
}

}  // namespace

extern "C" {

size_t ckv_workspace_bytes(const ckv_layout* layout, const ckv_lrfu_params* params) {
  std::string why;
  if (!layout_ok(layout, &why) || !params_ok(layout, params, &why)) return 0;
  return carve(layout, make_decay_table(params->lambda).size()).total;
}

int ckv_init(ckv_ctx** out, const ckv_layout* layout, const int32_t* budgets, const ckv_lrfu_params* params,
             const ckv_buffers* b, void* stream) {
  if (!out) return CKV_EINVAL;
  *out = nullptr;
  std::string why;
  if (!layout_ok(layout, &why) || !params_ok(layout, params, &why)) return CKV_EINVAL;
  if (!b || !b->k_pool || !b->v_pool || !b->crf || !b->tau || !b->pos || !b->flags || !b->workspace) return CKV_EINVAL;
  if (int rc = check_budgets(nullptr, layout, params, budgets)) return rc;
  std::vector<float> tab = make_decay_table(params->lambda);
  const Carve cv = carve(layout, tab.size());
  if (b->workspace_bytes < cv.total || ((uintptr_t)b->workspace % kAlign) != 0) return CKV_EWORKSPACE;
  if (((uintptr_t)b->k_pool | (uintptr_t)b->v_pool | (uintptr_t)b->crf | (uintptr_t)b->tau | (uintptr_t)b->pos) % 16 != 0)
    return CKV_EINVAL;

  ckv_ctx* c = new (std::nothrow) ckv_ctx();
  if (!c) return CKV_EINVAL;
  c->lay = *layout;
  c->par = *params;
  c->buf = *b;
  c->units_per_layer = layout->batch * layout->n_kv_heads;
  c->units = layout->n_layers * c->units_per_layer;
  c->prompt_loaded.assign(layout->n_layers, 0);
  c->prompt_len.assign(layout->n_layers, -1);
  hipStream_t s = (hipStream_t)stream;

  int devid = 0;
  hipError_t e = hipGetDevice(&devid);
  int max_lds = 65536;
  if (e == hipSuccess) {
    if (hipDeviceGetAttribute(&c->n_cu, hipDeviceAttributeMultiprocessorCount, devid) != hipSuccess) c->n_cu = 0;
    if (hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, devid) != hipSuccess) max_lds = 65536;
  }
  if (e != hipSuccess || c->n_cu <= 0) {
    delete c;
    return CKV_EHIP;
  }
  c->device = devid;
  if (int rc = scratch_setup(devid)) {        // the static scratch of ckv_probe_noalloc: its address on this device
    delete c;
    return rc;
  }
  c->finish_lds = std::max(sizeof(TopBuf), (size_t)layout->cap * 4 + (size_t)((layout->cap + 31) / 32) * 4);
  if (c->finish_lds + 12288 > (size_t)max_lds) {   // static LDS of the kernels stays below 12 KB
    delete c;
    return CKV_EINVAL;
  }
  c->layer_lds = std::max((size_t)kLayerScanLds, c->finish_lds);
  bool lds_ok = true;
  for (const void* fn : {reinterpret_cast<const void*>(layer_step_kernel<false, 4>), reinterpret_cast<const void*>(layer_step_kernel<true, 4>),
                         reinterpret_cast<const void*>(layer_step_kernel<false, 12>), reinterpret_cast<const void*>(layer_step_kernel<true, 12>)})
    lds_ok = lds_ok && allow_lds(devid, fn, c->layer_lds);
  for (const void* fn : {reinterpret_cast<const void*>(seed_scan_kernel), reinterpret_cast<const void*>(seed_weights_kernel)})
    lds_ok = lds_ok && allow_lds(devid, fn, kSeedTiles * 4096);
  for (const void* fn : {reinterpret_cast<const void*>(finish_kernel<kThreads>), reinterpret_cast<const void*>(finish_kernel<kWideThreads>),
                         reinterpret_cast<const void*>(seed_hits_kernel<0>)})
    lds_ok = lds_ok && allow_lds(devid, fn, c->finish_lds);
  if (!lds_ok) {
    delete c;
    return CKV_EHIP;
  }

  // fused kernel: 8 / W workgroups of W wavefronts per CU, each with its share of the CU's 160 KB of LDS
  for (int v = 0; v < 2; ++v) {
    ckv_ctx::Fused& f = c->fused[v];
    f.waves = v == 0 ? 4 : 2;
    const int wgs = 8 / f.waves;
    const int static_lds = v == 0 ? 11 * 1024 : 6 * 1024;      // upper bounds of unit_kernel<W>'s static LDS
    const int evm_bytes = ((layout->cap + 31) / 32) * 4;
    const int tbl_bytes = 2 * ((layout->cap + kSeg - 1) / kSeg) * 4;   // two rows of the segment table
    const int share = (160 * 1024 / wgs) & ~1023;
    const int per_wg = max_lds < share ? max_lds : share;
    const int main_bytes = (per_wg - static_lds - evm_bytes - tbl_bytes) & ~127;
    f.grid = wgs * c->n_cu;
    f.ok = main_bytes >= 4 * layout->cap;                       // every entry's value must fit
    f.lds_main = main_bytes;
    f.lds = (size_t)main_bytes + evm_bytes + tbl_bytes;
    const void* fn = v == 0 ? reinterpret_cast<const void*>(unit_kernel<4>) : reinterpret_cast<const void*>(unit_kernel<2>);
    if (f.ok && !allow_lds(devid, fn, f.lds)) f.ok = false;
  }
  Dev& d = c->dev;
  d.L = layout->n_layers;
  d.Bz = layout->batch;
  d.Hq = layout->n_q_heads;
  d.Hkv = layout->n_kv_heads;
  d.G = layout->n_q_heads / layout->n_kv_heads;
  d.cap = layout->cap;
  d.units = c->units;
  d.unit0 = 0;
  d.by_order = 1;
  d.max_chunks = (layout->cap + kChunk - 1) / kChunk;
  d.slots = d.max_chunks + 1;
  d.out_bf16 = layout->out_dtype == CKV_BF16;
  d.scale_log2e = params->softmax_scale * 1.44269504088896340736f;
  d.top_p = params->top_p;
  d.reward_mode = params->reward_mode;
  d.bmin = params->budget_min;
  d.bmax = params->budget_max;
  d.tab_last = (int32_t)tab.size() - 1;
  d.K = (uint16_t*)b->k_pool;
  d.V = (uint16_t*)b->v_pool;
  d.crf = b->crf;
  d.tau = b->tau;
  d.pos = b->pos;
  d.flags = b->flags;
  uint8_t* ws = (uint8_t*)b->workspace;
  d.n = (int32_t*)(ws + cv.n);
  d.budget = (int32_t*)(ws + cv.budget);
  d.t_unit = (int32_t*)(ws + cv.t_unit);
  d.nev = (int32_t*)(ws + cv.nev);
  d.window = (u64*)(ws + cv.window);
  d.sc = (int32_t*)(ws + cv.sc);
  d.tab = (const float*)(ws + cv.tab);
  d.partial = (float*)(ws + cv.partial);
  d.ml = (float*)(ws + cv.ml);
  d.logits = (float*)(ws + cv.logits);
  d.btotal = (long long*)(ws + cv.btotal);
  d.order = (int32_t*)(ws + cv.order);
  d.layer_ts = (int32_t*)(ws + cv.layer_ts);
  d.arrive = (int32_t*)(ws + cv.arrive);
  d.msum = (float*)(ws + cv.msum);
  d.tbl = (int32_t*)(ws + cv.tbl);
  d.owned = (int32_t*)(ws + cv.owned);
  d.spare = (int32_t*)(ws + cv.spare);
  d.max_seg = (int32_t)((layout->cap + kSeg - 1) / kSeg);
  c->seedmi = (float*)(ws + cv.seedmi);
  c->seedrw = (float*)(ws + cv.seedrw);

  auto bail = [&](int rc) {
    ckv_destroy(c);
    return rc;
  };
  c->books.reset(layout->n_layers);
  c->many.assign(layout->n_layers, 0);
  c->excess.assign(layout->n_layers, 0);
  for (int i = 0; i < kSide; ++i)
    if (take_stream(devid, &c->side[i]) != hipSuccess) return bail(CKV_EHIP);
  if (hipEventCreateWithFlags(&c->ev_out, hipEventDisableTiming) != hipSuccess) return bail(CKV_EHIP);
  for (int l = 0; l < layout->n_layers; ++l) {
    hipEvent_t e;
    if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) return bail(CKV_EHIP);
    c->ev_book.push_back(e);
  }
  // Segment table.  headroom 0: every unit owns room for cap entries for good.  Otherwise a unit starts with
  // the segments that budget + headroom entries need, handed out in unit order (so a unit's segments are
  // contiguous to begin with); the rest of the pool is spare.
  const size_t S = (size_t)layout->pool_slots, U = (size_t)c->units;
  std::vector<int32_t> stage;
  InitJob job{};
  try {
    const size_t totals_at = 3 * U + (U & 1), tab_at = totals_at + 2 * (size_t)layout->batch;
    const bool tab_staged = (tab_at + tab.size()) * 4 <= cv.ml - cv.partial;      // the staging place: the decode partials
    stage.assign(tab_at + (tab_staged ? tab.size() : 0), 0);
    std::vector<long long> tot(layout->batch, 0);
    job.pool_segs = layout->pool_slots / kSeg;
    for (size_t u = 0; u < U; ++u) {
      const int need = layout->headroom == 0 ? d.max_seg : std::min<long long>(d.max_seg, ((long long)budgets[u] + layout->headroom + kSeg - 1) / kSeg);
      if (job.given + need > job.pool_segs) return bail(CKV_EINVAL);       // pool_slots too small for these budgets: see ckv_pool_slots
      stage[u] = budgets[u];
      stage[U + u] = (int32_t)job.given;
      stage[2 * U + u] = need;
      job.given += need;
      tot[u / layout->n_kv_heads % layout->batch] += budgets[u];
    }
    for (long long t : tot) c->budget_total += t;
    std::memcpy(stage.data() + totals_at, tot.data(), tot.size() * 8);
    if (tab_staged) std::memcpy(stage.data() + tab_at, tab.data(), tab.size() * 4);
    job.tab_n = tab_staged ? (int)tab.size() : 0;
  } catch (const std::bad_alloc&) {
    return bail(CKV_EHIP);
  }
  const unsigned blocks = (unsigned)std::min<size_t>(8ull * c->n_cu, std::max<size_t>(1, (S * kDim / 8 + kThreads - 1) / kThreads));
  auto region = [&](void* p, size_t bytes, uint32_t v = 0u) {
    const size_t count = bytes / 16, rounds = count / ((size_t)blocks * kThreads);
    return InitFill{(u32x4*)p, v, count, rounds >= 16 ? rounds * kThreads : 0};
  };
  job.fill[0] = region(d.K, S * kDim * 2);
  job.fill[1] = region(d.V, S * kDim * 2);
  job.fill[2] = region(d.crf, S * 4);
  job.fill[3] = region(d.tau, S * 4);
  job.fill[4] = region(d.pos, S * 4);
  // (the flags are the one array that need not lie at a multiple of 16 bytes)
  if ((uintptr_t)d.flags % 16 == 0)
    job.fill[5] = region(d.flags, S);
  else if (int rc = fill32(c, d.flags, 0u, S / 4, s))
    return bail(rc);
  // per-unit state (everything up to the scalars, budgets excepted, which follow from the staged copy)
  job.fill[6] = region(ws + cv.n, cv.budget - cv.n);
  job.fill[7] = region(ws + cv.t_unit, cv.nev - cv.t_unit, (uint32_t)(params->t0 - 1));
  job.fill[8] = region(ws + cv.nev, cv.sc - cv.nev);
  job.stage = (const int32_t*)d.partial;
  job.tab = (int32_t*)d.tab;
  job.t0 = params->t0;
  if (hipMemcpyAsync(d.partial, stage.data(), stage.size() * 4, hipMemcpyHostToDevice, s) != hipSuccess) return bail(CKV_EHIP);
  if (!job.tab_n && hipMemcpyAsync((void*)d.tab, tab.data(), tab.size() * 4, hipMemcpyHostToDevice, s) != hipSuccess) return bail(CKV_EHIP);
  hipLaunchKernelGGL(init_kernel, dim3(blocks), dim3(kThreads), 0, s, d, job);
  if (hipGetLastError() != hipSuccess) return bail(CKV_EHIP);
  if (int rc = launch_schedule(c, s)) return bail(rc);
  if (hipStreamSynchronize(s) != hipSuccess) return bail(CKV_EHIP);
  *out = c;
  return CKV_OK;
}

void ckv_destroy(ckv_ctx* c) {
  if (!c) return;
  for (int i = 0; i < kSide; ++i)
    if (c->side[i]) give_stream(c->device, c->side[i]);
  if (c->ev_out) (void)hipEventDestroy(c->ev_out);
  for (hipEvent_t e : c->ev_book) (void)hipEventDestroy(e);
  for (hipEvent_t e : c->ev) (void)hipEventDestroy(e);
  delete c;
}

int ckv_load_cache(ckv_ctx* c, int32_t layer, const void* k, const void* v, int32_t P, const int32_t* lengths,
                   const float* crf0, const int32_t* tau0, const int32_t* pos0, void* stream) {
  if (!c) return CKV_EINVAL;
  if (layer < 0 || layer >= c->lay.n_layers) return fail(c, CKV_EINVAL, "layer out of range");
  if (!k || !v) return fail(c, CKV_EINVAL, "k or v is NULL");
  if (P <= 0 || P >= c->lay.cap) return fail(c, CKV_EINVAL, "need 0 < P < cap");
  if (c->next_layer != 0) return fail(c, CKV_ESTATE, "a per-layer step is in progress");
  if (c->prompt_loaded[layer]) return fail(c, CKV_ESTATE, "layer already holds entries");
  c->prompt_loaded[layer] = 1;
  c->prompt_len[layer] = (!lengths && !pos0) ? P : -1;
  c->excess[layer] = kManyEntries;
  if (int rc = join_side(c, (hipStream_t)stream)) return rc;
  if (c->lay.headroom > 0) {
    // shared pools: the layer's units get room for what is loaded (and an append behind it) from the spare list,
    // and whatever earlier layers no longer need goes back to it first; an eviction gives the surplus back
    c->due = false;
    c->dirty = true;
    if (int rc = launch_rebalance(c, (hipStream_t)stream, layer * c->units_per_layer, c->units_per_layer, (int)P + c->lay.headroom, lengths)) return rc;
  }
  dim3 grid((unsigned)((P + kBlk - 1) / kBlk), (unsigned)c->units_per_layer);
  auto load = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, (hipStream_t)stream, c->dev, layer * c->units_per_layer, (const uint16_t*)k,
                       (const uint16_t*)v, (int)P, lengths, crf0, tau0, pos0);
  };
  if (loads_past_caches((long long)c->units_per_layer * P)) load(load_cache_kernel<true>);
  else load(load_cache_kernel<false>);
  CKV_HIP(c, hipGetLastError());
  return CKV_OK;
}

int ckv_load_prompt(ckv_ctx* c, int32_t layer, const void* k, const void* v, int32_t P, const float* crf0,
                    const int32_t* tau0, void* stream) {
  if (!c) return CKV_EINVAL;
  if (P > c->par.t0) return fail(c, CKV_EINVAL, "need P <= t0");
  return ckv_load_cache(c, layer, k, v, P, nullptr, crf0, tau0, nullptr, stream);
}

int ckv_decode_step(ckv_ctx* c, int32_t layer, const void* q, const void* k_new, const void* v_new, void* out,
                    uint32_t flags, void* stream) {
  if (!c) return CKV_EINVAL;
  if (!q || !k_new || !v_new || !out) return fail(c, CKV_EINVAL, "q, k_new, v_new or out is NULL");
  if (flags & ~(CKV_FUSE_EVICT | CKV_ATTENTION_ONLY | CKV_DEFER_BOOKKEEPING)) return fail(c, CKV_EINVAL, "unknown flag bits");
  if ((flags & CKV_DEFER_BOOKKEEPING) && (layer == -1 || (flags & CKV_ATTENTION_ONLY)))
    return fail(c, CKV_EINVAL, "CKV_DEFER_BOOKKEEPING is for single-layer steps with bookkeeping");
  if ((flags & CKV_ATTENTION_ONLY) && (flags & CKV_FUSE_EVICT))
    return fail(c, CKV_EINVAL, "CKV_ATTENTION_ONLY excludes CKV_FUSE_EVICT");
  int begin, count;
  if (int rc = layer_range(c, layer, &begin, &count)) return rc;
  if (layer == -1) {
    if (c->next_layer != 0) return fail(c, CKV_ESTATE, "a per-layer step is in progress");
  } else {
    if (layer != c->next_layer) return fail(c, CKV_ESTATE, "layers must be stepped in order");
  }
  const int advance = (layer == -1 || layer == c->lay.n_layers - 1) ? 1 : 0;
  c->next_layer = advance ? 0 : layer + 1;
  for (int l = (layer == -1 ? 0 : layer); l < (layer == -1 ? c->lay.n_layers : layer + 1); ++l) {
    c->prompt_loaded[l] = 1;
    c->prompt_len[l] = -1;
    c->excess[l] = (flags & CKV_FUSE_EVICT) ? 0 : std::min(c->excess[l] + 1, kManyEntries);
  }
  hipStream_t s = (hipStream_t)stream;
  // The fused kernel takes whole units: all layers at once, or one layer that has at least a unit per
  // workgroup.  Such a layer it also finishes sooner than a scan with deferred bookkeeping would (Llama-8B
  // shape, 512 units per layer: 74 against 78 us), so there the flag is not followed.
  const ckv_ctx::Fused* fv = fused_variant(c);
  if (fv && (c->path_mode == 0 || layer >= 0) && count < fv->grid) fv = nullptr;   // fewer units than workgroups: split the units instead
  const bool fused = fv != nullptr;
  if (fused) flags &= ~CKV_DEFER_BOOKKEEPING;
  if (flags & CKV_FUSE_EVICT) {
    // After a change of budgets, once.  Not into a graph: replays would evict what is not there; the kernels' own
    // evictions, which do without the launches behind them, give the same.
    bool many = false;
    for (int l = (layer == -1 ? 0 : layer); l < (layer == -1 ? c->lay.n_layers : layer + 1); ++l) {
      many |= c->many[l] != 0;
      c->many[l] = 0;
    }
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    if (many) CKV_HIP(c, hipStreamIsCapturing(s, &capturing));
    if (many && capturing == hipStreamCaptureStatusNone && leave_many_pays(c, count, (flags & CKV_DEFER_BOOKKEEPING) != 0)) flags |= kLeaveMany;
  }
  if (layer <= 0)
    if (int rc = rebalance_if_due(c, s)) return rc;
  if (int rc = join_side(c, s, layer)) return rc;
  if (flags & CKV_DEFER_BOOKKEEPING) {
    // One kernel on the caller's stream: it appends, attends and writes the output; the bookkeeping (which also
    // records the append) follows on a side stream, a group of layers at a time.
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (c->profile) {
      if (int rc = profile_events(c, &e0, &e1)) return rc;
      CKV_HIP(c, hipEventRecord(e0, s));
    }
    if (int rc = launch_layer_step(c, s, begin, count, (const uint16_t*)q, (const uint16_t*)k_new, (const uint16_t*)v_new, out, flags, kScanOnly, advance))
      return rc;
    if (c->profile) CKV_HIP(c, hipEventRecord(e1, s));
    const uint32_t kflags = flags & (CKV_FUSE_EVICT | kLeaveMany);
    if (c->group_count && (c->group_flags != kflags || c->group_stream != s || c->group_first + c->group_count != layer))
      if (int rc = flush_group(c)) return rc;
    if (c->group_count == 0) {
      c->group_first = layer;
      c->group_flags = kflags;
      c->group_stream = s;
    }
    c->group_count += 1;
    if (advance && (flags & CKV_FUSE_EVICT))
      if (int rc = rebalance_after_eviction(c)) return rc;
    if (c->group_count == book_group(c->n_cu, c->units_per_layer) || advance) return flush_group(c);
    return CKV_OK;
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (c->profile) {
    if (int rc = profile_events(c, &e0, &e1)) return rc;
    CKV_HIP(c, hipEventRecord(e0, s));
  }
  if (fused) {
    // The kernel takes its units from the schedule (all layers: by descending budget) or, for a single layer, in
    // the layer's own order starting at its first unit, whose rows come first in q, k_new, v_new and out.
    Dev dv = c->dev;
    dv.units = count;
    dv.unit0 = layer >= 0 ? begin : 0;
    dv.by_order = layer >= 0 ? 0 : 1;
    const uint16_t* qb = (const uint16_t*)q;
    const uint16_t* vb = (const uint16_t*)v_new;
    const uint16_t* kb = (const uint16_t*)k_new;
    void* ob = out;
    if (fv->waves == 4)
      hipLaunchKernelGGL(unit_kernel<4>, dim3((unsigned)fv->grid), dim3(256), fv->lds, s, dv, qb, ob, flags, advance, fv->lds_main, vb, kb);
    else
      hipLaunchKernelGGL(unit_kernel<2>, dim3((unsigned)fv->grid), dim3(128), fv->lds, s, dv, qb, ob, flags, advance, fv->lds_main, vb, kb);
    CKV_HIP(c, hipGetLastError());
    if (c->profile) CKV_HIP(c, hipEventRecord(e1, s));
    if (flags & kLeaveMany)
      if (int rc = launch_evict(c, s, begin, count, -1, 1)) return rc;
    if (advance && (flags & CKV_FUSE_EVICT)) return rebalance_after_eviction(c);
    return CKV_OK;
  }
  // Few units: several workgroups per unit, what follows the attention by a unit's last one, or in a kernel of its own.
  const long long mean = mean_budget(c);
  const int mode = (flags & CKV_ATTENTION_ONLY) ? (attends_apart(mean, count, c->lay.cap, c->n_cu) ? kAttendOnly : kAttend)
                   : books_apart(mean, count, c->lay.cap, c->n_cu, kLayerThreads, 12 * kLayerThreads) ? kScanOnly : kWholeStep;
  const uint32_t kflags = flags & (CKV_FUSE_EVICT | kLeaveMany);
  if (int rc = launch_layer_step(c, s, begin, count, (const uint16_t*)q, (const uint16_t*)k_new, (const uint16_t*)v_new, out, kflags, mode, advance)) return rc;
  if (c->profile) CKV_HIP(c, hipEventRecord(e1, s));
  if (mode == kScanOnly)
    if (int rc = launch_finish(c, s, begin, count, kflags)) return rc;
  if (mode == kAttendOnly) {
    hipLaunchKernelGGL(append_kernel, dim3(1), dim3(kWideThreads), 0, s, c->dev, begin, count, advance);
    CKV_HIP(c, hipGetLastError());
  }
  if (flags & kLeaveMany)
    if (int rc = launch_evict(c, s, begin, count, -1, 1)) return rc;
  if (advance && (flags & CKV_FUSE_EVICT)) return rebalance_after_eviction(c);
  return CKV_OK;
}

int ckv_seed_prompt(ckv_ctx* c, int32_t layer, const void* q_obs, int32_t W, void* stream) {
  if (!c) return CKV_EINVAL;
  if (layer < 0 || layer >= c->lay.n_layers) return fail(c, CKV_EINVAL, "layer out of range");
  if (!q_obs) return fail(c, CKV_EINVAL, "q_obs is NULL");
  if (c->next_layer != 0) return fail(c, CKV_ESTATE, "a per-layer step is in progress");
  const int P = c->prompt_len[layer];
  if (P < 0) return fail(c, CKV_ESTATE, "needs a prompt loaded whole (ckv_load_prompt) and not touched since");
  if (W < 1 || W > P) return fail(c, CKV_EINVAL, "need 1 <= W <= P");
  hipStream_t s = (hipStream_t)stream;
  if (int rc = join_side(c, s)) return rc;
  const int begin = layer * c->units_per_layer, count = c->units_per_layer;
  // Groups of 16 queries fill G tiles of 16 columns each.  Per batch of groups: a pass over the keys for the softmax
  // partials of all its queries, their maxima and sums, a second pass for the mean weights, the hits (top-p rule),
  // the score recurrence.  The batch's softmax partials live in the decode paths' partials, its weights in their logits (a row
  // of cap floats per unit and query: G rows of every unit) when those hold at least two groups, else in the replay's own
  // buffer for one (partials and logits are idle here and rewritten by the next scan before anything reads them).
  const int G = c->dev.G;
  const int fit = std::min(c->lay.n_layers * G / kSeedGroup, kSeedTiles / G);
  float *ml = c->dev.partial, *rw = c->seedrw, *mi = c->seedmi;
  int groups = 1;
  if (fit >= 2) {
    groups = fit;
    rw = c->dev.logits;
  }
  const int batch = groups * kSeedGroup;
  const bool topp = c->par.reward_mode == CKV_REWARD_TOPP_HIT;
  for (int j0 = 0; j0 < W; j0 += batch) {
    const int nq = std::min(batch, (int)W - j0), nt = (nq + kSeedGroup - 1) / kSeedGroup * G;
    const int S = seed_spans(c, P - W + j0 + nq, count);
    const dim3 sgrid((unsigned)((S + 3) / 4), (unsigned)count);
    hipLaunchKernelGGL(seed_scan_kernel, sgrid, dim3(kThreads), (size_t)seed_scan_tiles(G, nq) * 4096, s, c->dev, begin, (const uint16_t*)q_obs, j0, nq, P, (int)W, S, ml);
    CKV_HIP(c, hipGetLastError());
    hipLaunchKernelGGL(seed_stats_kernel, dim3((unsigned)count, (unsigned)seed_scan_tiles(G, nq)), dim3(8 * kSeedCols), 0, s, S, (const float*)ml, mi);
    CKV_HIP(c, hipGetLastError());
    hipLaunchKernelGGL(seed_weights_kernel, sgrid, dim3(kThreads), (size_t)nt * 4096, s, c->dev, begin, (const uint16_t*)q_obs, j0, nq, P, (int)W, S,
                       (const float*)mi, rw);
    CKV_HIP(c, hipGetLastError());
    if (topp) {
      const int per = (P - W + j0 + nq + kSeedThreads - 1) / kSeedThreads;          // entries per thread of the longest row
      auto hits = [&](auto kernel, size_t lds) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)nq, (unsigned)count), dim3(kSeedThreads), lds, s, c->dev, begin, j0, P, (int)W, rw);
      };
      // The fewest registers that hold the row, in steps of four (one step more than needed costs the whole call 2-3 % at 32
      // queries: 6100 entries 181 us with 12, 185 with 16; 9350 entries 247 with 20, 252 with 24; 12000 entries 290 with 24,
      // 298 with 28; in LDS instead of 32 registers, 16384 entries, 562 against 355).
      constexpr size_t list = kSeedHitsLds;
      switch ((per + 3) / 4) {
        case 0: case 1: case 2: hits(seed_hits_kernel<8>, list); break;
        case 3: hits(seed_hits_kernel<12>, list); break;
        case 4: hits(seed_hits_kernel<16>, list); break;
        case 5: hits(seed_hits_kernel<20>, list); break;
        case 6: hits(seed_hits_kernel<24>, list); break;
        case 7: hits(seed_hits_kernel<28>, list); break;
        case 8: hits(seed_hits_kernel<32>, list); break;
        default: hits(seed_hits_kernel<0>, c->finish_lds);
      }
      CKV_HIP(c, hipGetLastError());
    }
    const dim3 cgrid((unsigned)((P + 4 * kThreads - 1) / (4 * kThreads)), (unsigned)count);
    if (topp && c->dev.tab_last < kTabLds)                 // LDS holds the whole table (lambda up to 0.7)
      hipLaunchKernelGGL(seed_crf_hits_kernel, cgrid, dim3(kThreads), 0, s, c->dev, begin, j0, nq, P, (int)W, c->par.t0 - 1, (const uint32_t*)rw);
    else if (topp)
      hipLaunchKernelGGL(seed_crf_kernel<true>, cgrid, dim3(kThreads), 0, s, c->dev, begin, j0, nq, P, (int)W, c->par.t0 - 1, (const float*)rw);
    else
      hipLaunchKernelGGL(seed_crf_kernel<false>, cgrid, dim3(kThreads), 0, s, c->dev, begin, j0, nq, P, (int)W, c->par.t0 - 1, (const float*)rw);
    CKV_HIP(c, hipGetLastError());
  }
  return CKV_OK;
}

int ckv_evict(ckv_ctx* c, int32_t layer, void* stream) {
  if (!c) return CKV_EINVAL;
  int begin, count;
  if (int rc = layer_range(c, layer, &begin, &count)) return rc;
  for (int l = (layer == -1 ? 0 : layer); l < (layer == -1 ? c->lay.n_layers : layer + 1); ++l) c->prompt_len[l] = -1;
  if (int rc = join_side(c, (hipStream_t)stream)) return rc;
  if (int rc = launch_evict(c, (hipStream_t)stream, begin, count, -1)) return rc;
  if (layer == -1 || layer == c->lay.n_layers - 1) return rebalance_after_eviction(c);
  return CKV_OK;
}

int ckv_evict_window(ckv_ctx* c, int32_t layer, int32_t n_sink, void* stream) {
  if (!c) return CKV_EINVAL;
  if (n_sink < 0) return fail(c, CKV_EINVAL, "n_sink is negative");
  int begin, count;
  if (int rc = layer_range(c, layer, &begin, &count)) return rc;
  for (int l = (layer == -1 ? 0 : layer); l < (layer == -1 ? c->lay.n_layers : layer + 1); ++l) c->prompt_len[l] = -1;
  if (int rc = join_side(c, (hipStream_t)stream)) return rc;
  if (int rc = launch_evict(c, (hipStream_t)stream, begin, count, (int)n_sink)) return rc;
  if (layer == -1 || layer == c->lay.n_layers - 1) return rebalance_after_eviction(c);
  return CKV_OK;
}

int ckv_rebudget(ckv_ctx* c, void* stream) {
  if (!c) return CKV_EINVAL;
  if (c->next_layer != 0) return fail(c, CKV_ESTATE, "a per-layer step is in progress");
  if (int rc = join_side(c, (hipStream_t)stream)) return rc;
  const size_t level2 = (size_t)c->lay.n_layers * c->lay.n_kv_heads * 25;
  const bool in_lds = level2 <= 48 * 1024;
  hipLaunchKernelGGL(rebudget_kernel, dim3((unsigned)c->lay.batch), dim3(kThreads), in_lds ? level2 : 0, (hipStream_t)stream, c->dev, in_lds ? 1 : 0);
  CKV_HIP(c, hipGetLastError());
  c->dirty = true;             // shared pools: the segments follow once the shrunken units have evicted
  c->many.assign(c->lay.n_layers, 1);
  c->excess.assign(c->lay.n_layers, kManyEntries);
  return launch_schedule(c, (hipStream_t)stream);
}

int ckv_rebalance(ckv_ctx* c, void* stream) {
  if (!c) return CKV_EINVAL;
  if (c->next_layer != 0) return fail(c, CKV_ESTATE, "a per-layer step is in progress");
  if (int rc = join_side(c, (hipStream_t)stream)) return rc;
  c->due = false;
  return launch_rebalance(c, (hipStream_t)stream);
}

int64_t ckv_pool_slots(const ckv_layout* l, const int32_t* budgets, int32_t prompt_len) {
  if (!l || !budgets || l->n_layers < 1 || l->batch < 1 || l->n_kv_heads < 1 || l->cap < kBlk || prompt_len < 0) return 0;
  const long long units = (long long)l->n_layers * l->batch * l->n_kv_heads, mseg = (l->cap + kSeg - 1) / kSeg;
  if (l->headroom <= 0) return units * mseg * kSeg;
  long long total = 0;
  for (long long u = 0; u < units; ++u) total += (long long)budgets[u] + l->headroom;
  // whatever Alg. 2 makes of the budgets, rounding to segments wastes less than one segment per unit
  long long segs = (total + kSeg - 1) / kSeg + units;
  if (prompt_len > 0) segs += (long long)l->batch * l->n_kv_heads * std::min<long long>(mseg, ((long long)prompt_len + l->headroom + kSeg - 1) / kSeg);
  return std::min(segs, units * mseg) * kSeg;
}

int ckv_probe(ckv_ctx* c, int32_t layer, const void* q_probe, uint8_t* classes, void* stream) {
  if (!c) return CKV_EINVAL;
  if (!q_probe || !classes) return fail(c, CKV_EINVAL, "q_probe or classes is NULL");
  if (layer < 0 || layer >= c->lay.n_layers) return fail(c, CKV_EINVAL, "layer out of range");
  if (c->next_layer != 0) return fail(c, CKV_ESTATE, "a per-layer step is in progress");
  const int begin = layer * c->units_per_layer, count = c->units_per_layer;
  hipStream_t s = (hipStream_t)stream;
  if (int rc = join_side(c, s)) return rc;
  return launch_probe(c, c->dev, begin, count, (const uint16_t*)q_probe, classes, s);
}

int ckv_probe_noalloc(ckv_ctx* c, int32_t layer, const void* q_probe, uint8_t* classes, void* stream) {
  if (!c) return CKV_EINVAL;
  if (!q_probe || !classes) return fail(c, CKV_EINVAL, "q_probe or classes is NULL");
  if (layer < 0 || layer >= c->lay.n_layers) return fail(c, CKV_EINVAL, "layer out of range");
  if (c->next_layer != 0) return fail(c, CKV_ESTATE, "a per-layer step is in progress");
  int devid = -1;
  if (hipGetDevice(&devid) != hipSuccess) return fail(c, CKV_EHIP, "hipGetDevice failed");
  if (devid != c->device) return fail(c, CKV_ESTATE, "the context's device is not the current one");
  unsigned char* base = g_scratch_ptr[devid];     // set by ckv_init on this device
  if (!base) return fail(c, CKV_ESTATE, "the library's scratch was not set up on this device");
  const int begin = layer * c->units_per_layer, count = c->units_per_layer;
  // The layer's logits and softmax statistics, carved from the static array instead of the context's workspace.
  // What a layer may need at most is a documented limit and stays what it was when the scan also kept a work list,
  // stamps and merged partials there.
  const size_t U = (size_t)count, G = (size_t)c->dev.G, mc = (size_t)c->dev.max_chunks, slots = mc + 1;
  const size_t o_partial = align_up(SC_COUNT * 4) + align_up(U * mc * 16) + align_up(U * slots * 4) + align_up(U * slots * G * 2 * 4),
               o_logits = o_partial + align_up(U * slots * G * kDim * 4), off = o_logits + align_up(U * G * (size_t)c->dev.cap * 4);
  if (off > kScratchBytes)
    return fail(c, CKV_EWORKSPACE, "one layer's scan scratch (" + std::to_string(off >> 20) + " MiB) exceeds the library's static scratch of " +
                                       std::to_string(kScratchBytes >> 20) + " MiB: use ckv_probe");
  // the layer's units as units 0 .. count-1 of a context of their own
  Dev ds = c->dev;
  ds.units = count;
  ds.tbl += (size_t)begin * c->dev.max_seg;      // the rows name pool segments: the pools stay where they are
  ds.n += begin;
  ds.partial = reinterpret_cast<float*>(base + o_partial);
  ds.logits = reinterpret_cast<float*>(base + o_logits);
  hipStream_t s = (hipStream_t)stream;
  if (int rc = join_side(c, s)) return rc;
  return launch_probe(c, ds, 0, count, (const uint16_t*)q_probe, classes, s);
}

int ckv_get_budgets(ckv_ctx* c, int32_t* budgets) {
  if (!c || !budgets) return CKV_EINVAL;
  if (int rc = flush_group(c)) return rc;
  CKV_HIP(c, hipDeviceSynchronize());
  CKV_HIP(c, hipMemcpy(budgets, c->dev.budget, (size_t)c->units * 4, hipMemcpyDeviceToHost));
  return CKV_OK;
}

int ckv_get_lengths(ckv_ctx* c, int32_t* lengths) {
  if (!c || !lengths) return CKV_EINVAL;
  if (int rc = flush_group(c)) return rc;
  CKV_HIP(c, hipDeviceSynchronize());
  CKV_HIP(c, hipMemcpy(lengths, c->dev.n, (size_t)c->units * 4, hipMemcpyDeviceToHost));
  return CKV_OK;
}

int ckv_get_segments(ckv_ctx* c, int32_t* owned, int32_t* rows, int32_t* spare, int32_t* n_spare) {
  if (!c || !n_spare) return CKV_EINVAL;
  if (int rc = flush_group(c)) return rc;
  CKV_HIP(c, hipDeviceSynchronize());
  CKV_HIP(c, hipMemcpy(n_spare, c->dev.sc + SC_SPARE, 4, hipMemcpyDeviceToHost));
  if (*n_spare < 0 || *n_spare > c->lay.pool_slots / kSeg) return fail(c, CKV_ESTATE, "corrupt spare list");
  if (owned) CKV_HIP(c, hipMemcpy(owned, c->dev.owned, (size_t)c->units * 4, hipMemcpyDeviceToHost));
  if (rows) CKV_HIP(c, hipMemcpy(rows, c->dev.tbl, (size_t)c->units * c->dev.max_seg * 4, hipMemcpyDeviceToHost));
  if (spare && *n_spare > 0) CKV_HIP(c, hipMemcpy(spare, c->dev.spare, (size_t)*n_spare * 4, hipMemcpyDeviceToHost));
  return CKV_OK;
}

int ckv_set_budgets(ckv_ctx* c, const int32_t* budgets) {
  if (!c) return CKV_EINVAL;
  if (int rc = check_budgets(c, &c->lay, &c->par, budgets)) return rc;
  if (int rc = flush_group(c)) return rc;
  CKV_HIP(c, hipDeviceSynchronize());
  c->dirty = true;
  c->many.assign(c->lay.n_layers, 1);
  c->excess.assign(c->lay.n_layers, kManyEntries);
  return upload_budgets(c, budgets, nullptr);
}

int ckv_get_time(ckv_ctx* c, int32_t* t) {
  if (!c || !t) return CKV_EINVAL;
  if (int rc = flush_group(c)) return rc;
  CKV_HIP(c, hipDeviceSynchronize());
  CKV_HIP(c, hipMemcpy(t, c->dev.sc + SC_T, 4, hipMemcpyDeviceToHost));
  return CKV_OK;
}

int ckv_set_time(ckv_ctx* c, int32_t t) {
  if (!c || t < 0) return CKV_EINVAL;
  if (c->next_layer != 0) return fail(c, CKV_ESTATE, "a per-layer step is in progress");
  CKV_HIP(c, hipDeviceSynchronize());
  int32_t zero = 0;
  CKV_HIP(c, hipMemcpy(c->dev.sc + SC_T, &t, 4, hipMemcpyHostToDevice));
  CKV_HIP(c, hipMemcpy(c->dev.sc + SC_WINDOW_STEPS, &zero, 4, hipMemcpyHostToDevice));
  if (int rc = fill32(c, c->dev.window, 0u, (size_t)c->units * 2, nullptr)) return rc;
  CKV_HIP(c, hipDeviceSynchronize());
  return CKV_OK;
}

int ckv_status(ckv_ctx* c) {
  if (!c) return CKV_EINVAL;
  CKV_HIP(c, hipDeviceSynchronize());
  int32_t st = 0, zero = 0;
  CKV_HIP(c, hipMemcpy(&st, c->dev.sc + SC_STATUS, 4, hipMemcpyDeviceToHost));
  if (st) {
    CKV_HIP(c, hipMemcpy(c->dev.sc + SC_STATUS, &zero, 4, hipMemcpyHostToDevice));
    if (st & 4) return fail(c, CKV_ECAPACITY, "the spare list ran short when the pool segments were dealt out: some units own less than budget + headroom needs");
    return fail(c, CKV_ECAPACITY, "an append found its unit full");
  }
  return CKV_OK;
}

// The unit's row of the segment table and the number of segments it owns (the device is idle).
static int read_row(ckv_ctx* c, size_t u, std::vector<int32_t>* row, int32_t* own) {
  row->resize((size_t)c->dev.max_seg);
  CKV_HIP(c, hipMemcpy(row->data(), c->dev.tbl + u * c->dev.max_seg, row->size() * 4, hipMemcpyDeviceToHost));
  CKV_HIP(c, hipMemcpy(own, c->dev.owned + u, 4, hipMemcpyDeviceToHost));
  if (*own < 0 || *own > c->dev.max_seg) return fail(c, CKV_ESTATE, "corrupt segment table");
  return CKV_OK;
}

int ckv_export_unit(ckv_ctx* c, int32_t layer, int32_t seq, int32_t head, int32_t* n_out, int32_t* nev_out,
                    int32_t* budget_out, uint16_t* K, uint16_t* V, float* crf, int32_t* tau, int32_t* pos,
                    uint8_t* flags) {
  if (!c) return CKV_EINVAL;
  if (layer < 0 || layer >= c->lay.n_layers || seq < 0 || seq >= c->lay.batch || head < 0 || head >= c->lay.n_kv_heads)
    return fail(c, CKV_EINVAL, "unit index out of range");
  const size_t u = ((size_t)layer * c->lay.batch + seq) * c->lay.n_kv_heads + head;
  const size_t cap = (size_t)c->lay.cap;
  if (int rc = flush_group(c)) return rc;
  CKV_HIP(c, hipDeviceSynchronize());
  // the unit's slots, segment by segment (what it does not own stays zero on the host side)
  std::vector<int32_t> row;
  int32_t own = 0;
  if (int rc = read_row(c, u, &row, &own)) return rc;
  auto fetch = [&](void* host, const void* pool, size_t elem_bytes) -> int {      // per-slot array
    std::memset(host, 0, cap * elem_bytes);
    for (int j = 0; j < own; ++j) {
      const size_t cnt = std::min<size_t>(kSeg, cap - (size_t)j * kSeg);
      CKV_HIP(c, hipMemcpy((char*)host + (size_t)j * kSeg * elem_bytes, (const char*)pool + (size_t)row[j] * kSeg * elem_bytes,
                           cnt * elem_bytes, hipMemcpyDeviceToHost));
    }
    return CKV_OK;
  };
  int32_t n = 0, nev = 0, bud = 0;
  CKV_HIP(c, hipMemcpy(&n, c->dev.n + u, 4, hipMemcpyDeviceToHost));
  CKV_HIP(c, hipMemcpy(&nev, c->dev.nev + u, 4, hipMemcpyDeviceToHost));
  CKV_HIP(c, hipMemcpy(&bud, c->dev.budget + u, 4, hipMemcpyDeviceToHost));
  if (n_out) *n_out = n;
  if (nev_out) *nev_out = nev;
  if (budget_out) *budget_out = bud;
  std::vector<uint16_t> tmp;
  for (int which = 0; which < 2; ++which) {
    uint16_t* dst = which == 0 ? K : V;
    if (!dst) continue;
    tmp.resize(kSegElems);
    std::memset(dst, 0, cap * kDim * 2);
    for (int j = 0; j < own; ++j) {
      CKV_HIP(c, hipMemcpy(tmp.data(), (which == 0 ? c->dev.K : c->dev.V) + (size_t)row[j] * kSegElems, (size_t)kSegElems * 2, hipMemcpyDeviceToHost));
      for (int rr = 0; rr < kSeg && (size_t)j * kSeg + rr < cap; ++rr)
        for (int col = 0; col < kDim; ++col)
          dst[((size_t)j * kSeg + rr) * kDim + col] = tmp[which == 0 ? k_offset(rr, col) : v_offset(rr, col)];
    }
  }
  if (crf) if (int rc = fetch(crf, c->dev.crf, 4)) return rc;
  if (tau) if (int rc = fetch(tau, c->dev.tau, 4)) return rc;
  if (pos) if (int rc = fetch(pos, c->dev.pos, 4)) return rc;
  if (flags) {
    if (int rc = fetch(flags, c->dev.flags, 1)) return rc;
    // the hit mark is not stored: in the top-p mode an entry was hit in the unit's last step iff its tau is that step
    int32_t tu = 0;
    CKV_HIP(c, hipMemcpy(&tu, c->dev.t_unit + u, 4, hipMemcpyDeviceToHost));
    if (c->dev.reward_mode == 0 && tu >= c->par.t0 && n > 0) {
      std::vector<int32_t> th(cap);
      if (int rc = fetch(th.data(), c->dev.tau, 4)) return rc;
      for (int i = 0; i < n; ++i)
        if (th[i] == tu) flags[i] |= CKV_FLAG_HIT;
    }
  }
  return CKV_OK;
}

int ckv_import_unit(ckv_ctx* c, int32_t layer, int32_t seq, int32_t head, int32_t n, const uint16_t* K,
                    const uint16_t* V, const float* crf, const int32_t* tau, const int32_t* pos, int32_t t_unit) {
  if (!c) return CKV_EINVAL;
  if (layer < 0 || layer >= c->lay.n_layers || seq < 0 || seq >= c->lay.batch || head < 0 || head >= c->lay.n_kv_heads)
    return fail(c, CKV_EINVAL, "unit index out of range");
  if (n < 0 || n >= c->lay.cap) return fail(c, CKV_EINVAL, "need 0 <= n < cap");
  if (n > 0 && (!K || !V || !crf || !tau || !pos)) return fail(c, CKV_EINVAL, "NULL state array");
  const size_t u = ((size_t)layer * c->lay.batch + seq) * c->lay.n_kv_heads + head;
  if (int rc = flush_group(c)) return rc;
  CKV_HIP(c, hipDeviceSynchronize());
  std::vector<int32_t> row;
  int32_t own = 0;
  if (int rc = read_row(c, u, &row, &own)) return rc;
  if (n >= std::min<long long>(c->lay.cap, (long long)own * kSeg)) return fail(c, CKV_ECAPACITY, "the unit's segments do not hold n + 1 entries");
  const int nseg = (n + kSeg - 1) / kSeg;
  std::vector<uint16_t> tmp((size_t)kSegElems);
  for (int which = 0; which < 2 && n > 0; ++which) {
    const uint16_t* src = which == 0 ? K : V;
    for (int j = 0; j < nseg; ++j) {
      std::fill(tmp.begin(), tmp.end(), (uint16_t)0);
      for (int rr = 0; rr < kSeg && j * kSeg + rr < n; ++rr)
        for (int col = 0; col < kDim; ++col)
          tmp[which == 0 ? k_offset(rr, col) : v_offset(rr, col)] = src[((size_t)j * kSeg + rr) * kDim + col];
      const size_t used = (size_t)((std::min(n - j * kSeg, kSeg) + kBlk - 1) / kBlk) * kBlkElems;      // whole blocks
      CKV_HIP(c, hipMemcpy((which == 0 ? c->dev.K : c->dev.V) + (size_t)row[j] * kSegElems, tmp.data(), used * 2, hipMemcpyHostToDevice));
    }
  }
  if (n > 0) {
    std::vector<uint8_t> zf(kSeg, 0);
    for (int j = 0; j < nseg; ++j) {
      const size_t cnt = (size_t)std::min(n - j * kSeg, kSeg), s0 = (size_t)row[j] * kSeg, h0 = (size_t)j * kSeg;
      CKV_HIP(c, hipMemcpy(c->dev.crf + s0, crf + h0, cnt * 4, hipMemcpyHostToDevice));
      CKV_HIP(c, hipMemcpy(c->dev.tau + s0, tau + h0, cnt * 4, hipMemcpyHostToDevice));
      CKV_HIP(c, hipMemcpy(c->dev.pos + s0, pos + h0, cnt * 4, hipMemcpyHostToDevice));
      CKV_HIP(c, hipMemcpy(c->dev.flags + s0, zf.data(), cnt, hipMemcpyHostToDevice));
    }
  }
  int32_t zero = 0;
  CKV_HIP(c, hipMemcpy(c->dev.n + u, &n, 4, hipMemcpyHostToDevice));
  CKV_HIP(c, hipMemcpy(c->dev.nev + u, &zero, 4, hipMemcpyHostToDevice));
  CKV_HIP(c, hipMemcpy(c->dev.t_unit + u, &t_unit, 4, hipMemcpyHostToDevice));
  c->prompt_loaded[layer] = 1;
  c->prompt_len[layer] = -1;
  c->excess[layer] = kManyEntries;
  return CKV_OK;
}

int ckv_profile_enable(ckv_ctx* c, int32_t on) {
  if (!c) return CKV_EINVAL;
  if (int rc = flush_group(c)) return rc;
  CKV_HIP(c, hipDeviceSynchronize());
  c->profile = on != 0;
  c->ev_used = 0;
  c->scan_ms = 0.0;
  c->scan_launches = 0;
  return CKV_OK;
}

int ckv_profile_read(ckv_ctx* c, double* scan_ms, int32_t* launches) {
  if (!c) return CKV_EINVAL;
  CKV_HIP(c, hipDeviceSynchronize());
  for (size_t i = 0; i + 1 < c->ev_used; i += 2) {
    float ms = 0.f;
    CKV_HIP(c, hipEventElapsedTime(&ms, c->ev[i], c->ev[i + 1]));
    c->scan_ms += ms;
    c->scan_launches += 1;
  }
  c->ev_used = 0;
  if (scan_ms) *scan_ms = c->scan_ms;
  if (launches) *launches = c->scan_launches;
  return CKV_OK;
}

int ckv_bandwidth_probe(const void* src, void* dst, size_t bytes, void* sink, void* stream) {
  if (!src || !sink || bytes < (1u << 20) || ((uintptr_t)src % 16) != 0 || ((uintptr_t)dst % 16) != 0) return CKV_EINVAL;
  int devid = 0, n_cu = 0;
  if (hipGetDevice(&devid) != hipSuccess ||
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, devid) != hipSuccess || n_cu <= 0)
    return CKV_EHIP;
  const size_t n_vec = bytes / 16;
  if (dst)
    hipLaunchKernelGGL(probe_copy_kernel, dim3((unsigned)(n_cu * 32)), dim3(kThreads), 0, (hipStream_t)stream,
                       (const u32x4*)src, (u32x4*)dst, n_vec);
  else
    hipLaunchKernelGGL(probe_read_kernel, dim3((unsigned)n_cu), dim3(kThreads), 0, (hipStream_t)stream,
                       (const u32x4*)src, n_vec, (uint32_t*)sink);
  return hipGetLastError() == hipSuccess ? CKV_OK : CKV_EHIP;
}

int ckv_set_path(ckv_ctx* c, int32_t mode) {
  if (!c || mode < 0 || mode > 4) return CKV_EINVAL;
  const bool any = c->fused[0].ok || c->fused[1].ok;
  if ((mode == 2 && !any) || (mode == 3 && !c->fused[0].ok) || (mode == 4 && !c->fused[1].ok))
    return fail(c, CKV_EINVAL, "cap too large for the fused kernel's LDS");
  c->path_mode = mode;
  return CKV_OK;
}

int ckv_path_info(ckv_ctx* c, int32_t* fused_waves, int32_t* lds_main_bytes) {
  if (!c) return CKV_EINVAL;
  const ckv_ctx::Fused* f = fused_variant(c);
  if (f && c->path_mode == 0 && c->units < f->grid) f = nullptr;
  if (fused_waves) *fused_waves = f ? f->waves : 0;
  if (lds_main_bytes) *lds_main_bytes = f ? f->lds_main : 0;
  return CKV_OK;
}

int ckv_join(ckv_ctx* c, void* stream) {
  if (!c) return CKV_EINVAL;
  return join_side(c, (hipStream_t)stream);
}

const char* ckv_strerror(int code) {
  switch (code) {
    case CKV_OK: return "ok";
    case CKV_EINVAL: return "invalid argument";
    case CKV_ECAPACITY: return "unit full at append";
    case CKV_ESTATE: return "call not valid in this state";
    case CKV_EHIP: return "HIP runtime error";
    case CKV_EWORKSPACE: return "workspace too small or misaligned";
    default: return "unknown error";
  }
}

const char* ckv_last_error(const ckv_ctx* c) { return c ? c->err.c_str() : ""; }


}  // extern "C"
