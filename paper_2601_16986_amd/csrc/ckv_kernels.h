// Device code of the Crystal-KV decode path for gfx950 (64-lane wavefronts,
// v_mfma_f32_16x16x32_bf16).  One decode step runs as one of
//
//   unit_kernel<W> (ckv_unit_kernel.h)  everything in one persistent kernel, a workgroup per unit at a time
//   layer_step_kernel (ckv_layer_kernel.h)  the units of one layer, or of a small context: append, attention and output with
//                  several workgroups per unit, then the bookkeeping (mean attention weight per entry, top-p hit mask, CRF
//                  update, aggregated CRF, and, optionally, eviction + compaction) by the workgroup that finishes the unit
//   layer_step_kernel, finish_kernel   the same with the bookkeeping in a kernel of its own, one workgroup per unit: straight behind
//                  where that is faster (books_apart), or later, on a stream of the context's (deferred)
//   layer_step_kernel, append_kernel   an attention-only step whose records have a launch of their own (attends_apart)
//
// and beside the step:
//
//   load_cache_kernel   fills a layer's caches
//   seed_scan_kernel, seed_stats_kernel, seed_weights_kernel, seed_hits_kernel, seed_crf_hits_kernel, seed_crf_kernel   scores of a loaded prompt from its last queries
//   evict_kernel, evict_move_kernel   eviction + compaction on its own (Alg. 1 Step 4, or the sink + recent window policy)
//   probe_scan_kernel, probe_kernel   answer-probe classes
//   rebudget_kernel  Alg. 2 with integer apportionment, one workgroup/sequence
//   rebalance_kernel pool segments between units after budgets have changed
//   schedule_kernel  (ckv_unit_kernel.h) the fused kernel's order of units
//
// All floating-point code is compiled with -ffp-contract=off: the CRF update
// and Alg. 2 must round exactly as their definitions say.
#pragma once
#include <hip/hip_runtime.h>
#include <float.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "ckv_layout.h"
#include "ckv_plan.h"

namespace ckv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned long long u64;

enum { SC_T = 0, SC_WINDOW_STEPS = 1, SC_DONE = 2, SC_STATUS = 3, SC_DONE_RB = 4, SC_QUEUE = 5, SC_SPARE = 6, SC_COUNT = 64 };
enum { FLAG_HIT = 1, FLAG_SLIP = 2 };
constexpr uint32_t kLeaveMany = 8u;       // a step's call flag: evictions of several entries from a unit are left to the evict_kernel that follows
// whether a step leaves a unit of so many entries above its budget to that kernel, which is faster at it
__device__ __forceinline__ bool leaves_unit(uint32_t call_flags, int excess) { return (call_flags & kLeaveMany) && excess > 1; }
constexpr int kThreads = 256;
constexpr int kWideThreads = 1024;        // kernels with one workgroup per unit and few units
constexpr int kMaxChunks = 128;           // cap <= 32768
constexpr float kFixedOne = 1048576.0f;   // 2^20: resolution of the aggregated-CRF accumulator
constexpr int kTabLds = 256;              // decay-table entries kept in LDS by the LRFU kernels

struct Dev {
  int32_t L, Bz, Hq, Hkv, G, cap, units, max_chunks, slots, out_bf16;   // slots = partial slots per unit
  int32_t unit0;         // fused kernel: unit whose rows come first in the call's q, k_new, v_new and out (a single layer's first unit)
  int32_t by_order;      // fused kernel: schedule slot i holds unit order[i] (all layers), else unit unit0 + i (one layer)
  float scale_log2e;     // softmax_scale * log2(e): logits are kept in the base-2 domain
  float top_p;
  int32_t reward_mode, bmin, bmax, tab_last;
  uint16_t* K;
  uint16_t* V;
  float* crf;
  int32_t* tau;
  int32_t* pos;
  uint8_t* flags;
  int32_t* tbl;          // [units][max_seg] segment table: the pool segments (256 slots each) a unit's entries live in, in order
  int32_t max_seg;       // cap / 256, rounded up: columns of tbl
  int32_t* owned;        // [units] segments the unit owns: the first owned[u] entries of its row (the others hold 0)
  int32_t* spare;        // pool segments no unit owns, a stack of sc[SC_SPARE] entries
  int32_t* n;            // [units] entries held
  int32_t* budget;       // [units]
  int32_t* t_unit;       // [units] time of the unit's last decode step
  int32_t* nev;          // [units] entries evicted by the last eviction
  u64* window;           // [units] fixed-point sum of aggregated CRF since the last re-allocation
  int32_t* sc;           // scalars, SC_*
  const float* tab;      // lambda^delta, delta = 0..tab_last
  float* partial;        // [units*slots][G][128] attention accumulated by one workgroup of a scan, a slot each
  float* ml;             // [units*slots][G][2] (running max, sum)
  float* logits;         // [units][cap/32][G][32] scaled logits (base-2 domain)
  long long* btotal;     // [Bz] budget total per sequence
  int32_t* order;        // [units] unit indices by descending budget (schedule of the fused kernel)
  int32_t* layer_ts;     // [layers] time of a layer's last step with its bookkeeping in a kernel of its own (layer_step_kernel -> finish_kernel)
  int32_t* arrive;       // [units] workgroups of the unit that have published their partial (zero between launches)
  float* msum;           // [units][8][2] softmax maximum (base-2 domain) and 1 / sum per query head, left by layer_step_kernel for finish_kernel
};



// Where a unit's entries live.  Pool memory (K, V and the per-slot arrays) is handed out in segments of 256
// slots; row u of the segment table names unit u's segments in order, so entry i sits in pool slot
// row[i / 256] * 256 + i % 256 and whole 256-entry chunks (what one wavefront or one workgroup of the
// single-layer scan, eight blocks of the fused kernel's stream cover) are contiguous.  `row` may point to a
// copy of the row in LDS.
struct Slots {
  const int32_t* row;
  // pool slot of entry i (index into crf / tau / pos / flags)
  __device__ __forceinline__ size_t operator+(int i) const { return (size_t)row[i >> 8] * kSeg + (size_t)(i & (kSeg - 1)); }
  // element offset in the K / V pool of block b (32 entries) of the unit
  __device__ __forceinline__ size_t blk(int b) const { return (size_t)row[b >> 3] * kSegElems + (size_t)(b & (kSegBlocks - 1)) * kBlkElems; }
  // element offset in the K / V pool of K[entry r][dim c] / V[entry r][dim c]
  __device__ __forceinline__ size_t k(int r, int c) const { return (size_t)row[r >> 8] * kSegElems + (size_t)k_offset(r & (kSeg - 1), c); }
  __device__ __forceinline__ size_t v(int r, int c) const { return (size_t)row[r >> 8] * kSegElems + (size_t)v_offset(r & (kSeg - 1), c); }
};
__device__ __forceinline__ Slots slots_of(const Dev& d, int u) { return Slots{d.tbl + (size_t)u * d.max_seg}; }
// entries unit u has room for: what its segments hold, `cap` at most
__device__ __forceinline__ int unit_cap(const Dev& d, int u) { return min(d.cap, d.owned[u] * kSeg); }

// ------------------------------------------------------------------ helpers
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Cross-lane moves inside a row of 16 lanes without going through LDS.
template <int kCtrl>
__device__ __forceinline__ int dpp_i32(int v) {
  return __builtin_amdgcn_update_dpp(0, v, kCtrl, 0xF, 0xF, true);
}
constexpr int kDppQuadSwap1 = 0xB1;      // quad_perm [1,0,3,2]
constexpr int kDppQuadSwap2 = 0x4E;      // quad_perm [2,3,0,1]
constexpr int kDppRowHalfMirror = 0x141;
constexpr int kDppRowMirror = 0x140;
constexpr int kDppRowShl = 0x100, kDppRowShr = 0x110;      // + 1 .. 15: from so many lanes up / down, 0 from beyond the row

// Lanes j, j + 16, j + 32 and j + 48 into one value, the same in all four: op(op(v0, v1), op(v2, v3)).  By swaps of rows, without a trip through LDS.
template <class Op>
__device__ __forceinline__ float rows_combine(float v, Op op) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(h[0]), __uint_as_float(h[1]));
}

// Maxima that are NaN if an operand is.
__device__ __forceinline__ float max2(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float max3(float a, float b, float c) { return max2(max2(a, b), c); }

// Sum over the 64 lanes, same fixed order in every lane: butterfly inside each
// row of 16 lanes, then the four row sums are read out and added.
__device__ __forceinline__ float wave_sum_f32(float v) {
  v += __int_as_float(dpp_i32<kDppQuadSwap1>(__float_as_int(v)));
  v += __int_as_float(dpp_i32<kDppQuadSwap2>(__float_as_int(v)));
  v += __int_as_float(dpp_i32<kDppRowHalfMirror>(__float_as_int(v)));
  v += __int_as_float(dpp_i32<kDppRowMirror>(__float_as_int(v)));
  const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
  const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
  const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
  const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
  return (r0 + r1) + (r2 + r3);
}

__device__ __forceinline__ int wave_sum_i32(int v) {
  v += dpp_i32<kDppQuadSwap1>(v);
  v += dpp_i32<kDppQuadSwap2>(v);
  v += dpp_i32<kDppRowHalfMirror>(v);
  v += dpp_i32<kDppRowMirror>(v);
  return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
         __builtin_amdgcn_readlane(v, 48);
}

template <int kCtrl>
__device__ __forceinline__ u64 dpp_u64(u64 v) {
  const uint32_t lo = (uint32_t)dpp_i32<kCtrl>((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)dpp_i32<kCtrl>((int)(uint32_t)(v >> 32));
  return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ u64 readlane_u64(u64 v, int lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
  return ((u64)hi << 32) | lo;
}

template <int kCtrl>
__device__ __forceinline__ double dpp_f64(double v) {
  return __longlong_as_double((long long)dpp_u64<kCtrl>((u64)__double_as_longlong(v)));
}
__device__ __forceinline__ double readlane_f64(double v, int lane) { return __longlong_as_double((long long)readlane_u64((u64)__double_as_longlong(v), lane)); }

__device__ __forceinline__ u64 wave_sum_u64(u64 v) {
  v += dpp_u64<kDppQuadSwap1>(v);
  v += dpp_u64<kDppQuadSwap2>(v);
  v += dpp_u64<kDppRowHalfMirror>(v);
  v += dpp_u64<kDppRowMirror>(v);
  return (readlane_u64(v, 0) + readlane_u64(v, 16)) + (readlane_u64(v, 32) + readlane_u64(v, 48));
}

// Sum over the lanes up to each: inside its row of 16, then the rows before.  (Six shuffles through LDS take 0.3 us, one after another.)
__device__ __forceinline__ int wave_scan_i32(int v, int lane) {
  v += dpp_i32<kDppRowShr + 1>(v);
  v += dpp_i32<kDppRowShr + 2>(v);
  v += dpp_i32<kDppRowShr + 4>(v);
  v += dpp_i32<kDppRowShr + 8>(v);
  const int row0 = __builtin_amdgcn_readlane(v, 15), row1 = row0 + __builtin_amdgcn_readlane(v, 31), row2 = row1 + __builtin_amdgcn_readlane(v, 47);
  return v + (lane < 16 ? 0 : lane < 32 ? row0 : lane < 48 ? row1 : row2);
}

__device__ __forceinline__ u64 min_u64(u64 a, u64 b) { return a < b ? a : b; }

__device__ __forceinline__ u64 wave_min_u64(u64 v) {
  v = min_u64(v, dpp_u64<kDppQuadSwap1>(v));
  v = min_u64(v, dpp_u64<kDppQuadSwap2>(v));
  v = min_u64(v, dpp_u64<kDppRowHalfMirror>(v));
  v = min_u64(v, dpp_u64<kDppRowMirror>(v));
  return min_u64(min_u64(readlane_u64(v, 0), readlane_u64(v, 16)), min_u64(readlane_u64(v, 32), readlane_u64(v, 48)));
}

// Barrier among the NT threads that work on one unit.  NT = 64: a single wavefront, which may be one of
// several in its workgroup and must not touch the workgroup barrier: its LDS and memory operations
// already execute in program order, only the compiler has to keep them so.
template <int NT>
struct alignas(16) RedBuf {
  u64 v[2][NT / 64];    // one slot per wavefront
  float t[2][NT / 64][4];
  int i[2][NT >= 512 ? NT / 64 : 1];
};

template <int NT>
__device__ __forceinline__ void block_sync(RedBuf<NT>& rb) {
  if constexpr (NT == 64) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// Block-wide reductions over NT threads with a fixed combination order
// (deterministic).  `rb` is a [2][NT/64] LDS array used alternately, so one
// barrier per call suffices.  NT = 64: the wavefront's own reduction, nothing else.
// With 8 or 16 wavefronts a lane reads one wavefront's value and the row of 16 lanes adds them up (every thread
// reading all 16 would put 256 LDS reads on the compute unit per call); with fewer every thread reads them all.
template <int NT>
constexpr bool kRowReduce = NT >= 512;

template <int NT, class T, class Op, class Dpp1, class Dpp2, class Dpp3, class Dpp4>
__device__ __forceinline__ T row_combine(T r, Op op, Dpp1 d1, Dpp2 d2, Dpp3 d3, Dpp4 d4) {
  static_assert(NT == 512 || NT == 1024, "8 or 16 wavefronts");
  r = op(r, d1(r));
  r = op(r, d2(r));
  r = op(r, d3(r));
  if constexpr (NT == 1024) r = op(r, d4(r));
  return r;
}

template <int NT = kThreads>
__device__ __forceinline__ u64 block_sum_u64(u64 v, RedBuf<NT>& rb, int& phase, int tid) {
  v = wave_sum_u64(v);
  if constexpr (NT == 64) return v;
  if ((tid & 63) == 0) rb.v[phase][tid >> 6] = v;
  block_sync<NT>(rb);
  u64 r;
  if constexpr (kRowReduce<NT>) {
    r = row_combine<NT>(rb.v[phase][tid & (NT / 64 - 1)], [](u64 a, u64 b) { return a + b; }, dpp_u64<kDppQuadSwap1>, dpp_u64<kDppQuadSwap2>,
                        dpp_u64<kDppRowHalfMirror>, dpp_u64<kDppRowMirror>);
  } else {
    r = rb.v[phase][0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) r += rb.v[phase][w];
  }
  phase ^= 1;
  return r;
}

template <int NT = kThreads>
__device__ __forceinline__ int block_sum_int(int v, RedBuf<NT>& rb, int& phase, int tid) {
  v = wave_sum_i32(v);
  if constexpr (NT == 64) return v;
  if ((tid & 63) == 0) rb.v[phase][tid >> 6] = (u64)(uint32_t)v;
  block_sync<NT>(rb);
  int r;
  if constexpr (kRowReduce<NT>) {
    r = row_combine<NT>((int)(uint32_t)rb.v[phase][tid & (NT / 64 - 1)], [](int a, int b) { return a + b; }, dpp_i32<kDppQuadSwap1>,
                        dpp_i32<kDppQuadSwap2>, dpp_i32<kDppRowHalfMirror>, dpp_i32<kDppRowMirror>);
  } else {
    r = (int)(uint32_t)rb.v[phase][0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) r += (int)(uint32_t)rb.v[phase][w];
  }
  phase ^= 1;
  return r;
}

// a value that is the same in all lanes, into scalar registers
__device__ __forceinline__ int uniform_i32(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform_f32(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }

template <int kCtrl>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(dpp_i32<kCtrl>(__float_as_int(v)));
}

template <int NT = kThreads>
__device__ __forceinline__ float block_sum_f32(float v, RedBuf<NT>& rb, int& phase, int tid) {
  v = wave_sum_f32(v);
  if constexpr (NT == 64) return v;
  if ((tid & 63) == 0) rb.v[phase][tid >> 6] = (u64)__float_as_uint(v);
  block_sync<NT>(rb);
  float r;
  if constexpr (kRowReduce<NT>) {
    r = row_combine<NT>(__uint_as_float((uint32_t)rb.v[phase][tid & (NT / 64 - 1)]), [](float a, float b) { return a + b; },
                        dpp_f32<kDppQuadSwap1>, dpp_f32<kDppQuadSwap2>, dpp_f32<kDppRowHalfMirror>, dpp_f32<kDppRowMirror>);
  } else {
    r = __uint_as_float((uint32_t)rb.v[phase][0]);
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) r += __uint_as_float((uint32_t)rb.v[phase][w]);
  }
  phase ^= 1;
  return r;
}

// Three sums at once (one barrier).
template <int NT = kThreads>
__device__ __forceinline__ void block_sum3_f32(float& x, float& y, float& z, RedBuf<NT>& rb, int& phase, int tid) {
  x = wave_sum_f32(x);
  y = wave_sum_f32(y);
  z = wave_sum_f32(z);
  if constexpr (NT == 64) return;
  if ((tid & 63) == 0) *reinterpret_cast<f32x4*>(rb.t[phase][tid >> 6]) = f32x4{x, y, z, 0.f};
  block_sync<NT>(rb);
  f32x4 r;
  if constexpr (kRowReduce<NT>) {
    r = *reinterpret_cast<const f32x4*>(rb.t[phase][tid & (NT / 64 - 1)]);
#pragma unroll
    for (int i = 0; i < 3; ++i)
      r[i] = row_combine<NT>(r[i], [](float a, float b) { return a + b; }, dpp_f32<kDppQuadSwap1>, dpp_f32<kDppQuadSwap2>,
                             dpp_f32<kDppRowHalfMirror>, dpp_f32<kDppRowMirror>);
  } else {
    r = *reinterpret_cast<const f32x4*>(rb.t[phase][0]);
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) {
      const f32x4 q = *reinterpret_cast<const f32x4*>(rb.t[phase][w]);
      r[0] += q[0];
      r[1] += q[1];
      r[2] += q[2];
    }
  }
  x = r[0];
  y = r[1];
  z = r[2];
  phase ^= 1;
}

template <int NT = kThreads>
__device__ __forceinline__ u64 block_min_u64(u64 v, RedBuf<NT>& rb, int& phase, int tid) {
  v = wave_min_u64(v);
  if constexpr (NT == 64) return v;
  if ((tid & 63) == 0) rb.v[phase][tid >> 6] = v;
  block_sync<NT>(rb);
  u64 r;
  if constexpr (kRowReduce<NT>) {
    r = row_combine<NT>(rb.v[phase][tid & (NT / 64 - 1)], [](u64 a, u64 b) { return min_u64(a, b); }, dpp_u64<kDppQuadSwap1>,
                        dpp_u64<kDppQuadSwap2>, dpp_u64<kDppRowHalfMirror>, dpp_u64<kDppRowMirror>);
  } else {
    r = rb.v[phase][0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) r = rb.v[phase][w] < r ? rb.v[phase][w] : r;
  }
  phase ^= 1;
  return r;
}

// The sum of `sum`, the smallest `key`, which comes back in every thread, and the `index` that came with it, in one barrier.
template <int NT>
__device__ __forceinline__ u64 block_sum_min(u64 sum, u64& key, int index, int& at, RedBuf<NT>& rb, int& phase, int tid) {
  constexpr int W = NT / 64;
  sum = wave_sum_u64(sum);
  const u64 least = wave_min_u64(key);
  const int mine = __builtin_amdgcn_readlane(index, __builtin_ctzll(__ballot(key == least)));
  if ((tid & 63) == 0) {
    *reinterpret_cast<u64*>(&rb.t[phase][tid >> 6][0]) = sum;
    *reinterpret_cast<u64*>(&rb.t[phase][tid >> 6][2]) = least;
    rb.i[phase][tid >> 6] = mine;
  }
  block_sync<NT>(rb);
  const int w = tid & (W - 1);                     // lane l looks at wavefront l % W
  sum = *reinterpret_cast<const u64*>(&rb.t[phase][w][0]);
  key = *reinterpret_cast<const u64*>(&rb.t[phase][w][2]);
  const int there = rb.i[phase][w];
  const u64 own = key;
  sum += dpp_u64<kDppQuadSwap1>(sum);
  key = min_u64(key, dpp_u64<kDppQuadSwap1>(key));
  if constexpr (W >= 4) {
    sum += dpp_u64<kDppQuadSwap2>(sum);
    key = min_u64(key, dpp_u64<kDppQuadSwap2>(key));
  }
  if constexpr (W >= 8) {
    sum += dpp_u64<kDppRowHalfMirror>(sum);
    key = min_u64(key, dpp_u64<kDppRowHalfMirror>(key));
  }
  if constexpr (W >= 16) {
    sum += dpp_u64<kDppRowMirror>(sum);
    key = min_u64(key, dpp_u64<kDppRowMirror>(key));
  }
  at = __builtin_amdgcn_readlane(there, __builtin_ctzll(__ballot(own == key)));
  phase ^= 1;
  return sum;
}

// ------------------------------------------------------------------ fill
__global__ void fill_u32_kernel(uint32_t* p, uint32_t v, size_t count) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < count; i += stride) p[i] = v;
}

// Everything a new context's device buffers start with, in one launch (nine fills, seven copies of a few hundred bytes, each
// staged by the runtime, and three waits were half of what making a small context took: a pass that makes one, admits a prompt of 777 tokens
// to four layers and takes three steps 487 -> 387 us, the step's shorter way through the binding included): regions of one value, 16 bytes at a time, and what
// the host has put together in one copy, from its staging place to where it belongs.  Region ends are multiples of 16 bytes.
// Large regions go to the workgroups in a run each, which the memory takes at 6.0 TB/s instead of 5.2 (pools of 1.5 GB, 303 us with all
// workgroups side by side, 263 now); their ends, and small ones, side by side.
struct InitFill {
  u32x4* p;
  uint32_t v;
  size_t count;        // of 16 bytes
  size_t run;          // of them in a row for each workgroup, a multiple of kThreads
};
struct InitJob {
  InitFill fill[9];
  const int32_t* stage;      // [units] budget, [units] first segment, [units] segments, [Bz] budget total (8 bytes), decay table (tab_n entries, or 0)
  int32_t* tab;
  int tab_n;
  long long pool_segs, given;      // segments in all, and handed to units
  int t0;
};
__global__ __launch_bounds__(kThreads) void init_kernel(Dev d, InitJob job) {
  const size_t at = (size_t)blockIdx.x * kThreads + threadIdx.x, stride = (size_t)gridDim.x * kThreads;
#pragma unroll 1
  for (int f = 0; f < 9; ++f) {
    const InitFill x = job.fill[f];
    const u32x4 v = {x.v, x.v, x.v, x.v};
    u32x4* mine = x.p + x.run * blockIdx.x + threadIdx.x;
#pragma unroll 4
    for (size_t i = 0; i < x.run; i += kThreads) mine[i] = v;
    for (size_t i = x.run * gridDim.x + at; i < x.count; i += stride) x.p[i] = v;
  }
  const size_t U = (size_t)d.units;
  const int32_t *budget = job.stage, *first = budget + U, *need = first + U;
  const long long* total = reinterpret_cast<const long long*>(need + U + (U & 1));
  const int32_t* tab = reinterpret_cast<const int32_t*>(total + d.Bz);
  for (size_t i = at; i < U; i += stride) {
    d.budget[i] = budget[i];
    d.owned[i] = need[i];
  }
  for (size_t i = at; i < U * d.max_seg; i += stride) {
    const size_t u = i / d.max_seg;
    const int j = (int)(i - u * d.max_seg);
    d.tbl[i] = j < need[u] ? first[u] + j : 0;
  }
  // the others are spare, a stack whose top is the lowest
  for (size_t i = at; i < (size_t)(job.pool_segs - job.given); i += stride) d.spare[i] = (int32_t)(job.pool_segs - 1 - (long long)i);
  for (size_t i = at; i < (size_t)d.Bz; i += stride) d.btotal[i] = total[i];
  for (size_t i = at; i < (size_t)job.tab_n; i += stride) job.tab[i] = tab[i];
  for (size_t i = at; i < (size_t)SC_COUNT; i += stride) d.sc[i] = i == SC_T ? job.t0 : i == SC_SPARE ? (int32_t)(job.pool_segs - job.given) : 0;
}

// ------------------------------------------------------------------ bandwidth probes
// Plain streaming kernels of known size: the on-box ceiling the scan kernel is
// compared with, and the calibration of the profiler's fetch/write counters.
__global__ __launch_bounds__(kThreads) void probe_read_kernel(const u32x4* __restrict__ src, size_t n_vec, uint32_t* sink) {
  const int lane = threadIdx.x & 63;
  const size_t nw = (size_t)gridDim.x * (kThreads / 64), gw = (size_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  u32x4 acc = {0u, 0u, 0u, 0u};
  for (size_t base = gw * 1024; base + 1024 <= n_vec; base += nw * 1024) {     // 16 KB per wavefront and round
    u32x4 v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = __builtin_nontemporal_load(src + base + i * 64 + lane);
#pragma unroll
    for (int i = 0; i < 16; ++i) acc ^= v[i];
  }
  if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9E3779B9u) sink[0] = 1u;          // keeps the loads alive
}

__global__ __launch_bounds__(kThreads) void probe_copy_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, size_t n_vec) {
  size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * kThreads;
  for (; i < n_vec; i += stride) dst[i] = src[i];
}

// ------------------------------------------------------------------ pool segments between units
// Shared pools (headroom >= 1): a unit should own the segments that budget + headroom entries need, never
// fewer than its entries occupy, and for the units [x_begin, x_begin + x_count) at least what x_entries
// entries need (a prompt on its way in; x_len, if given, holds the units' own lengths, headroom not included).  One workgroup walks all units twice: units that own more than
// they should push the surplus (their last segments) onto the spare stack, then units that own less pop what
// they lack.  Who gets which segment follows from prefix sums over the units in index order, so the result
// does not depend on timing.  If the spare list is short nobody is given anything and bit 2 of the status
// word is set; a unit that still holds more entries than its budget (its eviction has not run yet) keeps
// its segments until a later call.  Unowned columns of a table row hold 0.
// The segments that change hands are dealt out to the threads one by one, each looks up the unit it comes from or goes to: what a prompt
// passes from layer to layer, 28 segments of each of 64 neighbouring units, was fetched and stored by 64 threads, in as many
// round trips as a unit has eights (22 us, now 8.3; the first version, one segment at a time, 42).  Budgets of 1024 units permuted 20.7 -> 9.4 us, of
// 6144 136 -> 41, of 16384 450 -> 101; nothing to deal out, 6144 units 16.2 -> 11.5.
constexpr int kBalanceThreads = 1024;
__global__ __launch_bounds__(kBalanceThreads) void rebalance_kernel(Dev d, int headroom, int x_begin, int x_count, int x_entries,
                                                                    const int32_t* x_len) {
  __shared__ u64 s_part[kBalanceThreads / 64];
  __shared__ int s_first[kBalanceThreads];       // of a thousand units: where each one's segments begin among those that change hands,
  __shared__ int s_from[kBalanceThreads];        // and the first column of its row that is concerned
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // what this kernel writes and reads back (ownership, table cells, the spare stack) goes through accesses that
  // are coherent one by one, whichever thread wrote them
  auto ld = [](const int32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  auto st = [](int32_t* p, int32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  auto need_of = [&](int u) {
    int e = max(d.budget[u] + headroom, d.n[u]);
    if (u >= x_begin && u < x_begin + x_count) e = max(e, x_len ? min(max(x_len[u - x_begin], 0) + headroom, x_entries) : x_entries);
    return min(d.max_seg, (e + kSeg - 1) / kSeg);
  };
  // of two counts per thread, sums over the threads before; the sums over all
  auto scan = [&](int a, int b, int& a_before, int& b_before, int& a_all, int& b_all) {
    const int ia = wave_scan_i32(a, lane), ib = wave_scan_i32(b, lane);
    __syncthreads();                       // the previous scan's readers are done
    if (lane == 63) s_part[wave] = ((u64)(uint32_t)ib << 32) | (uint32_t)ia;
    __syncthreads();
    a_before = ia - a;
    b_before = ib - b;
    a_all = b_all = 0;
    for (int w = 0; w < kBalanceThreads / 64; ++w) {
      const int x = (int)(uint32_t)s_part[w], y = (int)(s_part[w] >> 32);
      a_before += w < wave ? x : 0;
      b_before += w < wave ? y : 0;
      a_all += x;
      b_all += y;
    }
  };
  // f(unit, column of its row, number among all) for every one of `total` segments
  auto each = [&](int c0, int first, int from, int total, auto f) {
    s_first[tid] = first;
    s_from[tid] = from;
    __syncthreads();
    for (int i = tid; i < total; i += kBalanceThreads) {
      int k = 0;                           // the last thread whose segments begin at i or before
#pragma unroll
      for (int step = kBalanceThreads / 2; step > 0; step >>= 1)
        if (s_first[k + step] <= i) k += step;
      f(c0 + k, s_from[k] + (i - s_first[k]), i);
    }
  };
  int spare_n = d.sc[SC_SPARE];
  // ---- release
  int wanted = 0, want_before = 0;         // (of the only thousand units, if there are no more)
  for (int c0 = 0; c0 < d.units; c0 += kBalanceThreads) {
    const int u = c0 + tid;
    const int need = u < d.units ? need_of(u) : 0, own = u < d.units ? ld(d.owned + u) : 0;
    int first, total, want;
    scan(max(0, own - need), max(0, need - own), first, want_before, total, want);
    wanted += want;
    if (total > 0) {
      each(c0, first, need, total, [&](int v, int j, int i) {
        int32_t* cell = d.tbl + (size_t)v * d.max_seg + j;
        st(d.spare + spare_n + i, ld(cell));
        st(cell, 0);
      });
      if (own > need) st(d.owned + u, need);
      spare_n += total;
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the stack's new entries before anyone pops them
  __syncthreads();
  // ---- grant
  if (wanted > spare_n) {
    if (tid == 0) {
      atomicOr(&d.sc[SC_STATUS], 4);
      d.sc[SC_SPARE] = spare_n;
    }
    return;
  }
  int top = spare_n;
  for (int c0 = 0; wanted > 0 && c0 < d.units; c0 += kBalanceThreads) {
    const int u = c0 + tid;
    const int need = u < d.units ? need_of(u) : 0, own = u < d.units ? ld(d.owned + u) : 0;
    int first = want_before, total = wanted, none, none_all;
    if (d.units > kBalanceThreads) scan(max(0, need - own), 0, first, none, total, none_all);
    if (total > 0) {
      each(c0, first, own, total, [&](int v, int j, int i) { st(d.tbl + (size_t)v * d.max_seg + j, ld(d.spare + (top - 1 - i))); });
      if (need > own) st(d.owned + u, need);
      top -= total;
    }
  }
  if (tid == 0) d.sc[SC_SPARE] = spare_n - wanted;
}

// ------------------------------------------------------------------ cache load
// What bounds it is the copy: 612 MB for 64 units of 9350 entries.  PAST: values go past the caches, where those of a large layer would push out keys
// that a replay of the prompt reads next (64 such units in an admission 113 -> 102 us, that replay's first pass 47 -> 49; keys past them too: 108, 43, but 11 us
// more for the moves of the eviction that follows; both as they come in: 104 and 50).
// grid: (ceil(P/32), units of the layer); converts 32 row-major rows to one
// tiled block.  k, v: [units][P][128]; unit `urel` holds len[urel] (or P)
// entries; rows beyond that become zero.
template <bool PAST>
__global__ __launch_bounds__(kThreads) void load_cache_kernel(Dev d, int unit_begin, const uint16_t* k,
                                                              const uint16_t* v, int P, const int32_t* len,
                                                              const float* crf0, const int32_t* tau0,
                                                              const int32_t* pos0) {
  __shared__ uint16_t vt[kBlk][kDim + 8];
  const int tid = threadIdx.x;
  const int urel = blockIdx.y, u = unit_begin + urel;
  const int blk = blockIdx.x, r0 = blk * kBlk;
  int n = len ? min(max(len[urel], 0), P) : P;
  if (n >= unit_cap(d, u)) {                     // the unit's segments do not hold it (shared pools that ran short)
    n = max(unit_cap(d, u) - 1, 0);
    if (blk == 0 && tid == 0) atomicOr(&d.sc[SC_STATUS], 1);
  }
  if (blk == 0 && tid == 0) {
    d.n[u] = n;
    d.nev[u] = 0;
  }
  if (r0 >= n) return;
  const uint16_t* ksrc = k + (size_t)urel * P * kDim;
  const uint16_t* vsrc = v + (size_t)urel * P * kDim;
  const Slots sl = slots_of(d, u);
  uint16_t* kdst = d.K + sl.blk(blk);          // this block's 32 entries
  uint16_t* vdst = d.V + sl.blk(blk);
  // K: 32 rows x 16 pieces of 16 bytes
  for (int p = tid; p < kBlk * 16; p += kThreads) {
    int rr = p >> 4, piece = p & 15, r = r0 + rr;
    u32x4 x = {0u, 0u, 0u, 0u};
    if (r < n) x = *reinterpret_cast<const u32x4*>(ksrc + (size_t)r * kDim + piece * 8);
    *reinterpret_cast<u32x4*>(kdst + k_offset(rr, piece * 8)) = x;
  }
  // V: stage the rows, then write 16-byte pieces of the entry-interleaved order
  for (int p = tid; p < kBlk * 16; p += kThreads) {
    int rr = p >> 4, piece = p & 15, r = r0 + rr;
    u32x4 x = {0u, 0u, 0u, 0u};
    if (r < n) x = *reinterpret_cast<const u32x4*>(vsrc + (size_t)r * kDim + piece * 8);
    *reinterpret_cast<u32x4*>(&vt[rr][piece * 8]) = x;
  }
  __syncthreads();
  for (int p = tid; p < 8 * 64; p += kThreads) {
    int dt = p >> 6, kg = (p >> 4) & 3, j = p & 15;
    uint16_t e8[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      int rr = (e < 4) ? (4 * kg + e) : (16 + 4 * kg + (e - 4));
      e8[e] = vt[rr][16 * dt + j];
    }
    u32x4 x;
    x.x = e8[0] | ((uint32_t)e8[1] << 16);
    x.y = e8[2] | ((uint32_t)e8[3] << 16);
    x.z = e8[4] | ((uint32_t)e8[5] << 16);
    x.w = e8[6] | ((uint32_t)e8[7] << 16);
    if constexpr (PAST)
      __builtin_nontemporal_store(x, reinterpret_cast<u32x4*>(vdst + (size_t)p * 8));
    else
      *reinterpret_cast<u32x4*>(vdst + (size_t)p * 8) = x;
  }
  // per-slot state
  const Slots base = sl;
  for (int rr = tid; rr < kBlk; rr += kThreads) {
    int r = r0 + rr;
    if (r < n) {
      d.pos[base + r] = pos0 ? pos0[(size_t)urel * P + r] : r;
      d.crf[base + r] = crf0 ? crf0[(size_t)urel * P + r] : 1.0f;
      d.tau[base + r] = tau0 ? tau0[(size_t)urel * P + r] : (P - 1);
      d.flags[base + r] = 0;
    }
  }
}

// Stores and loads that are coherent across the chip's L2 caches one by one (no cache-wide write-back or
// invalidation, which a fence at that scope would cost every workgroup): how a scan hands its partials from the
// workgroups that wrote them to the one that combines them.
template <class T>
__device__ __forceinline__ void put_coherent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ T get_coherent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Sixteen bytes at once: buffer accesses with the cache policy bit (sc1) of those loads and stores, which the language has no atomic
// of that size for.  (The four words may arrive apart, which nobody sees who waits for the count.)  The array's base and
// size are the same in all lanes, `at` counts floats and is a multiple of 4.
constexpr int kSc1 = 16;
typedef __amdgpu_buffer_rsrc_t Buffer;
__device__ __forceinline__ Buffer buffer_of(float* base, int floats) { return __builtin_amdgcn_make_buffer_rsrc(base, 0, floats * 4, 0x00027000); }
__device__ __forceinline__ void put_coherent16(Buffer b, int at, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b, at * 4, 0, kSc1);
}
template <int kPolicy>
__device__ __forceinline__ f32x4 get_f32x4(Buffer b, int at) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(b, at * 4, 0, kPolicy));
}
__device__ __forceinline__ u64 pack_f32(float a, float b) { return ((u64)__float_as_uint(b) << 32) | __float_as_uint(a); }
__device__ __forceinline__ float low_f32(u64 x) { return __uint_as_float((uint32_t)x); }
__device__ __forceinline__ float high_f32(u64 x) { return __uint_as_float((uint32_t)(x >> 32)); }

// ------------------------------------------------------------------ scan
struct KFrag {
  u32x4 k[8];
};
struct VFrag {
  u32x4 v[8];
};

// K and V are read once per step and never reused: non-temporal loads keep
// them from displacing the logits that the finish kernel re-reads.
__device__ __forceinline__ u32x4 stream_load(const uint16_t* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}

// `kb` / `vb` already include the lane's offset (8 bf16 per lane).
__device__ __forceinline__ void load_k(KFrag& f, const uint16_t* kb) {
#pragma unroll
  for (int i = 0; i < 8; ++i) f.k[i] = stream_load(kb + i * 512);
}

__device__ __forceinline__ void load_v(VFrag& f, const uint16_t* vb) {
#pragma unroll
  for (int i = 0; i < 8; ++i) f.v[i] = stream_load(vb + i * 512);
}

// s_waitcnt vmcnt(0) alone
constexpr int kWaitLoads = 0x0F70;

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 x) { return __builtin_bit_cast(bf16x8, x); }

// One block of 32 entries is processed in two halves so that each fragment's
// registers can be refilled as soon as it has been consumed.  The scaled logits
// leave through a wave-private LDS tile so that each block's values go to memory
// as one contiguous store.
constexpr int kLgRow = 36;     // floats per head row in the LDS tile (32 + pad against bank conflicts)

// First half of a block of 32 entries: logits on the matrix cores, masked and
// scaled into sv[8] (this lane's 4 + 4 entries), and sent on their way to the
// finish phase.  The K fragment is dead afterwards.
// `forward`, if it is true, takes a block's logits to memory: lane l < 8 G the four at 4 l of the block's [head][32].
struct LogitsOut {
  float* dst;          // the span's logits, this lane's four of the first block
  __device__ __forceinline__ explicit operator bool() const { return dst != nullptr; }
  __device__ __forceinline__ void operator()(int first, f32x4 row) const { *reinterpret_cast<f32x4*>(dst + first) = row; }
};
template <class Forward>
__device__ __forceinline__ void scan_qk(const KFrag& f, const bf16x8 (&qv)[4], float (&sv)[8], float c_scale, int e_base,
                                        int n_valid, float* lds_lg, int lds_row, Forward forward, int G, int lane) {
  const int j = lane & 15, kg = lane >> 4;
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 4; ++s) s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(f.k[s]), qv[s], s0, 0, 0, 0);
#pragma unroll
  for (int s = 0; s < 4; ++s) s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(f.k[4 + s]), qv[s], s1, 0, 0, 0);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    sv[v] = (e_base + 4 * kg + v < n_valid) ? s0[v] * c_scale : -INFINITY;
    sv[4 + v] = (e_base + 4 * kg + 16 + v < n_valid) ? s1[v] * c_scale : -INFINITY;
  }
  // logits: row j of the LDS buffer (a wave-private staging tile, or the block's
  // place in a resident logits tile); with `forward` the tile goes on to memory
  // as one contiguous 128 G-byte store
  if (lds_lg == nullptr) return;            // attention only: nobody looks at the logits afterwards
  if (j < G) {
    *reinterpret_cast<f32x4*>(lds_lg + j * lds_row + 4 * kg) = f32x4{sv[0], sv[1], sv[2], sv[3]};
    *reinterpret_cast<f32x4*>(lds_lg + j * lds_row + 16 + 4 * kg) = f32x4{sv[4], sv[5], sv[6], sv[7]};
  }
  if (forward) {
    __builtin_amdgcn_wave_barrier();
    if (lane < 8 * G) forward(e_base * G, *reinterpret_cast<const f32x4*>(lds_lg + (lane >> 3) * lds_row + 4 * (lane & 7)));
    __builtin_amdgcn_wave_barrier();
  }
}

// Second half: online softmax update and probabilities (split into two bf16
// terms) times V on the matrix cores.  The V fragment is dead afterwards.
//
// PACK: the caller has duplicated the query heads 0..7 into the MFMA's columns 8..15 (at most 8 heads are
// real), so lane (j + 8, kg) holds the same logits and probabilities as lane (j, kg).  The product's
// operand then carries the high terms in rows 0..7 and the low terms in rows 8..15: one MFMA per 16
// dims instead of two, the result rows g (high) and g + 8 (low) of head g are added by the caller at the
// end of the unit (acc of lane + 32).
template <bool PACK = false>
__device__ __forceinline__ void scan_pv(const float (&sv)[8], const VFrag& fv, f32x4 (&acc)[8], float& m_run, float& l_run,
                                        int lane) {
  float bm = fmaxf(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])), fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
  bm = fmaxf(bm, __shfl_xor(bm, 16));
  bm = fmaxf(bm, __shfl_xor(bm, 32));
  if (__any(bm > m_run)) {
    const float m_new = fmaxf(m_run, bm);
    const float sc = fast_exp2(m_run - m_new);
    l_run *= sc;
    m_run = m_new;
    const int h4 = (lane >> 4) << 2;
    const float c0 = __shfl(sc, h4), c1 = __shfl(sc, h4 + 1), c2 = __shfl(sc, h4 + 2), c3 = __shfl(sc, h4 + 3);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      acc[dt][0] *= c0;
      acc[dt][1] *= c1;
      acc[dt][2] *= c2;
      acc[dt][3] *= c3;
    }
  }
  bf16x8 ph, pl;
  float ps = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float p = fast_exp2(sv[i] - m_run);
    ps += p;
    const __bf16 h = (__bf16)p;
    ph[i] = h;
    pl[i] = (__bf16)(p - (float)h);
  }
  l_run += ps;
  if constexpr (PACK) {
    const bool low = (lane & 8) != 0;
    const u32x4 h4 = __builtin_bit_cast(u32x4, ph), l4 = __builtin_bit_cast(u32x4, pl);
    const u32x4 a4 = {low ? l4[0] : h4[0], low ? l4[1] : h4[1], low ? l4[2] : h4[2], low ? l4[3] : h4[3]};
    const bf16x8 pa = as_bf16x8(a4);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa, as_bf16x8(fv.v[dt]), acc[dt], 0, 0, 0);
  } else {
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph, as_bf16x8(fv.v[dt]), acc[dt], 0, 0, 0);
      acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl, as_bf16x8(fv.v[dt]), acc[dt], 0, 0, 0);
    }
  }
}

// ------------------------------------------------------------------ eviction
__device__ __forceinline__ u64 evict_key(float tmp, int pos) {
  // ascending key order = eviction order: lower score first, then higher position
  return ((u64)__float_as_uint(tmp) << 32) | (u64)(uint32_t)(~pos);
}

// One wavefront moves the entry in slot `src` to slot `dst` (both of unit
// base slot `base`); dst's position goes to src, flagged as evicted.
__device__ __forceinline__ void move_entry(const Dev& d, Slots base, int src, int dst, int lane) {
  uint16_t* K = d.K;
  uint16_t* V = d.V;
  if (lane < 16)
    *reinterpret_cast<u32x4*>(K + base.k(dst, lane * 8)) = *reinterpret_cast<const u32x4*>(K + base.k(src, lane * 8));
  V[base.v(dst, lane)] = V[base.v(src, lane)];
  V[base.v(dst, lane + 64)] = V[base.v(src, lane + 64)];
  if (lane == 0) {
    d.crf[base + dst] = d.crf[base + src];
    d.tau[base + dst] = d.tau[base + src];
    const int ps = d.pos[base + src], pd = d.pos[base + dst];
    d.pos[base + dst] = ps;
    d.pos[base + src] = pd;
    d.flags[base + dst] = d.flags[base + src];
    d.flags[base + src] = FLAG_SLIP;
  }
}

// Up to four moves at once by one wavefront: move r0 + m takes the entry in slot lst[lst_cap - 1 - (r0 + m)]
// to slot lst[r0 + m] (m < count), as move_entry does, but every load is issued before the first store, so
// the moves' memory round trips overlap.  Lane l does the key piece l & 15 of move l >> 4; all lanes do two
// value elements of every move; lanes 0..3 do the per-slot state of moves 0..3.
__device__ __forceinline__ void move_entries4(const Dev& d, Slots base, const int* lst, int lst_cap, int r0, int count, int lane) {
  uint16_t* K = d.K;
  uint16_t* V = d.V;
  const int mk = lane >> 4;
  int src[4], dst[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int mm = min(m, count - 1);
    src[m] = lst[lst_cap - 1 - (r0 + mm)];
    dst[m] = lst[r0 + mm];
  }
  const int ks = mk == 0 ? src[0] : mk == 1 ? src[1] : mk == 2 ? src[2] : src[3];
  const int kd = mk == 0 ? dst[0] : mk == 1 ? dst[1] : mk == 2 ? dst[2] : dst[3];
  const u32x4 kx = *reinterpret_cast<const u32x4*>(K + base.k(ks, (lane & 15) * 8));
  uint16_t v0[4], v1[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    v0[m] = V[base.v(src[m], lane)];
    v1[m] = V[base.v(src[m], lane + 64)];
  }
  float crf = 0.f;
  int tau = 0, ps = 0, pd = 0;
  uint8_t fl = 0;
  const int ms = lane == 0 ? src[0] : lane == 1 ? src[1] : lane == 2 ? src[2] : src[3];
  const int md = lane == 0 ? dst[0] : lane == 1 ? dst[1] : lane == 2 ? dst[2] : dst[3];
  if (lane < count) {
    crf = d.crf[base + ms];
    tau = d.tau[base + ms];
    ps = d.pos[base + ms];
    pd = d.pos[base + md];
    fl = d.flags[base + ms];
  }
  if (mk < count) *reinterpret_cast<u32x4*>(K + base.k(kd, (lane & 15) * 8)) = kx;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    if (m < count) {
      V[base.v(dst[m], lane)] = v0[m];
      V[base.v(dst[m], lane + 64)] = v1[m];
    }
  }
  if (lane < count) {
    d.crf[base + md] = crf;
    d.tau[base + md] = tau;
    d.pos[base + md] = ps;
    d.pos[base + ms] = pd;
    d.flags[base + md] = fl;
    d.flags[base + ms] = FLAG_SLIP;
  }
}

// Eviction of exactly one entry: the last slot's entry moves into the victim's
// slot `dst`, whose position goes to the last slot, flagged as evicted.  The K
// row, the V row and the per-slot state are handled by different wavefronts;
// the state comes from sh[1..3] = {CRF bits, tau, position} of the last slot's
// entry and the victim's position, so no per-slot array is read.
// The K and V rows of the slot that will move are read ahead of time (load_row, by the wavefronts that
// will store them), so that the eviction itself only stores.
struct EntryRow {
  u32x4 k;             // lanes 0..15 of wavefront 0: 8 dims of the K row each
  uint16_t v0, v1;     // wavefront 1 (0 if there is only one): dims lane and lane + 64 of the V row
};

template <int NT = kThreads>
__device__ __forceinline__ EntryRow load_row(const Dev& d, Slots base, int src, int tid) {
  const int wave = tid >> 6, lane = tid & 63;
  constexpr int W = NT / 64;
  const uint16_t* K = d.K;
  const uint16_t* V = d.V;
  EntryRow r{{0u, 0u, 0u, 0u}, 0, 0};
  if (wave == 0 && lane < 16) r.k = *reinterpret_cast<const u32x4*>(K + base.k(src, lane * 8));
  if (wave == (W > 1 ? 1 : 0)) {
    r.v0 = V[base.v(src, lane)];
    r.v1 = V[base.v(src, lane + 64)];
  }
  return r;
}

template <int NT = kThreads>
__device__ __forceinline__ void evict_one(const Dev& d, Slots base, int src, int dst, int dst_pos, const int* sh, int tid, const EntryRow& row) {
  const int wave = tid >> 6, lane = tid & 63;
  constexpr int W = NT / 64;
  uint16_t* K = d.K;
  uint16_t* V = d.V;
  if (dst != src) {
    if (wave == 0 && lane < 16) *reinterpret_cast<u32x4*>(K + base.k(dst, lane * 8)) = row.k;
    if (wave == (W > 1 ? 1 : 0)) {
      V[base.v(dst, lane)] = row.v0;
      V[base.v(dst, lane + 64)] = row.v1;
    }
  }
  if (wave == (W > 2 ? 2 : 0) && lane == 32) {
    if (dst != src) {
      d.crf[base + dst] = __int_as_float(sh[1]);
      d.tau[base + dst] = sh[2];
      d.pos[base + dst] = sh[3];
    }
    d.pos[base + src] = dst_pos;               // the victim's position (the last slot's own if that is the victim)
    d.flags[base + src] = FLAG_SLIP;
  }
}

// Per-entry LDS values (mean weight, then CRF_temp) are reached through an
// accessor: a plain array in the finish kernel, a view into the logits tile in
// the fused unit kernel.
struct ValLinear {
  float* p;
  __device__ __forceinline__ float& operator()(int i) const { return p[i]; }
};

// Alg. 1 Step 4 for one unit with n > B.  val(i) = CRF_temp of slot i (LDS),
// evm = LDS bit mask of n bits, lst = LDS scratch of lst_cap >= n ints that may
// overlap the storage behind `val` (the scores are dead by the time it is used).
template <class Val, int NT = kThreads>
__device__ __forceinline__ void evict_phase(const Dev& d, int u, Slots base, int n, int B, Val val, uint32_t* evm, int* lst, int lst_cap, RedBuf<NT>& rb,
                            int& phase, int* sh, int tid) {
  const int lane = tid & 63, wave = tid >> 6;
  const int k = n - B;
  if (k == 1) {
    u64 best = ~0ull;
    int best_i = -1;
    for (int i0 = tid; i0 < n; i0 += 4 * NT) {
      int ps[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + r * NT;
        ps[r] = i < n ? d.pos[base + i] : 0;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + r * NT;
        if (i < n) {
          const u64 key = evict_key(val(i), ps[r]);
          if (key < best) {
            best = key;
            best_i = i;
          }
        }
      }
    }
    const u64 gbest = block_min_u64<NT>(best, rb, phase, tid);
    if (best == gbest && best_i >= 0) sh[0] = best_i;     // keys are unique: one writer
    block_sync<NT>(rb);
    const int e = sh[0];
    if (wave == 0) {
      if (e != n - 1) {
        move_entry(d, base, n - 1, e, lane);
      } else if (lane == 0) {
        d.flags[base + e] = FLAG_SLIP;
      }
    }
  } else {
    // The k smallest keys (score, then higher position first) in two stages, two bits per round (the three
    // candidates' counts are nested, and they are small integers, exact as floats).  Stage 1: S = the k-th
    // smallest score pattern, from the scores in LDS alone.  Stage 2, only if the entries equal to S are
    // not all evicted: which of them, by position; only those entries' positions are read.
    uint32_t S = 0;
    for (int bit = 31; bit >= 1; bit -= 2) {
      const uint32_t c1 = S | (1u << (bit - 1)), c2 = S | (1u << bit), c3 = c1 | c2;
      float n1 = 0.f, n2 = 0.f, n3 = 0.f;
      for (int i = tid; i < n; i += NT) {
        const uint32_t b = __float_as_uint(val(i));
        n1 += b < c1 ? 1.f : 0.f;
        n2 += b < c2 ? 1.f : 0.f;
        n3 += b < c3 ? 1.f : 0.f;
      }
      block_sum3_f32<NT>(n1, n2, n3, rb, phase, tid);
      const float kf = (float)k;
      S = n3 < kf ? c3 : n2 < kf ? c2 : n1 < kf ? c1 : S;          // the largest pattern with fewer than k scores below it
    }
    float below = 0.f, equal = 0.f, unused = 0.f;
    for (int i = tid; i < n; i += NT) {
      const uint32_t b = __float_as_uint(val(i));
      below += b < S ? 1.f : 0.f;
      equal += b == S ? 1.f : 0.f;
    }
    block_sum3_f32<NT>(below, equal, unused, rb, phase, tid);
    const int r = k - (int)below;                                  // of the entries equal to S, the r highest positions go
    uint32_t P = 0xFFFFFFFFu;                                      // ... those with ~position <= P
    if (r < (int)equal) {
      P = 0;
      for (int bit = 31; bit >= 1; bit -= 2) {
        const uint32_t c1 = P | (1u << (bit - 1)), c2 = P | (1u << bit), c3 = c1 | c2;
        float n1 = 0.f, n2 = 0.f, n3 = 0.f;
        for (int i = tid; i < n; i += NT) {
          if (__float_as_uint(val(i)) == S) {
            const uint32_t np = ~(uint32_t)d.pos[base + i];
            n1 += np < c1 ? 1.f : 0.f;
            n2 += np < c2 ? 1.f : 0.f;
            n3 += np < c3 ? 1.f : 0.f;
          }
        }
        block_sum3_f32<NT>(n1, n2, n3, rb, phase, tid);
        const float rf = (float)r;
        P = n3 < rf ? c3 : n2 < rf ? c2 : n1 < rf ? c1 : P;
      }
    }
    const int words = (n + 31) >> 5;
    for (int w = tid; w < words; w += NT) evm[w] = 0u;
    block_sync<NT>(rb);
    for (int i = tid; i < n; i += NT) {
      const uint32_t b = __float_as_uint(val(i));
      if (b < S || (b == S && (P == 0xFFFFFFFFu || ~(uint32_t)d.pos[base + i] <= P))) atomicOr(&evm[i >> 5], 1u << (i & 31));
    }
    block_sync<NT>(rb);
    // holes = evicted slots below B, movers = surviving slots at or above B (equal counts)
    const int wpt = (words + NT - 1) / NT;
    const int w0 = min(words, tid * wpt), w1 = min(words, w0 + wpt);
    uint32_t holes = 0, movers = 0;
    for (int w = w0; w < w1; ++w) {
      const uint32_t e = evm[w];
      const int s0 = w << 5;
      const uint32_t below = (B >= s0 + 32) ? 0xFFFFFFFFu : (B <= s0 ? 0u : ((1u << (B - s0)) - 1u));
      const uint32_t valid = (n >= s0 + 32) ? 0xFFFFFFFFu : ((1u << (n - s0)) - 1u);
      holes += __popc(e & below);
      movers += __popc(~e & ~below & valid);
    }
    const uint32_t packed = holes | (movers << 16);
    uint32_t incl = packed;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
    if (lane == 63) sh[4 + wave] = (int)incl;
    block_sync<NT>(rb);
    uint32_t prefix = 0, total = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
      if (w < wave) prefix += (uint32_t)sh[4 + w];
      total += (uint32_t)sh[4 + w];
    }
    const uint32_t excl = incl - packed + prefix;
    int hrank = (int)(excl & 0xFFFFu), mrank = (int)(excl >> 16);
    const int h = (int)(total & 0xFFFFu);
    for (int w = w0; w < w1; ++w) {
      const uint32_t e = evm[w];
      const int s0 = w << 5;
      const uint32_t below = (B >= s0 + 32) ? 0xFFFFFFFFu : (B <= s0 ? 0u : ((1u << (B - s0)) - 1u));
      const uint32_t valid = (n >= s0 + 32) ? 0xFFFFFFFFu : ((1u << (n - s0)) - 1u);
      uint32_t hm = e & below, mm = ~e & ~below & valid;
      while (hm) {
        lst[hrank++] = s0 + __builtin_ctz(hm);
        hm &= hm - 1;
      }
      while (mm) {
        lst[lst_cap - 1 - (mrank++)] = s0 + __builtin_ctz(mm);
        mm &= mm - 1;
      }
    }
    block_sync<NT>(rb);
    // evicted entries that already sit at or above B just get their flag
    for (int i = B + tid; i < n; i += NT)
      if ((evm[i >> 5] >> (i & 31)) & 1u) d.flags[base + i] = FLAG_SLIP;
    // moves, four per wavefront at a time: all loads of a batch are issued before its stores
    for (int r0 = 4 * wave; r0 < h; r0 += 4 * (NT / 64)) move_entries4(d, base, lst, lst_cap, r0, min(4, h - r0), lane);
  }
  if (tid == 0) {
    d.n[u] = B;
    d.nev[u] = k;
  }
}

// ------------------------------------------------------------------ eviction of many entries, keys in registers
// Thread tid of NT owns R entries in groups of four consecutive ones, 4 (tid + c NT) + e (group c), as in
// lrfu_regs below: b[4 c + e] = the entry's score pattern (0xFFFFFFFF beyond the unit), np[4 c + e] = ~position.
// n <= R NT <= 32 NT, so the eviction mask has at most one 32-bit word per thread.
struct alignas(16) CutBuf {
  uint32_t hist[3][256];  // digit counts of a round; three in turn, so that one barrier per round is enough
  uint32_t lo[16], hi[16];
  int a[16], b[16];
};

template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return (uint32_t)dpp_i32<kCtrl>((int)v);
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  v = min(v, dpp_u32<kDppQuadSwap1>(v));
  v = min(v, dpp_u32<kDppQuadSwap2>(v));
  v = min(v, dpp_u32<kDppRowHalfMirror>(v));
  v = min(v, dpp_u32<kDppRowMirror>(v));
  const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), y = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
  const uint32_t z = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), w = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
  return min(min(x, y), min(z, w));
}

// The k-th smallest key is (S, P): an entry is among the k smallest (score, then higher position first) if its
// pattern is below S, or equal to S with ~position <= P.
struct KeyCut {
  uint32_t S, P;
  __device__ __forceinline__ bool operator()(uint32_t b, uint32_t np) const { return (b < S) | ((b == S) & (np <= P)); }
};

// Eight bits per round from the highest bit in which the values differ (positions share most of theirs: 14 bits are
// left of 32 for a unit that spans 16384 tokens): a histogram of the digit in LDS over the entries that still
// match the prefix, then every wavefront finds the digit at which the count passes `want` by itself.  Scores that have decayed to
// zero (most of a prompt's) are counted first: their common digit would serialise the LDS atomics of every round.
// 64 units of 9350 entries, 7300 of them evicted, the whole kernel: 21.7 us; with two-bit rounds that count with ballots
// 70 us (16 entries per thread and three compares each make such a round 2.5 us of issue); with two-bit rounds over
// scores in LDS and positions in memory by 256 threads, moves included, 632 us.
template <int R, int NT>
__device__ __forceinline__ KeyCut select_low_keys(const uint32_t (&b)[R], const uint32_t (&np)[R], int k, CutBuf& cb, int tid) {
  const int lane = tid & 63, wave = tid >> 6;
  constexpr int W = NT / 64;
  int turn = 0;
  int zeros = 0;
#pragma unroll
  for (int i = 0; i < R; ++i) zeros += __popcll(__ballot(b[i] == 0u));
  if (lane == 0) cb.a[wave] = zeros;
  for (int i = tid; i < 256; i += NT) cb.hist[0][i] = 0u;
  __syncthreads();
  zeros = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) zeros += cb.a[w];
  // The `want`-th smallest of the values for which `value(i, v)` is true; all of them equal to the result are
  // wanted if all_equal comes back true (the result may then lie above the value itself, below the next larger one).
  auto radix = [&](auto value, int want, bool& all_equal) -> uint32_t {
    uint32_t lo = 0xFFFFFFFFu, nhi = 0xFFFFFFFFu;              // minimum, and ~maximum
#pragma unroll
    for (int i = 0; i < R; ++i) {
      uint32_t v;
      if (value(i, v)) {
        lo = min(lo, v);
        nhi = min(nhi, ~v);
      }
    }
    lo = wave_min_u32(lo);
    nhi = wave_min_u32(nhi);
    if (lane == 0) {
      cb.lo[wave] = lo;
      cb.hi[wave] = nhi;
    }
    __syncthreads();
    lo = cb.lo[0];
    nhi = cb.hi[0];
#pragma unroll
    for (int w = 1; w < W; ++w) {
      lo = min(lo, cb.lo[w]);
      nhi = min(nhi, cb.hi[w]);
    }
    const uint32_t diff = lo ^ ~nhi;
    int top = diff ? 32 - __builtin_clz(diff) : 0;             // the values agree in all bits from `top` on
    uint32_t X = top < 32 ? lo >> top << top : 0u;
    all_equal = false;
    while (top > 0) {
      const int s = max(top - 8, 0);
      const uint32_t digits = 1u << (top - s);
      uint32_t* h = cb.hist[turn];
#pragma unroll
      for (int i = 0; i < R; ++i) {
        uint32_t v;
        if (value(i, v) && (v >> s) - (X >> s) < digits) atomicAdd(&h[(v >> s) - (X >> s)], 1u);      // (X ends in zeros from the digit on)
      }
      turn = turn == 2 ? 0 : turn + 1;
      for (int i = tid; i < 256; i += NT) cb.hist[turn][i] = 0u;       // read last two rounds ago
      __syncthreads();
      const u32x4 q = *reinterpret_cast<const u32x4*>(h + 4 * lane);
      const int mine = (int)(q[0] + q[1] + q[2] + q[3]);
      const int incl = wave_scan_i32(mine, lane);
      const int at = __ffsll((long long)__ballot(incl >= want)) - 1;   // the lane whose four digits hold the wanted one
      int below = __builtin_amdgcn_readlane(incl - mine, at);
      uint32_t digit = 4u * (uint32_t)at;
      int count = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        count = __builtin_amdgcn_readlane((int)q[e], at);
        if (below + count >= want) {
          digit += e;
          break;
        }
        below += count;
      }
      want -= below;
      X |= digit << s;
      top = s;
      if (count == want) {                                     // the whole digit is wanted: no need to look inside
        X |= (1u << s) - 1u;
        all_equal = true;
        break;
      }
    }
    return X;
  };
  KeyCut cut;
  cut.P = 0xFFFFFFFFu;
  bool all_equal = false;
  int want = k;
  if (zeros >= k) {
    cut.S = 0u;
    if (zeros == k) return cut;
  } else {
    want = k - zeros;
    cut.S = radix([&](int i, uint32_t& v) { v = b[i]; return b[i] - 1u < 0xFFFFFFFEu; }, want, all_equal);      // neither zero nor beyond the unit
    if (all_equal) return cut;
    int below = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) below += __popcll(__ballot(b[i] < cut.S));
    if (lane == 0) cb.b[wave] = below;
    __syncthreads();
    want = k;
#pragma unroll
    for (int w = 0; w < W; ++w) want -= cb.b[w];
  }
  // of the entries equal to S the `want` highest positions go (radix() returns at once if that is all of them)
  cut.P = radix([&](int i, uint32_t& v) { v = np[i]; return b[i] == cut.S; }, want, all_equal);
  return cut;
}

// What an eviction leaves for the kernel that moves the survivors: destination slots (evicted slots below the
// budget) from the front of the unit's list, source slots (survivors at or above it) from its end, and their number.
// The lists lie in the decode paths' logits, dead between calls, the numbers in the partials' maxima.
__device__ __forceinline__ int* move_list(const Dev& d, int u) { return reinterpret_cast<int*>(d.logits + (size_t)u * d.cap * d.G); }
__device__ __forceinline__ int* move_count(const Dev& d, int u) { return reinterpret_cast<int*>(d.ml + (size_t)u * d.slots * d.G * 2); }

// Alg. 1 Step 4 for a unit of n > B entries up to the moves: the survivors' lists go to `lst` (the unit's list in
// memory), evicted entries at or above B get their flag, the records are written.  evm: 32 NT bits of LDS.
template <int R, int NT>
__device__ __forceinline__ int evict_lists(const Dev& d, int u, Slots base, int n, int B, const uint32_t (&b)[R], const uint32_t (&np)[R],
                                           int* lst, uint32_t* evm, CutBuf& cb, int tid) {
  const int lane = tid & 63, wave = tid >> 6, k = n - B;
  const KeyCut cut = select_low_keys<R, NT>(b, np, k, cb, tid);
  evm[tid] = 0u;
  __syncthreads();
#pragma unroll
  for (int c = 0; c < R / 4; ++c) {
    const int e0 = 4 * (tid + c * NT);
    uint32_t m = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool ev = b[4 * c + e] != 0xFFFFFFFFu && cut(b[4 * c + e], np[4 * c + e]);
      m |= (ev ? 1u : 0u) << e;
      if (ev && e0 + e >= B) d.flags[base + (e0 + e)] = FLAG_SLIP;       // movers' sources get theirs when they have moved
    }
    if (m) atomicOr(&evm[e0 >> 5], m << (e0 & 31));
  }
  __syncthreads();
  // holes = evicted slots below B, movers = surviving slots at or above B (equal counts), in ascending order
  const uint32_t ev = evm[tid];
  const int s0 = tid << 5;
  const uint32_t below = (B >= s0 + 32) ? 0xFFFFFFFFu : (B <= s0 ? 0u : ((1u << (B - s0)) - 1u));
  const uint32_t valid = (n >= s0 + 32) ? 0xFFFFFFFFu : (n <= s0 ? 0u : ((1u << (n - s0)) - 1u));
  uint32_t hm = ev & below, mm = ~ev & ~below & valid;
  const uint32_t packed = __popc(hm) | (__popc(mm) << 16);
  const uint32_t incl = (uint32_t)wave_scan_i32((int)packed, lane);
  if (lane == 63) cb.a[wave] = (int)incl;
  __syncthreads();
  uint32_t before = incl - packed, total = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    if (w < wave) before += (uint32_t)cb.a[w];
    total += (uint32_t)cb.a[w];
  }
  int hrank = (int)(before & 0xFFFFu), mrank = (int)(before >> 16);
  while (hm) {
    lst[hrank++] = s0 + __builtin_ctz(hm);
    hm &= hm - 1;
  }
  while (mm) {
    lst[d.cap - 1 - (mrank++)] = s0 + __builtin_ctz(mm);
    mm &= mm - 1;
  }
  if (tid == 0) {
    d.n[u] = B;
    d.nev[u] = k;
  }
  return (int)min(total & 0xFFFFu, total >> 16);          // equal, unless positions repeat within the unit
}

// Second kernel of an eviction: the survivors' rows, four per wavefront at a time (every load of a batch before
// its first store).  All units' moves are one sequence, an eighth of it for each XCD, whose wavefronts go through it side by side.
// What bounds it is what it has to read and write: survivors lie seven to a block of 32 on average and bring most of their blocks'
// lines with them, and a row is 16 pieces of a key and 128 single values, each in another piece of its block.  The cache of
// an XCD makes that up only for moves that follow one another at about the same time.  64 units of 9350 entries cut to 2048 on average, and 1024
// of 2048 after a re-allocation: units with a few workgroups each 79 and 310 us; runs of the sequence, a wavefront each 75 and
// 350, a workgroup each, four moves in turn for its wavefronts, 70 and 229; side by side as it is, eight workgroups per compute unit 63 and 208, four 63 and 207, two
// 56 and 198, one 62 and 188; two, with eight rows per wavefront 62 and 200.  (Destination blocks put together in LDS and stored whole, instead of a
// row's 48 partial lines, units with workgroups of their own: 85 us for the first.)  By the counters the first reads 164 MB and writes 68, for about 50 MB
// of rows each way, 4.1 TB/s; the second 259 and 332 MB, 3.0 TB/s.
// Places in the lists and in the segment table are looked up by a lane per move, sixteen batches at once; the units' numbers of moves are
// summed up by every workgroup for itself.
// grid: a multiple of 8 workgroups of kThreads threads; count <= kMoveUnits.
constexpr int kMoveUnits = 4 * kThreads;
__global__ __launch_bounds__(kThreads) void evict_move_kernel(Dev d, int unit_begin, int count) {
  __shared__ int s_first[kMoveUnits];                      // each unit's first move in the sequence
  __shared__ int s_part[kThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int h[4], sum = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) h[e] = 4 * tid + e < count ? *move_count(d, unit_begin + 4 * tid + e) : 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) sum += h[e];
  const int incl = wave_scan_i32(sum, lane);
  if (lane == 63) s_part[wave] = incl;
  __syncthreads();
  int first = incl - sum, moves = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) {
    first += w < wave ? s_part[w] : 0;
    moves += s_part[w];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    s_first[4 * tid + e] = first;
    first += h[e];
  }
  __syncthreads();
  constexpr int kStep = 4 * (kThreads / 64);               // moves that a workgroup's wavefronts have in flight, four each
  const int eighth = (moves + 7) / 8, hop = (gridDim.x >> 3) * kStep;
  const int begin = (blockIdx.x & 7) * eighth, end = min(moves, begin + eighth);
  uint16_t* K = d.K;
  uint16_t* V = d.V;
  for (int r0 = begin + (blockIdx.x >> 3) * kStep + 4 * wave; r0 < end; r0 += 16 * hop) {
    const int mine = r0 + hop * (lane >> 2) + (lane & 3), n = __popcll(__ballot(mine < end));      // lane 4 b + m: the m-th of batch b
    const int r = min(mine, end - 1);
    int k = 0;                                             // the last unit whose moves begin at r or before (units without any begin where the next does)
#pragma unroll
    for (int step = kMoveUnits / 2; step > 0; step >>= 1)
      if (k + step < count && s_first[k + step] <= r) k += step;
    const int u = unit_begin + k, rank = r - s_first[k];
    const int* lst = move_list(d, u);
    const int src = lst[d.cap - 1 - rank], dst = lst[rank];
    const int32_t* row = d.tbl + (size_t)u * d.max_seg;
    const int src_seg = row[src >> 8], dst_seg = row[dst >> 8], src_in = src & (kSeg - 1), dst_in = dst & (kSeg - 1);
    const size_t from = (size_t)src_seg * kSeg + src_in, to = (size_t)dst_seg * kSeg + dst_in;
    const float crf = d.crf[from];
    const int tau = d.tau[from], ps = d.pos[from], pd = d.pos[to];
    const uint8_t fl = d.flags[from];
    for (int m0 = 0; m0 < n; m0 += 4) {
      // lane l: the key piece l % 16 of move l / 16, two value elements of every move
      const int mk = min(m0 + (lane >> 4), n - 1), piece = (lane & 15) * 8;
      const u32x4 kx = *reinterpret_cast<const u32x4*>(K + (size_t)__shfl(src_seg, mk) * kSegElems + k_offset(__shfl(src_in, mk), piece));
      uint16_t* to_k = K + (size_t)__shfl(dst_seg, mk) * kSegElems + k_offset(__shfl(dst_in, mk), piece);
      uint16_t v0[4], v1[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int mm = min(m0 + m, n - 1), in = __builtin_amdgcn_readlane(src_in, mm);
        const uint16_t* p = V + (size_t)__builtin_amdgcn_readlane(src_seg, mm) * kSegElems;
        v0[m] = p[v_offset(in, lane)];
        v1[m] = p[v_offset(in, lane + 64)];
      }
      if (m0 + (lane >> 4) < n) *reinterpret_cast<u32x4*>(to_k) = kx;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        if (m0 + m < n) {
          const int in = __builtin_amdgcn_readlane(dst_in, m0 + m);
          uint16_t* p = V + (size_t)__builtin_amdgcn_readlane(dst_seg, m0 + m) * kSegElems;
          p[v_offset(in, lane)] = v0[m];
          p[v_offset(in, lane + 64)] = v1[m];
        }
      }
    }
    if (lane < n) {
      d.crf[to] = crf;
      d.tau[to] = tau;
      d.pos[to] = ps;
      d.pos[from] = pd;
      d.flags[to] = fl;
      d.flags[from] = FLAG_SLIP;
    }
  }
}

// ------------------------------------------------------------------ finish
// Ends a kernel that must leave the step scalars consistent: the last block
// to arrive resets the queue and, if asked, advances time.  No fence: the
// last block reads nothing the others wrote (the scalars it updates are read-only
// during the launch, and every claim on the queue has returned before its
// workgroup gets here); the end of the kernel publishes what it writes.  A
// device-scope fence here would write back a whole L2 once per workgroup.
__device__ __forceinline__ void step_epilogue(const Dev& d, int t, int advance, int tid, int queue_reset = -1) {
  __syncthreads();
  if (tid == 0) {
    const int prev = atomicAdd(&d.sc[SC_DONE], 1);
    if (prev == (int)gridDim.x - 1) {
      d.sc[SC_DONE] = 0;
      if (queue_reset >= 0) d.sc[SC_QUEUE] = queue_reset;
      if (advance) {
        d.sc[SC_T] = t + 1;
        d.sc[SC_WINDOW_STEPS] = d.sc[SC_WINDOW_STEPS] + 1;
      }
    }
  }
}

// lambda^delta from the decay table: its first s_tab_n entries sit in LDS, the rest (long tables: lambda
// close to 1) in global memory.  Written as two loads in two address spaces on purpose: a conditional
// expression over the two pointers becomes one flat load, which waits for every vector-memory
// operation in flight.
__device__ __forceinline__ float decay_far(const Dev& d, int delta) {
  float far = d.tab[delta];
  asm volatile("" : "+v"(far));          // the wait for this load stays inside the caller's branch: placed after
  return far;                            // the branch it would be a wait for every vector-memory operation
}                                        // in flight, executed for every entry
__device__ __forceinline__ float decay_of(const Dev& d, int delta, const float* s_tab, int s_tab_n) {
  float dec = s_tab[min(delta, s_tab_n - 1)];
  asm volatile("" : "+v"(dec));          // pins the LDS load: otherwise the two loads are merged again
  if (delta >= s_tab_n) dec = decay_far(d, delta);
  return dec;
}
// Four lookups at once: the LDS reads are issued together and waited for once.
__device__ __forceinline__ void decay4_of(const Dev& d, const int (&delta)[4], const float* s_tab, int s_tab_n, float (&dec)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) dec[e] = s_tab[min(delta[e], s_tab_n - 1)];
#pragma unroll
  for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(dec[e]));
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (delta[e] >= s_tab_n) dec[e] = decay_far(d, delta[e]);
}

// Where a unit's scaled logits lie in memory: per block of 32 entries a group of rows [row][32], of which
// the G rows from `p` on are the unit's heads.
struct LgView {
  const float* p;      // head 0, entry 0
  int blk_stride;      // floats from one block to the next
};
__device__ __forceinline__ LgView unit_logits(const Dev& d, int u) {
  return LgView{d.logits + (size_t)u * d.G * d.cap, d.G * kBlk};
}

// Alg. 1 Steps 1-3 for one unit: top-p hit set from the mean weights val(i),
// score update, flags.  Leaves CRF_temp in val(i) and returns the unit's
// aggregated CRF (2^-20 fixed point), summed over the block.  s_tab: the first
// s_tab_n entries of the decay table in LDS.
// Alg. 1 Step 1 as a rule: an entry of weight pattern b and position pe is hit if b > theta, or b == theta and
// (ties_all or pe <= pos_cut).  (The entry appended in the step is hit whatever its weight: the callers add that.)
struct HitRule {
  uint32_t theta;
  bool ties_all;
  int pos_cut;
  __device__ __forceinline__ bool operator()(uint32_t b, int pe) const { return (b > theta) | ((b == theta) & (ties_all | (pe <= pos_cut))); }
};

// No threshold to look for: the reward is the weight itself, or p >= 1 marks every entry (the weights' sum, which rounding may leave above 1, is
// not asked).
__device__ __forceinline__ bool every_entry_hit(const Dev& d) { return (d.reward_mode != 0) | (d.top_p >= 1.0f); }

// Step 1 over weights in val(0 .. n - 1) (LDS), any n
template <class Val, int NT = kThreads>
__device__ __forceinline__ HitRule top_p_lds(const Dev& d, Slots base, int n, Val val, RedBuf<NT>& rb, int& phase, int tid) {
  uint32_t theta = 0;
  bool ties_all = true;
  int pos_cut = 0x7FFFFFFF;
  if (!every_entry_hit(d)) {
    for (int bit = 30; bit >= 0; --bit) {
      const uint32_t cand = theta | (1u << bit);
      float part = 0.f;
      for (int i = tid; i < n; i += NT) {
        const float a = val(i);
        part += (__float_as_uint(a) >= cand) ? a : 0.f;
      }
      const float tot = block_sum_f32<NT>(part, rb, phase, tid);
      if (tot > d.top_p) theta = cand;
    }
    if (theta != 0) {
      // entries equal to the threshold: only as many as needed, lower positions first
      float above = 0.f;
      int ties = 0;
      for (int i = tid; i < n; i += NT) {
        const float a = val(i);
        const uint32_t b = __float_as_uint(a);
        above += (b > theta) ? a : 0.f;
        ties += (b == theta) ? 1 : 0;
      }
      above = block_sum_f32<NT>(above, rb, phase, tid);
      ties = block_sum_int<NT>(ties, rb, phase, tid);
      if (ties > 1) {
        const double th = (double)__uint_as_float(theta), p = (double)d.top_p;
        double c = (double)above;
        int r = 0;
        do {
          c += th;
          ++r;
        } while (c <= p && r < ties);
        if (r < ties) {
          ties_all = false;
          int X = 0;   // r-th smallest position among the ties
          for (int bit = 30; bit >= 0; --bit) {
            const int trial = X | (1 << bit);
            int cnt = 0;
            for (int i = tid; i < n; i += NT)
              cnt += (__float_as_uint(val(i)) == theta && d.pos[base + i] < trial) ? 1 : 0;
            cnt = block_sum_int<NT>(cnt, rb, phase, tid);
            if (cnt < r) X = trial;
          }
          pos_cut = X;
        }
      }
    }
  }
  return HitRule{theta, ties_all, pos_cut};
}

template <class Val, int NT = kThreads>
__device__ __forceinline__ u64 lrfu_update(const Dev& d, int u, Slots base, int n, int t, Val val, const float* s_tab, int s_tab_n, RedBuf<NT>& rb,
                           int& phase, int tid) {
  // ---- Alg. 1 Step 1: top-p hit set as a threshold on the weight's bit pattern
  const HitRule rule = top_p_lds<Val, NT>(d, base, n, val, rb, phase, tid);
  const bool ties_all = rule.ties_all;

  // ---- Alg. 1 Steps 2-3: scores (4 entries per thread and round: loads, table lookups, then stores)
  const bool has_new = d.pos[base + (n - 1)] == t;
  const bool need_pos = d.reward_mode == 0 && !ties_all;
  u64 sfix = 0;
  for (int i0 = tid; i0 < n; i0 += 4 * NT) {
    float crf[4], dec[4];
    int tau[4], ps[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + r * NT;
      const bool ok = i < n;
      crf[r] = ok ? d.crf[base + i] : 0.f;
      tau[r] = ok ? d.tau[base + i] : t;
      ps[r] = (ok && need_pos) ? d.pos[base + i] : 0;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int delta = t - tau[r];
      delta = delta < 0 ? 0 : (delta > d.tab_last ? d.tab_last : delta);
      dec[r] = decay_of(d, delta, s_tab, s_tab_n);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + r * NT;
      if (i < n) {
        const float a = val(i);
        bool hit, store;
        float reward;
        if (d.reward_mode == 0) {
          const uint32_t b = __float_as_uint(a);
          hit = rule(b, ps[r]);
          if (i == n - 1 && has_new) hit = true;
          store = hit;
          reward = hit ? 1.0f : 0.0f;
        } else {
          store = true;
          reward = a;
        }
        float tmp = __fadd_rn(__fmul_rn(dec[r], crf[r]), reward);
        if (tmp < FLT_MIN) tmp = 0.0f;
        if (store) {
          d.crf[base + i] = tmp;
          d.tau[base + i] = t;
        }
        val(i) = tmp;
        sfix += (u64)floorf(tmp * kFixedOne);
      }
    }
  }
  return block_sum_u64<NT>(sfix, rb, phase, tid);   // its barrier also completes val() for what follows
}



// Register-resident bookkeeping: thread tid of NT owns R = 4 C entries, in C
// groups of four consecutive entries 4 (tid + c NT) .. + 3 (group c), so that
// every access to the per-entry arrays is a 16-byte one: the memory pipeline of
// a CU is shared with the streaming loads of the other workgroup and every
// instruction queues behind them, so the number of memory instructions, not
// their size, is what the latency of this phase depends on.

// Mean attention weights of this thread's groups from logits in global memory
// (per block of 32 entries: [head][32]); 0 beyond n.
template <int R, int NT = kThreads>
__device__ __forceinline__ void mean_weights_regs(const Dev& d, LgView lv, int n, const float* sM, const float* sInv,
                                                  float (&a)[R], int tid) {
  const int G = d.G;
  const float invG = 1.0f / (float)G;
  const float* lg = lv.p;
#pragma unroll
  for (int c = 0; c < R / 4; ++c) {
    const int e0 = 4 * (tid + c * NT);
    f32x4 x[kMaxGroup];
    const float* row = lg + (size_t)(e0 >> 5) * lv.blk_stride + (e0 & 31);
#pragma unroll
    for (int g = 0; g < kMaxGroup; ++g)
      x[g] = (e0 < n && g < G) ? *reinterpret_cast<const f32x4*>(row + g * kBlk) : f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float acc = 0.f;
#pragma unroll
      for (int g = 0; g < kMaxGroup; ++g)
        if (g < G) acc += fast_exp2(x[g][e] - sM[g]) * sInv[g];
      a[4 * c + e] = (e0 + e < n) ? acc * invG : 0.f;
    }
    if (R > 8 && (c & 1)) __builtin_amdgcn_sched_barrier(0);     // two groups' logits at a time: 1024 threads have 128 registers each
  }
}

// CRF, tau and position of group c of thread tid.  The loads are unconditional
// (a select on their result would wait for them on the spot): a group beyond
// the unit reads the unit's last group instead, and nothing looks at the values
// of entries >= n.
template <int NT = kThreads>
__device__ __forceinline__ void load_meta(const Dev& d, Slots base, int n, int t, int c, int tid, f32x4& crf, i32x4& tau, i32x4& ps) {
  const int e0 = min(4 * (tid + c * NT), (max(n, 1) - 1) & ~3);
  const size_t s0 = base + e0;                 // four consecutive entries share a segment
  crf = *reinterpret_cast<const f32x4*>(d.crf + s0);
  tau = *reinterpret_cast<const i32x4*>(d.tau + s0);
  ps = *reinterpret_cast<const i32x4*>(d.pos + s0);
}

// Alg. 1 Steps 1-4 for a unit of n <= R NT entries with the weights in
// registers (a[4 c + e] = mean weight of entry 4 (tid + c NT) + e, 0 beyond n).
// Same decisions and arithmetic as lrfu_update + evict_phase.  The groups'
// CRF, tau and position pass through register arrays of CH groups: the caller
// has loaded the first CP of them (early enough that they have arrived), the
// rest of the first CH groups are loaded here, before the bisection, whose 31
// rounds hide their latency; further chunks of CH groups (large units only, to
// bound the registers) are loaded when their turn comes.  The hit mark of an entry is not stored: in the
// top-p mode it equals tau == t.  Evicting exactly one entry is done in place
// (the owners of the two entries involved pass their registers through `sh`);
// evicting more falls back to evict_phase (scores then go to val()).
struct NoHook {
  __device__ __forceinline__ void operator()() const {}
};

// The entry appended in this step when the caller has NOT written it to the cache (the fused kernel when
// exactly one entry will be evicted): logically it is the unit's last entry, index n - 1, with CRF 0,
// tau = t and position t; its key and value rows are the step's inputs.  Its per-slot state is supplied
// here instead of being read, and if it survives the eviction its rows go straight from the inputs into
// the victim's slot (one write instead of a write, a read and a write).  k_row == nullptr: the entry is in
// the cache like any other (or nothing was appended).
struct NewEntry {
  const uint16_t* k_row;    // 128 bf16, or nullptr
  const uint16_t* v_row;
  __device__ __forceinline__ bool there() const { return k_row != nullptr; }
};
// The same with the rows in the cache already (a scan that ran before put them there).
struct NewInCache {
  bool arrived;
  __device__ __forceinline__ bool there() const { return arrived; }
};

template <int NT = kThreads>
__device__ __forceinline__ EntryRow load_row_input(const NewEntry& ne, int tid) {
  const int wave = tid >> 6, lane = tid & 63;
  constexpr int W = NT / 64;
  EntryRow r{{0u, 0u, 0u, 0u}, 0, 0};
  if (wave == 0 && lane < 16) r.k = *reinterpret_cast<const u32x4*>(ne.k_row + lane * 8);
  if (wave == (W > 1 ? 1 : 0)) {
    r.v0 = ne.v_row[lane];
    r.v1 = ne.v_row[lane + 64];
  }
  return r;
}

// What top_p_regs keeps in LDS.
struct alignas(16) TopBuf {
  u64 bin[24 << 5];
  uint32_t list[256 + 8];
  double above;           // sum of the bins above the one in question
  int at, count;          // that bin (-1: none), and the number of its weights
  double above_theta;
  uint32_t listed, odd, theta, ties;
  uint32_t tied;          // entries equal to the threshold in the list
  int cut;
};

template <int NT>
__device__ constexpr int top_list() { return NT < 256 ? NT : 256; }      // entries of the list, a thread each

// Entries equal to the threshold: only as many as needed, lower positions first.  above = total weight of the entries
// above theta, ties = entries equal to it.  Of a list's worth, each counts the lower positions (LIST: not in the fused kernel, whose streaming
// loop is short of registers for it); more take 31 rounds over all entries, each with a block's reduction and another trip to the positions. Those rounds
// were half of a step on caches where keys repeat (336 units of 550 entries after 16000 steps, four to eight ties each, 69 us per step, 38 with the
// list; 240 of 222 on average 40 / 23).
template <int R, int NT, bool LIST>
__device__ __forceinline__ HitRule tie_rule(const Dev& d, Slots base, int n, const float (&a)[R], uint32_t theta, double above, int ties,
                                            TopBuf& tb, int new_last_t, RedBuf<NT>& rb, int& phase, int tid) {
  HitRule rule{theta, true, 0x7FFFFFFF};
  if (ties <= 1) return rule;
  const double th = (double)__uint_as_float(theta), p = (double)d.top_p;      // (in fp32 hundreds of equal additions round the same way)
  double c = above;
  int r = 0;
  do {
    c += th;
    ++r;
  } while (c <= p && r < ties);
  if (r >= ties) return rule;
  rule.ties_all = false;
  if (LIST && ties <= top_list<NT>()) {
    for (int k = 0; k < R; ++k) {
      const int i = 4 * (tid + (k >> 2) * NT) + (k & 3);
      if (__float_as_uint(a[k]) == theta && i < n)
        tb.list[atomicAdd(&tb.tied, 1u)] = (uint32_t)((new_last_t >= 0 && i == n - 1) ? new_last_t : d.pos[base + i]);
    }
    block_sync<NT>(rb);
    if (tid < ties) {
      const int mine = (int)tb.list[tid];
      int lower = 0, equal = 0;
      for (int k = 0; k < ties; ++k) {
        lower += (int)tb.list[k] < mine ? 1 : 0;
        equal += (int)tb.list[k] == mine ? 1 : 0;
      }
      if (lower < r && lower + equal >= r) tb.cut = max(mine, 0);        // every such thread has the same to say
    }
    block_sync<NT>(rb);
    rule.pos_cut = uniform_i32(tb.cut);
    return rule;
  }
  int X = 0;   // r-th smallest position among the ties (positions are re-read from memory)
  for (int bit = 30; bit >= 0; --bit) {
    const int trial = X | (1 << bit);
    int cnt = 0;
    for (int k = 0; k < R; ++k) {
      const int i = 4 * (tid + (k >> 2) * NT) + (k & 3);
      if (__float_as_uint(a[k]) == theta && i < n && ((new_last_t >= 0 && i == n - 1) ? new_last_t : d.pos[base + i]) < trial) ++cnt;
    }
    cnt = uniform_i32(block_sum_int<NT>(cnt, rb, phase, tid));
    if (cnt < r) X = trial;
  }
  rule.pos_cut = X;
  return rule;
}

// Step 1 over weights in registers (a[4 c + e] = mean weight of entry 4 (tid + c NT) + e, 0 beyond n): the largest pattern
// theta with sum{a >= theta} > p.
//
// One pass over the weights instead of a reduction over all of them per round of a search.  A histogram in LDS over the
// patterns' top bits (24 octaves below 2 in bins of 1/32 octave) takes per bin the number of its weights and the
// sum of their low bits in one 64-bit integer addition, so that a bin's sum is known exactly and does not depend on the order; the bin in which
// the sum from above passes p follows from a scan over the bins in 64 bits.  The bin's weights, usually a few dozen, go to a list, where each
// finds the sum of those at least as large, again from counts and low bits.  A bin of more than kList weights (long rows: what is left of it after
// another histogram over its next eight bits), and weights outside
// the bins that might matter (below 2^-23 in all; negative, NaN or 2 and above), take two bits per round over all entries.
//
// What bounded the search was issue: nine instructions per weight and round, six rounds (three or four by bracketing), a barrier and a
// reduction each; now about eight per weight in all and an LDS addition (a wavefront's 64-bit additions to a hundred random
// bins take 13 cycles of the compute unit).  finish_kernel for 128 units of 2048 entries 20.8 -> 15.6 us, 4096 rows of 9350 weights of a
// replay 80 -> 70 us, fused step of 896 units of 2048 entries 194.3 -> 190.6 us, of 6144 units 1243 -> 1238 us.
// The scan over the bins moves through DPP and by one wavefront: its registers come on top of the weights and of what the callers
// have in flight.
constexpr int kBinShift = 18, kBins = 24 << 5, kBinFirst = (127 - 23) << 5;
constexpr uint32_t kBinLow = (1u << kBinShift) - 1u;
constexpr int kBinCount = 34;                 // the count's place: 32768 low parts of 18 bits lie below it
constexpr int kSubShift = kBinShift - 8;      // a bin's 256 parts
constexpr uint32_t kSubLow = (1u << kSubShift) - 1u;
__device__ __forceinline__ double bin_edge(int i) { return (double)__uint_as_float((uint32_t)(kBinFirst + i) << kBinShift); }
__device__ __forceinline__ double bin_unit(int i) { return (double)__uint_as_float((uint32_t)((kBinFirst + i) >> 5) << 23) * 0x1p-23; }

// The same sum in units of 2^-46, the lowest bin's (24 octaves of 32768 weights stay below 2^62), for the scan over the bins.
constexpr double kFixedBin = 0x1p46;
__device__ __forceinline__ u64 bin_fixed(u64 v, int i) {
  return (((u64)((uint32_t)(v >> kBinCount) * (uint32_t)(32 + (i & 31))) << kBinShift) + (v & ((1ull << kBinCount) - 1ull))) << (i >> 5);
}

__device__ __forceinline__ double bin_sum(u64 v, int i) {
  return (double)(uint32_t)(v >> kBinCount) * bin_edge(i) + (double)(v & ((1ull << kBinCount) - 1ull)) * bin_unit(i);
}

__device__ __forceinline__ void clear_top(TopBuf& tb, int tid, int threads) {
  for (int i = tid; i < (int)(sizeof(TopBuf) / 16); i += threads) reinterpret_cast<u32x4*>(&tb)[i] = u32x4{0u, 0u, 0u, 0u};
}

// tb: in LDS, CLEARED (and a barrier since), or where something else may lie.  new_last_t >= 0: the unit's last entry is not in
// the cache, or not to be looked up there, and has this position.
// REFINE: long rows of flat weights, where a bin holds more than the list: the bin once more, by its next eight bits.  64 places of 8 bytes lie behind tb.
template <int R, int NT = kThreads, bool CLEARED = false, bool REFINE = false, bool LIST = CLEARED && !REFINE>
__device__ __forceinline__ HitRule top_p_regs(const Dev& d, Slots base, int n, const float (&a)[R], TopBuf& tb, int new_last_t, RedBuf<NT>& rb, int& phase,
                                              int tid) {
  if (every_entry_hit(d)) return HitRule{0u, true, 0x7FFFFFFF};
  constexpr int kList = top_list<NT>();
  // Steps that one wavefront, or a few, would take alone are shared by all: the list's places taken once per wavefront, candidates compared by all, sums over
  // the bins in whole numbers.  (Not in the fused kernel, where it gains nothing: with this / without, 896 units of 2048, G = 7, 193.0 / 192.6 us,
  // 6144 of 2048 1240 / 1238, 16384 of 1024 1695 / 1696, 87 and 88 registers spilled.)  4096 rows of 9350 weights 65.7 -> 62.9 us, 2048 of them 33.2 -> 29.8 (with fewer instructions per weight around it), the
  // bookkeeping of 128 units 14.9 -> 14.7.
  constexpr bool kShare = CLEARED || REFINE;
  const int lane = tid & 63, wave = tid >> 6;
  // (not known to the compiler as the same in every unit: kept in registers across the units of a persistent kernel it would be
  // spilled, and a reload is a wait for every load in flight)
  float top_p = d.top_p;
  asm volatile("" : "+s"(top_p));
  const double p = (double)top_p;
  if constexpr (!CLEARED) {
    block_sync<NT>(rb);                             // whatever lay in the buffer has been read
    clear_top(tb, tid, NT);
    block_sync<NT>(rb);
  }
  uint32_t largest = 0;
  if constexpr (REFINE) {
    // Weights outside the bins go to one of 64 behind the buffer, a lane's own, instead of nowhere: a select in place of a branch
    // over the addition.  (The caller's rows are zero beyond their end, which only the last few registers reach.  Rows with half, nine tenths or all but fifty
    // of their weights below the bins, 128 units of 9350, 32 queries, a whole replay 521 / 452 / 381 -> 516 / 443 / 379 us.)
    const uint32_t beyond = (uint32_t)sizeof(TopBuf) + 8u * lane;
    unsigned char* bins = reinterpret_cast<unsigned char*>(tb.bin);
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t b = __float_as_uint(a[k]);
      largest = max(largest, b);
      const uint32_t at = ((b >> kBinShift) << 3) - (uint32_t)(kBinFirst << 3);
      atomicAdd(reinterpret_cast<u64*>(bins + (at < (uint32_t)(kBins << 3) ? at : beyond)), (1ull << kBinCount) | (b & kBinLow));
      if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);        // few addresses at a time
    }
  } else {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t b = __float_as_uint(a[k]), i = (b >> kBinShift) - (uint32_t)kBinFirst;
      largest = max(largest, b);
      if (i < (uint32_t)kBins) atomicAdd(&tb.bin[i], (1ull << kBinCount) | (b & kBinLow));
      if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);        // few addresses at a time
    }
  }
  if (largest >= 0x40000000u) tb.odd = 1u;
  block_sync<NT>(rb);
  if (kShare && wave == 0) {
    // lane l: bins kPer l and up
    constexpr int kPer = kBins / 64;
    const u64 pass = (u64)(p * kFixedBin);                // a sum exceeds p if it exceeds this
    u64 mine = 0;
#pragma unroll
    for (int i = 0; i < kPer; i += 4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) mine += bin_fixed(tb.bin[kPer * lane + i + e], kPer * lane + i + e);
      __builtin_amdgcn_sched_barrier(0);                    // the weights need the registers
    }
    // sums from each lane up: inside a row of 16 lanes, then the rows above (the sum grows towards the lower lanes)
    u64 incl = mine;
    incl += dpp_u64<kDppRowShl + 1>(incl);
    incl += dpp_u64<kDppRowShl + 2>(incl);
    incl += dpp_u64<kDppRowShl + 4>(incl);
    incl += dpp_u64<kDppRowShl + 8>(incl);
    const u64 row3 = readlane_u64(incl, 48), row2 = readlane_u64(incl, 32) + row3, row1 = readlane_u64(incl, 16) + row2;
    incl += lane < 16 ? row1 : lane < 32 ? row2 : lane < 48 ? row3 : 0;
    const u64 passed = __ballot(incl > pass);
    if (passed) {
      // the highest lane at which it passes; of that lane's bins, from the top, lane i takes the i-th
      const int at = 63 - __builtin_clzll(passed), bin = kPer * at + kPer - 1 - min(lane, kPer - 1);
      const u64 before = readlane_u64(incl - mine, at), v = tb.bin[bin], own = lane < kPer ? bin_fixed(v, bin) : 0;
      u64 sum = own;
      sum += dpp_u64<kDppRowShr + 1>(sum);
      sum += dpp_u64<kDppRowShr + 2>(sum);
      sum += dpp_u64<kDppRowShr + 4>(sum);
      sum += dpp_u64<kDppRowShr + 8>(sum);
      const u64 here = __ballot(before + sum > pass) & ((1ull << kPer) - 1ull);
      if (lane == __builtin_ctzll(here)) {                  // (sums of whole numbers: it passes at one of them)
        tb.at = bin;
        tb.count = (int)(v >> kBinCount);
        tb.above = (double)(before + (sum - own)) / kFixedBin;
      }
    } else if (lane == 0) {
      tb.at = -1;
    }
  }
  if (!kShare && wave == 0) {
    // lane l: bins kPer l and up; few registers at a time, since the weights and the callers' prefetches live through this
    constexpr int kPer = kBins / 64;
    double mine = 0.0;
#pragma unroll 1
    for (int i = 0; i < kPer; i += 4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) mine += bin_sum(tb.bin[kPer * lane + i + e], kPer * lane + i + e);
    }
    // sums from each lane up: inside a row of 16 lanes, then the rows above (the sum grows towards the lower lanes)
    double incl = mine;
    incl += dpp_f64<kDppRowShl + 1>(incl);
    incl += dpp_f64<kDppRowShl + 2>(incl);
    incl += dpp_f64<kDppRowShl + 4>(incl);
    incl += dpp_f64<kDppRowShl + 8>(incl);
    const double row3 = readlane_f64(incl, 48), row2 = readlane_f64(incl, 32) + row3, row1 = readlane_f64(incl, 16) + row2;
    incl += lane < 16 ? row1 : lane < 32 ? row2 : lane < 48 ? row3 : 0.0;
    const u64 passed = __ballot(incl > p);
    if (passed) {
      // the highest lane at which it passes; of that lane's bins, from the top, lane i takes the i-th
      const int at = 63 - __builtin_clzll(passed), bin = kPer * at + kPer - 1 - min(lane, kPer - 1);
      const double before = at == 63 ? 0.0 : readlane_f64(incl, min(at + 1, 63));
      const u64 v = tb.bin[bin];
      double sum = lane < kPer ? bin_sum(v, bin) : 0.0;
      sum += dpp_f64<kDppRowShr + 1>(sum);
      sum += dpp_f64<kDppRowShr + 2>(sum);
      sum += dpp_f64<kDppRowShr + 4>(sum);
      sum += dpp_f64<kDppRowShr + 8>(sum);
      const double above = before + dpp_f64<kDppRowShr + 1>(sum);
      const u64 here = __ballot(before + sum > p) & ((1ull << kPer) - 1ull);
      if (lane == (here ? __builtin_ctzll(here) : kPer - 1)) {        // (none only by rounding)
        tb.at = bin;
        tb.count = (int)(v >> kBinCount);
        tb.above = above;
      }
    } else if (lane == 0) {
      tb.at = -1;
    }
  }
  block_sync<NT>(rb);
  // what every thread reads from LDS is made uniform: the branches on it are then scalar
  const int bin = uniform_i32(tb.at);
  int m = uniform_i32(tb.count);
  uint32_t theta = 0, low_bits = kBinLow;         // the pattern's bits below `theta` that are still open
  int bit = 29;
  if (bin >= 0 && uniform_i32((int)tb.odd) == 0) {
    theta = (uint32_t)(kBinFirst + bin) << kBinShift;
    bit = kBinShift - 1;
    if constexpr (REFINE) {
      if (__builtin_expect(m > kList, 0)) {
        for (int i = tid; i < 256; i += NT) tb.bin[i] = 0ull;
        block_sync<NT>(rb);
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const uint32_t b = __float_as_uint(a[k]);
          if ((b ^ theta) <= kBinLow) atomicAdd(&tb.bin[(b & kBinLow) >> kSubShift], (1ull << kBinCount) | (b & kSubLow));
          if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        block_sync<NT>(rb);
        if (wave == 0) {
          // lane l: the four parts from 4 (63 - l) up, the highest first
          const double unit = bin_unit(bin);
          double part[4], mine = 0.0;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int i = 4 * (63 - lane) + 3 - e;
            const u64 v = tb.bin[i];
            part[e] = (double)(uint32_t)(v >> kBinCount) * (double)__uint_as_float(theta | ((uint32_t)i << kSubShift)) +
                      (double)(v & ((1ull << kBinCount) - 1ull)) * unit;
            mine += part[e];
          }
          double incl = mine;                              // sums up to each lane: inside a row of 16 lanes, then the rows before
          incl += dpp_f64<kDppRowShr + 1>(incl);
          incl += dpp_f64<kDppRowShr + 2>(incl);
          incl += dpp_f64<kDppRowShr + 4>(incl);
          incl += dpp_f64<kDppRowShr + 8>(incl);
          const double row0 = readlane_f64(incl, 15), row1 = row0 + readlane_f64(incl, 31), row2 = row1 + readlane_f64(incl, 47);
          incl += lane < 16 ? 0.0 : lane < 32 ? row0 : lane < 48 ? row1 : row2;
          const double from = readlane_f64(tb.above, 0);
          const u64 passed = __ballot(from + incl > p);
          if (lane == (passed ? __builtin_ctzll(passed) : 63)) {        // (none only by rounding)
            double above = from + (incl - mine);
            int e = 0;
            while (e < 3 && above + part[e] <= p) above += part[e++];
            const int i = 4 * (63 - lane) + 3 - e;
            tb.at = i;
            tb.count = (int)(tb.bin[i] >> kBinCount);
            tb.above = above;
          }
        }
        block_sync<NT>(rb);
        theta |= (uint32_t)uniform_i32(tb.at) << kSubShift;
        m = uniform_i32(tb.count);
        low_bits = kSubLow;
        bit = kSubShift - 1;
      }
    }
    if (m <= kList) {
      if constexpr (kShare) {
        // a wavefront's places in the list are taken by one addition (one per register, each waited for: 1.4 us of a workgroup's 10 on rows of 9350)
        for (int i = tid; i < kList; i += NT) tb.bin[i] = 0ull;            // the bins have been read: what follows adds up here
        int mine = 0;
#pragma unroll
        for (int k = 0; k < R; ++k) mine += __popcll(__ballot((__float_as_uint(a[k]) ^ theta) <= low_bits));
        int at = 0;
        if (lane == 0 && mine > 0) at = (int)atomicAdd(&tb.listed, (uint32_t)mine);
        at = uniform_i32(at);
        if (mine > 0) {
#pragma unroll
          for (int k = 0; k < R; ++k) {
            const uint32_t b = __float_as_uint(a[k]);
            const u64 here = __ballot((b ^ theta) <= low_bits);
            if (here) {                                      // uniform
              const int before = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(here >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)here, 0u));
              if ((b ^ theta) <= low_bits) tb.list[at + before] = b;
              at += __popcll(here);
            }
          }
        }
        block_sync<NT>(rb);
        // every wavefront compares all candidates with its part of the list
        const int part = ((m + NT / 64 - 1) / (NT / 64) + 3) & ~3, k0 = wave * part, k1 = min(m, k0 + part);
        for (int c0 = 0; c0 < m && k0 < m; c0 += 64) {
          const uint32_t mine = tb.list[min(c0 + lane, m - 1)];
          uint32_t larger = 0u, equal = 0u, low = 0u;
          for (int k = k0; k < k1; k += 4) {               // the list ends in zeros
            const u32x4 four = *reinterpret_cast<const u32x4*>(tb.list + k);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              larger += four[e] > mine ? 1u : 0u;
              low += four[e] > mine ? four[e] & low_bits : 0u;
              equal += four[e] == mine ? 1u : 0u;
            }
          }
          if (c0 + lane < m) atomicAdd(&tb.bin[c0 + lane], (u64)low | (u64)larger << 32 | (u64)equal << 48);      // low: 256 parts of 18 bits
        }
      } else {
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const uint32_t b = __float_as_uint(a[k]);
          if ((b ^ theta) <= low_bits) tb.list[atomicAdd(&tb.listed, 1u)] = b;
          if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
      }
      block_sync<NT>(rb);
      // A candidate per thread: theta is the largest of them whose sum of those at least as large, on top of the bins above, exceeds p.
      const double edge = REFINE ? (double)__uint_as_float(theta) : bin_edge(bin), unit = bin_unit(bin), above = tb.above;
      uint32_t mine = 0u, th = 0u, equal = 0u, larger = 0u, low = 0u;
      if (64 * wave < m) {
        mine = tb.list[tid];
        if constexpr (kShare) {
          const u64 v = tid < m ? tb.bin[tid] : 0ull;
          low = (uint32_t)v;
          larger = (uint32_t)(v >> 32) & 0xFFFFu;
          equal = (uint32_t)(v >> 48);
        } else {
          for (int k = 0; k < m; k += 4) {                 // the list ends in zeros
            const u32x4 four = *reinterpret_cast<const u32x4*>(tb.list + k);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              larger += four[e] > mine ? 1u : 0u;
              low += four[e] > mine ? four[e] & low_bits : 0u;
              equal += four[e] == mine ? 1u : 0u;
            }
          }
        }
        const double sum = above + ((double)(larger + equal) * edge + (double)(low + equal * (mine & low_bits)) * unit);
        th = ~wave_min_u32(~((tid < m && sum > p) ? mine : 0u));
        if (m > 64 && lane == 0) atomicMax(&tb.theta, th);
      }
      if (m > 64) {
        block_sync<NT>(rb);
        th = tb.theta;
      }
      if (tid < m && mine == th) {                         // every such thread has the same to say
        tb.theta = th;
        tb.ties = equal;
        tb.above_theta = above + ((double)larger * edge + (double)low * unit);
      }
      block_sync<NT>(rb);
      const uint32_t found = (uint32_t)uniform_i32((int)tb.theta);
      if (found == 0u) return HitRule{theta, true, 0x7FFFFFFF};
      return tie_rule<R, NT, LIST>(d, base, n, a, found, readlane_f64(tb.above_theta, 0), uniform_i32((int)tb.ties), tb, new_last_t, rb, phase, tid);
    }
  }
  // two bits per round (one barrier each): the three candidates' sums are nested, so the largest candidate that passes is
  // what bit-by-bit bisection would reach.  Bit 30 is never set: the weights are <= 1.
  for (; bit >= 1; bit -= 2) {
    const uint32_t c1 = theta | (1u << (bit - 1)), c2 = theta | (1u << bit), c3 = c1 | c2;
    float p1 = 0.f, p2 = 0.f, p3 = 0.f;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t b = __float_as_uint(a[k]);
      p1 += (b >= c1) ? a[k] : 0.f;
      p2 += (b >= c2) ? a[k] : 0.f;
      p3 += (b >= c3) ? a[k] : 0.f;
    }
    block_sum3_f32<NT>(p1, p2, p3, rb, phase, tid);
    theta = uniform_f32(p3) > d.top_p ? c3 : uniform_f32(p2) > d.top_p ? c2 : uniform_f32(p1) > d.top_p ? c1 : theta;
  }
  if (theta == 0) return HitRule{0u, true, 0x7FFFFFFF};
  float above = 0.f;
  int ties = 0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const uint32_t b = __float_as_uint(a[k]);
    above += (b > theta) ? a[k] : 0.f;
    ties += (b == theta) ? 1 : 0;
  }
  above = uniform_f32(block_sum_f32<NT>(above, rb, phase, tid));
  ties = uniform_i32(block_sum_int<NT>(ties, rb, phase, tid));
  return tie_rule<R, NT, LIST>(d, base, n, a, theta, above, ties, tb, new_last_t, rb, phase, tid);
}

// `after_step1` runs once between Step 1 and the score update (the fused kernel
// picks up its queue claim there).
template <int R, int CH, int CP, class Val, int NT = kThreads, bool TOP_CLEARED = false, class Hook = NoHook, class New = NewEntry>
__device__ __forceinline__ void lrfu_regs(const Dev& d, int u, Slots base, int n, int B, int t, float (&a)[R], f32x4 (&crf)[CH],
                                          i32x4 (&tau)[CH], i32x4 (&ps)[CH], Val val, bool evict, uint32_t* evm, int* lst,
                                          int lst_cap, const float* s_tab, int s_tab_n, RedBuf<NT>& rb, int& phase, int* sh,
                                          int tid, Hook after_step1 = Hook{}, New ne = New{}, TopBuf* top = nullptr) {
  constexpr int C = R / 4;
  static_assert(C % CH == 0 && CP <= CH, "groups come in chunks of CH");
  const bool new_last = ne.there();                      // uniform
#pragma unroll
  for (int c = CP; c < CH; ++c) load_meta<NT>(d, base, n, t, c, tid, crf[c], tau[c], ps[c]);
  // what the end of the step would otherwise wait for: the unit's running sum, and the last slot's rows
  // (the entry that moves if exactly one entry is evicted)
  const u64 window0 = d.window[u];
  const bool evict_single = evict && n - B == 1;
  EntryRow last_row{{0u, 0u, 0u, 0u}, 0, 0};
  if (evict_single) {
    if constexpr (std::is_same_v<New, NewEntry>)
      last_row = new_last ? load_row_input<NT>(ne, tid) : load_row<NT>(d, base, n - 1, tid);
    else
      last_row = load_row<NT>(d, base, n - 1, tid);
  }
  // ---- Step 1: top-p hit set as a threshold on the weight's bit pattern
  const HitRule rule = top_p_regs<R, NT, TOP_CLEARED>(d, base, n, a, TOP_CLEARED ? *top : *reinterpret_cast<TopBuf*>(lst), new_last ? t : -1, rb, phase, tid);
  after_step1();
  // ---- Steps 2-3: scores; a[k] becomes CRF_temp.  The candidate for Step 4 (lowest score, then
  // highest position) is tracked on the way.
  u64 sfix = 0;
  u64 best = ~0ull;
  int best_i = -1;
#pragma unroll
  for (int cc = 0; cc < C; ++cc) {
    const int c = cc % CH;                  // register slot of group cc
    if (cc >= CH && c == 0) {               // next chunk of groups: its state is requested only now
      __builtin_amdgcn_sched_barrier(0);    // (and not earlier: hoisted, the chunks' registers would all be live at once)
#pragma unroll
      for (int k = 0; k < CH; ++k) load_meta<NT>(d, base, n, t, cc + k, tid, crf[k], tau[k], ps[k]);
    }
    // Straight-line, predicated code (selects instead of branches; entries beyond n compute on
    // whatever was loaded and are masked out of every result): branchy per-entry code ran at a small
    // fraction of the issue rate.
    const int e0 = 4 * (tid + cc * NT);
    f32x4 ncrf = crf[c];
    i32x4 ntau = tau[c];
    uint32_t stored = 0;                    // bit e: entry e0 + e gets a new (CRF, tau)
    const bool topp = d.reward_mode == 0;
    int delta4[4];
    float dec4[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) delta4[e] = min(max(t - tau[c][e], 0), d.tab_last);
    decay4_of(d, delta4, s_tab, s_tab_n, dec4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = e0 + e;
      const bool ok = i < n;
      const bool fresh = new_last & (i == n - 1);                    // the new entry: CRF 0, tau = position = t
      const int pe = fresh ? t : ps[c][e];
      const float w = a[4 * cc + e];
      const float dec = fresh ? 1.0f : dec4[e];
      const float crf_old = fresh ? 0.0f : crf[c][e];
      const uint32_t b = __float_as_uint(w);
      const bool hit = topp & (rule(b, pe) | ((i == n - 1) & (pe == t)));          // the entry appended this step is always hit
      const bool store = ok & (hit | !topp);
      const float reward = topp ? (hit ? 1.0f : 0.0f) : w;
      float tmp = __fadd_rn(__fmul_rn(dec, crf_old), reward);
      tmp = tmp < FLT_MIN ? 0.0f : tmp;
      ncrf[e] = store ? tmp : ncrf[e];
      ntau[e] = store ? t : ntau[e];
      stored |= (store ? 1u : 0u) << e;
      a[4 * cc + e] = ok ? tmp : 0.0f;
      // 2^-20 fixed point of the score: the scaling is exact, the split into two 32-bit halves too
      const float fx = floorf(tmp * kFixedOne);
      const uint32_t fhi = (uint32_t)(fx * 2.3283064365386963e-10f);
      const uint32_t flo = (uint32_t)(fx - (float)fhi * 4294967296.0f);
      sfix += ok ? (((u64)fhi << 32) | flo) : 0ull;
      const u64 key = ok ? evict_key(tmp, pe) : ~0ull;
      best_i = key < best ? i : best_i;
      best = key < best ? key : best;
      if (i == n - 1) {                     // the last slot's final state, for the in-place eviction
        sh[1] = __float_as_int(ncrf[e]);
        sh[2] = ntau[e];
        sh[3] = pe;
      }
    }
    if (e0 + 3 < n) {
      if (stored) {
        const size_t s0 = base + e0;
        *reinterpret_cast<f32x4*>(d.crf + s0) = ncrf;
        *reinterpret_cast<i32x4*>(d.tau + s0) = ntau;
      }
    } else if (e0 < n) {                     // the unit's last, partial group: entry by entry
      for (int e = 0; e < 4 && e0 + e < n; ++e) {
        if ((stored >> e) & 1u) {
          d.crf[base + (e0 + e)] = ncrf[e];
          d.tau[base + (e0 + e)] = t;
        }
      }
    }
  }
  // one reduction for both (in the fused kernel, which holds the next unit's first blocks beside this, it costs registers)
  constexpr bool kOneReduction = NT >= 512;
  int victim = -1;
  if (kOneReduction && evict_single)
    sfix = block_sum_min<NT>(sfix, best, best_i, victim, rb, phase, tid);
  else
    sfix = block_sum_u64<NT>(sfix, rb, phase, tid);
  if (tid == 0) {
    d.window[u] = window0 + sfix;
    d.t_unit[u] = t;
  }
  // ---- Step 4
  if (!(evict && n > B)) {
    if (tid == 0) d.nev[u] = 0;
    return;
  }
  if (evict_single) {
    int dst_pos;
    if constexpr (kOneReduction) {
      // (an entry has no key below the largest only if its score is a NaN of all ones: then the last one goes)
      dst_pos = victim < 0 ? sh[3] : ~(int)(uint32_t)best;
      victim = victim < 0 ? n - 1 : victim;
    } else {
      const u64 gbest = block_min_u64<NT>(best, rb, phase, tid);
      if (best == gbest && best_i >= 0) {   // keys are unique: one writer
        sh[0] = best_i;
        sh[4] = ~(int)(uint32_t)best;       // the victim's position
      }
      block_sync<NT>(rb);
      victim = sh[0];
      dst_pos = sh[4];
    }
    evict_one<NT>(d, base, n - 1, victim, dst_pos, sh, tid, last_row);
    if (tid == 0) {
      d.n[u] = B;
      d.nev[u] = 1;
    }
  } else {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const int i = 4 * (tid + (k >> 2) * NT) + (k & 3);
      if (i < n) val(i) = a[k];
    }
    block_sync<NT>(rb);
    evict_phase<Val, NT>(d, u, base, n, B, val, evm, lst, lst_cap, rb, phase, sh, tid);
  }
}

// Bookkeeping (Alg. 1 Steps 1-4) of a unit of n <= RMAX NT entries by one workgroup, from its logits in memory: a chain of memory
// round trips and block reductions, and what a whole step waits for.  So the entries' scores, times and positions and the first logits are asked for before
// `merge` (the unit's output and softmax statistics, whose own loads are on their way), later logits two groups ahead.  ne: the unit's last
// entry arrived in this step (its rows; what the cache says of it is not looked at), or nothing did.  COHERENT: the logits were written within
// the same launch, perhaps on another XCD.  top: cleared.
template <int NT, int RMAX, bool COHERENT, bool LEAN, class New, class Merge>
__device__ __forceinline__ void finish_unit(const Dev& d, int u, Slots base, int n, int B, int t, const float* sM, const float* sInv, uint32_t call_flags,
                                            float* val, uint32_t* evm, TopBuf* top, const float* s_tab, int s_tab_n, RedBuf<NT>& rb, int* sh, int tid,
                                            New ne, Merge merge) {
  int phase = 0;
  const int G = d.G;
  const Buffer logits = buffer_of(d.logits + (size_t)u * d.cap * G, d.cap * G);
  auto regs = [&](auto rc) {
    // (LEAN: few registers, as at logit_groups)
    constexpr int R = decltype(rc)::value, C = R / 4;
    constexpr int CH = C <= 2 ? C : LEAN ? (C % 2 == 0 ? 2 : 1) : C <= 4 ? C : 4, CG = logit_groups(C, NT, LEAN);
    static_assert(C % CG == 0, "groups come in chunks of CG");
    f32x4 crf[CH];
    i32x4 tau[CH], ps[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) load_meta<NT>(d, base, n, t, c, tid, crf[c], tau[c], ps[c]);
    f32x4 x[2][CG][kMaxGroup];
    auto request = [&](int c0, f32x4 (&to)[CG][kMaxGroup]) {
#pragma unroll
      for (int c = 0; c < CG; ++c) {
        const int e0 = 4 * (tid + (c0 + c) * NT), at = (e0 >> 5) * (G * kBlk) + (e0 & 31);      // beyond the unit: some value, or 0 from beyond its logits
#pragma unroll
        for (int g = 0; g < kMaxGroup; ++g)
          if (g < G) to[c][g] = get_f32x4<COHERENT ? kSc1 : 0>(logits, at + g * kBlk);
      }
    };
    request(0, x[0]);
    merge();
    const float invG = 1.0f / (float)G;
    float a[R];
#pragma unroll
    for (int c0 = 0; c0 < C; c0 += CG) {
      if (c0 + CG < C) request(c0 + CG, x[(c0 / CG + 1) & 1]);
      const auto& from = x[(c0 / CG) & 1];
#pragma unroll
      for (int c = 0; c < CG; ++c) {
        const int e0 = 4 * (tid + (c0 + c) * NT);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < kMaxGroup; ++g) {
          if (g < G) {                      // uniform; heads in ascending order, as everywhere
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += fast_exp2(from[c][g][e] - sM[g]) * sInv[g];
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) a[4 * (c0 + c) + e] = (e0 + e < n) ? acc[e] * invG : 0.f;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    lrfu_regs<R, CH, CH, ValLinear, NT, true>(d, u, base, n, leaves_unit(call_flags, n - B) ? n : B, t, a, crf, tau, ps, ValLinear{val},
                                              (call_flags & 1u) != 0, evm, reinterpret_cast<int*>(val), d.cap, s_tab, s_tab_n, rb, phase, sh, tid, NoHook{}, ne, top);
  };
  if constexpr (RMAX > 16)
    if (n > 16 * NT) return regs(std::integral_constant<int, 32>{});
  if constexpr (RMAX > 12)
    if (n > 8 * NT) return regs(std::integral_constant<int, 16>{});
  if constexpr (RMAX == 12)
    if (n > 8 * NT) return regs(std::integral_constant<int, 12>{});
  if constexpr (RMAX > 4)
    if (n > 4 * NT) return regs(std::integral_constant<int, 8>{});
  regs(std::integral_constant<int, 4>{});
}

// The bookkeeping of a step in a kernel of its own, deferred or straight behind layer_step_kernel, one workgroup per unit, at the time that the scan
// left for the unit's layer: the new entry's rows are in the cache and its logits with the others, the unit's records still describe the step
// before.  A unit is a chain of about ten block reductions and memory round trips, so few units take 1024 threads each
// (at most 8 entries per thread up to 8192).
template <int NT>
__global__ __launch_bounds__(NT) void finish_kernel(Dev d, int unit_begin, uint32_t call_flags) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* val = reinterpret_cast<float*>(smem);
  uint32_t* evm = reinterpret_cast<uint32_t*>(smem + (size_t)d.cap * 4);
  __shared__ TopBuf top;
  __shared__ float sM[kMaxGroup], sInv[kMaxGroup];
  __shared__ int32_t s_row[kMaxChunks];
  __shared__ RedBuf<NT> rb;
  __shared__ int sh[4 + (NT / 64 < 4 ? 4 : NT / 64)];
  __shared__ float s_tab[kTabLds];
  const int tid = threadIdx.x;
  const int u = unit_begin + blockIdx.x;
  const int n_old = d.n[u];
  const int t = d.layer_ts[u / (d.Bz * d.Hkv)];
  const int B = d.budget[u];
  const int s_tab_n = min(kTabLds, d.tab_last + 1);
  const bool room = n_old < unit_cap(d, u);
  if (tid < d.max_seg) s_row[tid] = d.tbl[(size_t)u * d.max_seg + tid];
  if (tid < s_tab_n) s_tab[tid] = d.tab[tid];
  if (tid < d.G) {
    sM[tid] = d.msum[((size_t)u * kMaxGroup + tid) * 2];
    sInv[tid] = d.msum[((size_t)u * kMaxGroup + tid) * 2 + 1];
  }
  clear_top(top, tid, NT);
  // Every wavefront has read the stored length before the first thread replaces it: a wavefront that started late
  // would otherwise count the new entry twice and part ways with the others.
  __syncthreads();
  const Slots base{s_row};
  const int n = n_old + (room ? 1 : 0);
  if (room && tid == NT - 1) {                             // (its score and time are written with the others')
    const size_t s = base + n_old;
    d.pos[s] = t;
    d.flags[s] = 0;
    d.n[u] = n;
  }
  // the new entry's rows are in the last slot like any other's, but nothing else there is yet
  if (n > 0)
    finish_unit<NT, NT == kWideThreads ? 32 : 8, false, NT == kWideThreads>(d, u, base, n, B, t, sM, sInv, call_flags, val, evm, &top, s_tab, s_tab_n, rb, sh, tid,
                                                        NewInCache{room}, []() {});
}

// What an attention-only step leaves besides the new entry's rows, behind a scan that leaves the records alone.
// grid: one workgroup.
__global__ __launch_bounds__(kWideThreads) void append_kernel(Dev d, int unit_begin, int count, int advance) {
  const int t = d.sc[SC_T];
  for (int u = unit_begin + (int)threadIdx.x; u < unit_begin + count; u += kWideThreads) {
    const int n = d.n[u];
    if (n < unit_cap(d, u)) {
      const size_t s = slots_of(d, u) + n;
      d.crf[s] = 0.0f;
      d.tau[s] = t;
      d.pos[s] = t;
      d.flags[s] = 0;
      d.n[u] = n + 1;
    }
  }
  __syncthreads();                                       // every wavefront has read the time
  if (advance && threadIdx.x == 0) {
    d.sc[SC_T] = t + 1;
    d.sc[SC_WINDOW_STEPS] = d.sc[SC_WINDOW_STEPS] + 1;
  }
}

// ------------------------------------------------------------------ prompt replay (scores of a loaded prompt)
// The prompt's last W queries in a few kernels per batch of queries.  What a query does to the scores splits
// into a part that does not depend on the scores - its mean attention weights over the entries it sees and,
// from them, the reward of every entry (Alg. 1 Steps 1-2: hit or not; or the weight itself) - and the score
// recurrence (Step 3), which is sequential over the queries but independent per entry.  So:
//   seed_scan_kernel     a pass over the keys for all queries of the batch: softmax partials per span of blocks
//   seed_stats_kernel    per query head: softmax maximum and 1 / sum over the entries the query sees
//   seed_weights_kernel  a second pass: the logits again, normalised, the mean over the heads -> weights
//   seed_hits_kernel     per (unit, query): hit rule, a bit per entry in place of the weights (top-p rule only)
//   seed_crf_kernel      per entry: the queries' rewards applied in order, from the state before the replay (seed_crf_hits_kernel: hits, short decay tables)
// (Two passes over the keys, 256 B per entry each, instead of the logits of every query head going through
// memory, 4 G B per entry and query written and read back.)  Only the weights are wanted (no output), so V is
// never read.
//
// Columns: the matrix-core tile has 16 query columns.  In the first pass, to which heads are all alike, column c of tile k is
// head i % G of query i / G, i = 16 k + c: ceil(G queries / 16) tiles.  In the second pass sixteen queries (a group) fill G
// tiles, column c of tile k
//   k < 4 (G / 4):  head 4 (k / 4) + c % 4 of the group's query 4 (k % 4) + c / 4
//   else:           head k of the group's query 4 (c % 4) + c / 4
// so that with the queries as the product's rows (the second pass) lane (j, kg) holds, of entry j, four heads of one
// query, or one head of the four queries whose other heads it also holds: the sum over a query's heads, in head
// order, never leaves the lane; the tiles of four heads that hold no query of a short group are left out.  (The second
// pass's columns in the first one too: a single query on G = 8 heads is 8 tiles instead of 1, of which the leftover heads' stay
// even if tiles without queries are skipped.  With the heads of 16 / G queries side by side in a tile, the sum took G - 1 lane
// shifts per logit, of which one lane in G was used, and a G that does not divide 16 left columns empty.)
// Both passes share a unit's blocks out over S wavefronts, as many as fill the chip evenly: with a wavefront per chunk of
// 256 entries, 128 units of 9350 entries were 1280 workgroups on 768 places.  Measured on that shape, 32 queries,
// G = 5: first pass 111 -> 88 us, second pass 163 -> 97 us.
// Then, the same shape: results of the products in ordinary registers (a compiler option), queries staged with all loads in flight, the
// segment table in a register, and in the second pass two tiles at a time with registers for three wavefronts per SIMD: 92 -> 88 and 98 -> 95 us.
// The first pass waits for its keys and for the issue of vector instructions in turn (with one tile in place of ten 56 us, without the
// exponentials 64); the second is bound by the products and by its stores (without them 77, without the products 66, without the exponentials 92 us).
// With three-operand maxima, the first keys asked for beside the queries and no divisions in front: first pass 79 -> 75 us, 64 such units 48.8 -> 47.2, 4
// units of 777 entries, 16 queries 9.1 -> 7.6.  (Two tiles at a time there: 78; keys two blocks ahead: 79; blocks dealt evenly to a block: no change.)
// Buffers of a batch of nq queries for the UL units of a layer (tiles and columns as in the first pass):
//   sml [tile][unit][span][column][2]     maximum (rounded up) and sum of the softmax over a wavefront's blocks
//   smi [tile][unit][column][2]           maximum (rounded up) and 1 / sum over all the entries the column's query sees
//   srw [query][unit][cap]                mean weights, then hits (a bit per entry at the start of the row)
constexpr int kSeedCols = 16;
constexpr int kSeedGroup = 16;         // queries that share G tiles
constexpr int kSeedTiles = 16;         // tiles of a batch, at most
constexpr float kNoMax = -FLT_MAX;     // maximum of no logit: finite, so that exponents relative to it are zeros, not NaNs
// Exponents are one fused multiply-add per logit (scale, minus the scaled maximum), while the maximum itself is a rounded
// product.  Up to 2^24 the two are within a half of each other; from 2^31 on within more than the exponential's
// range, and the sum of a column would be 0 or infinite.  Columns whose maximum lies beyond this bound take the product
// rounded, as the decode path does (which is exact at the maximum).
constexpr float kFarMax = 16777216.0f;
__device__ __forceinline__ bool is_far(float max) { return fabsf(max) > kFarMax && max != kNoMax; }
template <bool ROUNDED>
__device__ __forceinline__ float seed_exp(float logit, float scale, float max) {
  if constexpr (ROUNDED) return fast_exp2(logit * scale - max);
  return fast_exp2(__builtin_fmaf(logit, scale, -max));
}

// Tiles of the first pass.
__host__ __device__ __forceinline__ int seed_scan_tiles(int G, int nq) { return (nq * G + kSeedCols - 1) / kSeedCols; }

// Columns by the group size, as a product: exact for 0 <= i < 2^13 and G <= 8.  (A division is twenty instructions, and each wavefront
// had one per tile for its lanes' queries and another for their limits.)
struct PerGroup {
  int m;
  __device__ __forceinline__ explicit PerGroup(int G) : m(65536 / G + 1) {}
  __device__ __forceinline__ int operator()(int i) const { return (i * m) >> 16; }
};
static_assert(kSeedCols * (kSeedTiles + 1) <= 8192 && kMaxGroup <= 8, "what PerGroup divides");

// Query (of the batch) and head of column c of tile tl: first pass (of any tile's columns those beyond the batch have queries
// from nq on), second pass.
__device__ __forceinline__ int seed_scan_column(int G, PerGroup per_group, int tl, int c, int& head) {
  const int i = kSeedCols * tl + c, q = per_group(i);
  head = i - q * G;
  return q;
}
__device__ __forceinline__ int seed_column(int G, PerGroup per_group, int tl, int c, int& head) {
  const int group = per_group(tl), k = tl - group * G;
  const bool four = k < (G & ~3);
  head = four ? (k & ~3) + (c & 3) : k;
  return kSeedGroup * group + (four ? 4 * (k & 3) + (c >> 2) : 4 * (c & 3) + (c >> 2));
}

// The batch's queries as operands in LDS ([tile][32-dim slice][lane], 16 bytes each); 0 in columns without a query.
// `meanwhile` runs when they have been asked for.
template <class Column, class Meanwhile>
__device__ __forceinline__ void seed_stage_queries(const Dev& d, const uint16_t* q_obs, int urel, int j0, int nq, int nt, Column column, u32x4* s_q, Meanwhile meanwhile) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, b = urel / d.Hkv, h = urel % d.Hkv;
  const PerGroup per_group(d.G);
  u32x4 x[kSeedTiles];                                    // all asked for before the first is stored
#pragma unroll
  for (int tl = 0; tl < kSeedTiles; ++tl) {
    x[tl] = u32x4{0u, 0u, 0u, 0u};
    if (tl < nt) {
      int head;
      const int qi = column(d.G, per_group, tl, lane & 15, head);
      if (qi < nq)
        x[tl] = *reinterpret_cast<const u32x4*>(q_obs + ((((size_t)(j0 + qi) * d.Bz + b) * d.Hq) + (size_t)h * d.G + head) * kDim + 32 * wave + 8 * (lane >> 4));
    }
  }
  meanwhile();
#pragma unroll
  for (int tl = 0; tl < kSeedTiles; ++tl)
    if (tl < nt) s_q[(tl * 4 + wave) * 64 + lane] = x[tl];
}

// This wavefront's blocks [b, b1) of the unit, and where they lie: the segments of up to 512 blocks sit in a register, one per lane (a look at
// the table per block was a vector load, since the kernel stores elsewhere, and the wait for it one for every store before it).
struct SeedSpan {
  int segs, first;
  int b, b1;
  __device__ __forceinline__ SeedSpan(const Dev& d, int u, int slot, int S, int n_last) {
    const int blocks = (n_last + kBlk - 1) / kBlk, per = (blocks + S - 1) / S;
    b = min(slot * per, blocks);
    b1 = min(b + per, blocks);
    first = b / kSegBlocks;
    segs = d.tbl[(size_t)u * d.max_seg + min(first + (int)(threadIdx.x & 63), d.max_seg - 1)];
  }
  __device__ __forceinline__ size_t off(int blk) const {
    const int seg = __builtin_amdgcn_readlane(segs, blk / kSegBlocks - first);
    return (size_t)seg * kSegElems + (size_t)(blk & (kSegBlocks - 1)) * kBlkElems;
  }
};

// seed_scan_kernel: per span and column the maximum and sum of the softmax over the entries the column's query sees:
// query j of the window sees the entries of positions <= its own, i.e. indices < P - W + j + 1 (the prompt's entries
// sit in position order).
// grid: (ceil(S / 4), units of the layer), kThreads threads, nt * 4096 bytes of dynamic LDS.
__global__ __launch_bounds__(kThreads) void seed_scan_kernel(Dev d, int unit_begin, const uint16_t* __restrict__ q_obs, int j0, int nq, int P, int W,
                                                             int S, float* __restrict__ sml) {
  extern __shared__ unsigned char smem[];
  u32x4* s_q = reinterpret_cast<u32x4*>(smem);
  const int lane = threadIdx.x & 63;
  const int slot = __builtin_amdgcn_readfirstlane(blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6));
  const int urel = blockIdx.y, u = unit_begin + urel, UL = gridDim.y;
  const int j = lane & 15, kg = lane >> 4;
  const int G = d.G, nt = seed_scan_tiles(G, nq);
  const int n_first = P - W + j0 + 1;                     // entries the batch's first query sees
  SeedSpan sp(d, u, slot, S, n_first + nq - 1);
  const uint16_t* kp = d.K + lane * 8;
  KFrag ka;
  // the first keys (of a wavefront without blocks, some that nobody looks at) are on their way before the queries are there
  seed_stage_queries(d, q_obs, urel, j0, nq, nt, seed_scan_column, s_q, [&]() { load_k(ka, kp + sp.off(sp.b)); });
  __syncthreads();
  if (slot >= S) return;
  const PerGroup per_group(G);
  int q_lo[kSeedTiles + 1];                               // the tiles' first queries
#pragma unroll
  for (int tl = 0; tl <= kSeedTiles; ++tl) q_lo[tl] = per_group(kSeedCols * tl);
  float m_run[kSeedTiles], l_run[kSeedTiles];             // of this lane's entries; the four lanes of a column meet at the end
#pragma unroll
  for (int tl = 0; tl < kSeedTiles; ++tl) {
    m_run[tl] = kNoMax;
    l_run[tl] = 0.f;
  }
  const float c = d.scale_log2e;
  auto sweep = [&](auto rounded) {
    KFrag kn;
    for (int blk = sp.b; blk < sp.b1; ++blk) {
      load_k(kn, kp + sp.off(min(blk + 1, sp.b1 - 1)));
      const int e0 = blk * kBlk + 4 * kg;
#pragma unroll
      for (int tl = 0; tl < kSeedTiles; ++tl) {
        if (tl < nt && blk * kBlk < n_first + min(q_lo[tl + 1], nq - 1)) {     // uniform: else no query of the tile sees the block
          bf16x8 qv[4];
#pragma unroll
          for (int s4 = 0; s4 < 4; ++s4) qv[s4] = as_bf16x8(s_q[(tl * 4 + s4) * 64 + lane]);
          f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s4 = 0; s4 < 4; ++s4) s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ka.k[s4]), qv[s4], s0, 0, 0, 0);
#pragma unroll
          for (int s4 = 0; s4 < 4; ++s4) s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ka.k[4 + s4]), qv[s4], s1, 0, 0, 0);
          float sv[8];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            sv[v] = s0[v];
            sv[4 + v] = s1[v];
          }
          if ((blk + 1) * kBlk > n_first + q_lo[tl]) {      // a block that the tile's first query sees whole needs no mask
            const int lim = n_first + per_group(kSeedCols * tl + j);       // entries this column's query sees
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              sv[v] = (e0 + v < lim) ? sv[v] : -INFINITY;
              sv[4 + v] = (e0 + 16 + v < lim) ? sv[4 + v] : -INFINITY;
            }
          }
          // The maximum is kept rounded up to a whole number: sums are then rescaled by exact powers of two, here and
          // where partials meet.  Every tile looks for it, so that the exponents of what weighs are small and carry the rounding of
          // small numbers.  (Looked for in a span's first block alone, sums redone from 2^60 on: 12 us less, but weights off by
          // 1.6e-6 where logits rise by 40 behind that block, else by 3e-7.  Tiles done again where eight exponentials pass 16:
          // no slower on even prompts, 22 us slower on ones with heavy entries here and there.)
          // (Of a maximum that propagates NaN there is an instruction for three, and its operands need no look at signalling ones.)
          const float bm = c * max3(max3(sv[0], sv[1], sv[2]), max3(sv[3], sv[4], sv[5]), max2(sv[6], sv[7]));
          const float m_new = max2(m_run[tl], ceilf(bm));
          l_run[tl] *= fast_exp2(m_run[tl] - m_new);        // 0 the first time
          m_run[tl] = m_new;
          float p[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) p[i] = seed_exp<decltype(rounded)::value>(sv[i], c, m_run[tl]);
          l_run[tl] += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
        }
      }
      ka = kn;
    }
  };
  sweep(std::false_type{});
  bool far = false;
#pragma unroll
  for (int tl = 0; tl < kSeedTiles; ++tl) far |= is_far(m_run[tl]);
  if (__any(far)) {                                       // the maxima stand; the sums once more
#pragma unroll
    for (int tl = 0; tl < kSeedTiles; ++tl) l_run[tl] = 0.f;
    if (sp.b < sp.b1) load_k(ka, kp + sp.off(sp.b));
    sweep(std::true_type{});
  }
  // per tile, the column's four lanes (kg = 0..3): maximum, then the sums rescaled to it
#pragma unroll
  for (int tl = 0; tl < kSeedTiles; ++tl) {
    if (tl < nt) {
      auto max_of = [](float x, float y) { return fmaxf(x, y); };
      const float M = rows_combine(m_run[tl], max_of);
      const float l = rows_combine(l_run[tl] * fast_exp2(m_run[tl] - M), [](float x, float y) { return x + y; });
      if (kg == 0)
        *reinterpret_cast<float2*>(sml + ((((size_t)tl * UL + urel) * S + slot) * kSeedCols + j) * 2) = make_float2(M, l);
    }
  }
}

// seed_stats_kernel: maximum and 1 / sum of a column's softmax over the spans.  Eight threads per column, thread k takes spans
// k, k + 8, .. in order, and the eight sums are added up in pairs (one chain of all spans would round as often as there are
// spans, in the same direction for every weight of the column).  Sixteen partials are asked for at a time: by one thread per
// column, eight at a time, eight units of 32000 entries (500 spans) took 30 us, now 6.
// grid: (units of the layer, tiles of the first pass), 8 kSeedCols threads.
__global__ __launch_bounds__(8 * kSeedCols) void seed_stats_kernel(int S, const float* __restrict__ sml, float* __restrict__ smi) {
  const int urel = blockIdx.x, UL = gridDim.x, tl = blockIdx.y;
  const int lane = threadIdx.x & 63, col = (threadIdx.x >> 6) * 8 + (lane & 7), k = lane >> 3;
  const float* ml = sml + ((((size_t)tl * UL + urel) * S) * kSeedCols + col) * 2;
  constexpr int kAhead = 16;
  float2 p[kAhead];
  auto request = [&](int c0) {
#pragma unroll
    for (int i = 0; i < kAhead; ++i) p[i] = *reinterpret_cast<const float2*>(ml + (size_t)min(c0 + 8 * i, S - 1) * kSeedCols * 2);
  };
  float M = kNoMax;
  for (int c0 = k; c0 < S; c0 += 8 * kAhead) {
    request(c0);
#pragma unroll
    for (int i = 0; i < kAhead; ++i) M = fmaxf(M, p[i].x);
  }
  M = fmaxf(M, __shfl_xor(M, 8));
  M = fmaxf(M, __shfl_xor(M, 16));
  M = fmaxf(M, __shfl_xor(M, 32));
  float l = 0.f;
  for (int c0 = k; c0 < S; c0 += 8 * kAhead) {
    if (S > 8 * kAhead) request(c0);                       // a column of 128 spans is still there
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
      if (c0 + 8 * i < S) l += p[i].y * fast_exp2(p[i].x - M);
  }
  l += __shfl_xor(l, 8);
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  // a head none of whose logits is above -inf weighs nothing
  if (k == 0) *reinterpret_cast<float2*>(smi + (((size_t)tl * UL + urel) * kSeedCols + col) * 2) = make_float2(M, l == 0.0f ? 0.0f : 1.0f / l);
}

// seed_weights_kernel: every logit normalised with its column's maximum and 1 / sum, the mean over a query's heads
// (summed in head order, as the decode path's mean weights are) to `srw`; entries that a query does not see, but others of the
// batch in the same block do, get 0.  Grid and LDS as seed_scan_kernel.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void seed_weights_kernel(Dev d, int unit_begin, const uint16_t* __restrict__ q_obs, int j0, int nq, int P,
                                                                int W, int S, const float* __restrict__ smi, float* __restrict__ srw) {
  extern __shared__ unsigned char smem[];
  u32x4* s_q = reinterpret_cast<u32x4*>(smem);
  __shared__ __align__(16) float s_M[kSeedTiles * kSeedCols], s_I[kSeedTiles * kSeedCols];      // every column's maximum and 1 / (G sum)
  const int lane = threadIdx.x & 63;
  const int slot = __builtin_amdgcn_readfirstlane(blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6));
  const int urel = blockIdx.y, u = unit_begin + urel, UL = gridDim.y;
  const int j = lane & 15, kg = lane >> 4;
  const int G = d.G, groups = (nq + kSeedGroup - 1) / kSeedGroup, nt = groups * G;
  const int n_first = P - W + j0 + 1;
  const float invG = 1.0f / (float)G;
  SeedSpan sp(d, u, slot, S, n_first + nq - 1);
  float2 mi = make_float2(0.f, 0.f);
  if ((int)threadIdx.x < nt * kSeedCols) {
    int head;
    const int i = seed_column(G, PerGroup(G), threadIdx.x / kSeedCols, threadIdx.x % kSeedCols, head) * G + head;         // the column's place in the first pass
    if (i < nq * G) mi = *reinterpret_cast<const float2*>(smi + (((size_t)(i / kSeedCols) * UL + urel) * kSeedCols + i % kSeedCols) * 2);
  }
  const uint16_t* kp = d.K + lane * 8;
  KFrag k0, k1;
  seed_stage_queries(d, q_obs, urel, j0, nq, nt, seed_column, s_q, [&]() { load_k(k0, kp + sp.off(sp.b)); });
  if ((int)threadIdx.x < nt * kSeedCols) {
    s_M[threadIdx.x] = mi.x;
    s_I[threadIdx.x] = mi.y * invG;
  }
  __syncthreads();
  if (slot >= S) return;
  bool far = false;
  for (int i = lane; i < nt * kSeedCols; i += 64) far |= is_far(s_M[i]);
  const float c = d.scale_log2e;
  const size_t lane_row = (size_t)kg * UL * d.cap + j;
  auto sweep = [&](auto rounded) {
    auto block = [&](const KFrag& ka, int blk) {
#pragma unroll 1
      for (int gr = 0; gr < groups; ++gr) {
        const int q0 = kSeedGroup * gr;
        if (blk * kBlk >= n_first + min(q0 + kSeedGroup - 1, nq - 1)) continue;      // uniform: no query of the group sees the block
        float mean[4][2];                                   // queries q0 + 4 t + kg, entries j and 16 + j of the block
#pragma unroll
        for (int t = 0; t < 4; ++t) mean[t][0] = mean[t][1] = 0.f;
        struct Tile {
          f32x4 s0, s1;
        };
        auto products = [&](int tl) -> Tile {
          Tile x{{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
          for (int s4 = 0; s4 < 4; ++s4) {
            const bf16x8 qv = as_bf16x8(s_q[(tl * 4 + s4) * 64 + lane]);
            x.s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qv, as_bf16x8(ka.k[s4]), x.s0, 0, 0, 0);
            x.s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qv, as_bf16x8(ka.k[4 + s4]), x.s1, 0, 0, 0);
          }
          return x;
        };
        // four heads of one query
        auto heads = [&](int tl, const Tile& x, float (&m)[2]) {
          const f32x4 M = *reinterpret_cast<const f32x4*>(s_M + tl * kSeedCols + 4 * kg), I = *reinterpret_cast<const f32x4*>(s_I + tl * kSeedCols + 4 * kg);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            m[0] = __builtin_fmaf(seed_exp<decltype(rounded)::value>(x.s0[v], c, M[v]), I[v], m[0]);
            m[1] = __builtin_fmaf(seed_exp<decltype(rounded)::value>(x.s1[v], c, M[v]), I[v], m[1]);
          }
        };
#pragma unroll 1
        for (int h = 0; h + 4 <= G; h += 4) {
          const int tl = gr * G + h;
          if (q0 + 12 < nq) {                             // no tile without queries: two at a time, one's products under the other's exponentials
            const Tile x0 = products(tl), x1 = products(tl + 1);
            heads(tl, x0, mean[0]);
            heads(tl + 1, x1, mean[1]);
            const Tile x2 = products(tl + 2), x3 = products(tl + 3);
            heads(tl + 2, x2, mean[2]);
            heads(tl + 3, x3, mean[3]);
          } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              if (q0 + 4 * t >= nq) continue;             // uniform
              heads(tl + t, products(tl + t), mean[t]);
            }
          }
        }
#pragma unroll 1
        for (int h = G & ~3; h < G; ++h) {
          const int tl = gr * G + h;
          const Tile x = products(tl);
          const f32x4 M = *reinterpret_cast<const f32x4*>(s_M + tl * kSeedCols + 4 * kg), I = *reinterpret_cast<const f32x4*>(s_I + tl * kSeedCols + 4 * kg);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            mean[v][0] = __builtin_fmaf(seed_exp<decltype(rounded)::value>(x.s0[v], c, M[v]), I[v], mean[v][0]);
            mean[v][1] = __builtin_fmaf(seed_exp<decltype(rounded)::value>(x.s1[v], c, M[v]), I[v], mean[v][1]);
          }
        }
        // The next block's keys, on their way since this one began, and the last group's stores are waited for here: a wait for the keys
        // behind stores whose number the compiler does not know would be a wait for those stores, just issued.
        __builtin_amdgcn_s_waitcnt(kWaitLoads);
        // (a lane's rows are 4 queries apart: one 64-bit addition each to addresses that are the same in all lanes)
        if ((blk + 1) * kBlk <= n_first + q0 && q0 + kSeedGroup <= nq) {       // every query of the group is there and sees the block whole
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            float* dst = srw + ((size_t)(q0 + 4 * t) * UL + urel) * d.cap + blk * kBlk + lane_row;
            dst[0] = mean[t][0];
            dst[16] = mean[t][1];
          }
        } else {
          const int e0 = blk * kBlk + j;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int qi = q0 + 4 * t + kg;
            if (qi < nq) {
              const int lim = n_first + qi;                   // entries the query sees
              float* dst = srw + ((size_t)(q0 + 4 * t) * UL + urel) * d.cap + blk * kBlk + lane_row;
              dst[0] = e0 < lim ? mean[t][0] : 0.f;
              dst[16] = e0 + 16 < lim ? mean[t][1] : 0.f;
            }
          }
        }
      }
    };
    // two blocks in turn, the next always on its way
    for (int blk = sp.b; blk < sp.b1; blk += 2) {
      load_k(k1, kp + sp.off(min(blk + 1, sp.b1 - 1)));
      block(k0, blk);
      if (blk + 1 < sp.b1) {
        load_k(k0, kp + sp.off(min(blk + 2, sp.b1 - 1)));
        block(k1, blk + 1);
      }
    }
  };
  if (__any(far))
    sweep(std::true_type{});
  else
    sweep(std::false_type{});
}

// seed_hits_kernel (top-p rule only): one workgroup per (query of the batch, unit).  The query's mean weights
// from `srw`, the hit rule, and in their place the hits, a bit per entry at the start of the row (the query's own entry,
// the last it sees, is always hit): every thread has its weights in registers (or LDS) before the first bit is written.
// (As rewards of 4 bytes they were 153 MB per layer of 128 units of 9350 entries and 32 queries, written and read.)
// grid: (queries of the batch, units of the layer), kSeedThreads threads, kSeedHitsLds of dynamic LDS (R = 0: cap floats).
constexpr int kSeedThreads = 512;      // prompts are long
constexpr size_t kSeedHitsLds = sizeof(TopBuf) + 64 * 8;

template <int R>
__device__ __forceinline__ void seed_rewards_regs(const Dev& d, Slots base, int n, bool last_new, float* rw, int* lst, RedBuf<kSeedThreads>& rb, int& phase,
                                                  int tid) {
  float a[R];
  f32x4 x[R / 4];
#pragma unroll
  for (int c = 0; c < R / 4; ++c) {
    const int e0 = 4 * (tid + c * kSeedThreads);
    x[c] = *reinterpret_cast<const f32x4*>(rw + min(e0, (n - 1) & ~3));
  }
  clear_top(*reinterpret_cast<TopBuf*>(lst), tid, kSeedThreads);            // while the weights are on their way
#pragma unroll
  for (int c = 0; c < R / 4; ++c) {
    const int left = n - 4 * (tid + c * kSeedThreads);
    if (4 * kSeedThreads * (c + 1) <= n) {                   // uniform: the row goes on behind them
#pragma unroll
      for (int e = 0; e < 4; ++e) a[4 * c + e] = x[c][e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) a[4 * c + e] = e < left ? x[c][e] : 0.f;
    }
  }
  block_sync<kSeedThreads>(rb);
  const HitRule rule = top_p_regs<R, kSeedThreads, true, true>(d, base, n, a, *reinterpret_cast<TopBuf*>(lst), -1, rb, phase, tid);
  uint32_t* bits = reinterpret_cast<uint32_t*>(rw);
#pragma unroll
  for (int c = 0; c < R / 4; ++c) {
    const int e0 = 4 * (tid + c * kSeedThreads);
    uint32_t word = 0;
    if (rule.ties_all) {                                   // uniform, nearly always
#pragma unroll
      for (int e = 3; e >= 0; --e) word += word + (__float_as_uint(a[4 * c + e]) >= rule.theta ? 1u : 0u);      // an addition with carry each
    } else if (e0 < n) {
      const i32x4 ps = *reinterpret_cast<const i32x4*>(d.pos + (base + e0));
#pragma unroll
      for (int e = 0; e < 4; ++e) word |= (rule(__float_as_uint(a[4 * c + e]), ps[e]) ? 1u : 0u) << e;
    }
    // the query's own entry, the row's last; nothing beyond it
    const int left = n - e0;
    if (left < 4) word &= left <= 0 ? 0u : (1u << left) - 1u;
    if (left >= 1 && left <= 4 && last_new) word |= 1u << (left - 1);
    // the word's eight nibbles sit in eight consecutive lanes
    word <<= 4 * (tid & 7);
    word |= dpp_u32<kDppQuadSwap1>(word);
    word |= dpp_u32<kDppQuadSwap2>(word);
    word |= dpp_u32<kDppRowHalfMirror>(word);
    if ((tid & 7) == 0 && e0 < n) bits[e0 >> 5] = word;
  }
}

// R: entries per thread, in registers, chosen by the longest row of the launch (a multiple of four), so that short rows do not
// pay for the registers of long ones: up to 16 four workgroups per compute unit, up to 24 three, up to 32 two; 0: weights in
// LDS, any length.
template <int R>
__global__ __launch_bounds__(kSeedThreads, R == 0 || R > 24 ? 4 : R > 16 ? 6 : 8) void seed_hits_kernel(Dev d, int unit_begin, int j0, int P, int W,
                                                                                                      float* __restrict__ srw) {
  extern __shared__ unsigned char smem[];
  __shared__ RedBuf<kSeedThreads> rb;
  const int tid = threadIdx.x;
  const int ql = blockIdx.x, urel = blockIdx.y, u = unit_begin + urel;
  const int UL = gridDim.y;
  const int t = P - W + j0 + ql;                          // the query's position = its time
  const int n = t + 1;
  const Slots base = slots_of(d, u);
  const bool last_new = d.pos[base + (n - 1)] == t;       // the query's own entry (asked for early: nothing waits for it until the end)
  int phase = 0;
  float* rw = srw + ((size_t)ql * UL + urel) * d.cap;
  if constexpr (R > 0) {
    seed_rewards_regs<R>(d, base, n, last_new, rw, reinterpret_cast<int*>(smem), rb, phase, tid);
  } else {
    float* val = reinterpret_cast<float*>(smem);
    for (int i = tid; i < n; i += kSeedThreads) val[i] = rw[i];
    __syncthreads();
    const HitRule rule = top_p_lds<ValLinear, kSeedThreads>(d, base, n, ValLinear{val}, rb, phase, tid);
    uint32_t* bits = reinterpret_cast<uint32_t*>(rw);
    for (int i0 = tid & ~63; i0 < n; i0 += kSeedThreads) {          // a wavefront's 64 entries are two words
      const int i = i0 + (tid & 63), ic = min(i, n - 1);
      const int pe = !rule.ties_all ? d.pos[base + ic] : 0;
      const u64 mask = __ballot(i < n && (rule(__float_as_uint(val[ic]), pe) | ((i == n - 1) & last_new)));
      if ((tid & 31) == 0 && i < n) bits[i >> 5] = (uint32_t)(mask >> (tid & 32));
    }
  }
}

// seed_crf_kernel: Alg. 1 Step 3 for the batch's queries in order, four consecutive entries per thread: an entry
// takes part from the query of its own position on; under the top-p rule only a hit replaces (CRF, tau).
// BITS: the queries' hits, a bit per entry at the start of each query's row (the top-p rule); else the weights themselves.
// (Hits under a table that LDS holds whole: seed_crf_hits_kernel.)
// The replay's first batch starts from the state before it (every entry referenced once, on arrival: CRF 1, tau =
// position; the W entries of the window not yet arrived: CRF 0), the last one leaves the units' records as a fresh
// context has them: no trace in the aggregated-CRF window, last-step time t_unit.
// grid: (ceil(P / (4 kThreads)), units of the layer), kThreads threads.
template <bool BITS>
__global__ __launch_bounds__(kThreads) void seed_crf_kernel(Dev d, int unit_begin, int j0, int nq, int P, int W, int t_unit,
                                                            const float* __restrict__ srw) {
  __shared__ float s_tab[kTabLds];
  const int tid = threadIdx.x;
  const int urel = blockIdx.y, u = unit_begin + urel;
  const int UL = gridDim.y;
  const int s_tab_n = min(kTabLds, d.tab_last + 1);
  if (tid < s_tab_n) s_tab[tid] = d.tab[tid];
  if (j0 + nq == W && blockIdx.x == 0 && tid == 0) {
    d.window[u] = 0;
    d.t_unit[u] = t_unit;
  }
  __syncthreads();
  const int e0 = 4 * (blockIdx.x * kThreads + tid);
  if (e0 >= P) return;
  const Slots base = slots_of(d, u);
  const size_t s0 = base + e0;                            // four consecutive entries share a segment
  f32x4 crf;
  i32x4 tau;
  if (j0 == 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      crf[e] = e0 + e < P - W ? 1.0f : 0.0f;
      tau[e] = e0 + e;
    }
  } else {
    crf = *reinterpret_cast<const f32x4*>(d.crf + s0);
    tau = *reinterpret_cast<const i32x4*>(d.tau + s0);
  }
  const float* rw = srw + (size_t)urel * d.cap + (BITS ? e0 >> 5 : e0);
  const size_t q_stride = (size_t)UL * d.cap;
  const int t_first = P - W + j0;
  bool changed = j0 == 0;
  // the four entries' updates at time t, side by side; entry e takes part if bit e of m is set
  auto update = [&](uint32_t m, int t, f32x4 reward) {
    int delta[4];
    float dec[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) delta[e] = min(max(t - tau[e], 0), d.tab_last);
    decay4_of(d, delta, s_tab, s_tab_n, dec);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = (m >> e) & 1u;
      float tmp = __fadd_rn(__fmul_rn(dec[e], crf[e]), reward[e]);
      tmp = tmp < FLT_MIN ? 0.0f : tmp;
      crf[e] = in ? tmp : crf[e];
      tau[e] = in ? t : tau[e];
    }
    changed |= m != 0u;
  };
  // bits of the entries that the query at time t sees: positions 0 .. t
  auto seen = [&](int t) -> uint32_t { return t >= e0 + 3 ? 0xFu : t < e0 ? 0u : (2u << (t - e0)) - 1u; };
  for (int q0 = 0; q0 < nq; q0 += 8) {
    if constexpr (BITS) {
      uint32_t r[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) r[k] = __float_as_uint(rw[(size_t)min(q0 + k, nq - 1) * q_stride]);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int t = t_first + q0 + k;
        update(q0 + k < nq ? (r[k] >> (e0 & 31)) & seen(t) : 0u, t, f32x4{1.0f, 1.0f, 1.0f, 1.0f});
      }
    } else {
      f32x4 r[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) r[k] = *reinterpret_cast<const f32x4*>(rw + (size_t)min(q0 + k, nq - 1) * q_stride);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int t = t_first + q0 + k;
        update(q0 + k < nq ? seen(t) : 0u, t, r[k]);
      }
    }
  }
  if (!changed) return;
  if (e0 + 3 < P) {
    *reinterpret_cast<f32x4*>(d.crf + s0) = crf;
    *reinterpret_cast<i32x4*>(d.tau + s0) = tau;
  } else {
    for (int e = 0; e < 4 && e0 + e < P; ++e) {
      d.crf[s0 + e] = crf[e];
      d.tau[s0 + e] = tau[e];
    }
  }
}

// The same for hits where LDS holds the whole decay table (a score that 1 is added to needs no look at the smallest number, and an entry's
// time is within the table's reach or clamped to its end).  A lane has four entries 64 apart, so that a wavefront's hits of a query are
// eight words in scalar registers, whose pairs are the selects' conditions as they are: no bit is tested per lane.  An entry's time is kept as its
// place in the table at the chunk's first query; later queries read on from there, at an offset known when it is compiled.  Four vector
// instructions and an LDS read per entry and query; with four consecutive entries per lane, bits and times looked at in vector registers, it
// took 14, and their issue was what bounded it.  128 units of 9350 entries, 32 queries: 20.3 -> 12.7 us,
// 64 such units 14.3 -> 9.2, 4 units of 777, 16 queries 6.1 -> 4.8.  (Words through scalar loads, eight queries at a time: no faster than before, and 8.6 for
// the last; the trips to memory follow one another.)
// An entry that has not arrived has score 0, so that its time, which starts at its position, does not matter before its first hit.
// grid: (ceil(P / (4 kThreads)), units of the layer), kThreads threads.
constexpr int kCrfChunk = 8;                              // queries per vector register of hits
constexpr int kMaxSeedBatch = kSeedTiles * kSeedGroup;    // queries of a batch, at most (G = 1)
__global__ __launch_bounds__(kThreads) void seed_crf_hits_kernel(Dev d, int unit_begin, int j0, int nq, int P, int W, int t_unit, const uint32_t* __restrict__ hits) {
  __shared__ float s_tab[kTabLds + kMaxSeedBatch + kCrfChunk];      // no time of the batch lies beyond it
  const int tid = threadIdx.x, lane = tid & 63;
  const int urel = blockIdx.y, u = unit_begin + urel;
  const int first = __builtin_amdgcn_readfirstlane((blockIdx.x * (kThreads / 64) + (tid >> 6)) * 256);      // the wavefront's first entry
  const int t_first = P - W + j0;
  const size_t q_stride = (size_t)gridDim.y * d.cap;
  const uint32_t* row = hits + (size_t)urel * d.cap + min(first, P - 1) / 32 + (lane & 7);
  for (int i = tid; i < d.tab_last + nq + kCrfChunk; i += kThreads) s_tab[i] = d.tab[min(i, d.tab_last)];
  // four registers of hits: lane l has word l % 8 of query l / 8 of its eight
  constexpr int kRegs = 4;
  uint32_t w[kRegs];
  auto request = [&](int q0) {
#pragma unroll
    for (int i = 0; i < kRegs; ++i) w[i] = row[(size_t)min(q0 + kCrfChunk * i + (lane >> 3), nq - 1) * q_stride];
  };
  request(0);
  if (j0 + nq == W && blockIdx.x == 0 && tid == 0) {
    d.window[u] = 0;
    d.t_unit[u] = t_unit;
  }
  const size_t s0 = (size_t)d.tbl[(size_t)u * d.max_seg + min(first / kSeg, d.max_seg - 1)] * kSeg + lane;      // its entries are a segment
  __syncthreads();
  if (first >= P) return;
  float crf[4];
  int at[4];                                              // place in the table at the chunk's first query, in bytes
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i = first + 64 * e + lane;
    int tau = i;
    if (j0 == 0) {
      crf[e] = i < P - W ? 1.0f : 0.0f;
    } else {
      crf[e] = d.crf[s0 + 64 * e];                        // (the whole segment is the unit's)
      tau = d.tau[s0 + 64 * e];
    }
    at[e] = 4 * min(max(t_first - tau, 0), d.tab_last);
  }
  u64 any[4] = {0, 0, 0, 0};
  int q_end = 0;                                          // the query at which `at` is the entry's age
  for (int q0 = 0; q0 < nq; q0 += kRegs * kCrfChunk) {
    uint32_t seen[kRegs];
#pragma unroll
    for (int i = 0; i < kRegs; ++i) {                     // positions 0 .. t; what lies beyond a row's hits is not theirs
      const int q = q0 + kCrfChunk * i + (lane >> 3), left = t_first + q + 1 - (first + 32 * (lane & 7));
      seen[i] = q >= nq || left <= 0 ? 0u : left >= 32 ? w[i] : w[i] & ((1u << left) - 1u);
    }
    if (q0 + kRegs * kCrfChunk < nq) request(q0 + kRegs * kCrfChunk);
#pragma unroll
    for (int i = 0; i < kRegs; ++i) {
      if (q0 + kCrfChunk * i >= nq) break;                // uniform
#pragma unroll
      for (int k = 0; k < kCrfChunk; ++k) {
        float dec[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) dec[e] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(s_tab) + at[e] + 4 * k);
#pragma unroll
        for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(dec[e]));      // by every lane: else each becomes a branch, with a wait of its own
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const u64 m = ((u64)(uint32_t)__builtin_amdgcn_readlane((int)seen[i], 8 * k + 2 * e + 1) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane((int)seen[i], 8 * k + 2 * e);
          any[e] |= m;
          const bool in = __builtin_amdgcn_inverse_ballot_w64(m);
          const float tmp = __fadd_rn(__fmul_rn(dec[e], crf[e]), 1.0f);
          crf[e] = in ? tmp : crf[e];
          at[e] = in ? -4 * k : at[e];                    // read again from the next query on
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) at[e] += 4 * kCrfChunk;
      q_end += kCrfChunk;
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i = first + 64 * e + lane;
    const bool hit = __builtin_amdgcn_inverse_ballot_w64(any[e]);
    if (i < P && (hit || j0 == 0)) {
      d.crf[s0 + 64 * e] = crf[e];
      d.tau[s0 + 64 * e] = hit ? t_first + q_end - at[e] / 4 : i;
    }
  }
}

// Alg. 1 Step 4 on its own: scores decayed to the unit's last step, no update.  One workgroup per unit; what is to
// move follows in evict_move_kernel, except a single entry (one eviction per step), which moves here.
// n_sink < 0: Alg. 1 Step 4 (retain the highest CRF_temp).  n_sink >= 0: the comparison policy of Sec. 2.3
// that keeps the initial and the most recent tokens; the retention key is then the position itself, carried
// as a bit pattern (the eviction only ever compares the bits), and the largest pattern for positions below n_sink.
template <int R, int NT>
__device__ __forceinline__ void evict_unit(const Dev& d, int u, Slots base, int n, int B, int n_sink, int moves_follow, const float* s_tab, int s_tab_n,
                                           uint32_t* evm, CutBuf& cb, RedBuf<NT>& rb, int* sh, int tid) {
  const int t = d.t_unit[u];
  uint32_t b[R], np[R];
#pragma unroll
  for (int c = 0; c < R / 4; ++c) {
    const int e0 = 4 * (tid + c * NT);
    f32x4 crf;
    i32x4 tau, ps;
    if (n_sink < 0)
      load_meta<NT>(d, base, n, t, c, tid, crf, tau, ps);
    else
      ps = *reinterpret_cast<const i32x4*>(d.pos + (base + min(e0, (n - 1) & ~3)));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t key;
      if (n_sink >= 0) {
        key = ps[e] < n_sink ? 0x7FFFFFFFu : (uint32_t)ps[e];
      } else {
        const int delta = min(max(t - tau[e], 0), d.tab_last);
        const float tmp = __fmul_rn(decay_of(d, delta, s_tab, s_tab_n), crf[e]);
        // a score may be any pattern, a NaN of all ones among them: an entry must not look like none
        key = tmp < FLT_MIN ? 0u : min(__float_as_uint(tmp), 0xFFFFFFFEu);
      }
      b[4 * c + e] = e0 + e < n ? key : 0xFFFFFFFFu;
      np[4 * c + e] = ~(uint32_t)ps[e];
    }
    if (R > 16 && (c & 1)) __builtin_amdgcn_sched_barrier(0);          // two groups' state in flight: the keys need the registers
  }
  if (n - B == 1) {
    u64 best = ~0ull;
    int best_i = -1;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const u64 key = ((u64)b[i] << 32) | np[i];
      if (b[i] != 0xFFFFFFFFu && key < best) {
        best = key;
        best_i = 4 * (tid + (i >> 2) * NT) + (i & 3);
      }
    }
    int phase = 0;
    const u64 gbest = block_min_u64<NT>(best, rb, phase, tid);
    if (best == gbest && best_i >= 0) sh[0] = best_i;     // keys are unique: one writer
    __syncthreads();
    const int e = sh[0];
    if (tid < 64) {
      if (e != n - 1)
        move_entry(d, base, n - 1, e, tid);
      else if (tid == 0)
        d.flags[base + e] = FLAG_SLIP;
    }
    if (tid == 0) {
      d.n[u] = B;
      d.nev[u] = 1;
      *move_count(d, u) = 0;
    }
    return;
  }
  const int h = evict_lists<R, NT>(d, u, base, n, B, b, np, move_list(d, u), evm, cb, tid);
  if (moves_follow) {
    if (tid == 0) *move_count(d, u) = h;
    return;
  }
  __syncthreads();                                         // the lists are there (and visible inside the workgroup)
  for (int r0 = 4 * (tid >> 6); r0 < h; r0 += 4 * (NT / 64)) move_entries4(d, base, move_list(d, u), d.cap, r0, min(4, h - r0), tid & 63);
}

// after_step: behind a decode step that has evicted single entries itself and left the rest (units that it dealt with keep
// their record).  moves_follow = 0: evict_move_kernel does not run, and a unit moves its survivors here.
// RMAX: entries per thread of the longest unit that the capacity allows.  The widest branch decides the registers of the
// whole kernel, and with them how many short units are on the chip side by side (256 threads, window policy, two evicted each, with 32 / as
// chosen: 4096 units of 1000 entries 75.5 / 58.7 us, 8192 of 500 101 / 66).
// Units take 4, 8, 12, 16, 24 or 32, the least that hold them: what bounds a round is its sixteen wavefronts' issue on one compute unit
// (64 units of 9350 entries, ten per thread, 23.3 us with 16, 21.7 with 12; 512 units of 9351, window policy, one evicted each, 14.8 / 13.4).
template <int NT, int RMAX>
__global__ __launch_bounds__(NT) void evict_kernel(Dev d, int unit_begin, int n_sink, int after_step, int moves_follow) {
  __shared__ uint32_t evm[NT];
  __shared__ int32_t s_row[kMaxChunks];
  __shared__ float s_tab[kTabLds];
  __shared__ CutBuf cb;
  __shared__ RedBuf<NT> rb;
  __shared__ int sh[1];
  const int tid = threadIdx.x;
  const int u = unit_begin + blockIdx.x;
  const int n = d.n[u], B = d.budget[u];
  if (n <= B) {
    if (tid == 0) {
      if (!after_step) d.nev[u] = 0;
      *move_count(d, u) = 0;
    }
    return;
  }
  const int s_tab_n = min(kTabLds, d.tab_last + 1);
  for (int i = tid; i < s_tab_n; i += NT) s_tab[i] = d.tab[i];
  if (tid < d.max_seg) s_row[tid] = d.tbl[(size_t)u * d.max_seg + tid];
  __syncthreads();
  const Slots base{s_row};
  auto unit = [&](auto r) {
    evict_unit<decltype(r)::value, NT>(d, u, base, n, B, n_sink, moves_follow, s_tab, s_tab_n, evm, cb, rb, sh, tid);
  };
  if constexpr (RMAX > 16) {
    if (n > 24 * NT) return unit(std::integral_constant<int, 32>{});
    if (n > 16 * NT) return unit(std::integral_constant<int, 24>{});
  }
  if constexpr (RMAX > 8) {
    if (n > 12 * NT) return unit(std::integral_constant<int, 16>{});
    if (n > 8 * NT) return unit(std::integral_constant<int, 12>{});
  }
  if constexpr (RMAX > 4)
    if (n > 4 * NT) return unit(std::integral_constant<int, 8>{});
  unit(std::integral_constant<int, 4>{});
}

// ------------------------------------------------------------------ probe
// Sec. 3 needs the probe query's weights only: a pass over the keys (values are never read), then one workgroup per
// unit for the classes.  Before, the probe ran the decode path's scan (keys and values, behind a kernel that built its work list)
// and found the two class boundaries with 126 one-bit rounds over weights in LDS and positions in memory: 5 + 29 +
// 390 us for a layer of 128 units of 2048 entries on average (up to 8192); now 16.5 + 14.4 us.
//
// probe_scan_kernel: one wavefront per 128 entries, whose four blocks of keys are requested at once (the pass is a
// single round trip to memory per wavefront: a layer is too little work for a pipeline to fill).  Leaves the scaled
// logits where the decode path does, and per span and head the softmax maximum and sum in the partials' place.
// grid: (units of the layer, ceil(spans / 4)), kThreads threads.
constexpr int kProbeBlks = 4, kProbeSpan = kProbeBlks * kBlk;
__device__ __forceinline__ float* probe_stats(const Dev& d, int u) { return d.partial + (size_t)u * d.slots * d.G * kDim; }

__global__ __launch_bounds__(kThreads, 2) void probe_scan_kernel(Dev d, int unit_begin, const uint16_t* __restrict__ q) {
  __shared__ float s_lg[kThreads / 64][kMaxGroup * kLgRow];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int urel = blockIdx.x, u = unit_begin + urel;
  const int span = blockIdx.y * (kThreads / 64) + w, e0 = span * kProbeSpan;
  const int seg = d.tbl[(size_t)u * d.max_seg + min(e0 / kSeg, d.max_seg - 1)];
  const int nv = d.n[u] - e0;
  if (nv <= 0) return;
  const int G = d.G, j = lane & 15, kg = lane >> 4;
  const int nb = min(kProbeBlks, (nv + kBlk - 1) / kBlk);
  const uint16_t* kb = d.K + (size_t)seg * kSegElems + (size_t)((e0 % kSeg) / kBlk) * kBlkElems + lane * 8;
  KFrag k[kProbeBlks];
#pragma unroll
  for (int b = 0; b < kProbeBlks; ++b) load_k(k[b], kb + (size_t)min(b, nb - 1) * kBlkElems);
  bf16x8 qv[4];
  const uint16_t* qrow = q + ((size_t)urel * G + (j < G ? j : 0)) * kDim + 8 * kg;     // columns beyond the group: never looked at
#pragma unroll
  for (int s = 0; s < 4; ++s) qv[s] = as_bf16x8(*reinterpret_cast<const u32x4*>(qrow + 32 * s));
  float* lg_dst = d.logits + ((size_t)u * d.cap + (size_t)e0) * G + 4 * min(lane, 8 * G - 1);
  float m = -INFINITY, l = 0.f;
#pragma unroll
  for (int b = 0; b < kProbeBlks; ++b) {
    if (b < nb) {
      float sv[8];
      scan_qk(k[b], qv, sv, d.scale_log2e, b * kBlk, nv, s_lg[w], kLgRow, LogitsOut{lg_dst}, G, lane);
      const float bm = fmaxf(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])), fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
      if (bm > m) {
        l *= fast_exp2(m - bm);
        m = bm;
      }
      if (m > -INFINITY) {
#pragma unroll
        for (int i = 0; i < 8; ++i) l += fast_exp2(sv[i] - m);
      }
    }
  }
  // the column's four lanes (kg = 0..3), in a fixed order
  float M = fmaxf(m, __shfl_xor(m, 16));
  M = fmaxf(M, __shfl_xor(M, 32));
  const float mine = m > -INFINITY ? l * fast_exp2(m - M) : 0.f;
  const float l0 = __shfl(mine, j), l1 = __shfl(mine, j + 16), l2 = __shfl(mine, j + 32), l3 = __shfl(mine, j + 48);
  if (kg == 0 && j < G) *reinterpret_cast<float2*>(probe_stats(d, u) + ((size_t)span * G + j) * 2) = make_float2(M, (l0 + l1) + (l2 + l3));
}

// Classes of the entries of a unit of n <= R NT entries.  Both boundaries come from the eviction's selection
// (ascending keys: lower weight first, then higher position).
template <int R, int NT>
__device__ __forceinline__ void probe_unit(const Dev& d, int u, Slots base, int n, const float* sM, const float* sInv, uint8_t* cls, CutBuf& cb,
                                           int tid) {
  uint32_t b[R], np[R];
  {
    float a[R];
    mean_weights_regs<R, NT>(d, unit_logits(d, u), n, sM, sInv, a, tid);
#pragma unroll
    for (int c = 0; c < R / 4; ++c) {
      const int e0 = 4 * (tid + c * NT);
      const i32x4 ps = *reinterpret_cast<const i32x4*>(d.pos + (base + min(e0, (n - 1) & ~3)));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        b[4 * c + e] = e0 + e < n ? __float_as_uint(a[4 * c + e]) : 0xFFFFFFFFu;
        np[4 * c + e] = ~(uint32_t)ps[e];
      }
    }
  }
  const int kq = (3 * n) / 10;
  KeyCut slip{0u, 0u}, rest{0u, 0u};
  if (kq > 0) {
    slip = select_low_keys<R, NT>(b, np, kq, cb, tid);
    __syncthreads();                                       // the first selection's buffers are free
    rest = select_low_keys<R, NT>(b, np, n - kq, cb, tid);
  }
#pragma unroll
  for (int c = 0; c < R / 4; ++c) {
    const int e0 = 4 * (tid + c * NT);
    uint32_t packed = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t bb = b[4 * c + e], pp = np[4 * c + e];
      const uint32_t k = kq == 0 ? 1u : slip(bb, pp) ? 0u : rest(bb, pp) ? 1u : 2u;
      packed |= k << (8 * e);
    }
    if (e0 + 3 < n && (reinterpret_cast<uintptr_t>(cls) & 3) == 0) {
      *reinterpret_cast<uint32_t*>(cls + e0) = packed;
    } else {
      for (int e = 0; e < 4 && e0 + e < n; ++e) cls[e0 + e] = (uint8_t)(packed >> (8 * e));
    }
  }
}

template <int NT>
__global__ __launch_bounds__(NT) void probe_kernel(Dev d, int unit_begin, uint8_t* classes) {
  __shared__ float sM[kMaxGroup], sInv[kMaxGroup];
  __shared__ int32_t s_row[kMaxChunks];
  __shared__ CutBuf cb;
  const int tid = threadIdx.x, lane = tid & 63;
  const int urel = blockIdx.x, u = unit_begin + urel;
  const int n = d.n[u];
  if (n <= 0) return;
  if (tid < d.max_seg) s_row[tid] = d.tbl[(size_t)u * d.max_seg + tid];
  // softmax maximum and 1 / sum of every head over the unit's spans: a wavefront per head
  const int G = d.G, spans = (n + kProbeSpan - 1) / kProbeSpan;
  for (int g = tid >> 6; g < G; g += NT / 64) {
    const float* st = probe_stats(d, u) + 2 * g;
    float M = -INFINITY, L = 0.f;
    for (int s = lane; s < spans; s += 64) M = fmaxf(M, st[(size_t)s * G * 2]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o));
    for (int s = lane; s < spans; s += 64) L += st[(size_t)s * G * 2 + 1] * fast_exp2(st[(size_t)s * G * 2] - M);
    L = wave_sum_f32(L);
    if (lane == 0) {
      sM[g] = M;
      sInv[g] = 1.0f / L;
    }
  }
  __syncthreads();
  const Slots base{s_row};
  uint8_t* cls = classes + (size_t)urel * d.cap;
  if (n <= 4 * NT)
    probe_unit<4, NT>(d, u, base, n, sM, sInv, cls, cb, tid);
  else if (n <= 8 * NT)
    probe_unit<8, NT>(d, u, base, n, sM, sInv, cls, cb, tid);
  else if (n <= 16 * NT)
    probe_unit<16, NT>(d, u, base, n, sM, sInv, cls, cb, tid);
  else
    probe_unit<32, NT>(d, u, base, n, sM, sInv, cls, cb, tid);
}

// ------------------------------------------------------------------ Alg. 2
// Integers val[k] in [lo, hi] summing to `total`, proportional to x[k] >= 0 as
// far as the bounds allow: water-filling on the reals, floor, remainder by
// largest fractional part (lower index first on ties), final spill in index order.
__device__ __forceinline__ void apportion(const double* x, int m, long long total, long long lo, long long hi, long long* val, double* y,
                          unsigned char* fixed) {
  for (int k = 0; k < m; ++k) {
    fixed[k] = 0;
    val[k] = 0;
    y[k] = 0.0;
  }
  for (int iter = 0; iter < m + 1; ++iter) {
    long long R = total;
    int n_free = 0;
    double X = 0.0;
    for (int k = 0; k < m; ++k) {
      if (fixed[k]) R -= val[k];
      else {
        ++n_free;
        X += x[k];
      }
    }
    if (n_free == 0) break;
    double over = 0.0, under = 0.0;
    for (int k = 0; k < m; ++k) {
      if (fixed[k]) continue;
      y[k] = (X > 0.0) ? (double)R * (x[k] / X) : (double)R / (double)n_free;
      if (y[k] > (double)hi) over += y[k] - (double)hi;
      if (y[k] < (double)lo) under += (double)lo - y[k];
    }
    if (over == 0.0 && under == 0.0) break;
    if (over >= under) {
      for (int k = 0; k < m; ++k)
        if (!fixed[k] && y[k] > (double)hi) {
          fixed[k] = 1;
          val[k] = hi;
        }
    } else {
      for (int k = 0; k < m; ++k)
        if (!fixed[k] && y[k] < (double)lo) {
          fixed[k] = 1;
          val[k] = lo;
        }
    }
  }
  long long sum = 0;
  for (int k = 0; k < m; ++k) {
    if (!fixed[k]) {
      const double f = floor(y[k]);
      long long fi = (long long)f;
      fi = fi < lo ? lo : (fi > hi ? hi : fi);
      val[k] = fi;
      y[k] = y[k] - f;         // fractional part
    }
    sum += val[k];
  }
  long long rem = total - sum;
  // fixed[k]: 0 = free and not yet visited, 1 = fixed at a bound, 2 = free and visited
  while (rem > 0) {
    int best = -1;
    for (int k = 0; k < m; ++k)
      if (fixed[k] == 0 && (best < 0 || y[k] > y[best])) best = k;
    if (best < 0) break;
    fixed[best] = 2;
    if (val[best] < hi) {
      val[best] += 1;
      rem -= 1;
    }
  }
  while (rem < 0) {
    int best = -1;
    for (int k = 0; k < m; ++k)
      if (fixed[k] == 0 && (best < 0 || y[k] <= y[best])) best = k;
    if (best < 0) break;
    fixed[best] = 2;
    if (val[best] > lo) {
      val[best] -= 1;
      rem += 1;
    }
  }
  while (rem != 0) {
    bool moved = false;
    for (int k = 0; k < m; ++k) {
      if (rem > 0 && val[k] < hi) {
        val[k] += 1;
        rem -= 1;
        moved = true;
      } else if (rem < 0 && val[k] > lo) {
        val[k] -= 1;
        rem += 1;
        moved = true;
      }
      if (rem == 0) break;
    }
    if (!moved) break;
  }
}

constexpr int kMaxLayers = 256;
constexpr int kMaxKvHeads = 32;

// One workgroup per sequence.  in_lds: there are 25 bytes of dynamic LDS per (layer, head) for the second level; else
// its arrays are the threads' own, in scratch memory, where every indexed access is a trip to memory: 28 us for 4
// layers of 4 heads, 16 in LDS; 60 us for 16 layers of 8, 35 in LDS).
__global__ __launch_bounds__(kThreads) void rebudget_kernel(Dev d, int in_lds) {
  extern __shared__ unsigned char smem[];
  __shared__ double eta_l[kMaxLayers], y_l[kMaxLayers];
  __shared__ long long tot_l[kMaxLayers];
  __shared__ unsigned char fx_l[kMaxLayers];
  __shared__ int ok;
  const int tid = threadIdx.x, b = blockIdx.x;
  const int L = d.L, H = d.Hkv;
  const int steps = d.sc[SC_WINDOW_STEPS];
  if (steps > 0) {
    const double denom = 1048576.0 * (double)steps;
    if (tid < L) {
      double sc = 0.0, sb = 0.0;
      for (int j = 0; j < H; ++j) {
        const int u = (tid * d.Bz + b) * H + j;
        sc += (double)d.window[u] / denom;
        sb += (double)d.budget[u];
      }
      eta_l[tid] = sc / sb;
    }
    __syncthreads();
    if (tid == 0) {
      double sum_eta = 0.0;
      for (int i = 0; i < L; ++i) sum_eta += eta_l[i];
      if (!(sum_eta > 0.0) || !isfinite(sum_eta)) {
        ok = 0;
      } else {
        apportion(eta_l, L, d.btotal[b], (long long)H * d.bmin, (long long)H * d.bmax, tot_l, y_l, fx_l);
        ok = 1;
      }
    }
    __syncthreads();
    auto second_level = [&](double* eta_h, double* y_h, long long* val_h, unsigned char* fx_h) {
      for (int j = 0; j < H; ++j) {
        const int u = (tid * d.Bz + b) * H + j;
        eta_h[j] = ((double)d.window[u] / denom) / (double)d.budget[u];
      }
      apportion(eta_h, H, tot_l[tid], d.bmin, d.bmax, val_h, y_h, fx_h);
      for (int j = 0; j < H; ++j) d.budget[(tid * d.Bz + b) * H + j] = (int32_t)val_h[j];
    };
    if (ok && tid < L) {
      if (in_lds) {
        double* eta = reinterpret_cast<double*>(smem);
        double* y = eta + L * H;
        long long* val = reinterpret_cast<long long*>(y + L * H);
        second_level(eta + tid * H, y + tid * H, val + tid * H, reinterpret_cast<unsigned char*>(val + L * H) + tid * H);
      } else {
        double eta_h[kMaxKvHeads], y_h[kMaxKvHeads];
        long long val_h[kMaxKvHeads];
        unsigned char fx_h[kMaxKvHeads];
        second_level(eta_h, y_h, val_h, fx_h);
      }
    }
    __syncthreads();
    for (int i = tid; i < L * H; i += kThreads) d.window[((i / H) * d.Bz + b) * H + (i % H)] = 0ull;
  }
  __syncthreads();
  if (tid == 0) {
    __threadfence();
    const int prev = atomicAdd(&d.sc[SC_DONE_RB], 1);
    if (prev == (int)gridDim.x - 1) {
      d.sc[SC_DONE_RB] = 0;
      d.sc[SC_WINDOW_STEPS] = 0;
    }
  }
}

}  // namespace ckv
