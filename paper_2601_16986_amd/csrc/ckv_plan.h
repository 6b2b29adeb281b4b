// Choices that kernels and host make by sizes alone.  Plain C++, no HIP, so that a host program can include it.
#pragma once
#include "ckv_layout.h"

#if defined(__HIPCC__)
#define CKV_PLAN __host__ __device__ constexpr
#else
#define CKV_PLAN constexpr
#endif

namespace ckv {

// Bookkeeping of a unit from its logits (finish_unit): a thread owns `groups` groups of four entries and asks for the logits of so
// many of them at a time, a number that divides them.  Two, as registers allow: 1024 threads have 128 each, and so have the 512 of a
// workgroup that shares its compute unit with another (`lean`).
CKV_PLAN int logit_groups(int groups, int threads, bool lean) {
  if (groups % 2 != 0 || (lean && (groups > 2 || threads < 1024))) return 1;
  return 2;
}

// A step of few units: a block of 32 entries per wavefront while two workgroups per compute unit cover the entries that the budgets (`mean`
// each, on average) allow, else eight (figures at layer_step_kernel).
CKV_PLAN bool one_block_each(long long mean, int count, int n_cu) { return mean * count <= 2ll * n_cu * kChunk; }
// Its workgroups per unit, by the capacity: most of them have nothing to do where the budgets stay far below it.
CKV_PLAN int step_pieces(int cap, bool one_block) {
  const int piece = kChunk * (one_block ? 1 : kChunkBlocks);
  return (cap + piece - 1) / piece;
}

// Workgroups of a step that run about at once: with a block per wavefront two fit on a compute unit, but only one each is as good as alone.
CKV_PLAN long long at_once(bool one_block, int n_cu) { return (one_block ? 1ll : 2ll) * n_cu; }
// Whether the workgroups look at their unit's counter of arrivals before they publish their own part: only if none has to wait for its place
// (figures at layer_step_kernel; eight blocks each, attention only, with the look / without: 64 units of 2000 entries, 256 workgroups, 26.8 / 28.7 us,
// 200 of 600, 400 workgroups, 17.7 / 18.8; a block per wavefront, 128 units of 100 at capacity 448, 256 workgroups, 7.7 / 9.1).
CKV_PLAN bool looks_early(long long workgroups, bool one_block, int n_cu) { return workgroups <= at_once(one_block, n_cu); }

// An attention-only step leaves its records to a launch of their own (append_kernel) where the capacity makes many more workgroups than the
// budgets have work for. In one launch these must arrive at their unit's counter like the others before its length may change, and queue for their
// places to do so; a second launch costs 1.2 us, 3 where the host waits for it. Us per layer, captured, one launch / two:
//  - a block per wavefront, units of one workgroup (its busy one often ends behind the idle ones): 128 of 100 entries at capacity 448, 128 idle, 7.7 / 8.7,
//    200 of 150 at 512, 200 idle, 11.1 / 10.1, 400 of 100 at 448, 400 idle, 16.3 / 12.6;
//  - longer units: 128 of 600 at 1408, 384 idle, 13.9 / 15.9, 104 of 1000 at 2240, 416 idle, 16.0 / 17.2, 32 of 1000 at 4096, 384 idle, 12.4 / 12.9; but
//    16 of 2000 at 8192, 352 idle, 13.6 / 12.8, 32 of 200 at 4096, 416 idle, 10.7 / 8.4, 8 of 1000 at 32768, 976 idle, 18.5 / 11.9, 64 of 200, 8000 idle, 45 / 12.4;
//  - eight blocks: 64 of 5000 at 10240, 128 idle, 34.8 / 36.0, 200 of 2500 at 5248, 200 idle, 53.3 / 55.1, 256 of 1000 at 2240, 256 idle, 30.2 / 28.8,
//    256 of 200 at 4096, 256 idle, 17.8 / 15.0, 400 of 1000 at 32768, 6000 idle, 67 / 46;
//  - short units of one workgroup of eight blocks, more of them than compute units, none idle: the busy ones share a compute unit, and the records keep
//    registers from the next: 400 of 300 at 416 25.8 / 23.4, 400 of 600 at 704 31.8 / 31.3, 256 of 600 20.1 / 19.9.
CKV_PLAN bool attends_apart(long long mean, int count, int cap, int n_cu) {
  const bool one_block = one_block_each(mean, count, n_cu);
  const int piece = kChunk * (one_block ? 1 : kChunkBlocks);
  if (!one_block && count > n_cu && cap <= piece && mean <= 3 * kChunk) return true;
  const long long idle = (step_pieces(cap, one_block) - (mean + piece - 1) / piece) * count;
  return 4 * idle >= (!one_block ? 4 : mean <= kChunk ? 3 : 6) * n_cu;
}

// A whole step leaves its bookkeeping to a kernel of its own (finish_kernel):
//  - where units may be longer than `most` entries, what the workgroup that finishes a unit has registers for. 1024 threads per unit are
//    also the faster way then (us per layer, captured, one kernel / two: 64 units of 2048 entries, up to 8192, 51 / 44, 16 of 8000, up to 32000, 104 / 76);
//  - where workgroups without work, which must arrive in one kernel and pass through in rounds of two per compute unit at 1.3 us each, cost more
//    than the second kernel does. That is 3 us where units have one workgroup each, 7 where more of them meet (capacity 6144: 64 units of 200 19.5 / 18.5,
//    256 of 200 34.4 / 27.0, under the attention-weighted reward 31.3 / 23.6 and at capacity 2048 21.0 / 17.3; but 56 of 200 17.7 / 18.6, 128 of 700
//    27.4 / 28.6, 104 of 1200 30.6 / 32.4);
//  - where few long units leave compute units idle, which 1024 threads per unit then use better than 512 (48 .. 85 units of at least six entries per
//    thread on average: 64 of 3700 47.5 / 45.4, 72 of 3700 49.8 / 46.8, weighted 45.9 / 43.4, 56 of 5900 56.9 / 53.9; but 32 of 5900 45.6 / 47.9, 104 of
//    5900 91.0 / 96.4, 72 of 2000 34.8 / 39.7).
CKV_PLAN bool books_apart(long long mean, int count, int cap, int n_cu, int threads, int most) {
  if (cap > most) return true;
  if (!one_block_each(mean, count, n_cu)) return mean >= 6 * threads && 16 * count >= 3 * n_cu && 3 * count <= n_cu;
  const long long idle = (long long)count * step_pieces(cap, true) - count * (mean / kChunk + 1);
  return idle > (mean <= kChunk ? 5 : 11) * n_cu;
}

// Loading a layer stores its values past the caches where keys and values together fill the last cache (256 MiB): they would push out keys
// that a replay of the prompt reads next. Of a smaller layer the next step, or the moves of an eviction, still find the values there. Whole admissions (per
// layer load, replay of 16 queries, eviction to a quarter, then a step; 3 .. 8 layers, us, values kept / past the caches): 8 units of 9350 entries 821 / 838,
// 32 of 3000 732 / 759, 128 of 2048 (134 MB a layer) 1389 / 1407, 32 of 9350 (153) 1630 / 1650, 40 of 9350 (191) 1852 / 1850, 48 of 9350 (230) 2185 / 2183, 64 of
// 9350 (306) 2723 / 2663, 512 of 1024 (268) 2621 / 2575, 128 of 9350 (612) 5112 / 5008; a load and a step behind it, 4 units of 777 25.6 / 26.5, 32 of 777 30.8 / 31.9.
// (`entries`: units times the longest's length, which is all that the host knows of a ragged load.)
CKV_PLAN bool loads_past_caches(long long entries) { return entries * kDim * 4 >= (256ll << 20); }

}  // namespace ckv
