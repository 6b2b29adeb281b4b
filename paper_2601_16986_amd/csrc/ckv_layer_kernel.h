// A step of few units (one layer, or a small context) in one kernel: append, attention and output with several workgroups per
// unit, then, by the workgroup that finishes the unit, the bookkeeping (Alg. 1 Steps 1-4).
//
// The shape a model imposes is one call per layer, a few hundred units at most: too few for the fused kernel (a workgroup per
// unit).  The grid itself is the work list: workgroup (x, y) of eight wavefronts takes the y-th 256 or 2048 entries of the
// call's unit x, a wavefront one block of 32 or eight, and has nothing to stream if the unit is shorter.  (Units along x:
// consecutive workgroups go to different XCDs, so the workgroups that have work - every unit's first, most units' second -
// spread over all of them; with the pieces of a unit along x, and eight or a multiple of them, each XCD would get one index, the first few all the
// work, and a step takes 1.6 times as long.)  Nothing has to run before it: every workgroup derives the unit's length
// after the append from the stored one, and the wavefront whose span receives the new entry puts its key and
// value rows into the block it has just loaded, so that the entry takes part like any cached one.
//
// The wavefronts combine their softmax states in LDS, a unit's workgroups through one partial each (coherent stores and
// loads): the last of them to arrive at the unit's counter merges the partials in index order, writes the output and, in a
// whole step, goes on with the bookkeeping from the unit's logits, which therefore went to memory the coherent way.  It
// changes the unit's length, so every workgroup of the unit arrives, those without work too (unless what follows has another
// launch, see books_apart and attends_apart): none can start late and take the new length for the old one.  A workgroup that finds all others arrived before it publishes
// its own partial keeps it in registers, if it looks at all: where the whole work list runs at once, a workgroup per compute unit,
// that saves a unit's last workgroup a round trip (2 units of 200 entries, attention only, 7.3 against 8.2 us per layer, 8 units of 700, whole
// step, 16.3 / 18.3); with more of them the looks, past every cache at words that the others are counting on, hold everybody up (16 units
// of 5000 entries, scan alone, 23.4 / 18.4 us, 32 of 3700, deferred, 29.7 / 22.5, 56 of 2000, whole step, 38.2 / 28.9).
//
// Two shapes, <true, .> a block per wavefront, a single round trip to memory, two workgroups per compute unit, while the entries that the
// budgets allow are no more than those hold (us per layer, scan alone, one block / eight: 8 units of 2048 entries 10 / 23, 32 units
// 17 / 25, 64 units of 1024 12 / 15, 64 units of 2048 25 / 28, 128 units of 2048 41 / 34, 256 units of 1024 32 / 28); <false, .>
// eight blocks, streamed one ahead (four 44, five 46, six 47, seven 38 for 128 units of 2048 on average, where eight take 36: the workgroups of a unit
// meet on one XCD, and more of them than it has compute units take a second round).
//
// What bounds a whole step of few units is the chain behind the scan: a unit of 129 entries takes 2.5 us to its last block, 1.5 to
// its output's inputs, 1 for the output, 0.8 for the mean weights, 2 for the threshold, 0.8 for the scores, 1 for the eviction; a second
// kernel for the bookkeeping added its start, the logits' way and the wait between the two.  Us per layer, captured, in two
// kernels / in one: 2 units of 128 entries 15.3 / 11.0, 2 of 1000 19.1 / 13.7, 32 of 300 19.9 / 14.8, 64 of 1024 28.5 / 20.9, 128 of
// 1000 (250 .. 4000) 41 / 37, 128 of 2048 53 / 48, 256 of 1024 47 / 38.
#pragma once
#include "ckv_kernels.h"

namespace ckv {

// What a launch does: a whole step; attention alone and the append's records; or either without what follows in another launch
// (kScanOnly: the bookkeeping, in finish_kernel; kAttendOnly: the records, in append_kernel).
enum { kAttend = 0, kWholeStep = 1, kScanOnly = 2, kAttendOnly = 3 };
constexpr int kLayerWaves = 8, kLayerThreads = 64 * kLayerWaves;
static_assert(kLayerWaves * kBlk == kChunk, "a workgroup's pieces as step_pieces counts them");

struct LayerCall {
  const uint16_t* q;
  const uint16_t* k_new;
  const uint16_t* v_new;
  void* out;
  int unit_begin;
  uint32_t flags;        // the step's call flags (bookkeeping)
  int mode;
  int layer, layers;     // kScanOnly: the first layer, and how many
  int advance;           // the time moves on with this launch
  int early;             // a workgroup looks at its unit's counter before it publishes (looks_early)
};

// Entry rr of the block in (ka, va) is replaced by the rows in `rows` (LDS: 128 bf16 of the key, then 128 of the
// value), piece by piece, so that few registers are live at a time.
__device__ __forceinline__ void inject_entry(KFrag& ka, VFrag& va, int rr, const uint16_t* rows, int lane) {
  const int j = lane & 15, kg = lane >> 4;
  const int tt = rr >> 4;
  const bool krow = j == (rr & 15);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const u32x4 kn = *reinterpret_cast<const u32x4*>(rows + 32 * s + 8 * kg);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (krow && h == tt) ka.k[h * 4 + s] = kn;
  }
  const bool vrow = kg == ((rr & 15) >> 2);
  const int e = tt * 4 + (rr & 3);
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) {
    const uint32_t vn = rows[kDim + 16 * dt + j];
#pragma unroll
    for (int wi = 0; wi < 4; ++wi) {
      const uint32_t old = va.v[dt][wi];
      const uint32_t nw = (e & 1) ? ((old & 0x0000FFFFu) | (vn << 16)) : ((old & 0xFFFF0000u) | vn);
      va.v[dt][wi] = (vrow && wi == (e >> 1)) ? nw : old;
    }
  }
}

// The span's logits on their way to memory: the coherent way if the bookkeeping reads them within this launch.
struct LayerLogits {
  Buffer unit;
  int at;
  int mode;
  __device__ __forceinline__ explicit operator bool() const { return mode == kWholeStep || mode == kScanOnly; }
  __device__ __forceinline__ void operator()(int first, f32x4 row) const {
    if (mode == kWholeStep)
      put_coherent16(unit, at + first, row);
    else
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, row), unit, (at + first) * 4, 0, 0);
  }
};

// LDS of the scan: the wavefronts' accumulators, staging tiles of their logits, the new entry's rows.  The bookkeeping's
// values (4 bytes per entry of cap, and a bit) take its place.
constexpr int kLayerScanLds = kLayerWaves * (kMaxGroup * kDim * 4 + kMaxGroup * kLgRow * 4 + 2 * kDim * 2);

// kOne: a block per wavefront (span = 1), requested at once, and registers for two workgroups per compute unit; else the span's
// blocks stream one ahead.  RMAX: entries per thread that the bookkeeping may have to hold, by the capacity (0: no
// bookkeeping here).
// grid: (units of the call, workgroups per unit by the capacity), kLayerThreads threads.
template <bool kOne, int RMAX>
__global__ __launch_bounds__(kLayerThreads, kOne ? 4 : 2) void layer_step_kernel(Dev d, LayerCall call) {
  constexpr int NT = kLayerThreads;
  extern __shared__ __align__(16) unsigned char smem[];
  float(*s_acc)[kMaxGroup * kDim] = reinterpret_cast<float(*)[kMaxGroup * kDim]>(smem);
  float(*s_lg)[kMaxGroup * kLgRow] = reinterpret_cast<float(*)[kMaxGroup * kLgRow]>(s_acc + kLayerWaves);
  uint16_t(*s_new)[2 * kDim] = reinterpret_cast<uint16_t(*)[2 * kDim]>(s_lg + kLayerWaves);
  float* val = reinterpret_cast<float*>(smem);
  uint32_t* evm = reinterpret_cast<uint32_t*>(smem + (size_t)d.cap * 4);
  __shared__ TopBuf top[1];
  __shared__ float s_m[kLayerWaves][kMaxGroup], s_l[kLayerWaves][kMaxGroup];
  __shared__ float sM[kMaxGroup], sInv[kMaxGroup];
  __shared__ int32_t s_row[kMaxChunks];
  __shared__ RedBuf<NT> rb;
  __shared__ int sh[4 + NT / 64];
  __shared__ float s_tab[kTabLds];
  __shared__ int s_seen, s_last;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int urel = blockIdx.x, u = call.unit_begin + urel, cg = blockIdx.y;
  const int G = d.G, mode = RMAX > 0 ? (int)kWholeStep : call.mode;
  constexpr int span = kOne ? 1 : kChunkBlocks;            // blocks per wavefront, all in one segment
  const int n_old = d.n[u];
  // where this wavefront's blocks lie (asked for beside the length: neither waits for the other)
  const int b0 = (cg * kLayerWaves + w) * span;
  const int32_t* row = d.tbl + (size_t)u * d.max_seg;
  const int seg = row[min(b0 / kSegBlocks, d.max_seg - 1)];
  const bool full = n_old >= unit_cap(d, u);
  const int n = n_old + (full ? 0 : 1);
  const int nblk = (n + kBlk - 1) / kBlk;
  const int nwg = (nblk + kLayerWaves * span - 1) / (kLayerWaves * span);
  const bool apart = mode == kScanOnly || mode == kAttendOnly;      // nothing in this launch changes a unit's length
  const int arrivals = apart ? nwg : (int)gridDim.y;
  if (cg == 0) {
    // the bookkeeping in another launch finds the step's time at its layer; nothing else in this launch reads the time
    if (urel == 0 && mode == kScanOnly) {
      const int t = d.sc[SC_T];
      if (tid < call.layers) d.layer_ts[call.layer + tid] = t;
      __syncthreads();
      if (call.advance && tid == 0) {
        d.sc[SC_T] = t + 1;
        d.sc[SC_WINDOW_STEPS] = d.sc[SC_WINDOW_STEPS] + 1;
      }
    }
    if (full && tid == 0) atomicOr(&d.sc[SC_STATUS], 1);
  }
  const bool active = cg < nwg;
  if (!active && apart) return;
  // what the finishing workgroup needs of the unit and of the decay table
  const int s_tab_n = min(kTabLds, d.tab_last + 1);
  if (!apart) {
    if (tid < d.max_seg) s_row[tid] = row[tid];
    if (tid < s_tab_n) s_tab[tid] = d.tab[tid];
    if (mode == kWholeStep) clear_top(*top, tid, NT);
  }
  const int j = lane & 15, kg = lane >> 4;
  const bool head_lane = j < G;
  int seen = 0;                        // workgroups of the unit that have arrived so far
  float Mg = -INFINITY, Lg = 0.f;      // this workgroup's state of head w: maximum, sum,
  float o0 = 0.f, o1 = 0.f;            // and the accumulated dims 2 lane, 2 lane + 1
  if (active) {
    f32x4 acc[8];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;
    if (b0 < nblk) {
      const int e0 = b0 * kBlk;
      const int nb = min(span, nblk - b0), nv = min(n - e0, span * kBlk);
      const bool inject = !full && n_old >= e0 && n_old < e0 + span * kBlk;      // the new entry is then the span's last
      auto off = [&](int blk) -> size_t { return (size_t)seg * kSegElems + (size_t)((b0 + blk) & (kSegBlocks - 1)) * kBlkElems + lane * 8; };
      KFrag ka;
      VFrag va;
      load_k(ka, d.K + off(0));
      load_v(va, d.V + off(0));
      bf16x8 qv[4];
      {
        const uint16_t* qrow = call.q + ((size_t)urel * G + (head_lane ? j : 0)) * kDim + 8 * kg;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          u32x4 x = *reinterpret_cast<const u32x4*>(qrow + 32 * s);
          if (!head_lane) x = u32x4{0u, 0u, 0u, 0u};
          qv[s] = as_bf16x8(x);
        }
      }
      // The new entry's rows wait in LDS for their block's turn (the span's last): held in registers through the
      // loop they would cost the kernel a third wavefront per SIMD.  Where no bookkeeping follows in this launch they also
      // go into the cache here.
      if (inject) {
        if (lane < 32) {
          const int piece = lane & 15;
          const uint16_t* src = (lane < 16 ? call.k_new : call.v_new) + (size_t)urel * kDim + piece * 8;
          const u32x4 x = *reinterpret_cast<const u32x4*>(src);
          *reinterpret_cast<u32x4*>(&s_new[w][(lane < 16 ? 0 : kDim) + piece * 8]) = x;
          if (mode != kWholeStep && lane < 16)
            *reinterpret_cast<u32x4*>(d.K + (size_t)seg * kSegElems + k_offset(n_old & (kSeg - 1), piece * 8)) = x;
        }
        if (mode != kWholeStep) {
          const int at = n_old & (kSeg - 1);
          uint16_t* vdst = d.V + (size_t)seg * kSegElems;
          vdst[v_offset(at, lane)] = call.v_new[(size_t)urel * kDim + lane];
          vdst[v_offset(at, lane + 64)] = call.v_new[(size_t)urel * kDim + lane + 64];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      }
      float* lds_lg = mode == kAttend || mode == kAttendOnly ? nullptr : s_lg[w];
      const LayerLogits lg{buffer_of(d.logits + (size_t)u * d.cap * G, d.cap * G), e0 * G + 4 * lane, mode};
      if constexpr (kOne) {
        if (inject) {
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          inject_entry(ka, va, (n_old - e0) & 31, s_new[w], lane);
        }
        float sv[8];
        scan_qk(ka, qv, sv, d.scale_log2e, 0, nv, lds_lg, kLgRow, lg, G, lane);
        scan_pv(sv, va, acc, m_run, l_run, lane);
      } else {
        // one block ahead (two ahead is slower here as well); the loads stay unconditional (the
        // last block is read twice), so that the waits the compiler inserts are exact
        for (int blk = 0; blk < nb; ++blk) {
          const bool last = blk + 1 == nb;
          const size_t nxt = off(last ? blk : blk + 1);
          if (last && inject) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            inject_entry(ka, va, (n_old - e0) & 31, s_new[w], lane);
          }
          float sv[8];
          scan_qk(ka, qv, sv, d.scale_log2e, blk * kBlk, nv, lds_lg, kLgRow, lg, G, lane);
          load_k(ka, d.K + nxt);
          scan_pv(sv, va, acc, m_run, l_run, lane);
          load_v(va, d.V + nxt);
        }
      }
      l_run += __shfl_xor(l_run, 16);
      l_run += __shfl_xor(l_run, 32);
    }
    if (tid == 0 && arrivals > 1 && call.early) seen = get_coherent(&d.arrive[u]);
    // ---- the workgroup's states into one: wavefront w takes head w
    if (head_lane && kg == 0) {
      s_m[w][j] = m_run;
      s_l[w][j] = l_run;
    }
    if (b0 < nblk) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int head = 4 * kg + v;
        if (head < G) {
#pragma unroll
          for (int dt = 0; dt < 8; ++dt) s_acc[w][head * kDim + 16 * dt + j] = acc[dt][v];
        }
      }
    }
    if (tid == 0) s_seen = seen;
    __syncthreads();
    seen = s_seen;
    if (w < G) {
#pragma unroll
      for (int ww = 0; ww < kLayerWaves; ++ww) Mg = fmaxf(Mg, s_m[ww][w]);
#pragma unroll
      for (int ww = 0; ww < kLayerWaves; ++ww) {
        const float m = s_m[ww][w];
        if (m > -INFINITY) {
          const float wt = fast_exp2(m - Mg);
          const float2 x = *reinterpret_cast<const float2*>(&s_acc[ww][w * kDim + 2 * lane]);
          o0 += x.x * wt;
          o1 += x.y * wt;
          Lg += s_l[ww][w] * wt;
        }
      }
    }
  }
  // ---- one partial per workgroup; the last to arrive goes on
  const size_t slot0 = (size_t)u * d.slots;
  if (arrivals > 1) {
    if (seen != arrivals - 1) {
      if (active && w < G) {
        put_coherent(reinterpret_cast<u64*>(&d.partial[((slot0 + cg) * G + w) * kDim]) + lane, pack_f32(o0, o1));
        if (lane == 0) put_coherent(reinterpret_cast<u64*>(&d.ml[((slot0 + cg) * G + w) * 2]), pack_f32(Mg, Lg));
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // partial and logits before the count (coherent stores: completed is enough)
      __syncthreads();
      if (tid == 0) s_last = atomicAdd(&d.arrive[u], 1) == arrivals - 1;
      __syncthreads();
      if (!s_last) return;
    }
    if (tid == 0) put_coherent(&d.arrive[u], 0);
  }
  if (mode == kWholeStep) {                                   // this workgroup's own logits are there, and s_row and s_tab
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }
  const int t = d.sc[SC_T];
  const int B = d.budget[u];
  // ---- the partials into one: wavefront g combines head g, lane l holds the states of partials l and l + 64, and dims 2 l, 2 l + 1
  // of the output
  constexpr int kRound = kOne && RMAX > 0 ? 8 : 16;     // partials asked for at a time: what the registers hold
  u64 x[kRound], st[2];
  const bool partials = w < G && (nwg > 1 || !active) && nwg > 0;
  auto request = [&](int r0) {
#pragma unroll
    for (int i = 0; i < kRound; ++i)
      x[i] = get_coherent(reinterpret_cast<const u64*>(&d.partial[((slot0 + min(r0 + i, nwg - 1)) * G + w) * kDim]) + lane);
  };
  if (partials) {
#pragma unroll
    for (int k = 0; k < 2; ++k) st[k] = get_coherent(reinterpret_cast<const u64*>(&d.ml[((slot0 + min(lane + 64 * k, nwg - 1)) * G + w) * 2]));
    request(0);
  }
  auto merge = [&]() {
    if (w < G && nwg > 0) {
      float M = Mg, L = Lg;
      if (partials) {
        float m[2], l[2], wt[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int r = lane + 64 * k;
          m[k] = r == cg ? Mg : r < nwg ? low_f32(st[k]) : -INFINITY;       // (cg < nwg or nothing of this workgroup's own)
          l[k] = r == cg ? Lg : high_f32(st[k]);
        }
        M = fmaxf(m[0], m[1]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o));
#pragma unroll
        for (int k = 0; k < 2; ++k) wt[k] = m[k] > -INFINITY ? fast_exp2(m[k] - M) : 0.f;
        L = wave_sum_f32((m[0] > -INFINITY ? l[0] * wt[0] : 0.f) + (m[1] > -INFINITY ? l[1] * wt[1] : 0.f));
        float v0 = 0.f, v1 = 0.f;
        for (int r0 = 0; r0 < nwg; r0 += kRound) {
#pragma unroll
          for (int i = 0; i < kRound; ++i) {
            const int r = r0 + i;
            if (r < nwg) {
              const float wr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r < 64 ? wt[0] : wt[1]), r & 63));
              const bool own = r == cg;
              if (wr != 0.f) {
                v0 += (own ? o0 : low_f32(x[i])) * wr;
                v1 += (own ? o1 : high_f32(x[i])) * wr;
              }
            }
          }
          if (r0 + kRound < nwg) request(r0 + kRound);
        }
        o0 = v0;
        o1 = v1;
      }
      const float inv = 1.0f / L;
      const size_t oi = ((size_t)urel * G + w) * kDim + 2 * lane;
      if (d.out_bf16) {
        reinterpret_cast<__bf16*>(call.out)[oi] = (__bf16)(o0 * inv);
        reinterpret_cast<__bf16*>(call.out)[oi + 1] = (__bf16)(o1 * inv);
      } else {
        reinterpret_cast<float*>(call.out)[oi] = o0 * inv;
        reinterpret_cast<float*>(call.out)[oi + 1] = o1 * inv;
      }
      if (lane == 0) {
        if (mode == kScanOnly) {
          d.msum[((size_t)u * kMaxGroup + w) * 2] = M;
          d.msum[((size_t)u * kMaxGroup + w) * 2 + 1] = inv;
        } else if (mode == kWholeStep) {
          sM[w] = M;
          sInv[w] = inv;
        }
      }
    }
    if (mode == kWholeStep) __syncthreads();                 // the statistics are there, and the scan's LDS is free
  };
  if (apart) {
    merge();
    return;
  }
  const Slots base{s_row};
  const bool room = !full, evict = (call.flags & 1u) != 0;
  // In the steady state (exactly one entry to evict) the new entry goes straight into the victim's slot, else behind the unit's
  // entries.  (Its score and time are written with the others'.)
  const bool new_in_regs = mode == kWholeStep && room && evict && n - B == 1;
  if (room && !new_in_regs) {
    if (mode == kWholeStep) {
      if (tid < 16)
        *reinterpret_cast<u32x4*>(d.K + base.k(n_old, tid * 8)) = *reinterpret_cast<const u32x4*>(call.k_new + (size_t)urel * kDim + tid * 8);
      if (tid >= 64 && tid < 192) d.V[base.v(n_old, tid - 64)] = call.v_new[(size_t)urel * kDim + (tid - 64)];
    }
    if (tid == 256) {
      const size_t s = base + n_old;
      if (mode == kAttend) {
        d.crf[s] = 0.0f;
        d.tau[s] = t;
      }
      d.pos[s] = t;
      d.flags[s] = 0;
      d.n[u] = n;
    }
  }
  if (mode == kAttend) {
    merge();
  } else if constexpr (RMAX > 0) {
    if (n > 0) {
      const NewEntry ne{room ? call.k_new + (size_t)urel * kDim : nullptr, call.v_new + (size_t)urel * kDim};
      finish_unit<NT, RMAX, true, kOne>(d, u, base, n, B, t, sM, sInv, call.flags, val, evm, top, s_tab, s_tab_n, rb, sh, tid, ne, merge);
    }
  }
  if (call.advance) step_epilogue(d, t, 1, tid);
}

}  // namespace ckv
