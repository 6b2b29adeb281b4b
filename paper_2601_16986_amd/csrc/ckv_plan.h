// Choices that kernels and host make by sizes alone.  Plain C++, no HIP, so that a host program can include it.
#pragma once

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

// Whether the workgroups of a step look at their unit's counter of arrivals before they publish their own part: only if all of them run at
// once, one per compute unit (figures at layer_step_kernel).
CKV_PLAN bool looks_early(long long workgroups, int n_cu) { return workgroups < n_cu; }

}  // namespace ckv
