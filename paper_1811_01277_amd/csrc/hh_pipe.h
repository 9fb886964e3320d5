// Pipelined schedule of the stripe kernels: a call's tiles in one launch.
//
// A unit is one sweep block m of one stripe, all its chase steps in order, on
// one wave.  Block m's step j needs block m+1's step j stored (and nothing
// else: the diagonal launch schedule keeps the same order with kernel
// boundaries), so the blocks of a stripe run side by side, each a step or two
// behind the next.  Two forms:
//
//   * local: a workgroup of W waves carries one stripe, wave w the blocks
//     M-1-w, M-1-w-W, ...; the steps done are counted in LDS and the rows pass
//     through the compute unit's own cache.  A hand-over costs a fraction of a
//     microsecond, but a stripe has one compute unit.
//   * device: one-wave workgroups take units by a ticket, block by block and
//     stripe by stripe inside a block; the counts are in device memory and the
//     stripes' rows are read and written with device-scope accesses.  A
//     hand-over costs two to three microseconds, and few stripes fill the
//     device.
//
// Waiting always ends: a unit waits only for the unit of the same stripe one
// block above, which in the local form belongs to a wave of the same
// workgroup that waits in the same way only for a block still further up, and
// in the device form has an earlier ticket, so a running wave holds it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "hh_common.h"
#include "hh_sched.h"

namespace ehh {

// No waiting: kernel boundaries order the tiles.
struct NoSync {
  static constexpr bool kDev = false;
  __device__ __forceinline__ bool ready(int64_t) const { return true; }
  __device__ __forceinline__ void wait(int64_t) const {}
  __device__ __forceinline__ void done(int64_t) const {}
};

// Counts in LDS: cnt[w] = o * span + steps done of the wave's block of order o
// (= M-1-m); span exceeds every block's steps.
struct LocalSync {
  static constexpr bool kDev = false;
  int* mine;
  const int* before;  // null: order 0
  int base, before_base, before_steps;
  __device__ __forceinline__ int target(int64_t j) const {
    return before_base + ((int)j + 1 < before_steps ? (int)j + 1 : before_steps);
  }
  __device__ __forceinline__ bool ready(int64_t j) const {
    if (!before) return true;
    const bool ok = __hip_atomic_load(before, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >=
                    target(j);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    return __builtin_amdgcn_readfirstlane(ok) != 0;
  }
  __device__ __forceinline__ void wait(int64_t j) const {
    while (!ready(j)) __builtin_amdgcn_s_sleep(1);
  }
  __device__ __forceinline__ void done(int64_t j) const {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __hip_atomic_store(mine, base + (int)j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
};

// Counts in device memory, one word per unit, kPipeStride ints apart.
constexpr int kPipeStride = 8;
struct DevSync {
  static constexpr bool kDev = true;
  int* mine;
  const int* before;  // null: order 0
  int before_steps;
  __device__ __forceinline__ bool ready(int64_t j) const {
    if (!before) return true;
    const int need = (int)j + 1 < before_steps ? (int)j + 1 : before_steps;
    const bool ok =
        __hip_atomic_load(before, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= need;
    asm volatile("" ::: "memory");
    return __builtin_amdgcn_readfirstlane(ok) != 0;
  }
  __device__ __forceinline__ void wait(int64_t j) const {
    while (!ready(j)) __builtin_amdgcn_s_sleep(1);
  }
  __device__ __forceinline__ void raise(int64_t j) const {
    __hip_atomic_store(mine, (int)j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void done(int64_t j) const {
    // the rows' stores are acknowledged before the count is raised
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    raise(j);
  }
};

// Words of a device-form call: the ticket, then the units' counts.
inline size_t pipe_words(int64_t units) { return (size_t)(units + 1) * kPipeStride; }

// (a fill kernel: memset nodes of captured graphs are avoided)
static __global__ __launch_bounds__(256) void k_pipe_clear(int* __restrict__ w, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) w[i] = 0;
}

// Modelled time of the diagonal launch schedule in steps of one wave: a launch
// of N tiles takes ceil(N / slots) rounds of S + 1 steps and about 8 us to
// start and drain.
inline double diag_steps(const DiagPlan& pl, double slots, double step_us) {
  double t = 0.0;
  for (int64_t i = 0; i < pl.T; ++i) {
    int64_t m0, cnt;
    pl.active(i, &m0, &cnt);
    if (cnt) t += std::ceil(2.0 * (double)(cnt * pl.G) / slots) * (double)(pl.S + 1) +
                  8.0 / step_us;
  }
  return t;
}

// Form of a call that leaves the schedule open, by a model in steps of one
// wave that has a SIMD to itself (step_us microseconds each); H stripes of one
// wave's columns, M blocks, J steps of the longest.
//  * local: a compute unit runs four steps at a time, a stripe's chain is its
//    blocks' starts, a step or so apart, and one block's steps;
//  * device: all SIMDs share the work; the chain pays the hand-over at each
//    step, and the last block runs while the others have ended (half of its
//    steps with idle waves beside it);
//  * the diagonal launches where there is no room for the device form's counts
//    and the local form would leave most of the device idle.
struct PipeChoice {
  enum Form { kDiagonal, kLocal, kDevice } form;
  int waves;  // of a local workgroup
  double steps;
};
inline PipeChoice choose_pipe(int64_t H, int64_t M, int64_t J, double unit_steps, int cus,
                              double step_us, bool device_ok, double diag) {
  const double hand_local = 0.4 / step_us, hand_dev = 2.5 / step_us;
  PipeChoice c;
  c.form = PipeChoice::kLocal;
  // eight waves (two per SIMD) where a compute unit has one stripe anyway
  c.waves = H <= cus && M >= 8 ? 8 : 4;
  c.steps = std::max((double)((H + cus - 1) / cus) * unit_steps / 4.0,
                     (double)(M + J) * (1.0 + hand_local));
  if (device_ok) {
    const double dev = std::max((double)H * unit_steps / (4.0 * cus) + 0.5 * (double)J,
                                (double)(M + J) * (1.0 + hand_dev));
    if (dev < c.steps) {
      c.form = PipeChoice::kDevice;
      c.steps = dev;
    }
  } else if (diag < c.steps) {
    c.form = PipeChoice::kDiagonal;
    c.steps = diag;
  }
  return c;
}

}  // namespace ehh
