// Pipelined schedule of the stripe kernels: a call's tiles in one launch.
//
// A unit is one sweep block m of a group of columns, all its chase steps in
// order, on one wave or four.  Block m's step j needs block m+1's step j stored (and nothing
// else: the diagonal launch schedule keeps the same order with kernel
// boundaries), so the blocks of a stripe run side by side, each a step or two
// behind the next.  Two forms:
//
//   * local: a workgroup of W waves carries one stripe, wave w the blocks
//     M-1-w, M-1-w-W, ...; the steps done are counted in LDS and the rows pass
//     through the compute unit's own cache.  A hand-over costs a fraction of a
//     microsecond, but a stripe has one compute unit.
//   * device: workgroups of four waves, 64 columns, take units by a ticket,
//     block by block and column group by column group inside a block; the
//     counts are in device memory and the rows are read and written with
//     device-scope accesses.  A hand-over costs about three microseconds, and
//     few stripes fill the device.
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
  __device__ __forceinline__ bool ready(int64_t) const { return true; }
  __device__ __forceinline__ void wait(int64_t) const {}
  __device__ __forceinline__ void done(int64_t) const {}
};

// Counts in LDS: cnt[w] = o * span + steps done of the wave's block of order o
// (= M-1-m); span exceeds every block's steps.
struct LocalSync {
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
};

// Words of a device-form call: the ticket, then the units' counts.
inline size_t pipe_words(int64_t units) { return (size_t)(units + 1) * kPipeStride; }

// (a fill kernel: memset nodes of captured graphs are avoided)
static __global__ __launch_bounds__(256) void k_pipe_clear(int* __restrict__ w, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) w[i] = 0;
}

// Modelled time in microseconds of the diagonal launch schedule: a launch of N
// tiles takes ceil(N / slots) rounds of S + 1 steps and about 8 us to start and
// drain.
inline double diag_us(const DiagPlan& pl, double slots, double step_us) {
  double t = 0.0;
  for (int64_t i = 0; i < pl.T; ++i) {
    int64_t m0, cnt;
    pl.active(i, &m0, &cnt);
    if (cnt) t += std::ceil(2.0 * (double)(cnt * pl.G) / slots) * (double)(pl.S + 1) * step_us +
                  8.0;
  }
  return t;
}

// Form of a call that leaves the schedule open, by a model in microseconds:
// H tiles of 16 columns, M blocks, J steps of the longest, unit_steps steps of
// all blocks, step_us the products of one step of one wave.
//  * local: M + J steps of a stripe's chain, and its other steps shared by the
//    four SIMDs of one compute unit;
//  * device: M + J steps with their hand-overs through memory, and all steps
//    shared by the device (64 columns to a unit);
//  * the diagonal launches where there is no room for the device form's counts
//    and the local form would leave most of the device idle.
// Measured, local and device, us: nbw 64, n = 300: 96, 121; 700: 214, 235;
// 1000: 362, 329; 1500: 626, 566; 2900: 1922, 1622; 8192 with 819 columns:
// 13100, 4060; nbw 32, n = 512: 155, 173; 1000: 395, 321; 1999: 1216, 843 (the
// model is within 15 % of these).
struct PipeChoice {
  enum Form { kDiagonal, kLocal, kDevice } form;
  int waves;  // of a local workgroup
};
inline PipeChoice choose_pipe(int64_t H, int64_t M, int64_t J, double unit_steps, int cus,
                              double step_us, bool device_ok, double diag) {
  PipeChoice c;
  c.form = PipeChoice::kLocal;
  // eight waves (two per SIMD) where a compute unit has one stripe anyway
  c.waves = H <= cus && M >= 8 ? 8 : 4;
  const double local = 40.0 + (double)(M + J) * step_us +
                       (double)((H + cus - 1) / cus) * unit_steps * step_us / 4.0;
  const double dev = 50.0 + (double)(M + J) * (1.35 * step_us + 1.0) +
                     (double)((H + 3) / 4) * unit_steps * step_us / cus;
  if (device_ok) {
    if (dev < local) c.form = PipeChoice::kDevice;
  } else if (diag < local) {
    c.form = PipeChoice::kDiagonal;
  }
  return c;
}

}  // namespace ehh
