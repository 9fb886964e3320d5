// Workgroup ids of a one-launch batched call.
//
// Ids are dealt to the dies round robin (id -> die id % kDies), and the host's
// unit map sends entry x + kDies i to the i-th unit of die x, so that a
// problem's units, which read the same operands, run on one die.  Kernels that
// split a unit's columns over two workgroups keep both on the unit's die: the
// first halves of kDies entries have consecutive ids, then their second halves.
#pragma once

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define EHH_HOST_DEVICE __host__ __device__
#else
#define EHH_HOST_DEVICE
#endif

namespace ehh {

constexpr int kDies = 8;

struct HalfUnit {
  int entry, half;
};

// Entry and half of a workgroup; mapped: the entries are the unit map's (their
// number is a multiple of kDies), else plain unit numbers.
EHH_HOST_DEVICE constexpr HalfUnit half_unit(int id, bool mapped) {
  return mapped ? HalfUnit{id / (2 * kDies) * kDies + id % kDies, id / kDies & 1}
                : HalfUnit{id >> 1, id & 1};
}

}  // namespace ehh
