// Band -> tridiagonal reduction by bulge chasing (C ABI in
// include/elpa_b2t.h; Kus et al., Sec. 2), one column per chase step, with
// the reflectors written in the slot layout of the tridiagonal -> band
// back-transformation.  Bands up to 64 wide run the whole chase in one launch
// (k_chase_resident, or k_chase_sweeps, below); wider ones run the launch
// schedule described here.
//
// Schedule.  Chase step (s, j) (row r = s+1+j*nbw, length L <= nbw) reads and
// writes only entries of the square [r-nbw, r+L+nbw)^2 that lie in rows
// [r, r+L) or in columns [r, r+L).  A step (s+1, j') with j' <= j-3 stays
// within indices up to r-nbw, and meets index r-nbw only in rows and columns
// below r, so it shares no entry with (s, j); steps further apart share none
// either.  So with the launch index
//   t(s, j) = j + 3 s
// every pair that shares entries runs in launches ordered as in the
// sequential reduction (sweep by sweep, step by step), and the steps of one
// launch (same t, distinct s) touch disjoint entries.  One workgroup per step;
// kernel boundaries order the launches.  There is no waiting between
// workgroups.
//
// A step: the reflector from column c (= s for j = 0, else r - nbw), rows
// [r, r+L) (LAPACK's larfg convention), then the left update of rows
// [r, r+L) over the window's columns (one wave per column, lanes over rows)
// and the right update of columns [r, r+L) over the window's rows (one
// thread per row), then the eliminated entries written exactly.  The step is
// bound by memory latency, so both updates issue a chunk of independent
// loads before using any of them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "../../include/elpa_b2t.h"
#include "../../include/elpa_hh.h"
#include "hh_common.h"
#include "hh_sched.h"
#include "lane_ops.h"

namespace eb2t {

using ehh::z64;

// scalar operations on double / complex double
__device__ __forceinline__ double conj_(double a) { return a; }
__device__ __forceinline__ z64 conj_(z64 a) { return z64{a.re, -a.im}; }
__device__ __forceinline__ double mul(double a, double b) { return a * b; }
__device__ __forceinline__ z64 mul(z64 a, z64 b) {
  return z64{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ double add(double a, double b) { return a + b; }
__device__ __forceinline__ z64 add(z64 a, z64 b) { return z64{a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ double sub(double a, double b) { return a - b; }
__device__ __forceinline__ z64 sub(z64 a, z64 b) { return z64{a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ double abs2(double a) { return a * a; }
__device__ __forceinline__ double abs2(z64 a) { return a.re * a.re + a.im * a.im; }
__device__ __forceinline__ double re(double a) { return a; }
__device__ __forceinline__ double re(z64 a) { return a.re; }
__device__ __forceinline__ double im(double) { return 0.0; }
__device__ __forceinline__ double im(z64 a) { return a.im; }
template <typename E>
__device__ __forceinline__ E from_re(double x) {
  if constexpr (std::is_same<E, double>::value)
    return x;
  else
    return z64{x, 0.0};
}
template <typename E>
__device__ __forceinline__ E zero() {
  return from_re<E>(0.0);
}

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1) x += __shfl_xor(x, w, 64);
  return x;
}
__device__ __forceinline__ z64 wave_sum(z64 x) { return z64{wave_sum(x.re), wave_sum(x.im)}; }

constexpr int kMaxNb = 512;
// Launch t runs the steps (s, t - kLag s): two steps of one launch touch
// disjoint entries (the later sweep only rows and columns below r - nb, the
// earlier one only from r on, sharing index r - nb in different entries).
constexpr int64_t kLag = 3;

// one launch: the steps (s, t - kLag s) for s = s_lo .. s_lo + gridDim.x - 1, one
// 512-thread workgroup (8 waves) per step
template <typename E>
__global__ __launch_bounds__(512) void k_chase(E* __restrict__ A, int64_t lda, int64_t n,
                                               int64_t nb, int64_t t, int64_t s_lo,
                                               E* __restrict__ hh, E* __restrict__ tau) {
  __shared__ E v[kMaxNb];
  __shared__ double part[8];
  __shared__ E sh_tau, sh_sc;
  __shared__ double sh_beta;
  const int64_t s = s_lo + blockIdx.x;
  const int64_t j = t - kLag * s;
  const int64_t r = s + 1 + j * nb;
  const int64_t L = (nb < n - r) ? nb : n - r;
  const int64_t c = (j == 0) ? s : r - nb;
  const int64_t lo = (r - nb > 0) ? r - nb : 0;
  const int64_t hi = (r + L + nb < n) ? r + L + nb : n;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto at = [&](int64_t i, int64_t k) -> E& { return A[i + k * lda]; };

  // reflector: x = A[r .. r+L, c]
  double ss = 0.0;
  for (int64_t i = tid; i < L; i += blockDim.x) {
    const E x = at(r + i, c);
    v[i] = x;
    if (i >= 1) ss += abs2(x);
  }
  ss = wave_sum(ss);
  if (lane == 0) part[wave] = ss;
  __syncthreads();
  if (tid == 0) {
    double sum = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) sum += part[w];
    const E alpha = v[0];
    const double ar = re(alpha), ai = im(alpha);
    if (sum == 0.0 && ai == 0.0) {
      sh_tau = zero<E>();
      sh_beta = ar;
      part[0] = 0.0;  // no scaling needed
    } else {
      const double h = sqrt(ar * ar + ai * ai + sum);
      const double bt = (ar >= 0.0) ? -h : h;
      if constexpr (std::is_same<E, double>::value)
        sh_tau = (bt - ar) / bt;
      else
        sh_tau = z64{(bt - ar) / bt, -ai / bt};
      sh_beta = bt;
      part[0] = 1.0;
      // scale 1 / (alpha - beta)
      const E den = sub(alpha, from_re<E>(bt));
      if constexpr (std::is_same<E, double>::value) {
        sh_sc = 1.0 / den;
      } else {
        const double dd = den.re * den.re + den.im * den.im;
        sh_sc = z64{den.re / dd, -den.im / dd};
      }
    }
  }
  __syncthreads();
  const E tv = sh_tau;
  const bool act = part[0] != 0.0;
  {
    // v <- (1, x[1:] / (alpha - beta)); with tau = 0 the tail is already zero
    const E sc = sh_sc;
    for (int64_t i = tid; i < L; i += blockDim.x)
      v[i] = (i == 0) ? from_re<E>(1.0) : (act ? mul(v[i], sc) : v[i]);
  }
  __syncthreads();

  if (act) {
    // left: rows [r, r+L) of columns [lo, hi) <- H^H rows, H^H = I - conj(tau) v v^H.
    // A wave takes columns lo+wave, lo+wave+NW, ...; with L <= 64 a lane holds
    // one row, and the values of CH columns are loaded before any is used,
    // so CH loads are in flight at once.
    const E ct = conj_(tv);
    const int NW = (int)(blockDim.x >> 6);
    if (L <= 64) {
      constexpr int CH = 8;
      const E vl = lane < L ? v[lane] : zero<E>();
      const E cvl = conj_(vl);
      for (int64_t k0 = lo + wave; k0 < hi; k0 += (int64_t)NW * CH) {
        E x[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
          const int64_t k = k0 + (int64_t)NW * u;
          x[u] = (k < hi && lane < L) ? at(r + lane, k) : zero<E>();
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
          const int64_t k = k0 + (int64_t)NW * u;
          const E w = mul(ct, wave_sum(mul(cvl, x[u])));
          if (k < hi && lane < L) at(r + lane, k) = sub(x[u], mul(vl, w));
        }
      }
    } else {
      for (int64_t k = lo + wave; k < hi; k += NW) {
        E acc = zero<E>();
        for (int64_t i = lane; i < L; i += 64) acc = add(acc, mul(conj_(v[i]), at(r + i, k)));
        const E w = mul(ct, wave_sum(acc));
        for (int64_t i = lane; i < L; i += 64) at(r + i, k) = sub(at(r + i, k), mul(v[i], w));
      }
    }
    __syncthreads();
    // right: columns [r, r+L) of rows [lo, hi) <- cols H, H = I - tau v v^H.
    // Four adjacent threads per row, each with QC consecutive columns of every
    // 4 QC; their partial products are combined by lane shuffles (all four get
    // the same sum in the same order), and every thread updates the values it
    // loaded.  Rows with L > 4 QC reload their values for the update.
    constexpr int QC = 16;
    const int part4 = tid & 3;
    const int64_t rows_per_pass = blockDim.x >> 2;
    for (int64_t i0 = lo; i0 < hi; i0 += rows_per_pass) {
      const int64_t i = i0 + (tid >> 2);
      const bool row_ok = i < hi;
      E y[QC];
      E acc = zero<E>();
      for (int64_t q0 = 0; q0 < L; q0 += 4 * QC) {
        const int64_t qb = q0 + (int64_t)part4 * QC;
#pragma unroll
        for (int u = 0; u < QC; ++u)
          y[u] = (row_ok && qb + u < L) ? at(i, r + qb + u) : zero<E>();
#pragma unroll
        for (int u = 0; u < QC; ++u)
          if (qb + u < L) acc = add(acc, mul(y[u], v[qb + u]));
      }
      // sum over the four threads of the row (lanes 4m .. 4m+3 of one wave)
      E tot = acc;
      if constexpr (std::is_same<E, double>::value) {
        tot = tot + __shfl_xor(tot, 1, 64);
        tot = tot + __shfl_xor(tot, 2, 64);
      } else {
        tot = z64{tot.re + __shfl_xor(tot.re, 1, 64), tot.im + __shfl_xor(tot.im, 1, 64)};
        tot = z64{tot.re + __shfl_xor(tot.re, 2, 64), tot.im + __shfl_xor(tot.im, 2, 64)};
      }
      const E w = mul(tot, tv);
      if (L <= 4 * QC) {
        const int64_t qb = (int64_t)part4 * QC;
#pragma unroll
        for (int u = 0; u < QC; ++u)
          if (row_ok && qb + u < L) at(i, r + qb + u) = sub(y[u], mul(w, conj_(v[qb + u])));
      } else {
        for (int64_t q0 = 0; q0 < L; q0 += 4 * QC) {
          const int64_t qb = q0 + (int64_t)part4 * QC;
#pragma unroll
          for (int u = 0; u < QC; ++u)
            if (row_ok && qb + u < L)
              at(i, r + qb + u) = sub(at(i, r + qb + u), mul(w, conj_(v[qb + u])));
        }
      }
    }
  }
  __syncthreads();
  // eliminated entries, the reflector in its slot
  const E beta = from_re<E>(sh_beta);
  const int64_t slot = ehh::slot_offset(n, nb, s) + j;
  E* __restrict__ dst = hh + slot * nb;
  for (int64_t i = tid; i < nb; i += blockDim.x) {
    if (i < L) {
      const E z = (i == 0) ? beta : zero<E>();
      at(r + i, c) = z;
      at(c, r + i) = z;
    }
    dst[i] = (i < L) ? v[i] : zero<E>();
  }
  if (tid == 0) tau[slot] = tv;
}

// ---------------------------------------------------------------------------
// nb <= 64: the whole chase in one launch, lower triangle only, every block a
// step touches held in registers.
//
// A step (s, j) with H = I - tau v v^H on the indices [r, r+L) changes three
// lower-triangle blocks:
//   R = rows [r, r+L) x columns [r-nb, r)  <- H^H R  (column s alone for j = 0)
//   D = rows and columns [r, r+L)          <- H^H D H (with y = D v, mu = v^H y
//       and w = tau y - |tau|^2 mu / 2 v: D <- D - w v^H - v w^H)
//   C = rows [r+L, hi) x columns [r, r+L)  <- C H    (hi = min(r+L+nb, n))
// and C is the next step's R.  A workgroup carries one sweep from its first
// step to its last, so C passes on in registers: a step loads D and C, and
// stores R and D.
//
// Order between sweeps.  Step (s, j) reads what sweep s-1 wrote in its steps
// up to j+1 and one entry of step j+2, the subdiagonal value beta that its
// reflector leaves (row r+2nb-1, column r+nb-1).  So a workgroup forms the
// next step's reflector at the end of each step, stores beta and the zeros
// below it with the step's R and D, and then raises its progress count; sweep
// s may load step j once sweep s-1 has counted min(j+2, J(s-1)) steps.  What
// sweep s stores in step j lies in rows below r+nb, which sweep s-1 no longer
// reads or writes at that count.
//
// Waiting always ends: sweeps are handed out in order by a ticket counter, so
// the sweep a workgroup waits for is held by a workgroup that started
// earlier, is running and waits only for a still earlier sweep; sweep 0 waits
// for none.  (Should a wait last longer than kWaitTicks all the same, it is
// given up and d is set to NaN.)  Matrix entries that pass between workgroups
// are read and written with device-scope accesses, stores are acknowledged
// before the count is raised.
//
// Bound: the chain of two steps and one hand-over per sweep, all latency.
// One launch per step (3 n launches, 12.1 us each at any size) took 34 ms at
// n = 1000 and 148 ms at n = 4000 (nbw = 64, fp64); the one-launch chase takes
// 8.7 and 36 ms, about 9 us per sweep.  It runs where the resident form below
// (4.5 and 21.4 ms) does not: more positions than the device holds, or a busy
// device.
//
// Layout: lane i of each wave holds row i of the blocks, wave w of NW the
// columns w, w + NW, ... (8 per wave): each block is one coalesced access per
// column.  Row sums (the lower part of D v, C v) add the waves' partials
// through LDS.  Column sums (v^H R, the strictly lower part of D^H v) halve
// the eight values per lane with each exchange, so the eight sums of a wave
// take 15 exchanges and not 48, and lane 8 q ends with column q's.
constexpr int64_t kWaitTicks = int64_t(20) * 100000000;  // 20 s of the 100 MHz clock
constexpr int kProgStride = 16;                          // counts 64 bytes apart
constexpr int64_t kGatherTicks = 100000;                 // 1 ms

using elane::dpp_mov;
using elane::kHalfMirror;
using elane::kMirror;
using elane::kRor8;
using elane::kXor1;
using elane::kXor2;
using elane::pair16;
using elane::pair32;
using elane::read_lane;

// sum over the wave, the same bits in every lane
__device__ __forceinline__ double wave_sum_dpp(double x) {
  x += dpp_mov<kXor1>(x);
  x += dpp_mov<kXor2>(x);
  x += dpp_mov<kHalfMirror>(x);
  x += dpp_mov<kMirror>(x);
  x = pair16(x, x);
  return pair32(x, x);
}
// x[0..7] per lane -> lane l returns the wave's sum of x[l / 8]
__device__ __forceinline__ double wave_sum8(const double (&x)[8]) {
  double y[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) y[i] = pair32(x[i], x[i + 4]);
  const double z0 = pair16(y[0], y[2]), z1 = pair16(y[1], y[3]);
  const bool up = (threadIdx.x & 8) != 0;
  double t = (up ? z1 : z0) + dpp_mov<kRor8>(up ? z0 : z1);
  t += dpp_mov<kXor1>(t);
  t += dpp_mov<kXor2>(t);
  return t + dpp_mov<kHalfMirror>(t);
}
__device__ __forceinline__ z64 wave_sum8(const z64 (&x)[8]) {
  double a[8], b[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    a[i] = x[i].re;
    b[i] = x[i].im;
  }
  return z64{wave_sum8(a), wave_sum8(b)};
}
__device__ __forceinline__ z64 read_lane(z64 x, int l) {
  return z64{read_lane(x.re, l), read_lane(x.im, l)};
}
// device-scope accesses of matrix entries
__device__ __forceinline__ double load_dev(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ z64 load_dev(const z64* p) {
  return z64{load_dev(&p->re), load_dev(&p->im)};
}
__device__ __forceinline__ void store_dev(double* p, double x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_dev(z64* p, z64 x) {
  store_dev(&p->re, x.re);
  store_dev(&p->im, x.im);
}
// the eliminated diagonal block stays exactly Hermitian
__device__ __forceinline__ double real_part(double a) { return a; }
__device__ __forceinline__ z64 real_part(z64 a) { return z64{a.re, 0.0}; }

// keeps a product out of a fused multiply-add
__device__ __forceinline__ double rounded(double x) {
  asm("" : "+v"(x));
  return x;
}
__device__ __forceinline__ z64 rounded(z64 x) { return z64{rounded(x.re), rounded(x.im)}; }
// a conj(b) + c conj(d), in one way in both chases
__device__ __forceinline__ double rank2(double a, double b, double c, double d) {
  return __builtin_fma(a, b, rounded(c * d));
}
__device__ __forceinline__ z64 rank2(z64 a, z64 b, z64 c, z64 d) {
  return add(mul(a, conj_(b)), mul(c, conj_(d)));
}

// progress counts, ticket, failure word and messages of one call
using u64 = unsigned long long;
struct ChaseState {
  int* prog;  // [n - 1] counts, kProgStride apart
  int* ticket;
  int* failed;
  int* arrived;  // resident form: workgroups that are there
  int* state;    // kOpen, kGo, kAlone
  u64* words;    // its messages
  int64_t nwords;
};
constexpr int kOpen = 0, kGo = 1, kAlone = 2;

__global__ __launch_bounds__(256) void k_chase_clear(ChaseState c, int64_t n, int open) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n - 1) c.prog[i * kProgStride] = 0;
  for (int64_t w = i; w < c.nwords; w += (int64_t)gridDim.x * blockDim.x) c.words[w] = 0;
  if (i == 0) {
    *c.ticket = 0;
    *c.failed = 0;
    *c.arrived = 0;
    *c.state = open;
  }
}

// waits until *p >= need; false when the wait was given up
__device__ __forceinline__ bool wait_for(const int* p, int need, int* failed) {
  if (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= need) return true;
  const int64_t t0 = (int64_t)wall_clock64();
  for (;;) {
#pragma unroll 1
    for (int k = 0; k < 64; ++k) {
      if (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= need) return true;
      __builtin_amdgcn_s_sleep(1);
    }
    if (__hip_atomic_load(failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return false;
    if ((int64_t)wall_clock64() - t0 > kWaitTicks) {
      __hip_atomic_store(failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return false;
    }
  }
}

// nb <= 8 NW
template <typename E, int NW>
__global__ __launch_bounds__(64 * NW) void k_chase_sweeps(E* __restrict__ A, int64_t lda,
                                                          int64_t n, int64_t nb, ChaseState st,
                                                          E* __restrict__ hh,
                                                          E* __restrict__ tau) {
  constexpr int NQ = 8;
  __shared__ E vs[64], ys[64], py[NW][64], pu[NW][64];
  __shared__ E sh_tau;
  __shared__ int sh_s, sh_arrived, sh_ok[NW];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // row i0 + lane of column k: a wave-uniform base and a 32-bit lane offset
  auto at = [&](int64_t i0, int64_t k) -> E* { return A + (i0 + k * lda) + (unsigned)lane; };

  // the resident form did the whole chase
  if (__hip_atomic_load(st.state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kGo) return;

  for (;;) {
    __syncthreads();
    if (tid == 0) {
      sh_s = __hip_atomic_fetch_add(st.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      sh_arrived = 0;
    }
    __syncthreads();
    const int64_t s = __builtin_amdgcn_readfirstlane(sh_s);
    if (s >= n - 1) return;
    const int64_t J = (n - 1 - s + nb - 1) / nb, Jp = (n - s + nb - 1) / nb;
    const int64_t slot0 = ehh::slot_offset(n, nb, s);
    const int* before = st.prog + (s - 1) * kProgStride;
    E xr[NQ], xd[NQ], xc[NQ];

    // reflector of the column x (wave 0; rows r .. r+L-1 in its lanes, the
    // column at c): v into LDS, beta and zeros into the matrix
    auto reflect = [&](E x, int64_t r, int L, int64_t c, int64_t j) {
      const double ss = wave_sum_dpp(lane >= 1 && lane < L ? abs2(x) : 0.0);
      const E alpha = read_lane(x, 0);
      const double ar = re(alpha), ai = im(alpha);
      E tv = zero<E>(), sc = zero<E>();
      double beta = ar;
      if (ss != 0.0 || ai != 0.0) {
        const double h = sqrt(ar * ar + ai * ai + ss);
        beta = ar >= 0.0 ? -h : h;
        if constexpr (std::is_same<E, double>::value) {
          tv = (beta - ar) / beta;
          sc = 1.0 / (ar - beta);
        } else {
          tv = z64{(beta - ar) / beta, -ai / beta};
          const double dr = ar - beta, dd = dr * dr + ai * ai;
          sc = z64{dr / dd, -ai / dd};
        }
      }
      const E v = lane == 0 ? from_re<E>(1.0) : (lane < L ? mul(x, sc) : zero<E>());
      vs[lane] = v;
      if (lane == 0) sh_tau = tv;
      xr[0] = lane == 0 ? from_re<E>(beta) : zero<E>();
      if (lane < L) store_dev(at(r, c), xr[0]);
      if (lane < nb) hh[(slot0 + j) * nb + lane] = v;
      if (lane == 0) tau[slot0 + j] = tv;
    };

    for (int64_t j = 0; j < J; ++j) {
      const int64_t r = s + 1 + j * nb;
      const int L = (int)((nb < n - r) ? nb : n - r);
      const int nR = j == 0 ? 1 : (int)nb;
      const int nC = (int)(((r + L + nb < n) ? r + L + nb : n) - r - L);
      bool ok = true;
      if (s > 0) ok = wait_for(before, (int)(j + 2 < Jp ? j + 2 : Jp), st.failed);
      asm volatile("" ::: "memory");
      if (lane == 0) sh_ok[wave] = ok ? 1 : 0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int k = wave + NW * q;
        xd[q] = (k < L && lane < L && lane >= k) ? load_dev(at(r, r + k)) : zero<E>();
        xc[q] = (k < L && lane < nC) ? load_dev(at(r + L, r + k)) : zero<E>();
      }
      if (j == 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) xr[q] = zero<E>();
        if (wave == 0) reflect(lane < L ? load_dev(at(r, s)) : zero<E>(), r, L, s, 0);
      }
      __syncthreads();
      {
        int all = 1;
#pragma unroll
        for (int w = 0; w < NW; ++w) all &= sh_ok[w];
        if (!__builtin_amdgcn_readfirstlane(all)) return;  // the same in every wave
      }
      const E tv = sh_tau, vl = vs[lane];
      const bool act = __builtin_amdgcn_readfirstlane(re(tv) != 0.0 || im(tv) != 0.0) != 0;
      E vk[NQ], wr;
#pragma unroll
      for (int q = 0; q < NQ; ++q) vk[q] = read_lane(vl, wave + NW * q);
      if (act) {
        const E cvl = conj_(vl);
        E p[NQ], ry = zero<E>(), ru = zero<E>();
#pragma unroll
        for (int q = 0; q < NQ; ++q) p[q] = mul(cvl, xr[q]);
        wr = wave_sum8(p);
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          p[q] = lane > wave + NW * q ? mul(cvl, xd[q]) : zero<E>();
        const E cs = wave_sum8(p);
        // (v^H D)_k = conj((D v)_k)
        if ((lane & 7) == 0) ys[wave + NW * (lane >> 3)] = conj_(cs);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          ry = add(ry, mul(xd[q], vk[q]));
          ru = add(ru, mul(xc[q], vk[q]));
        }
        py[wave][lane] = ry;
        pu[wave][lane] = ru;
      }
      __syncthreads();
      if (act) {
        // every wave forms y and u of its rows (the same bits in each)
        E yl = lane < 8 * NW ? ys[lane] : zero<E>(), us = zero<E>();
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          yl = add(yl, py[w][lane]);
          us = add(us, pu[w][lane]);
        }
        const E ul = mul(tv, us);
#pragma unroll
        for (int q = 0; q < NQ; ++q) xc[q] = sub(xc[q], mul(ul, conj_(vk[q])));
        const E ct = conj_(tv);
        const double mu = wave_sum_dpp(re(mul(conj_(vl), yl)));
        const double h2 = 0.5 * abs2(tv) * mu;
        const E wl = sub(mul(tv, yl), mul(from_re<E>(h2), vl));
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const int k = wave + NW * q;
          const E wk = read_lane(wl, k), rk = mul(ct, read_lane(wr, 8 * q));
          // column 0 is the reduced one (j = 0: the only one)
          if (k >= 1) xr[q] = sub(xr[q], mul(vl, rk));
          xd[q] = sub(xd[q], rank2(wl, vk[q], vl, wk));
          if (lane == k) xd[q] = real_part(xd[q]);
        }
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int k = wave + NW * q;
        if (lane < L && k >= 1 && k < nR) store_dev(at(r, r - nb + k), xr[q]);
        if (lane < L && k < L && lane >= k) store_dev(at(r, r + k), xd[q]);
        xr[q] = xc[q];
      }
      if (wave == 0 && nC > 0) reflect(xc[0], r + L, nC, r, j + 1);
      // every wave's stores are acknowledged, then the last one counts the step
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (lane == 0) {
        const int a = __hip_atomic_fetch_add(&sh_arrived, 1, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP);
        if (a == (int)(j + 1) * NW - 1)
          __hip_atomic_store(st.prog + s * kProgStride, (int)(j + 1), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// nb <= 64, all positions resident
// ---------------------------------------------------------------------------
// A workgroup stays at chase position j and holds its blocks R and D (as above)
// through all sweeps: the next sweep's blocks are the same ones, one row and
// one column further down.  Columns sit in the waves by their global index
// modulo nb, so the column that comes takes the place of the one that leaves;
// rows move up one lane.  Sums run in the order of the moving form's, which
// gives the same bits where the waves divide nb.  Per sweep two messages pass between neighbours:
//   forward   v and tau of position j, for the right update of R_{j+1};
//   backward  the row that position j+1 gives up, R_{j+1}'s first: beta, the
//             entries behind it, and D_{j+1}'s first entry: position j's new
//             last row.  (New entries left of beta are zero.)
// Position 0 gives its first row up to the result: e and d.
//
// A position's reflector needs the forward message, beta of the backward
// message of the sweep before, and its own blocks, so the chain is, per sweep,
// two hand-overs, two sums over the waves' columns and two reflectors; the
// rest of a step runs beside it.  Every wave receives for itself and forms the
// reflector for itself, which saves the barriers a broadcast would take.
//
// Words: an 8-byte word carries half a double and the sweep's tag, so a word
// that is there is whole.  Messages alternate between two places.  A forward
// place is written again two sweeps later, after the receiver's beta of the
// sweep between came back, which followed a barrier behind its waves' receipt;
// a backward place two sweeps later after the forward message of that sweep,
// which the receiver sent after the barriers of the sweep between.
//
// All J positions must be running: the workgroups count themselves, and the
// last one opens the chase (kGo).  If they do not come together in time the
// chase is left to k_chase_sweeps behind (kAlone), nothing having been written.
// A wait of more than kWaitTicks is given up as above, and then all are.
//
// Bound: the latency of that chain, and nearly as much the instructions of one
// position's step.  n = 1000 / 4000, nbw = 64: 4.5 / 21.4 ms, where workgroups
// that follow the sweeps take 8.7 / 36; complex, n = 700, nbw = 32: 4.1 ms
// against 7.1.  Selects in place of uniform branches and column numbers kept
// from sweep to sweep took 6.2 ms to 4.5 at n = 1000.
template <typename E>
struct ChaseWords {
  static constexpr int W = std::is_same<E, double>::value ? 2 : 4;  // words per value
  static constexpr int FWD = 64 * W, BACK = 65 * W, ALL = 2 * (FWD + BACK);
};
__device__ __forceinline__ void put_word(u64* p, unsigned half, unsigned tag) {
  __hip_atomic_store(p, ((u64)half << 32) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_value(u64* p, double x, unsigned tag) {
  put_word(p, (unsigned)__double2hiint(x), tag);
  put_word(p + 1, (unsigned)__double2loint(x), tag);
}
__device__ __forceinline__ void put_value(u64* p, z64 x, unsigned tag) {
  put_value(p, x.re, tag);
  put_value(p + 2, x.im, tag);
}
__device__ __forceinline__ u64 get_word(const u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool get_value(const u64* p, double& x, unsigned tag) {
  const u64 h = get_word(p), l = get_word(p + 1);
  x = __hiloint2double((int)(h >> 32), (int)(l >> 32));
  return (unsigned)h == tag && (unsigned)l == tag;
}
__device__ __forceinline__ bool get_value(const u64* p, z64& x, unsigned tag) {
  const bool a = get_value(p, x.re, tag), b = get_value(p + 2, x.im, tag);
  return a && b;
}
// the lanes with `mine` (`mine2`) receive their values; zero in the others
template <typename E>
__device__ __forceinline__ void receive(const u64* p, bool mine, unsigned tag, E& x, const u64* p2,
                                        bool mine2, unsigned tag2, E& x2, int* failed) {
  int64_t t0 = 0;
  x = x2 = zero<E>();
  for (int k = 0;; ++k) {
    E y = zero<E>(), y2 = zero<E>();
    bool ok = true;
    if (mine) ok = get_value(p, y, tag);
    if (mine2 && !get_value(p2, y2, tag2)) ok = false;
    if (__all(ok)) {
      x = y;
      x2 = y2;
      return;
    }
    if ((k & 63) == 63) {
      if (__hip_atomic_load(failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
      const int64_t t = (int64_t)wall_clock64();
      if (t0 == 0) t0 = t;
      if (t - t0 > kWaitTicks) {
        __hip_atomic_store(failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
      }
    }
  }
}

__device__ __forceinline__ double choose(bool c, double a, double b) { return c ? a : b; }
__device__ __forceinline__ z64 choose(bool c, z64 a, z64 b) {
  return z64{c ? a.re : b.re, c ? a.im : b.im};
}
// lane l takes lane l + 1's value, the last one zero
__device__ __forceinline__ double next_lane(double x) { return dpp_mov<0x130>(x); }
__device__ __forceinline__ z64 next_lane(z64 x) { return z64{next_lane(x.re), next_lane(x.im)}; }

template <typename E, int NW>
__global__ __launch_bounds__(64 * NW) void k_chase_resident(E* __restrict__ A, int64_t lda, int n,
                                                            int nb, ChaseState st,
                                                            int64_t gather_ticks,
                                                            E* __restrict__ hh,
                                                            E* __restrict__ tau) {
  constexpr int NQ = 8, W = ChaseWords<E>::W;
  __shared__ E cs[64], ys[64], py[NW][64], pu[NW][64], row[NW][NQ];
  __shared__ int sh_j, sh_state;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid == 0) {
    int now = __hip_atomic_load(st.state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (now == kOpen) {
      const int old =
          __hip_atomic_fetch_add(st.arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      sh_j = old;
      int expect = kOpen;
      if (old == (int)gridDim.x - 1)
        __hip_atomic_compare_exchange_strong(st.state, &expect, kGo, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int64_t t0 = (int64_t)wall_clock64();
      while ((now = __hip_atomic_load(st.state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) ==
             kOpen) {
        if ((int64_t)wall_clock64() - t0 > gather_ticks) {
          expect = kOpen;
          __hip_atomic_compare_exchange_strong(st.state, &expect, kAlone, __ATOMIC_RELAXED,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    sh_state = now;
  }
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(sh_state) != kGo) return;
  const int j = __builtin_amdgcn_readfirstlane(sh_j);
  u64* const out_fwd = st.words + (int64_t)j * ChaseWords<E>::ALL;   // to position j + 1
  u64* const out_back = out_fwd + 2 * ChaseWords<E>::FWD;            // to position j - 1
  const u64* const in_fwd = out_fwd - ChaseWords<E>::ALL;
  const u64* const in_back = out_back + ChaseWords<E>::ALL;

  const bool in_band = lane < nb;
  unsigned base = nb == 1 ? 0 : 1;  // place of columns r - nb and r
  int J = (n - 1 + nb - 1) / nb, last = n - 1 - (J - 1) * nb;  // of this sweep; its last length
  int64_t slot0 = 0;
  E xr[NQ], xd[NQ];
  // col[q]: the block's column at the wave's place q; nb, a lane of zeros, for
  // places past the band
  int col[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int k = wave + NW * q;
    col[q] = k >= nb ? nb : (k < (int)base ? k - (int)base + nb : k - (int)base);
    const int r = 1 + j * nb, c = col[q];
    const bool ok = in_band && k < nb && r + lane < n;
    xr[q] = ok && (j > 0 || c == nb - 1) ? A[r + lane + (int64_t)(r - nb + c) * lda] : zero<E>();
    xd[q] = ok && r + c < n && lane >= c ? A[r + lane + (int64_t)(r + c) * lda] : zero<E>();
  }
  for (int s = 0;; ++s) {
    const int r = s + 1 + j * nb;
    if (r >= n) return;
    const unsigned tag = (unsigned)s + 1u;
    const unsigned old = base == 0 ? nb - 1 : base - 1;  // place of the last column
    const int turn = nb - (int)base;  // columns from here on sit at places from 0
    // the sweep before: position j + 1 gave up row r + nb - 1
    const bool gained = s > 0 && r + nb - 1 < n;
    const u64* const bw = in_back + ((s - 1) & 1) * ChaseWords<E>::BACK;
    // the forward message, and beta of the last row for the wave that holds it
    // (together: they come at about the same time)
    E vp, last_beta;
    receive<E>(in_fwd + (s & 1) * ChaseWords<E>::FWD + lane * W, j > 0 && in_band, tag, vp,
               bw + old * W, gained && old % NW == (unsigned)wave && lane == nb - 1, tag - 1u, last_beta,
               st.failed);
    const bool newest = gained && old % NW == (unsigned)wave;
    if (newest) {
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        xr[q] = choose(col[q] == nb - 1 && lane == nb - 1, last_beta, xr[q]);
    }
    // right update of R with the reflector of position j - 1; sums in the
    // order of the columns, not of their places
    E tp = zero<E>(), ul = zero<E>();
    E vk[NQ];
    const unsigned red = j > 0 ? base : old;  // place of the column to reduce
    if (j > 0) {
      tp = read_lane(vp, 0);
      if (lane == 0) vp = from_re<E>(1.0);
      E ru = zero<E>();
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        vk[q] = read_lane(vp, col[q] & 63);
        ru = add(ru, mul(xr[q], choose(col[q] < turn, vk[q], zero<E>())));
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        ru = add(ru, mul(xr[q], choose(col[q] >= turn, vk[q], zero<E>())));
      pu[wave][lane] = ru;
    }
    if (red % NW == (unsigned)wave) {
      const int want = j > 0 ? 0 : nb - 1;
      E x = xr[0];
#pragma unroll
      for (int q = 1; q < NQ; ++q) x = choose(col[q] == want, xr[q], x);
      cs[lane] = x;
    }
    __syncthreads();
    E x = cs[lane];
    const bool right =
        j > 0 && __builtin_amdgcn_readfirstlane(re(tp) != 0.0 || im(tp) != 0.0) != 0;
    if (right) {
      E us = zero<E>();
#pragma unroll
      for (int w = 0; w < NW; ++w) us = add(us, pu[(base + w) % NW][lane]);
      // (rounded once, for the reduced column too, whose entry of v is 1)
      ul = rounded(mul(tp, us));
      x = sub(x, ul);
    }
    // the reflector, in every wave the same
    const double ss = wave_sum_dpp(in_band && lane >= 1 ? abs2(x) : 0.0);
    const E alpha = read_lane(x, 0);
    const double ar = re(alpha), ai = im(alpha);
    E tv = zero<E>(), sc = zero<E>();
    double beta = ar;
    const bool act = __builtin_amdgcn_readfirstlane(ss != 0.0 || ai != 0.0) != 0;
    if (act) {
      const double h = sqrt(ar * ar + ai * ai + ss);
      beta = ar >= 0.0 ? -h : h;
      if constexpr (std::is_same<E, double>::value) {
        tv = (beta - ar) / beta;
        sc = 1.0 / (ar - beta);
      } else {
        tv = z64{(beta - ar) / beta, -ai / beta};
        const double dr = ar - beta, dd = dr * dr + ai * ai;
        sc = z64{dr / dd, -ai / dd};
      }
    }
    const E vl = lane == 0 ? from_re<E>(1.0) : (in_band ? mul(x, sc) : zero<E>());
    if (wave == 0 && r + nb < n && in_band)
      put_value(out_fwd + (s & 1) * ChaseWords<E>::FWD + lane * W, lane == 0 ? tv : vl, tag);
    if (wave == 1 && lane == 0) {
      if (j > 0)
        put_value(out_back + (s & 1) * ChaseWords<E>::BACK + base * W, from_re<E>(beta), tag);
      else
        A[s + 1 + (int64_t)s * lda] = from_re<E>(beta);
    }
    if (wave == 2) {
      if (in_band) hh[(slot0 + j) * nb + lane] = vl;
      if (lane == 0) tau[slot0 + j] = tv;
    }
    if (right) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) xr[q] = sub(xr[q], mul(ul, conj_(vk[q])));
    }
    // the rest of the last row, in D: lane q receives this wave's column q
    const int kq = wave + NW * (lane & 7);
    if (gained) {
      E m, none;
      receive<E>(bw + (kq == (int)old ? 64 : kq) * W, lane < NQ && kq < nb, tag - 1u, m, nullptr, false,
                 0, none, st.failed);
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const E v = read_lane(m, q);
        xd[q] = choose(lane == nb - 1, v, xd[q]);
      }
    }
    // left update of R, two-sided update of D
    E wr = zero<E>();
    if (act) {
      const E cvl = conj_(vl);
      E p[NQ], ry = zero<E>();
      if (j > 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) p[q] = mul(cvl, xr[q]);
        wr = wave_sum8(p);
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        p[q] = choose(lane > col[q], mul(cvl, xd[q]), zero<E>());
        vk[q] = read_lane(vl, col[q] & 63);
        ry = add(ry, mul(xd[q], choose(col[q] < turn, vk[q], zero<E>())));
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        ry = add(ry, mul(xd[q], choose(col[q] >= turn, vk[q], zero<E>())));
      const E cd = wave_sum8(p);
      // (v^H D)_k = conj((D v)_k)
      const int k8 = wave + NW * (lane >> 3), c8 = k8 - (int)base;
      if ((lane & 7) == 0 && k8 < nb) ys[c8 < 0 ? c8 + nb : c8] = conj_(cd);
      py[wave][lane] = ry;
    }
    __syncthreads();
    if (act) {
      E yl = in_band ? ys[lane] : zero<E>();
#pragma unroll
      for (int w = 0; w < NW; ++w) yl = add(yl, py[(base + w) % NW][lane]);
      const double mu = wave_sum_dpp(re(mul(conj_(vl), yl)));
      const double h2 = 0.5 * abs2(tv) * mu;
      const E wl = sub(mul(tv, yl), mul(from_re<E>(h2), vl));
      if (j > 0) {
        const E ct = conj_(tv);
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          xr[q] = sub(xr[q], mul(vl, mul(ct, read_lane(wr, 8 * q))));
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const E wk = read_lane(wl, col[q] & 63);
        xd[q] = sub(xd[q], rank2(wl, vk[q], vl, wk));
        xd[q] = choose(lane < col[q], zero<E>(), xd[q]);
        if constexpr (!std::is_same<E, double>::value)
          xd[q] = choose(lane == col[q], real_part(xd[q]), xd[q]);
      }
    }
    // column r passes from D to R: its first entry is the last of row r that
    // leaves, the others follow in R
    if (base % NW == (unsigned)wave) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        xr[q] = choose(col[q] == 0, xd[q], xr[q]);
        xd[q] = choose(col[q] == 0, zero<E>(), xd[q]);
      }
    }
    // row r leaves
    {
      if (lane == 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) row[wave][q] = xr[q];
      }
      __builtin_amdgcn_wave_barrier();
      if (j > 0) {
        if (lane < NQ && kq < nb)
          put_value(out_back + (s & 1) * ChaseWords<E>::BACK + (kq == (int)base ? 64 : kq) * W,
                    row[wave][lane], tag);
      } else if (lane < NQ && kq == (int)base) {
        A[r + (int64_t)r * lda] = row[wave][lane];
      }
      __builtin_amdgcn_wave_barrier();
    }
    // the rows move up by one; row r + nb comes with the next sweep
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      xr[q] = next_lane(xr[q]);
      xd[q] = next_lane(xd[q]);
      const int c = col[q] == 0 ? nb - 1 : col[q] - 1;
      col[q] = col[q] == nb ? nb : c;
    }
    slot0 += J;
    if (--last == 0) {
      --J;
      last = nb;
    }
    base = base + 1 == (unsigned)nb ? 0 : base + 1;
  }
}

// The rest of the result (the one-launch chases leave the upper triangle, the
// resident one also the zeros of the lower): A[k-1, k] = e[k-1], zeros above it
// up to 2 nb rows; zeros in column k-1 below row k up to nb rows.
template <typename E>
__global__ __launch_bounds__(256) void k_upper_out(E* __restrict__ A, int64_t lda, int64_t n,
                                                   int64_t nb, const double* __restrict__ e) {
  const int64_t k = (int64_t)blockIdx.x + 1;   // columns 1 .. n-1
  const int64_t span = 2 * nb;
  for (int64_t q = threadIdx.x; q < span; q += blockDim.x) {
    const int64_t i = k - 1 - q;
    if (i < 0) break;
    A[i + k * lda] = from_re<E>(q == 0 ? e[k - 1] : 0.0);
  }
  for (int64_t i = k + 1 + threadIdx.x; i < n && i < k + nb; i += blockDim.x)
    A[i + (k - 1) * lda] = zero<E>();
}

template <typename E>
__global__ __launch_bounds__(256) void k_diag_out(const E* __restrict__ A, int64_t lda,
                                                  int64_t n, double* __restrict__ d,
                                                  double* __restrict__ e,
                                                  const int* __restrict__ failed) {
  const bool bad = failed && *failed != 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    d[i] = bad ? __builtin_nan("") : re(A[i + i * lda]);
    if (i + 1 < n) e[i] = re(A[i + 1 + i * lda]);
  }
}

// J(s) = ceil((n-1-s)/nb)
inline int64_t steps_of(int64_t n, int64_t nb, int64_t s) { return (n - 1 - s + nb - 1) / nb; }

// nb <= 64: the one-launch chase
template <typename E>
int run_sweeps(int64_t n, int64_t nb, E* A, int64_t lda, double* d, double* e, E* hh, E* tau,
               hipStream_t st, int64_t gather_ticks) {
  const auto resident = nb > 32 ? k_chase_resident<E, 8> : k_chase_resident<E, 4>;
  const int threads = nb > 32 ? 512 : 256;
  const int64_t J = n > 1 ? steps_of(n, nb, 0) : 0;
  // the resident form needs a place for every position on an idle device
  int dev = 0, cus = 0, per_cu = 0;
  const bool fits = gather_ticks >= 0 && n < (int64_t(1) << 30) &&
                    hipGetDevice(&dev) == hipSuccess &&
                    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) ==
                        hipSuccess &&
                    hipOccupancyMaxActiveBlocksPerMultiprocessor(
                        &per_cu, reinterpret_cast<const void*>(resident), threads, 0) ==
                        hipSuccess &&
                    J <= (int64_t)cus * per_cu;
  const unsigned g = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
  int* words = nullptr;
  const size_t counts = ((size_t)std::max<int64_t>(n - 1, 1) + 1) * kProgStride * sizeof(int);
  const int64_t nwords = fits ? J * ChaseWords<E>::ALL : 0;
  const hipError_t err = ehh::ws_alloc((void**)&words, counts + (size_t)nwords * sizeof(u64), st);
  if (err != hipSuccess)
    return err == hipErrorOutOfMemory ? ELPA_ERR_NOMEM : ELPA_ERR_DEVICE;
  const ChaseState cs{words + kProgStride, words,     words + 1, words + 2,
                      words + 3,           (u64*)((char*)words + counts), nwords};
  if (n > 1) {
    hipLaunchKernelGGL(k_chase_clear, dim3((unsigned)((n + 254) / 256)), dim3(256), 0, st, cs, n,
                       fits ? kOpen : kAlone);
    if (fits)
      hipLaunchKernelGGL(resident, dim3((unsigned)J), dim3(threads), 0, st, A, lda, (int)n,
                         (int)nb, cs, gather_ticks, hh, tau);
    // (returns at once where the resident form ran) a sweep lags two steps
    // behind the one before it, so at most about J / 2 are under way; the
    // tickets make any number of workgroups correct
    const unsigned wgs = (unsigned)std::min<int64_t>({n - 1, J / 2 + 2, 512});
    if (nb > 32)
      hipLaunchKernelGGL((k_chase_sweeps<E, 8>), dim3(wgs), dim3(512), 0, st, A, lda, n, nb, cs,
                         hh, tau);
    else
      hipLaunchKernelGGL((k_chase_sweeps<E, 4>), dim3(wgs), dim3(256), 0, st, A, lda, n, nb, cs,
                         hh, tau);
  }
  hipLaunchKernelGGL(k_diag_out<E>, dim3(g), dim3(256), 0, st, (const E*)A, lda, n, d, e,
                     (const int*)(n > 1 ? cs.failed : nullptr));
  if (n > 1)
    hipLaunchKernelGGL(k_upper_out<E>, dim3((unsigned)n - 1), dim3(256), 0, st, A, lda, n, nb,
                       (const double*)e);
  const bool ok = hipGetLastError() == hipSuccess;
  return ehh::ws_free(words, st) == hipSuccess && ok ? ELPA_OK : ELPA_ERR_DEVICE;
}

template <typename E>
int run(int64_t n, int64_t nb, E* A, int64_t lda, double* d, double* e, E* hh, E* tau,
        hipStream_t st, int64_t gather_ticks) {
  if (nb <= 64) return run_sweeps<E>(n, nb, A, lda, d, e, hh, tau, st, gather_ticks);
  // launches t = 0 .. T-1 with T = max_s (3 s + J(s)); the active sweeps of
  // launch t are s_lo(t) .. min(t / kLag, n - 2), s_lo the least s with
  // 3 s + J(s) > t (3 s + J(s) increases with s)
  int64_t T = 0;
  for (int64_t s = 0; s <= n - 2; ++s) T = std::max(T, kLag * s + steps_of(n, nb, s));
  int64_t s_lo = 0;
  for (int64_t t = 0; t < T; ++t) {
    while (s_lo <= n - 2 && kLag * s_lo + steps_of(n, nb, s_lo) <= t) ++s_lo;
    const int64_t s_hi = std::min<int64_t>(t / kLag, n - 2);
    if (s_hi < s_lo) continue;
    hipLaunchKernelGGL(k_chase<E>, dim3((unsigned)(s_hi - s_lo + 1)), dim3(512), 0, st, A, lda,
                       n, nb, t, s_lo, hh, tau);
  }
  const unsigned g = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_diag_out<E>, dim3(g), dim3(256), 0, st, (const E*)A, lda, n, d, e,
                     (const int*)nullptr);
  return hipGetLastError() == hipSuccess ? ELPA_OK : ELPA_ERR_DEVICE;
}

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

}  // namespace eb2t

extern "C" int elpa_band_to_tridiag_gather(int64_t n, int64_t nbw, void* A, int64_t lda,
                                           double* d, double* e, void* hh, void* tau,
                                           int32_t dtype, void* stream, int64_t gather_ticks) {
  if (dtype != ELPA_R64 && dtype != ELPA_C64) return ELPA_ERR_DTYPE;
  if (n < 1 || nbw < 1 || nbw > eb2t::kMaxNb || lda < n) return ELPA_ERR_ARG;
  if (!A || !d || (n > 1 && (!e || !hh || !tau))) return ELPA_ERR_ARG;
  const size_t es = dtype == ELPA_C64 ? 16 : 8;
  if (!eb2t::aligned(A, es) || !eb2t::aligned(d, 8) || (n > 1 && (!eb2t::aligned(e, 8) ||
      !eb2t::aligned(hh, es) || !eb2t::aligned(tau, es))))
    return ELPA_ERR_ALIGN;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (dtype == ELPA_R64)
    return eb2t::run<double>(n, nbw, (double*)A, lda, d, e, (double*)hh, (double*)tau, st,
                             gather_ticks);
  return eb2t::run<ehh::z64>(n, nbw, (ehh::z64*)A, lda, d, e, (ehh::z64*)hh, (ehh::z64*)tau,
                             st, gather_ticks);
}

extern "C" int elpa_band_to_tridiag(int64_t n, int64_t nbw, void* A, int64_t lda, double* d,
                                    double* e, void* hh, void* tau, int32_t dtype,
                                    void* stream) {
  return elpa_band_to_tridiag_gather(n, nbw, A, lda, d, e, hh, tau, dtype, stream,
                                     eb2t::kGatherTicks);
}
