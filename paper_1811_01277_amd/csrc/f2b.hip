// Full -> band reduction (C ABI in include/elpa_f2b.h; Kus et al., Sec. 2).
//
// Panel p: the m = n-p-nbw rows below the band of columns [p, p+nbw) get a
// Householder QR, one column at a time.  Bands up to 64 wide do a panel in one
// launch (k_panel below).  Wider ones spread each column over G workgroups of
// 256 rows, two launches per column and no waiting between workgroups:
//   reflect(i): every workgroup sums the G partial norms of column p+i in a
//     fixed order and derives the same larfg result (tau, beta, scale); it
//     scales its rows of the column into V (zeros above the unit lead) and
//     writes its partial products conj(v)^T A[:, p+j] for the panel's later
//     columns;
//   update(i): every workgroup sums those partials in a fixed order, applies
//     the reflector to its rows of the later columns, writes beta and the
//     zeros of column p+i, and the partial norms of column p+i+1.
// The panel is then mirrored into the rows above (Hermitian storage), and the
// trailing matrix A22 = A[p+nbw:, p+nbw:] is updated from both sides with the
// panel's compact-WY product Q = I - V T V^H, T = M^{-1} diag(tau),
// M = I + diag(tau) striu(V^H V), in the symmetric two-sided form:
//   X = A22 V T,  Y = T^H (V^H X),  W = X - V Y / 2,
//   Q^H A22 Q = A22 - V W^H - W V^H   (one product with inner dimension 2k),
// as GEMMs and triangular solves on the matrix cores (rocBLAS); with up to 64
// reflectors T and Y come from one small kernel instead (k_small_factors).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "../../include/elpa_f2b.h"
#include "../../include/elpa_hh.h"
#include "lane_ops.h"
#include "wy_blas.h"

namespace ef2b {

using ebt::Blas;
using ebt::Num;
using ebt::zc;

__device__ __forceinline__ double conj_(double a) { return a; }
__device__ __forceinline__ zc conj_(zc a) { return zc{a.re, -a.im}; }
__device__ __forceinline__ double sub(double a, double b) { return a - b; }
__device__ __forceinline__ zc sub(zc a, zc b) { return zc{a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ double abs2(double a) { return a * a; }
__device__ __forceinline__ double abs2(zc a) { return a.re * a.re + a.im * a.im; }
__device__ __forceinline__ double re(double a) { return a; }
__device__ __forceinline__ double re(zc a) { return a.re; }
__device__ __forceinline__ double im(double) { return 0.0; }
__device__ __forceinline__ double im(zc a) { return a.im; }
template <typename E>
__device__ __forceinline__ E from_re(double x) {
  if constexpr (std::is_same<E, double>::value)
    return x;
  else
    return zc{x, 0.0};
}

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1) x += __shfl_xor(x, w, 64);
  return x;
}
__device__ __forceinline__ zc wave_sum(zc x) { return zc{wave_sum(x.re), wave_sum(x.im)}; }

constexpr int kRows = 256;  // panel rows per workgroup (one per thread)
constexpr int kMaxNb = 256;

// sum over the workgroup's threads (4 waves); every thread gets the total
template <typename T>
__device__ __forceinline__ T block_sum(T x, T* red) {
  x = wave_sum(x);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = x;
  __syncthreads();
  T t = red[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) t = Num<T>::add(t, red[w]);
  return t;
}

// partial norms sum |A[r0+row, col]|^2 over the group's rows with row > i
template <typename E>
__global__ __launch_bounds__(kRows) void k_pnorm(const E* __restrict__ A, int64_t lda, int64_t r0,
                                                 int64_t col, int64_t m, int64_t i,
                                                 double* __restrict__ pn) {
  __shared__ double red[4];
  const int64_t row = (int64_t)blockIdx.x * kRows + threadIdx.x;
  const double x = (row < m && row > i) ? abs2(A[r0 + row + col * lda]) : 0.0;
  const double t = block_sum(x, red);
  if (threadIdx.x == 0) pn[blockIdx.x] = t;
}

// larfg of column p+i from the partial norms, called by a whole wave: the
// lanes add the partials in a fixed order (lane l takes l, l+64, ...; then a
// butterfly), so every workgroup derives the same (tau, beta, scale)
template <typename E>
__device__ __forceinline__ void larfg_from(const E* __restrict__ A, int64_t lda, int64_t r0,
                                           int64_t p, int64_t i, int G,
                                           const double* __restrict__ pn, E* tau_out,
                                           double* beta_out, E* scale_out) {
  double part = 0.0;
  for (int g = (int)(threadIdx.x & 63); g < G; g += 64) part += pn[g];
  const double sum = wave_sum(part);
  const E alpha = A[r0 + i + (p + i) * lda];
  const double ar = re(alpha), ai = im(alpha);
  if (sum == 0.0 && ai == 0.0) {
    *tau_out = from_re<E>(0.0);
    *beta_out = ar;
    *scale_out = from_re<E>(1.0);
    return;
  }
  const double h = sqrt(ar * ar + ai * ai + sum);
  const double bt = (ar >= 0.0) ? -h : h;
  if constexpr (std::is_same<E, double>::value) {
    *tau_out = (bt - ar) / bt;
    *scale_out = 1.0 / (alpha - bt);
  } else {
    *tau_out = zc{(bt - ar) / bt, -ai / bt};
    const zc den{alpha.re - bt, alpha.im};
    const double dd = den.re * den.re + den.im * den.im;
    *scale_out = zc{den.re / dd, -den.im / dd};
  }
  *beta_out = bt;
}

template <typename E>
__global__ __launch_bounds__(kRows) void k_reflect(const E* __restrict__ A, int64_t lda,
                                                   int64_t r0, int64_t p, int64_t m, int64_t b,
                                                   int64_t i, int G, const double* __restrict__ pn,
                                                   E* __restrict__ V, int64_t ldv,
                                                   E* __restrict__ tau, E* __restrict__ pd) {
  __shared__ E sh[2];
  __shared__ E wred[kRows / 64][kMaxNb];
  if (threadIdx.x < 64) {
    E t, s;
    double beta;
    larfg_from(A, lda, r0, p, i, G, pn, &t, &beta, &s);
    if (threadIdx.x == 0) {
      sh[0] = t;
      sh[1] = s;
      if (blockIdx.x == 0) tau[p + i] = t;
    }
  }
  __syncthreads();
  const E sc = sh[1];
  const int64_t row = (int64_t)blockIdx.x * kRows + threadIdx.x;
  E v = from_re<E>(0.0);
  if (row < m) {
    if (row > i)
      v = Num<E>::mul(A[r0 + row + (p + i) * lda], sc);
    else if (row == i)
      v = from_re<E>(1.0);
    V[r0 + row + (p + i) * ldv] = v;  // zeros above the unit lead
  }
  // partial products conj(v)^T A[:, p+j]: every wave reduces all columns with
  // shuffles (no barrier between columns, so their loads overlap), then the
  // four waves' sums are added in a fixed order
  const E cv = conj_(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool own = row < m && row >= i;
  // eight columns' values loaded before any is reduced, so their loads are
  // in flight together
  constexpr int CH = 8;
  for (int64_t j0 = i + 1; j0 < b; j0 += CH) {
    E x[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u)
      x[u] = (own && j0 + u < b) ? A[r0 + row + (p + j0 + u) * lda] : from_re<E>(0.0);
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const E t = wave_sum(Num<E>::mul(cv, x[u]));
      if (lane == 0 && j0 + u < b) wred[wave][j0 + u] = t;
    }
  }
  __syncthreads();
  for (int64_t j = i + 1 + threadIdx.x; j < b; j += blockDim.x) {
    E t = wred[0][j];
    for (int w = 1; w < kRows / 64; ++w) t = Num<E>::add(t, wred[w][j]);
    pd[(int64_t)blockIdx.x * b + j] = t;
  }
}

template <typename E>
__global__ __launch_bounds__(kRows) void k_update(E* __restrict__ A, int64_t lda, int64_t r0,
                                                  int64_t p, int64_t m, int64_t b, int64_t i,
                                                  int G, const E* __restrict__ V, int64_t ldv,
                                                  const E* __restrict__ tau,
                                                  const double* __restrict__ pn_in,
                                                  const E* __restrict__ pd,
                                                  double* __restrict__ pn_out, int64_t k) {
  __shared__ E coef[kMaxNb];
  __shared__ double shb;
  __shared__ double red[4];
  const E ct = conj_(tau[p + i]);
  // coef[j] = conj(tau) sum_g pd[g][j]: one wave per column, lanes over the
  // partials in a fixed order
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int64_t j = i + 1 + wave; j < b; j += kRows / 64) {
    E w = from_re<E>(0.0);
    for (int g = lane; g < G; g += 64) w = Num<E>::add(w, pd[(int64_t)g * b + j]);
    w = wave_sum(w);
    if (lane == 0) coef[j] = Num<E>::mul(ct, w);
  }
  if (threadIdx.x < 64) {
    E t, s;
    double beta;
    larfg_from(A, lda, r0, p, i, G, pn_in, &t, &beta, &s);
    if (threadIdx.x == 0) shb = beta;
  }
  __syncthreads();
  const int64_t row = (int64_t)blockIdx.x * kRows + threadIdx.x;
  if (row < m && row >= i) {
    const E v = (row == i) ? from_re<E>(1.0) : V[r0 + row + (p + i) * ldv];
    // eight columns loaded before any is written back: the stores could
    // alias the next loads as far as the compiler knows, which would
    // otherwise serialise every column's load behind the previous store
    constexpr int CH = 8;
    for (int64_t j0 = i + 1; j0 < b; j0 += CH) {
      E a[CH];
#pragma unroll
      for (int u = 0; u < CH; ++u)
        if (j0 + u < b) a[u] = A[r0 + row + (p + j0 + u) * lda];
#pragma unroll
      for (int u = 0; u < CH; ++u)
        if (j0 + u < b) A[r0 + row + (p + j0 + u) * lda] = sub(a[u], Num<E>::mul(v, coef[j0 + u]));
    }
    A[r0 + row + (p + i) * lda] = (row == i) ? from_re<E>(shb) : from_re<E>(0.0);
  }
  if (i + 1 < k) {  // partial norms of the next column, rows > i+1
    const double x = (row < m && row > i + 1) ? abs2(A[r0 + row + (p + i + 1) * lda]) : 0.0;
    const double t = block_sum(x, red);
    if (threadIdx.x == 0) pn_out[blockIdx.x] = t;
  }
}

// ---------------------------------------------------------------------------
// nb <= 64: a panel in one launch
//
// A workgroup of four waves keeps 64 RT rows of the panel in registers from
// its first column to its last: lane l holds rows l + 64 t (t < RT), wave w
// the columns 4 c + w (c < CW).  Per column i:
//   1. the wave that holds column i hands it to the others through LDS;
//   2. every wave forms the products S_j = sum over rows > i of conj(x) a_j
//      with the column as it is, not yet scaled to a reflector.  With the row i
//      itself (the head) they give the norm for larfg (S_i) and, since
//      v = (1, sc x), the update's coefficients v^H a_j = a_ij + conj(sc) S_j:
//      one exchange between workgroups per column, and no norm is downdated;
//   3. the workgroups' sums are exchanged and added in one fixed order, so all
//      derive the same bits;
//   4. larfg, update in registers; a column that has been reduced drops out by
//      writing the wave's updated columns one place further left.
//
// The exchange.  A sum goes out as two (real) or four (complex) 8-byte words,
// each half of a double and a tag that counts the columns of the call; a
// reader takes a word when its tag is the column's, so no flag or fence is
// needed.  Two sets of slots alternate: a workgroup writes a slot again two
// columns later, after it has read every other workgroup's sums of the column
// in between, which those send after they have read this slot.
//
// Waiting ends because all workgroups of the launch are resident together:
// each first registers, and only when all have done so does any of them start
// (state kGo).  Should they not come together within a millisecond (the device
// full of other work), the launch leaves the panel as it was (state kApart) and
// k_panel_crew, next on the stream, does it with as many workgroups as there is
// room for and the same arithmetic.  Panels of more workgroups than the device
// holds at all take the two launches per column.
//
// Bound: latency, about two microseconds a column for any number of rows up to
// kMaxGroups workgroups, half of it the exchange.  Two launches per column (a
// norm, then the coefficients; 12.5 and 9 us) took 21.5 us: the
// reduction went from 22.6 to 4.7 ms at n = 1000 and from 100 to 28 ms at
// n = 4000 (nbw = 64, fp64).
// ---------------------------------------------------------------------------
constexpr int kOpen = 0, kGo = 1, kApart = 2;
constexpr int64_t kSmall = 64;  // reflectors of k_small_factors
constexpr int kCtl = 32;  // words before the slots
constexpr int kMaxGroups = 256;               // every workgroup reads every other's sums
constexpr int64_t kGatherTicks = 100000;      // 1 ms of the 100 MHz clock, some five panels
constexpr int64_t kCrewTicks = 10000;         // 0.1 ms
constexpr int kClosed = 1 << 30;              // of a crew's count
constexpr int64_t kWaitTicks = int64_t(20) * 100000000;  // never reached once all are resident

using elane::dpp_mov;
using elane::kHalfMirror;
using elane::kRor8;
using elane::kXor1;
using elane::kXor2;
using elane::pair16;
using elane::pair32;
using elane::read_lane;

// pair32's sums for groups of 8 and of 4 lanes within a row of 16
template <int CTRL, int BIT>
__device__ __forceinline__ double pair_dpp(double a, double b) {
  const bool up = (threadIdx.x & BIT) != 0;
  return (up ? b : a) + dpp_mov<CTRL>(up ? a : b);
}
// x[0..CW) per lane -> lane l: the wave's sum of x[l / (64 / CW)]
template <int CW>
__device__ __forceinline__ double wave_sums(const double (&x)[CW]) {
  static_assert(CW == 8 || CW == 16, "8 or 16 columns per wave");
  double y[CW / 2], z[CW / 4];
#pragma unroll
  for (int i = 0; i < CW / 2; ++i) y[i] = pair32(x[i], x[i + CW / 2]);
#pragma unroll
  for (int i = 0; i < CW / 4; ++i) z[i] = pair16(y[i], y[i + CW / 4]);
  double t;
  if constexpr (CW == 16) {
    const double u0 = pair_dpp<kRor8, 8>(z[0], z[2]), u1 = pair_dpp<kRor8, 8>(z[1], z[3]);
    t = pair_dpp<kHalfMirror, 4>(u0, u1);
  } else {
    t = pair_dpp<kRor8, 8>(z[0], z[1]);
    t += dpp_mov<kHalfMirror>(t);
  }
  t += dpp_mov<kXor2>(t);
  return t + dpp_mov<kXor1>(t);
}
template <int CW>
__device__ __forceinline__ zc wave_sums(const zc (&x)[CW]) {
  double a[CW], b[CW];
#pragma unroll
  for (int i = 0; i < CW; ++i) {
    a[i] = x[i].re;
    b[i] = x[i].im;
  }
  return zc{wave_sums<CW>(a), wave_sums<CW>(b)};
}
// sum over the 64 / CW lanes that share a column, each with its own part
template <int CW>
__device__ __forceinline__ double lane_sum(double t) {
  if constexpr (CW == 8) t += dpp_mov<kHalfMirror>(t);
  t += dpp_mov<kXor2>(t);
  return t + dpp_mov<kXor1>(t);
}
template <int CW>
__device__ __forceinline__ zc lane_sum(zc t) {
  return zc{lane_sum<CW>(t.re), lane_sum<CW>(t.im)};
}
__device__ __forceinline__ zc read_lane(zc x, int l) {
  return zc{read_lane(x.re, l), read_lane(x.im, l)};
}

// Products with every rounding written out, so that all forms of a panel give the
// same bits: acc + conj(x) a, y - v w, a b.
__device__ __forceinline__ double dot_step(double x, double a, double acc) {
  return __builtin_fma(x, a, acc);
}
__device__ __forceinline__ zc dot_step(zc x, zc a, zc acc) {
  return zc{__builtin_fma(x.re, a.re, __builtin_fma(x.im, a.im, acc.re)),
            __builtin_fma(x.re, a.im, __builtin_fma(-x.im, a.re, acc.im))};
}
__device__ __forceinline__ double update(double y, double v, double w) {
  return __builtin_fma(-v, w, y);
}
__device__ __forceinline__ zc update(zc y, zc v, zc w) {
  return zc{__builtin_fma(-v.re, w.re, __builtin_fma(v.im, w.im, y.re)),
            __builtin_fma(-v.re, w.im, __builtin_fma(-v.im, w.re, y.im))};
}
__device__ __forceinline__ double times(double a, double b) { return a * b; }
__device__ __forceinline__ zc times(zc a, zc b) { return update(zc{0.0, 0.0}, zc{-a.re, -a.im}, b); }

typedef unsigned long long u64;
// a value as tagged words (2 per double)
__device__ __forceinline__ void send(u64* p, double x, unsigned tag) {
  const u64 t = (u64)tag << 32;
  __hip_atomic_store(p, t | (unsigned)__double2loint(x), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(p + 1, t | (unsigned)__double2hiint(x), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void send(u64* p, zc x, unsigned tag) {
  send(p, x.re, tag);
  send(p + 2, x.im, tag);
}
template <int NWORD>
struct Words {
  u64 w[NWORD];
  __device__ __forceinline__ void load(const u64* p) {
#pragma unroll
    for (int i = 0; i < NWORD; ++i)
      w[i] = __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ bool has(unsigned tag) const {
    bool ok = true;
#pragma unroll
    for (int i = 0; i < NWORD; ++i) ok = ok && (unsigned)(w[i] >> 32) == tag;
    return ok;
  }
  // The wait is given up after `limit` ticks; the lane's later ones end at the
  // first miss then (limit -1).
  __device__ __forceinline__ void wait(const u64* p, unsigned tag, int64_t& limit) {
    if (has(tag)) return;
    const int64_t t0 = (int64_t)wall_clock64();
    do {
      load(p);
      if (has(tag)) return;
    } while ((int64_t)wall_clock64() - t0 < limit);
    limit = -1;
  }
  __device__ __forceinline__ void get(double& x) const {
    x = __hiloint2double((int)(unsigned)w[1], (int)(unsigned)w[0]);
  }
  __device__ __forceinline__ void get(zc& x) const {
    x.re = __hiloint2double((int)(unsigned)w[1], (int)(unsigned)w[0]);
    x.im = __hiloint2double((int)(unsigned)w[NWORD - 1], (int)(unsigned)w[NWORD - 2]);
  }
};

// larfg of (alpha, tail) from alpha and the tail's squared norm
template <typename E>
__device__ __forceinline__ void larfg(E alpha, double ss, E* tau, double* beta, E* sc) {
  const double ar = re(alpha), ai = im(alpha);
  *tau = from_re<E>(0.0);
  *beta = ar;
  *sc = from_re<E>(1.0);
  if (ss == 0.0 && ai == 0.0) return;
  const double h = sqrt(ar * ar + ai * ai + ss);
  const double bt = ar >= 0.0 ? -h : h;
  if constexpr (std::is_same<E, double>::value) {
    *tau = (bt - ar) / bt;
    *sc = 1.0 / (ar - bt);
  } else {
    *tau = zc{(bt - ar) / bt, -ai / bt};
    const double dr = ar - bt, dd = dr * dr + ai * ai;
    *sc = zc{dr / dd, -ai / dd};
  }
  *beta = bt;
}

// Geometry of one panel and the exchange's memory.
template <typename E>
struct Panel {
  E* A;
  int64_t lda, r0, p, m;
  int b, k;  // columns, reflectors
  E* V;
  int64_t ldv;
  E* tau;
  u64* slots;   // [2][groups + 1][4 CW][words]: the groups' sums, then the head row;
                // before them kCtl words: whether a wait was given up, their limit
  int* state;   // arrived, state, crew's count
  int groups;
  unsigned tag0;
  int64_t gather_ticks;
};

template <typename E>
struct PanelTraits {
  static constexpr int RT = std::is_same<E, double>::value ? 4 : 2;  // rows per lane
  static constexpr int NWORD = std::is_same<E, double>::value ? 2 : 4;
  static constexpr int ROWS = 64 * RT;
};

template <typename E, int CW>
__device__ __forceinline__ u64* slot_of(const Panel<E>& P, unsigned tag, int g, int at) {
  constexpr int NWORD = PanelTraits<E>::NWORD;
  return P.slots + (((int64_t)(tag & 1) * (P.groups + 1) + g) * (4 * CW) + at) * NWORD;
}

__global__ __launch_bounds__(256) void k_panel_clear(u64* __restrict__ slots, int64_t words,
                                                     int* __restrict__ state, int64_t states,
                                                     int open, int64_t limit) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words;
       i += (int64_t)gridDim.x * blockDim.x)
    slots[i] = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < states;
       i += (int64_t)gridDim.x * blockDim.x)
    state[i] = (i & 3) == 1 ? open : 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    slots[-kCtl] = 0;
    slots[-kCtl + 1] = (u64)limit;
  }
}

// A call in which a wait was given up has no result: tau and the band's diagonal
// are set to NaN.
template <typename E>
__global__ __launch_bounds__(256) void k_failed_out(E* __restrict__ A, int64_t lda, int64_t n,
                                                    E* __restrict__ tau, int64_t N,
                                                    const u64* __restrict__ failed) {
  if (*failed == 0) return;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    A[i + i * lda] = from_re<E>(__builtin_nan(""));
    if (i < N) tau[i] = from_re<E>(__builtin_nan(""));
  }
}

// One wave's share of a workgroup's sums for one column: x its rows of the
// column (zero in the rows up to i).
template <typename E, int RT, int CW>
__device__ __forceinline__ E panel_sums(const E (&a)[RT][CW], const E (&x)[RT]) {
  E p[CW];
#pragma unroll
  for (int c = 0; c < CW; ++c) {
    p[c] = from_re<E>(0.0);
#pragma unroll
    for (int t = 0; t < RT; ++t) p[c] = dot_step(x[t], a[t][c], p[c]);
  }
  return wave_sums<CW>(p);
}

// The sums of all groups and, for those without the head row, its entry: lane
// (column, part) adds the groups part, part + SUB, ...; a batch of loads in flight
// at once.
template <typename E, int CW>
__device__ __forceinline__ void panel_gather(const Panel<E>& P, unsigned tag, int at, int part,
                                             bool far, E& S, E& head, int64_t& limit) {
  constexpr int NWORD = PanelTraits<E>::NWORD, SUB = 64 / CW, U = 4;
  const int G = P.groups;
  Words<NWORD> hw;
  if (far) hw.load(slot_of<E, CW>(P, tag, G, at));
  E acc = from_re<E>(0.0);
  for (int g0 = part; g0 < G; g0 += U * SUB) {
    Words<NWORD> w[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (g0 + u * SUB < G) w[u].load(slot_of<E, CW>(P, tag, g0 + u * SUB, at));
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (g0 + u * SUB < G) {
        w[u].wait(slot_of<E, CW>(P, tag, g0 + u * SUB, at), tag, limit);
        E y;
        w[u].get(y);
        acc = Num<E>::add(acc, y);
      }
  }
  S = lane_sum<CW>(acc);
  if (far) {
    hw.wait(slot_of<E, CW>(P, tag, G, at), tag, limit);
    hw.get(head);
  }
}

template <typename E, int CW>
__global__ __launch_bounds__(256, 1) void k_panel(Panel<E> P) {
  constexpr int RT = PanelTraits<E>::RT, ROWS = PanelTraits<E>::ROWS;
  constexpr int SUB = 64 / CW;  // lanes per column
  __shared__ E xs[ROWS];
  __shared__ E sh[2];
  __shared__ int sh_state;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = P.groups, grp = (int)blockIdx.x;
  const int64_t row0 = (int64_t)grp * ROWS;
  const int cl = lane / SUB, part = lane % SUB;

  if (G > 1) {
    if (tid == 0) {
      int st = __hip_atomic_load(P.state + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (P.slots[-kCtl] != 0) st = kApart;  // an earlier panel failed: no more
      if (st == kOpen) {
        const int old = __hip_atomic_fetch_add(P.state, 1, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
        int expect = kOpen;
        if (old == G - 1)
          __hip_atomic_compare_exchange_strong(P.state + 1, &expect, kGo, __ATOMIC_RELAXED,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int64_t t0 = (int64_t)wall_clock64();
        while ((st = __hip_atomic_load(P.state + 1, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT)) == kOpen) {
          if ((int64_t)wall_clock64() - t0 > P.gather_ticks) {
            expect = kOpen;
            __hip_atomic_compare_exchange_strong(P.state + 1, &expect, kApart, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      }
      sh_state = st;
    }
    __syncthreads();
    if (sh_state != kGo) return;
  }

  E a[RT][CW];
#pragma unroll
  for (int c = 0; c < CW; ++c)
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int64_t row = row0 + lane + 64 * t;
      const int j = 4 * c + wave;
      a[t][c] = (row < P.m && j < P.b) ? P.A[P.r0 + row + (P.p + j) * P.lda] : from_re<E>(0.0);
    }

  int gone = 0;  // of this wave's columns
  int64_t limit = (int64_t)P.slots[-kCtl + 1];
  for (int i = 0; i < P.k; ++i) {
    const bool own = (i & 3) == wave;
    const unsigned tag = P.tag0 + (unsigned)i;
    if (own) {
#pragma unroll
      for (int t = 0; t < RT; ++t) xs[lane + 64 * t] = a[t][0];
    }
    __syncthreads();
    E x[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      x[t] = xs[lane + 64 * t];
      if (row0 + lane + 64 * t <= i) x[t] = from_re<E>(0.0);
    }
    // sums of column 4 (cl + gone) + wave, the same in the SUB lanes of cl
    E S = panel_sums<E, RT, CW>(a, x), head = from_re<E>(0.0);
    if (grp == 0) {
      // row i is lane i's first row (i < 64)
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const E hc = read_lane(a[0][c], i);
        if (cl == c) head = hc;
      }
    }
    if (G > 1) {
      const int at = wave * CW + cl;
      if (part == 0) send(slot_of<E, CW>(P, tag, grp, at), S, tag);
      if (grp == 0 && part == 1) send(slot_of<E, CW>(P, tag, G, at), head, tag);
      panel_gather<E, CW>(P, tag, at, part, grp != 0, S, head, limit);
    }
    if (own) {  // lane 0 holds column i's sum and head
      E tv, sc;
      double beta;
      larfg(read_lane(head, 0), re(read_lane(S, 0)), &tv, &beta, &sc);
      if (lane == 0) {
        sh[0] = tv;
        sh[1] = sc;
        if (grp == 0) {
          P.tau[P.p + i] = tv;
          P.A[P.r0 + i + (P.p + i) * P.lda] = from_re<E>(beta);
        }
      }
    }
    __syncthreads();
    const E tv = sh[0], sc = sh[1];
    // coefficient of this lane's column: conj(tau) v^H a_j
    const E cw = times(conj_(tv), dot_step(sc, S, head));
    E v[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int64_t row = row0 + lane + 64 * t;
      v[t] = row == i ? from_re<E>(1.0) : times(x[t], sc);
      if (own && row < P.m) P.V[P.r0 + row + (P.p + i) * P.ldv] = v[t];
    }
    // row i of the result (v = 1 there), columns right of i
    if (grp == 0 && part == 0 && !(own && cl == 0)) {
      const int j = 4 * (cl + gone) + wave;
      if (j < P.b) P.A[P.r0 + i + (P.p + j) * P.lda] = sub(head, cw);
    }
    if (own) {
#pragma unroll
      for (int c = 1; c < CW; ++c) {
        const E w = read_lane(cw, c * SUB);
#pragma unroll
        for (int t = 0; t < RT; ++t) a[t][c - 1] = update(a[t][c], v[t], w);
      }
#pragma unroll
      for (int t = 0; t < RT; ++t) a[t][CW - 1] = from_re<E>(0.0);
      ++gone;
    } else {
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const E w = read_lane(cw, c * SUB);
#pragma unroll
        for (int t = 0; t < RT; ++t) a[t][c] = update(a[t][c], v[t], w);
      }
    }
  }
  if (limit < 0) P.slots[-kCtl] = 1;
  // zeros below the diagonal of the reduced columns; a panel with fewer rows
  // than columns has all its rows written above
  int first = lane;
  asm volatile("" : "+v"(first));  // addresses are formed anew, not kept from the loads above
#pragma unroll 1
  for (int j = wave; j < P.b; j += 4)
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int64_t row = row0 + first + 64 * t;
      if (row < P.m && row > j) P.A[P.r0 + row + (P.p + j) * P.lda] = from_re<E>(0.0);
    }
}

// The panel by a crew, where k_panel's workgroups did not come together (no work
// otherwise): the workgroups that are there when the last of them or the first
// whose time is up closes the count.  Later ones return, so all of the crew are
// running and their waits end as above.  Workgroup w of c does the groups w,
// w + c, ... with the panel in A: the same sums, sent and added in the same order.
// Per column two passes over the rows.  The reduction at n = 4000 / 12000, nbw = 64,
// fp64, with every panel done this way by as many workgroups as it has groups: 50 /
// 252 ms, where panels together take 19.1 / 152; two launches per column took 100 /
// 468, and all the panels' rows on one workgroup 245 ms at n = 4000.
template <typename E, int CW>
__global__ __launch_bounds__(256, 1) void k_panel_crew(Panel<E> P) {
  constexpr int RT = PanelTraits<E>::RT, ROWS = PanelTraits<E>::ROWS;
  constexpr int SUB = 64 / CW;
  __shared__ E sh[2];
  __shared__ int sh_me, sh_crew;
  if (__hip_atomic_load(P.state + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kGo) return;
  if (P.slots[-kCtl] != 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cl = lane / SUB, part = lane % SUB;
  if (tid == 0) {
    int* const count = P.state + 2;
    int v = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), me = -1;
    while (me < 0 && !(v & kClosed))
      if (__hip_atomic_compare_exchange_strong(count, &v, v + 1, __ATOMIC_RELAXED,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        me = v;
    if (me >= 0) {
      const int64_t t0 = (int64_t)wall_clock64();
      while (!((v = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) &
               kClosed))
        if (v == (int)gridDim.x || (int64_t)wall_clock64() - t0 > kCrewTicks)
          __hip_atomic_fetch_or(count, kClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    sh_me = me;
    sh_crew = v & ~kClosed;
  }
  __syncthreads();
  const int me = __builtin_amdgcn_readfirstlane(sh_me);
  const int crew = __builtin_amdgcn_readfirstlane(sh_crew);
  if (me < 0) return;
  const int at = wave * CW + cl;
  int64_t limit = (int64_t)P.slots[-kCtl + 1];
  for (int i = 0; i < P.k; ++i) {
    const bool own = (i & 3) == wave;
    const int gone = i > wave ? (i - wave + 3) / 4 : 0;
    const unsigned tag = P.tag0 + (unsigned)i;
    const int jl = 4 * (cl + gone) + wave;
    E head = from_re<E>(0.0), S;
    if (me == 0) {
      if (jl < P.b) head = P.A[P.r0 + i + (P.p + jl) * P.lda];
      if (part == 1) send(slot_of<E, CW>(P, tag, P.groups, at), head, tag);
    }
    for (int g = me; g < P.groups; g += crew) {
      E a[RT][CW], x[RT];
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const int64_t row = (int64_t)g * ROWS + lane + 64 * t;
        x[t] = row < P.m && row > i ? P.A[P.r0 + row + (P.p + i) * P.lda] : from_re<E>(0.0);
#pragma unroll
        for (int c = 0; c < CW; ++c) {
          const int j = 4 * (c + gone) + wave;
          a[t][c] = (row < P.m && j < P.b) ? P.A[P.r0 + row + (P.p + j) * P.lda]
                                           : from_re<E>(0.0);
        }
      }
      S = panel_sums<E, RT, CW>(a, x);
      if (part == 0) send(slot_of<E, CW>(P, tag, g, at), S, tag);
    }
    panel_gather<E, CW>(P, tag, at, part, me != 0, S, head, limit);
    double beta = 0.0;
    if (own) {
      E tv, sc;
      larfg(read_lane(head, 0), re(read_lane(S, 0)), &tv, &beta, &sc);
      if (lane == 0) {
        sh[0] = tv;
        sh[1] = sc;
        if (me == 0) P.tau[P.p + i] = tv;
      }
    }
    __syncthreads();
    const E tv = sh[0], sc = sh[1];
    const E cw = times(conj_(tv), dot_step(sc, S, head));
    E w[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) w[c] = read_lane(cw, c * SUB);
    for (int g = me; g < P.groups; g += crew)
#pragma unroll 1
      for (int t = 0; t < RT; ++t) {
        const int64_t row = (int64_t)g * ROWS + lane + 64 * t;
        if (row >= P.m) continue;
        const E x = P.A[P.r0 + row + (P.p + i) * P.lda];
        const E v = row == i ? from_re<E>(1.0) : (row > i ? times(x, sc) : from_re<E>(0.0));
        if (own) P.V[P.r0 + row + (P.p + i) * P.ldv] = v;
        if (row < i) continue;
        E y[CW];
#pragma unroll
        for (int c = 0; c < CW; ++c) {
          const int j = 4 * (c + gone) + wave;
          if (j > i && j < P.b) y[c] = P.A[P.r0 + row + (P.p + j) * P.lda];
        }
#pragma unroll
        for (int c = 0; c < CW; ++c) {
          const int j = 4 * (c + gone) + wave;
          if (j > i && j < P.b)
            P.A[P.r0 + row + (P.p + j) * P.lda] = update(y[c], v, w[c]);
        }
      }
    __syncthreads();
    if (own)
      for (int g = me; g < P.groups; g += crew)
        for (int t = 0; t < RT; ++t) {
          const int64_t row = (int64_t)g * ROWS + lane + 64 * t;
          if (row >= i && row < P.m)
            P.A[P.r0 + row + (P.p + i) * P.lda] = from_re<E>(row == i ? beta : 0.0);
        }
    __syncthreads();
  }
  if (limit < 0) P.slots[-kCtl] = 1;
}

// ---------------------------------------------------------------------------
// trailing update, up to 64 reflectors
// ---------------------------------------------------------------------------
// B = [V | W | V | Z] (m rows, ld mp, k columns each; rows m .. mp of the last
// two zero), Z = A22 V, GS = V^H [V | Z].  Then T from the first half of GS, Y =
// T^H (V^H Z) T and W = [V | Z] [-Y / 2; T] = A22 V T - V Y / 2, and A22 takes
// one product of the first half of B with its middle.  Four products, where
// the general order (below) has five, two triangular solves (each an inversion
// of diagonal blocks in launches of its own), two scalings and three copies: at
// n = 4000, nbw = 64 an update took 245 us on average with those and takes 108
// (all of f2b: 27.9 -> 19.4 ms; n = 1000: 4.6 -> 3.4; complex, n = 700, nbw = 32:
// 6.6 -> 3.7).

// The panel mirrored into the rows above, V into both its places, zeros.
template <typename E>
__global__ __launch_bounds__(256) void k_panel_out(E* __restrict__ A, int64_t lda, int64_t r0,
                                                   int64_t p, int64_t m, int64_t k, int64_t mp,
                                                   const E* __restrict__ V, int64_t ldv,
                                                   E* __restrict__ B) {
  const int64_t j = blockIdx.y;
  for (int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; row < mp;
       row += (int64_t)gridDim.x * blockDim.x) {
    if (row < m) A[p + j + (r0 + row) * lda] = conj_(A[r0 + row + (p + j) * lda]);
    if (j < k) {
      const E v = row < m ? V[r0 + row + (p + j) * ldv] : from_re<E>(0.0);
      B[row + j * mp] = v;
      B[row + (2 * k + j) * mp] = v;
      if (row >= m) B[row + (3 * k + j) * mp] = v;
    }
  }
}

// K chunks of Z = A22 V: its m / 64 output tiles fill a quarter of the device at
// m = 4000 (144 us in one product, 40 in eight chunks); at most 8, of 128
// columns or more, and about 512 tiles in all.
inline int64_t zsplit(int64_t m) {
  return std::max<int64_t>(1, std::min<int64_t>({8, m / 128, 512 / ((m + 63) / 64)}));
}

// Z = the sum of `chunks` partial products of kc columns of A22 each (m x k, in
// a fixed order) and the columns of A22 past them (fewer than chunks)
template <typename E>
__global__ __launch_bounds__(256) void k_sum_z(const E* __restrict__ part, int64_t chunks,
                                               int64_t kc, const E* __restrict__ A22, int64_t lda,
                                               const E* __restrict__ V, int64_t m, int64_t k,
                                               int64_t mp, E* __restrict__ Z) {
  const int64_t c = blockIdx.y;
  for (int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; row < m;
       row += (int64_t)gridDim.x * blockDim.x) {
    E acc = part[row + c * m];
    for (int64_t s = 1; s < chunks; ++s) acc = Num<E>::add(acc, part[s * m * k + row + c * m]);
    for (int64_t l = chunks * kc; l < m; ++l)
      acc = Num<E>::add(acc, Num<E>::mul(A22[row + l * lda], V[l + c * mp]));
    Z[row + c * mp] = acc;
  }
}

// C (2 k x k) = [-Y / 2; T] for k <= 64, one workgroup.  T by halves: the
// diagonal blocks of 16 by the forward recurrence, T_ii = tau_i, T[0:i, i] =
// -tau_i T[0:i, 0:i] G[0:i, i], a lane to a row; a block beside two of them as
// -T1 (G12 T2), and the two products of Y, on the matrix cores.  An MFMA result
// is the second operand of the next product as it lies in its registers (row q
// + 4 r of lane quad q, register r).  Planes of complex values apart.
// Bound: a chain of dependent products and LDS reads on one compute unit, 13 us
// (real); with the products in plain loops 29.
template <typename E>
__global__ __launch_bounds__(256) void k_small_factors(const E* __restrict__ GS,
                                                       const E* __restrict__ tau, int k,
                                                       E* __restrict__ C) {
  constexpr int PL = ebt::Planes<E>::PL, N = 64, LD = N + 1, I = PL - 1;
  using ebt::d4;
  __shared__ double G[PL][N * LD], T[PL][N * LD];
  const int tid = (int)threadIdx.x, lane = tid & 63, q = lane >> 4, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  E g[16], s[16];  // entries lane of columns wave, wave + 4, ...
#pragma unroll
  for (int x = 0; x < 16; ++x) {
    const int c = wave + 4 * x;
    const bool ok = lane < k && c < k;
    g[x] = ok ? GS[lane + (int64_t)c * k] : from_re<E>(0.0);
    s[x] = ok ? GS[lane + (int64_t)(k + c) * k] : from_re<E>(0.0);
  }
  E tk = lane < k ? tau[lane] : from_re<E>(0.0);
  auto put = [&](const E (&v)[16]) {
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      double y[2];
      ebt::split(v[x], &y[0], &y[1]);
#pragma unroll
      for (int p = 0; p < PL; ++p) G[p][lane * LD + wave + 4 * x] = y[p];
    }
  };
  put(g);
#pragma unroll
  for (int p = 0; p < PL; ++p)
#pragma unroll
    for (int x = 0; x < 16; ++x) T[p][lane * LD + wave + 4 * x] = 0.0;
  __syncthreads();
  double ty[2];
  ebt::split(tk, &ty[0], &ty[1]);
  ebt::tri_factor64<PL>(G, T, ty, wave, lane);
  put(s);
  __syncthreads();
  using ebt::mac;
  // this wave's 16 columns of U = S T, then of Y = T^H U
  d4 u[4][PL], y[4][PL];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int p = 0; p < PL; ++p) u[rt][p] = y[rt][p] = d4{0, 0, 0, 0};
  const int col = 16 * wave + c16;
#pragma unroll 4
  for (int kk = 0; kk < 16; ++kk) {
    const int l = 4 * kk + q;
    const double br = T[0][l * LD + col], bi = T[I][l * LD + col];
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
      const int at = (16 * rt + c16) * LD + l;
      mac(G[0][at], G[I][at], br, bi, u[rt]);
    }
  }
#pragma unroll
  for (int kk = 0; kk < 16; ++kk) {
    const int l = 4 * kk + q;
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
      if (kk / 4 > rt) continue;  // T is upper triangular
      const int at = l * LD + 16 * rt + c16;
      mac(T[0][at], -T[I][at], u[kk / 4][0][kk % 4], u[kk / 4][I][kk % 4], y[rt]);
    }
  }
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * rt + q + 4 * r;
      if (i >= k || col >= k) continue;
      double a[PL], t[PL];
#pragma unroll
      for (int p = 0; p < PL; ++p) {
        a[p] = -0.5 * y[rt][p][r];
        t[p] = T[p][i * LD + col];
      }
      C[i + (int64_t)col * 2 * k] = ebt::join<E>(a);
      C[k + i + (int64_t)col * 2 * k] = ebt::join<E>(t);
    }
}

// A[p+j, r0+row] = conj(A[r0+row, p+j]) for the panel
template <typename E>
__global__ __launch_bounds__(256) void k_mirror(E* __restrict__ A, int64_t lda, int64_t r0,
                                                int64_t p, int64_t m, int64_t b) {
  const int64_t j = blockIdx.y;
  for (int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; row < m;
       row += (int64_t)gridDim.x * blockDim.x)
    A[p + j + (r0 + row) * lda] = conj_(A[r0 + row + (p + j) * lda]);
}

// W (rows x cols, ld) scaled: by_rows: W[r, c] *= conj(tau[r]); else W[r, c] *= tau[c]
template <typename E>
__global__ __launch_bounds__(256) void k_scale(E* __restrict__ W, int64_t ld, int64_t rows,
                                               int64_t cols, const E* __restrict__ tau,
                                               bool by_rows) {
  const int64_t total = rows * cols;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = e % rows, c = e / rows;
    E& w = W[r + c * ld];
    w = Num<E>::mul(by_rows ? conj_(tau[r]) : tau[c], w);
  }
}

template <typename E>
int run(int64_t n, int64_t b, E* A, int64_t lda, E* V, int64_t ldv, E* tau, hipStream_t st,
        int64_t gather_ticks, int64_t wait_ticks, int64_t crew) {
  using S = typename std::conditional<std::is_same<E, float>::value, float, double>::type;
  const size_t es = sizeof(E);
  const int64_t mmax = n - b;
  const int Gmax = (int)((mmax + kRows - 1) / kRows);
  auto al = [](size_t x) { return (x + 255) / 256 * 256; };
  size_t part_e = 0;  // the largest set of K-chunk partial products over the panels
  for (int64_t p = 0; p + b < n; p += b) {
    const int64_t m = n - p - b, k = std::min(b, m);
    part_e = std::max(part_e, (size_t)ebt::ksplit(m, k, k, es) * k * k);
    if (b <= kSmall) part_e = std::max(part_e, (size_t)ebt::ksplit(m, k, 2 * k, es) * 2 * k * k);
    if (b <= kSmall && zsplit(m) > 1) part_e = std::max(part_e, (size_t)zsplit(m) * m * k);
  }
  // (the padded rows of a small update: fewer than its chunks, at most 768)
  const int64_t wrows = b <= kSmall ? mmax + 768 : mmax;
  const size_t off_pn = 0, off_pd = off_pn + al(2 * Gmax * sizeof(double) + 512),
               off_g = off_pd + al((size_t)Gmax * b * es),
               off_m = off_g + al((size_t)2 * b * b * es),
               off_w1 = off_m + al((size_t)2 * b * b * es),
               off_w2 = off_w1 + al((size_t)2 * b * wrows * es),
               off_part = off_w2 + al((size_t)2 * b * wrows * es), off_slot = off_part + al(part_e * es);
  // one-launch panels: their exchange slots and per-panel states
  constexpr int ROWS = PanelTraits<E>::ROWS, NWORD = PanelTraits<E>::NWORD;
  const int64_t groups = b <= 64 ? std::min<int64_t>((mmax + ROWS - 1) / ROWS, kMaxGroups) : 0;
  // the most workgroups of a panel: what an idle device holds at once
  int64_t most = std::min<int64_t>(groups, 1);
  if (groups > 1) {
    const auto panel = b > 32 ? k_panel<E, 16> : k_panel<E, 8>;
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per_cu, reinterpret_cast<const void*>(panel), 256, 0) == hipSuccess)
      most = std::max<int64_t>(1, std::min<int64_t>(groups, (int64_t)cus * per_cu));
  }
  const int64_t words = 2 * (groups + 1) * 64 * NWORD, panels = (n - 1) / b;
  const size_t off_state = off_slot + al((size_t)(kCtl + words) * 8), total = off_state + al((size_t)panels * 16);
  char* ws = nullptr;
  if (hipMallocAsync((void**)&ws, total, st) != hipSuccess) return ELPA_ERR_NOMEM;
  double* pn0 = (double*)(ws + off_pn);
  double* pn1 = pn0 + Gmax;
  E* pd = (E*)(ws + off_pd);
  E* Gm = (E*)(ws + off_g);
  E* M = (E*)(ws + off_m);
  E* W1 = (E*)(ws + off_w1);
  E* W2 = (E*)(ws + off_w2);
  E* part = (E*)(ws + off_part);
  u64* slots = (u64*)(ws + off_slot) + kCtl;
  int* states = (int*)(ws + off_state);
  if (groups > 0)
    hipLaunchKernelGGL(k_panel_clear, dim3((unsigned)std::min<int64_t>((words + 255) / 256, 256)),
                       dim3(256), 0, st, slots, words, states, 4 * panels,
                       gather_ticks < 0 ? kApart : kOpen, wait_ticks);
  int rc = ELPA_OK;
  {
    std::lock_guard<std::mutex> lock(ebt::Handles::get().mu);
    rocblas_handle h = ebt::handle_for(st);
    if (!h) rc = ELPA_ERR_DEVICE;
    const auto N_ = rocblas_operation_none;
    const auto C_ = Blas<E>::adj;
    for (int64_t p = 0; rc == ELPA_OK && p + b < n; p += b) {
      const int64_t r0 = p + b, m = n - r0, k = std::min(b, m);
      const int64_t wide = (m + ROWS - 1) / ROWS;  // workgroups of a one-launch panel
      if (b <= 64 && wide <= most) {
        const Panel<E> P{A,     lda, r0,    p, m, (int)b, (int)k, V, ldv,
                         tau,   slots, states + 4 * (p / b), (int)wide, (unsigned)(p + 1),
                         gather_ticks};
        const dim3 g((unsigned)wide), t(256);
        if (b > 32)
          hipLaunchKernelGGL((k_panel<E, 16>), g, t, 0, st, P);
        else
          hipLaunchKernelGGL((k_panel<E, 8>), g, t, 0, st, P);
        if (wide > 1) {
          const dim3 gc((unsigned)(crew > 0 ? std::min(crew, wide) : wide));
          if (b > 32)
            hipLaunchKernelGGL((k_panel_crew<E, 16>), gc, t, 0, st, P);
          else
            hipLaunchKernelGGL((k_panel_crew<E, 8>), gc, t, 0, st, P);
        }
      } else {
        const int G = (int)((m + kRows - 1) / kRows);
        double* pa = pn0;
        double* pb = pn1;
        hipLaunchKernelGGL(k_pnorm<E>, dim3(G), dim3(kRows), 0, st, (const E*)A, lda, r0, p, m,
                           (int64_t)0, pa);
        for (int64_t i = 0; i < k; ++i) {
          hipLaunchKernelGGL(k_reflect<E>, dim3(G), dim3(kRows), 0, st, (const E*)A, lda, r0, p,
                             m, b, i, G, (const double*)pa, V, ldv, tau, pd);
          hipLaunchKernelGGL(k_update<E>, dim3(G), dim3(kRows), 0, st, A, lda, r0, p, m, b, i, G,
                             (const E*)V, ldv, (const E*)tau, (const double*)pa, (const E*)pd, pb,
                             k);
          std::swap(pa, pb);
        }
      }
      // trailing update with the panel's k reflectors
      const E* Vp = V + r0 + p * ldv;
      E* A22 = A + r0 + r0 * lda;
      const E* tp = tau + p;
      if (b <= kSmall) {
        const int64_t chunks = ebt::ksplit(m, k, 2 * k, es), kc = (m + chunks - 1) / chunks;
        const int64_t mp = kc * chunks;
        E* VZ = W1 + 2 * k * mp;
        hipLaunchKernelGGL(k_panel_out<E>,
                           dim3((unsigned)std::min<int64_t>((mp + 255) / 256, 1024), (unsigned)b),
                           dim3(256), 0, st, A, lda, r0, p, m, k, mp, V, ldv, W1);
        E* Z = VZ + k * mp;
        const int64_t zc_ = zsplit(m), zk = m / zc_;
        bool ok;
        if (zc_ == 1) {
          ok = Blas<E>::gemm(h, N_, N_, m, k, m, S(1), A22, lda, VZ, mp, S(0), Z, mp) ==
               rocblas_status_success;
        } else {
          ok = Blas<E>::gemm_sb(h, N_, N_, m, k, zk, S(1), A22, lda, zk * lda, VZ, mp, zk, S(0),
                                part, m, m * k, zc_) == rocblas_status_success;
          if (ok)
            hipLaunchKernelGGL(k_sum_z<E>, dim3((unsigned)((m + 255) / 256), (unsigned)k),
                               dim3(256), 0, st, (const E*)part, zc_, zk, (const E*)A22, lda,
                               (const E*)VZ, m, k, mp, Z);
        }
        ok = ok && Blas<E>::gemm_sb(h, C_, N_, k, 2 * k, kc, S(1), VZ, mp, kc, VZ, mp, kc, S(0),
                                    part, k, 2 * k * k, chunks) == rocblas_status_success;
        if (ok) {
          hipLaunchKernelGGL(ebt::k_sum_parts<E>, dim3((unsigned)((2 * k * k + 255) / 256)),
                             dim3(256), 0, st, (const E*)part, chunks, 2 * k * k, Gm);
          hipLaunchKernelGGL(k_small_factors<E>, dim3(1), dim3(256), 0, st, (const E*)Gm, tp,
                             (int)k, M);
        }
        ok = ok && Blas<E>::gemm(h, N_, N_, m, k, 2 * k, S(1), VZ, mp, M, 2 * k, S(0), W1 + k * mp,
                                 mp) == rocblas_status_success;
        // A22 -= [V W] [W V]^H: one rank-2k product over both triangles
        ok = ok && Blas<E>::gemm(h, N_, C_, m, m, 2 * k, S(-1), W1, mp, W1 + k * mp, mp, S(1),
                                 A22, lda) == rocblas_status_success;
        if (!ok || hipGetLastError() != hipSuccess) rc = ELPA_ERR_DEVICE;
        continue;
      }
      hipLaunchKernelGGL(k_mirror<E>, dim3((unsigned)std::min<int64_t>((m + 255) / 256, 1024),
                                           (unsigned)b),
                         dim3(256), 0, st, A, lda, r0, p, m, b);
      bool ok = ebt::gemm_adj_splitk<E, S>(h, k, k, m, Vp, ldv, Vp, ldv,
                                           ebt::ksplit(m, k, k, es), part, Gm, st);
      if (ok)
        hipLaunchKernelGGL(ebt::k_unit_tri<E>, dim3((unsigned)((k * k + 255) / 256)), dim3(256),
                           0, st, (const E*)Gm, tp, k, M);
      // X = A22 V T (T = M^{-1} diag(tau)) into the W half of P = [V | W]
      E* Pv = W1;
      E* Pw = W1 + m * k;
      E* Rw = W2;
      E* Rv = W2 + m * k;
      const auto D2D = hipMemcpyDeviceToDevice;
      ok = ok && hipMemcpy2DAsync(Pv, (size_t)m * es, Vp, (size_t)ldv * es, (size_t)m * es,
                                  (size_t)k, D2D, st) == hipSuccess;
      ok = ok && hipMemcpy2DAsync(Rv, (size_t)m * es, Vp, (size_t)ldv * es, (size_t)m * es,
                                  (size_t)k, D2D, st) == hipSuccess;
      ok = ok && Blas<E>::gemm(h, N_, N_, m, k, m, S(1), A22, lda, Vp, ldv, S(0), Pw, m) ==
                     rocblas_status_success;
      ok = ok && Blas<E>::trsm(h, rocblas_side_right, N_, m, k, M, k, Pw, m) ==
                     rocblas_status_success;
      if (ok)
        hipLaunchKernelGGL(k_scale<E>, dim3((unsigned)std::min<int64_t>((k * m + 255) / 256, 4096)),
                           dim3(256), 0, st, Pw, m, m, k, tp, false);
      // Y = T^H V^H X = diag(conj tau) M^{-H} (V^H X), k x k (in Gm)
      ok = ok && ebt::gemm_adj_splitk<E, S>(h, k, k, m, Vp, ldv, Pw, m, ebt::ksplit(m, k, k, es),
                                            part, Gm, st);
      ok = ok && Blas<E>::trsm(h, rocblas_side_left, C_, k, k, M, k, Gm, k) ==
                     rocblas_status_success;
      if (ok)
        hipLaunchKernelGGL(k_scale<E>, dim3((unsigned)((k * k + 255) / 256)), dim3(256), 0, st,
                           Gm, k, k, k, tp, true);
      // W = X - V Y / 2, so that Q^H A22 Q = A22 - V W^H - W V^H
      ok = ok && Blas<E>::gemm(h, N_, N_, m, k, k, S(-0.5), Vp, ldv, Gm, k, S(1), Pw, m) ==
                     rocblas_status_success;
      ok = ok && hipMemcpyAsync(Rw, Pw, (size_t)m * k * es, D2D, st) == hipSuccess;
      // A22 -= [V W] [W V]^H: one rank-2k product over both triangles
      ok = ok && Blas<E>::gemm(h, N_, C_, m, m, 2 * k, S(-1), W1, m, W2, m, S(1), A22, lda) ==
                     rocblas_status_success;
      if (!ok || hipGetLastError() != hipSuccess) rc = ELPA_ERR_DEVICE;
    }
  }
  if (groups > 1) {
    hipLaunchKernelGGL(k_failed_out<E>, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1024)),
                       dim3(256), 0, st, A, lda, n, tau, mmax, (const u64*)(slots - kCtl));
    if (rc == ELPA_OK && hipGetLastError() != hipSuccess) rc = ELPA_ERR_DEVICE;
  }
  const hipError_t e2 = hipFreeAsync(ws, st);
  if (rc == ELPA_OK && e2 != hipSuccess) rc = ELPA_ERR_DEVICE;
  return rc;
}

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

}  // namespace ef2b

extern "C" int elpa_full_to_band_crew(int64_t n, int64_t nbw, void* A, int64_t lda, void* V,
                                      int64_t ldv, void* tau, int32_t dtype, void* stream,
                                      int64_t gather_ticks, int64_t wait_ticks, int64_t crew) {
  if (dtype != ELPA_R64 && dtype != ELPA_C64) return ELPA_ERR_DTYPE;
  if (n < 1 || nbw < 1 || nbw > ef2b::kMaxNb || lda < n || ldv < n) return ELPA_ERR_ARG;
  if (!A) return ELPA_ERR_ARG;
  if (n <= nbw) return ELPA_OK;
  if (!V || !tau) return ELPA_ERR_ARG;
  const size_t es = dtype == ELPA_C64 ? 16 : 8;
  if (!ef2b::aligned(A, es) || !ef2b::aligned(V, es) || !ef2b::aligned(tau, es))
    return ELPA_ERR_ALIGN;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (dtype == ELPA_R64)
    return ef2b::run<double>(n, nbw, (double*)A, lda, (double*)V, ldv, (double*)tau, st,
                             gather_ticks, wait_ticks, crew);
  return ef2b::run<ebt::zc>(n, nbw, (ebt::zc*)A, lda, (ebt::zc*)V, ldv, (ebt::zc*)tau, st,
                            gather_ticks, wait_ticks, crew);
}

extern "C" int elpa_full_to_band_limits(int64_t n, int64_t nbw, void* A, int64_t lda, void* V,
                                        int64_t ldv, void* tau, int32_t dtype, void* stream,
                                        int64_t gather_ticks, int64_t wait_ticks) {
  return elpa_full_to_band_crew(n, nbw, A, lda, V, ldv, tau, dtype, stream, gather_ticks,
                                wait_ticks, 0);
}

extern "C" int elpa_full_to_band_gather(int64_t n, int64_t nbw, void* A, int64_t lda, void* V,
                                        int64_t ldv, void* tau, int32_t dtype, void* stream,
                                        int64_t gather_ticks) {
  return elpa_full_to_band_limits(n, nbw, A, lda, V, ldv, tau, dtype, stream, gather_ticks,
                                  ef2b::kWaitTicks);
}

extern "C" int elpa_full_to_band(int64_t n, int64_t nbw, void* A, int64_t lda, void* V,
                                 int64_t ldv, void* tau, int32_t dtype, void* stream) {
  return elpa_full_to_band_gather(n, nbw, A, lda, V, ldv, tau, dtype, stream,
                                  ef2b::kGatherTicks);
}
