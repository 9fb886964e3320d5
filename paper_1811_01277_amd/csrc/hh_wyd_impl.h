// Compact-WY kernel of the two-lane family's place (path 3) for real fp64: the
// reflectors are read where the caller keeps them, only the triangular
// factors are packed.
//
//     Q <- H(0,0) H(0,1) ... H(n-2, J-1) Q       (Kus et al., Sec. 2, Sec. 3.1)
//
// Blocks of K sweeps slide a window of NB+K rows down a stripe, one chase step
// at a time; a step's K reflectors are applied as K/16 sub-groups
//
//     H(a) ... H(a+15) = I - V T V^T :   W = V^T X,  W' = -T W,  X += V W'
//
// on 16x16x4 fp64 MFMA tiles, the window in registers in the MFMA result
// layout (hh_wy_impl.h has the family that packs (-U)^T = -(V T^T)^T and V
// instead; it needs 2.3 times the space per reflector and a pre-pass to match,
// and saves the four MFMAs of -T W, a tenth of a sub-group's 44 at NB = 64).
//
// Why this and not fp64 FMAs on two lanes per column, which this family used
// to run: both units have the same peak here, but a lone wave issues a vector
// fp64 FMA only every eighth cycle and a 64-reflector step is one long chain
// for it, so problems of a few thousand rows ran at a fifth of the peak; an
// MFMA keeps the unit busy from one wave, and a wave covers 16 columns, so a
// stripe's step is four times shorter.  With the one-launch schedules of
// hh_pipe.h: n = 512, nbw = 32: 426 -> 152 us; n = 1000, nbw = 64: 637 -> 329
// us; n = 8192 with 819 columns: 6.6 -> 4.1 ms; 256 problems of n = 200 ..
// 2000, nbw = 32: 46.8 -> 40.5 ms.  A step of K = 80, NB = 64 takes about
// 10 us on a wave that has its SIMD to itself, 6.8 of them MFMAs (74 cycles
// each from one wave, 65 with two waves per SIMD).
//
// Rows within a 16-row tile: register r of lane quad q holds row 4q + r of the
// tile (an MFMA result's row label q + 4r stands for it), so a lane's four
// contraction rows are consecutive, in a reflector and in a column of Q.
#pragma once

#include "hh_batch_map.h"
#include "hh_common.h"
#include "hh_dispatch.h"
#include "hh_layout.h"
#include "hh_pipe.h"
#include "hh_sched.h"

namespace ehh {

typedef double wyd_d4 __attribute__((ext_vector_type(4)));

template <int NB, int K>
struct WydGeom {
  static_assert(NB == 32 || NB == 64, "NB = 32, 64");
  static_assert(K % 16 == 0 && K >= 16, "K must be a multiple of 16");
  static constexpr int SG = K / 16;          // sub-groups per step
  static constexpr int RT = NB / 16 + 1;     // 16-row tiles a sub-group touches
  static constexpr int RTW = (NB + K) / 16;  // 16-row tiles of the window
  static constexpr int RS = NB + 4;          // values per reflector in the packed area
  static constexpr int SW = 32;              // columns per stripe of the schedules; a wave takes 16
  // LDS of a wave: 16 reflectors, STR apart (STR - 1 = 17 mod 32: the 16 rows
  // of one reflector and of the next fall on different banks)
  static constexpr int STR = NB + 50, LDS = 16 * STR;
  static_assert(16 * RS >= 256, "a sub-group's area holds its T");
};

// T of sub-group u of (block m, step j), stored as the MFMA operand -T: value
// 64 kk + lane is -T[lane % 16][lane / 16 + 4 kk].  One 256-thread workgroup;
// the one of step 0, sub-group 0 also writes Bt[m].  Forward recurrence
// T_ii = tau_i, T[0:i, i] = -tau_i T[0:i, 0:i] (V^T v_i)[0:i] (LAPACK's larft).
// Bound by latency; the recurrence in registers, a lane to a row, instead of
// through LDS took the pre-pass at n = 8192 from 284 to 243 us.
template <int NB, int K>
__device__ __forceinline__ void wyd_prep_group(const double* __restrict__ hh,
                                               const double* __restrict__ tau, int64_t n,
                                               int64_t m, int64_t j, int u,
                                               double* __restrict__ P,
                                               int64_t* __restrict__ Bt) {
  using Gm = WydGeom<NB, K>;
  constexpr int RP = NB + 16;
  __shared__ double V[16][RP + 1], G[16][17], T[16][17], t_[16];
  __shared__ int64_t slot_[16], mb_;
  __shared__ int len_[16];
  const int64_t s0 = m * K;
  if (j >= block_steps(n, NB, K, m)) return;
  const int tid = threadIdx.x;
  if (tid == 64) {
    mb_ = block_base(n, NB, K, m);
    if (j == 0 && u == 0) Bt[m] = mb_;
  }
  if (tid < 16) {
    const int64_t s = s0 + 16 * u + tid, left = n - 1 - s - j * NB;
    const int L = (int)(left < 0 ? 0 : (left < NB ? left : NB));
    const int64_t slot = L > 0 ? slot_offset(n, NB, s) + j : 0;
    slot_[tid] = slot;
    len_[tid] = L;
    t_[tid] = L > 0 ? tau[slot] : 0.0;
  }
  __syncthreads();
  for (int e = tid; e < RP * 16; e += 256) {
    const int i = e / RP, rho = e % RP, d = rho - i;
    V[i][rho] = (d >= 0 && d < len_[i]) ? hh[slot_[i] * NB + d] : 0.0;
  }
  __syncthreads();
  {
    const int a = tid / 16, b = tid % 16;
    double g = 0.0;
    for (int rho = 0; rho < RP; ++rho) g += V[a][rho] * V[b][rho];
    G[a][b] = g;
  }
  __syncthreads();
  if (tid < 16) {  // row tid of T, in column order, in registers (T[a][l] = 0 for l < a)
    double t[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      double a = 0.0;
#pragma unroll
      for (int l = 0; l < i; ++l) a += t[l] * G[l][i];
      t[i] = i == tid ? t_[i] : (i > tid ? -(t_[i] * a) : 0.0);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) T[tid][i] = t[i];
  }
  __syncthreads();
  const int lane = tid & 63, kk = tid >> 6;
  P[((mb_ + j) * Gm::SG + u) * (16 * Gm::RS) + tid] = -T[lane & 15][(lane >> 4) + 4 * kk];
}

// Groups (block, step), existing or not, of one launch, a workgroup for each of
// their sub-groups: a launch holds fewer than 2^32 threads, and a large problem
// has more sub-groups than that (n = 131000 at K = 80).
constexpr int64_t kPrepGroups = int64_t(1) << 16;

// Groups g0 .. of a problem.
template <int NB, int K>
__global__ __launch_bounds__(256) void k_wyd_prep(const double* __restrict__ hh,
                                                  const double* __restrict__ tau, int64_t n,
                                                  int64_t Jmax, double* __restrict__ P,
                                                  int64_t* __restrict__ Bt, int64_t g0) {
  constexpr int SG = K / 16;
  static_assert(kPrepGroups * SG * 256 < int64_t(1) << 32, "threads of a launch");
  const int64_t g = g0 + blockIdx.x / SG;
  wyd_prep_group<NB, K>(hh, tau, n, g / Jmax, g % Jmax, (int)(blockIdx.x % SG), P, Bt);
}

template <int NB, int K>
__global__ __launch_bounds__(256) void k_wyd_prep_b(const ProblemDesc* __restrict__ d,
                                                    int count, int g0) {
  constexpr int SG = K / 16;
  const int b = g0 + (int)(blockIdx.x / SG);
  const ProblemDesc& D = d[find_by<ProblemDesc, &ProblemDesc::ptile0>(d, count, b)];
  const int64_t g = b - D.ptile0;
  wyd_prep_group<NB, K>((const double*)D.hh, (const double*)D.tau, D.n, g / D.Jmax, g % D.Jmax,
                        (int)(blockIdx.x % SG), (double*)D.P, (int64_t*)D.Bt);
}

__device__ __forceinline__ wyd_d4 wyd_mfma(double a, double b, wyd_d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Buffer accesses from a wave-uniform base: byte offsets of 32 bits, per lane
// and per wave, so that addresses take no registers.
typedef unsigned wyd_u2 __attribute__((ext_vector_type(2)));
typedef double wyd_u4 __attribute__((ext_vector_type(4), aligned(8)));
struct WydBuffer {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ explicit WydBuffer(const double* p)
      : r(__builtin_amdgcn_make_buffer_rsrc((void*)p, 0, 0x7fffffff, 0x00020000)) {}
  // zero, and nothing read, where the offset is not valid (past the range)
  __device__ __forceinline__ double get(bool valid, int off) const {
    const wyd_u2 w = __builtin_amdgcn_raw_buffer_load_b64(r, valid ? off : -1, 0, 0);
    return __hiloint2double((int)w[1], (int)w[0]);
  }
  __device__ __forceinline__ double load(int lane_off, int wave_off) const {
    const wyd_u2 w = __builtin_amdgcn_raw_buffer_load_b64(r, lane_off, wave_off, 0);
    return __hiloint2double((int)w[1], (int)w[0]);
  }
  // device scope
  __device__ __forceinline__ double load_dev(int lane_off, int wave_off) const {
    const wyd_u2 w = __builtin_amdgcn_raw_buffer_load_b64(r, lane_off, wave_off, 16);
    return __hiloint2double((int)w[1], (int)w[0]);
  }
  __device__ __forceinline__ void store_dev(double x, int lane_off, int wave_off) const {
    const wyd_u2 w{(unsigned)__double2loint(x), (unsigned)__double2hiint(x)};
    __builtin_amdgcn_raw_buffer_store_b64(w, r, lane_off, wave_off, 16);
  }
};

// W = V^T X and X += V (-T W) of a sub-group, tiles u .. of the window x; la,
// lb: the lane's operands in the staged reflectors, t: its -T fragments.
template <int NB, int u>
__device__ __forceinline__ wyd_d4 wyd_first(const wyd_d4* x, const double* la) {
  wyd_d4 w0{0, 0, 0, 0}, w1{0, 0, 0, 0};
#pragma unroll
  for (int rt = 0; rt < NB / 16 + 1; ++rt)
#pragma unroll
    for (int kk = 0; kk < 4; kk += 2) {
      w0 = wyd_mfma(la[16 * rt + kk], x[u + rt][kk], w0);
      w1 = wyd_mfma(la[16 * rt + kk + 1], x[u + rt][kk + 1], w1);
    }
  return w0 + w1;
}
template <int NB, int u>
__device__ __forceinline__ void wyd_second(wyd_d4* x, const double* lb, const double (&t)[4],
                                           wyd_d4 w) {
  // (two chains: each product waits for the one before it)
  wyd_d4 z0{0, 0, 0, 0}, z1{0, 0, 0, 0};
  z0 = wyd_mfma(t[0], w[0], z0);
  z1 = wyd_mfma(t[1], w[1], z1);
  z0 = wyd_mfma(t[2], w[2], z0);
  z1 = wyd_mfma(t[3], w[3], z1);
  const wyd_d4 z = z0 + z1;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
#pragma unroll
    for (int rt = 0; rt < NB / 16 + 1; ++rt)
      x[u + rt] = wyd_mfma(lb[4 * kk * (NB + 49) + 16 * rt], z[kk], x[u + rt]);
}

// The window rows of 16 columns: 16-row tiles [t0, t1) of the window at row w0.
// Plain form: the caller's column-major Q, where a lane's four rows of a tile
// are consecutive and a column's 16 rows one cache line, so no stripe copy is
// made (for n = 512 the two copies took 17 of 166 us, for the 256-problem batch
// 3 of 43 ms).  Rows past n and columns past nev are zero and not stored.
// Device form (Q, ldq: a stripe copy and its rows): the stores go through to
// memory, where a stripe's whole lines cost less than a column's 16-byte pieces
// (n = 8192, 819 columns: 4.5 ms against 5.3).
template <int NB, int K, bool DEV>
struct WydRows {
  using Gm = WydGeom<NB, K>;
  static constexpr int SW = Gm::SW;
  int64_t n;
  int q;
  bool col_ok;
  double* qp;    // column major: the lane's column
  double* sp;    // stripes
  int lane_off;
  __device__ __forceinline__ WydRows(double* Q, int64_t ldq, int64_t n_, int64_t nev, int64_t h,
                                     int lane)
      : n(n_),
        q(lane >> 4),
        col_ok(16 * h + (lane & 15) < nev),
        qp(Q + (16 * h + (lane & 15) < nev ? 16 * h + (lane & 15) : 0) * ldq + 4 * (lane >> 4)),
        sp(Q + (h >> 1) * ldq * SW + 16 * (h & 1)),
        lane_off((4 * (lane >> 4) * SW + (lane & 15)) * 8) {}
  __device__ __forceinline__ void load(wyd_d4* y, int t0, int t1, int64_t w0) const {
    if constexpr (DEV) {
      const WydBuffer win(sp + w0 * SW);
#pragma unroll
      for (int i = 0; i < t1 - t0; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          y[i][r] = win.load_dev(lane_off + r * SW * 8, 16 * (t0 + i) * SW * 8);
      return;
    }
    const double* __restrict__ p = qp + w0;
    if (w0 + 16 * t1 <= n) {
#pragma unroll
      for (int i = 0; i < t1 - t0; ++i) y[i] = wyd_d4{0, 0, 0, 0};
      if (col_ok) {
#pragma unroll
        for (int i = 0; i < t1 - t0; ++i) y[i] = *(const wyd_u4*)(p + 16 * (t0 + i));
      }
    } else {
      const int left = (int)(n - w0) - 4 * q;  // of this lane's rows
#pragma unroll
      for (int i = 0; i < t1 - t0; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          y[i][r] = (col_ok && 16 * (t0 + i) + r < left) ? p[16 * (t0 + i) + r] : 0.0;
    }
  }
  __device__ __forceinline__ void store(const wyd_d4* x, int t0, int t1, int64_t w0,
                                        bool skip_last) const {
    if constexpr (DEV) {
      const WydBuffer win(sp + w0 * SW);
#pragma unroll
      for (int tr = t0; tr < t1; ++tr)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (!(skip_last && tr == t1 - 1 && r == 3 && q == 3))
            win.store_dev(x[tr][r], lane_off + r * SW * 8, 16 * tr * SW * 8);
      return;
    }
    double* __restrict__ p = qp + w0;
    if (w0 + 16 * t1 <= n && !skip_last) {
      if (col_ok) {
#pragma unroll
        for (int tr = t0; tr < t1; ++tr) *(wyd_u4*)(p + 16 * tr) = x[tr];
      }
    } else {
      const int left = (int)(n - w0) - 4 * q;
#pragma unroll
      for (int tr = t0; tr < t1; ++tr)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (col_ok && 16 * tr + r < left && !(skip_last && tr == t1 - 1 && r == 3 && q == 3))
            p[16 * tr + r] = x[tr][r];
    }
  }
};

// Chase steps [j0, j1) of block m on the columns 16 h .. 16 h + 15 of Q.
// lv: WydGeom::LDS doubles of LDS of this wave's own, where it keeps the
// current sub-group's reflectors: reflector i at i STR + 16, zeros
// 16 places before and after it.  Both operands are read from there (row rho
// of the sub-group meets reflector i's entry rho - i), so the parallelogram
// needs no masks; reading them from the caller's array instead, 25 cache lines
// per load on average, kept the address units 85 % busy and ran the
// 256-problem batch at 57 ms.
template <int NB, int K, typename Sync>
__device__ __forceinline__ void run_wyd_steps(const double* __restrict__ P,
                                              const int64_t* __restrict__ Bt,
                                              const double* __restrict__ hh, int64_t n,
                                              int64_t nev, double* __restrict__ Q, int64_t ldq,
                                              int64_t h, int64_t m, int64_t j0, int64_t j1,
                                              const Sync& sync, double* __restrict__ lv) {
  using Gm = WydGeom<NB, K>;
  constexpr int SG = Gm::SG, RTW = Gm::RTW, STR = Gm::STR;
  constexpr int TN = NB / 16, TK = K / 16;
  constexpr int PER = 64 / NB;  // reflectors per load of the wave
  constexpr int LG = NB == 64 ? 6 : 5;
  const int lane = (int)(threadIdx.x & 63), q = lane >> 4, c = lane & 15;
  const int pc = 4 * (c & 3) + (c >> 2);  // matrix row of label c within a tile
  const int64_t s0 = m * K;
  const double* __restrict__ Pm = P + Bt[m] * (K * Gm::RS) + lane;
  const double* __restrict__ hb = hh + slot_offset(n, NB, s0) * NB;
  // zeros around the reflectors
  for (int e = lane; e < 16 * 32; e += 64) {
    const int i = e >> 5, t = e & 31;
    lv[i * STR + (t < 16 ? t : NB + t)] = 0.0;
  }
  double* const lw = lv + (lane / NB) * STR + 16 + lane % NB;  // staging
  const double* const la = lv + c * (STR - 1) + 4 * q + 16;    // V^T operand
  const double* const lb = lv + q * (STR - 1) + pc + 16;       // V operand
  const int reach = lane % NB + lane / NB;

  wyd_d4 x[RTW];
  double pre[16 / PER];
  // the next step's rows, loaded during the step's last sub-group where that
  // fits 256 registers without spilling
  constexpr bool kAhead = NB == 32;
  wyd_d4 nx[kAhead ? TN : 1];
  const WydRows<NB, K, false> rows(Q, ldq, n, nev, h, lane);
  // The sub-group's reflectors (s0 + 16 u + i, j) into registers.  Sweep s's
  // steps number (n - 1 - s + NB - 1) / NB, and that many slots lie between
  // its reflectors and the next sweep's; entry d exists for row r + d < n.
  auto fetch = [&](int64_t j, int u) {
    const WydBuffer src(hb + j * NB);
    const int steps0 = (int)(n - 1 - s0 + NB - 1), left = (int)(n - 1 - s0 - j * NB) - 16 * u;
    int off = (int)((slot_offset(n, NB, s0 + 16 * u) - slot_offset(n, NB, s0)) * (NB * 8));
    if (PER == 1 && left - 15 >= NB) {  // all of them whole
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        pre[i] = src.load(lane * 8, off);
        off += ((steps0 - 16 * u - i) >> LG) * (NB * 8);
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < 16; i += PER) {
      const int here = ((steps0 - 16 * u - i) >> LG) * (NB * 8);
      const int at = off + (PER == 2 && lane >= 32 ? here : 0) + (lane % NB) * 8;
      pre[i / PER] = src.get(reach < left - i, at);
      off += here;
      if constexpr (PER == 2) off += ((steps0 - 16 * u - i - 1) >> LG) * (NB * 8);
    }
  };

  sync.wait(j0);
  rows.load(x, 0, RTW, s0 + 1 + j0 * NB);
  fetch(j0, SG - 1);
  for (int64_t j = j0; j < j1; ++j) {
    const int64_t w0r = s0 + 1 + j * NB;
    const double* __restrict__ tp = Pm + j * (K * Gm::RS);
    [[maybe_unused]] bool ahead = false;
    RevFor<SG>::run([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      // (no load of a later sub-group moves up here: registers)
      __builtin_amdgcn_sched_barrier(0);
      double t[4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) t[kk] = tp[u * (16 * Gm::RS) + 64 * kk];
      // (one wave's LDS accesses run in order)
#pragma unroll
      for (int i = 0; i < 16; i += PER) lw[i * STR] = pre[i / PER];
      __builtin_amdgcn_wave_barrier();
      if constexpr (u > 0)
        fetch(j, u - 1);
      else if (j + 1 < j1)
        fetch(j + 1, SG - 1);
      if constexpr (kAhead && u == 0) {
        ahead = j + 1 < j1 && sync.ready(j + 1);
        if (ahead) rows.load(nx, TK, RTW, w0r + NB);
      }
      const wyd_d4 w = wyd_first<NB, u>(x, la);
      // the last step's stores are older than the loads of this product: by
      // now their acknowledgement costs no wait
      if constexpr (u == SG - 1)
        if (j > j0) sync.done(j);
      wyd_second<NB, u>(x, lb, t, w);
      __builtin_amdgcn_wave_barrier();
    });
    __builtin_amdgcn_sched_barrier(0);
    // rows final for this block
    rows.store(x, 0, TN, w0r, false);
    if (j + 1 < j1) {
#pragma unroll
      for (int tr = 0; tr < TK; ++tr) x[tr] = x[tr + TN];
      if constexpr (kAhead)
#pragma unroll
        for (int tr = 0; tr < TN; ++tr) x[TK + tr] = nx[tr];
      if (!ahead) {
        sync.wait(j + 1);
        rows.load(x + TK, TK, RTW, w0r + NB);
      }
    }
  }
  // carried rows; the window's last row (row NB+K-1, which no reflector of the
  // block touches) may belong to another tile and is not written
  rows.store(x, TN, RTW, s0 + 1 + (j1 - 1) * NB, true);
  sync.done(j1);
}

// A unit of the device form: all steps of block m on a workgroup of four waves,
// this wave on the 16-column tile h16 (live: it has columns).  The waves share
// the staged reflectors: each thread passes four (NB = 32: two) consecutive
// entries of one reflector per sub-group, fetched two sub-groups ahead, and the
// row waits of one workgroup overlap the products of the other on its compute
// unit.  (One wave to a unit, each staging for itself: n = 8192 with 819
// columns 4.45 ms instead of 4.06, n = 2900 1.9 instead of 1.6.  The same units
// without hand-overs for a batch ran 256 problems in 53.8 ms, the one-wave
// local form in 41.4 then: it loads the next rows ahead and has no barriers.)
// lds: 2 WydGeom::LDS doubles.
template <int NB, int K>
__device__ __forceinline__ void run_wyd_unit(const double* __restrict__ P,
                                             const int64_t* __restrict__ Bt,
                                             const double* __restrict__ hh, int64_t n,
                                             int64_t nev, double* __restrict__ Q, int64_t ldq,
                                             int64_t h16, bool live, int64_t m,
                                             const DevSync& sync, double* lds) {
  using Gm = WydGeom<NB, K>;
  constexpr int SG = Gm::SG, RTW = Gm::RTW, STR = Gm::STR, LDS = Gm::LDS;
  constexpr int TN = NB / 16, TK = K / 16;
  constexpr int PER = NB / 16;  // entries of a thread
  const int tid = (int)threadIdx.x, lane = tid & 63, q = lane >> 4, c = lane & 15;
  const int pc = 4 * (c & 3) + (c >> 2);  // matrix row of label c within a tile
  const int fi = tid >> 4, fd = (tid & 15) * PER;  // the thread's reflector and first entry
  const int64_t s0 = m * K, steps = block_steps(n, NB, K, m);
  const double* __restrict__ Pm = P + Bt[m] * (K * Gm::RS) + lane;
  const int64_t slot0 = slot_offset(n, NB, s0);
  const double* __restrict__ hb = hh + slot0 * NB;
  int off[SG];  // of the thread's reflectors of step 0, in bytes
#pragma unroll
  for (int u = 0; u < SG; ++u) {
    const int64_t s = s0 + 16 * u + fi;
    off[u] = s <= n - 2 ? (int)((slot_offset(n, NB, s) - slot0) * (NB * 8)) + fd * 8 : 0;
  }
  double pre[2][PER];
  auto fetch = [&](double (&d)[PER], int64_t j, int u) {
    const WydBuffer src(hb + j * NB);
    const int left = (int)(n - 1 - s0 - j * NB) - 16 * u - fi - fd;  // entries from fd on
#pragma unroll
    for (int e = 0; e < PER; ++e) d[e] = src.get(e < left, off[u] + 8 * e);
  };
  auto stage = [&](const double (&d)[PER], int buf) {
    double* p = lds + buf * LDS + fi * STR + 16 + fd;
#pragma unroll
    for (int e = 0; e < PER; ++e) p[e] = d[e];
  };
  const WydRows<NB, K, true> rows(Q, ldq, n, nev, h16, lane);
  wyd_d4 x[RTW];
#pragma unroll
  for (int tr = 0; tr < RTW; ++tr) x[tr] = wyd_d4{0, 0, 0, 0};
  // zeros around the reflectors
  for (int e = tid; e < 2 * 16 * 32; e += 256) {
    const int i = (e >> 5) & 15, t = e & 31;
    lds[(e >> 9) * LDS + i * STR + (t < 16 ? t : NB + t)] = 0.0;
  }
  fetch(pre[0], 0, SG - 1);
  fetch(pre[1], 0, SG - 2);
  stage(pre[0], 0);
  int buf = 0;
  sync.wait(0);
  if (live) rows.load(x, 0, RTW, s0 + 1);
  for (int64_t j = 0; j < steps; ++j) {
    const int64_t w0r = s0 + 1 + j * NB;
    const bool more = j + 1 < steps;
    const double* __restrict__ tp = Pm + j * (K * Gm::RS);
    RevFor<SG>::run([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      constexpr int cur = (SG - 1 - u) & 1;
      // the sub-group's reflectors are staged, its predecessor's place is
      // free; a step's first barrier follows the step before's stores'
      // acknowledgement too
      if constexpr (u == SG - 1)
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      else
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if constexpr (u == SG - 1) {
        if (j > 0) {
          if (tid == 0) sync.raise(j);
          sync.wait(j);
          if (live) rows.load(x + TK, TK, RTW, w0r);
        }
      }
      double t[4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) t[kk] = tp[u * (16 * Gm::RS) + 64 * kk];
      if constexpr (u > 1)
        fetch(pre[cur], j, u - 2);
      else if (more)
        fetch(pre[cur], j + 1, SG + u - 2);
      __builtin_amdgcn_sched_barrier(0);  // the loads stay up here
      const double* lv = lds + buf * LDS;
      const wyd_d4 w = wyd_first<NB, u>(x, lv + c * (STR - 1) + 4 * q + 16);
      wyd_second<NB, u>(x, lv + q * (STR - 1) + pc + 16, t, w);
      buf ^= 1;
      if (u > 0 || more) stage(pre[cur ^ 1], buf);
    });
    if constexpr ((SG & 1) == 1)
#pragma unroll
      for (int e = 0; e < PER; ++e) pre[1][e] = pre[0][e];
    // rows final for this block
    if (live) rows.store(x, 0, TN, w0r, false);
    if (more) {
#pragma unroll
      for (int tr = 0; tr < TK; ++tr) x[tr] = x[tr + TN];
    }
  }
  // carried rows; the window's last row (row NB+K-1, which no reflector of the
  // block touches) may belong to another unit and is not written
  if (live) rows.store(x, TN, RTW, s0 + 1 + (steps - 1) * NB, true);
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  if (tid == 0) sync.raise(steps);
}

// Diagonal schedule: launch t's tiles (16-column halves of the stripes c0 ..
// c0+G-1, blocks m0 ..).
template <int NB, int K>
__global__ __launch_bounds__(64, 2) void k_wyd(const double* __restrict__ P,
                                               const int64_t* __restrict__ Bt,
                                               const double* __restrict__ hh,
                                               double* __restrict__ Q, int64_t ldq,
                                               int64_t n, int64_t nev, int c0, int G, int M, int t,
                                               int m0, int S, int xcd) {
  __shared__ double lv[WydGeom<NB, K>::LDS];
  const int b = tile_of((int)blockIdx.x, (int)gridDim.x, xcd);
  const int64_t h = 2 * (int64_t)c0 + b % (2 * G);
  if (16 * h >= nev) return;
  const int m = m0 + b / (2 * G);
  const int64_t J0 = block_steps(n, NB, K, m);
  const int64_t j0 = (int64_t)(t - (M - 1 - m)) * S;
  run_wyd_steps<NB, K>(P, Bt, hh, n, nev, Q, ldq, h, m, j0,
                       j0 + S < J0 ? j0 + S : J0, NoSync{}, lv);
}

template <int NB, int K>
__global__ __launch_bounds__(64, 2) void k_wyd_b(const ProblemDesc* __restrict__ d,
                                                 const DiagEntry* __restrict__ e, int ecount,
                                                 int t, int xcd) {
  __shared__ double lv[WydGeom<NB, K>::LDS];
  const int b = tile_of((int)blockIdx.x, (int)gridDim.x, xcd);
  const DiagEntry& E0 = e[find_by<DiagEntry, &DiagEntry::tile0>(e, ecount, b >> 1)];
  const ProblemDesc& D = d[E0.p];
  const int local = b - 2 * E0.tile0;
  const int64_t h = local % (2 * D.G);
  if (16 * h >= D.nev) return;
  const int m = E0.m0 + local / (2 * D.G);
  const int64_t J0 = block_steps(D.n, NB, K, m);
  const int64_t j0 = (int64_t)(t - (D.M - 1 - m)) * D.S;
  run_wyd_steps<NB, K>((const double*)D.P, (const int64_t*)D.Bt, (const double*)D.hh, D.n,
                       D.nev, (double*)D.Q, D.ldq, h, m, j0,
                       j0 + D.S < J0 ? j0 + D.S : J0, NoSync{}, lv);
}

// One workgroup's 16 columns through every block (local form).
template <int NB, int K>
__device__ __forceinline__ void wyd_local(const double* P, const int64_t* Bt, const double* hh,
                                          double* Q, int64_t ldq, int64_t n, int64_t nev,
                                          int64_t h, int64_t M, int* cnt, double* lv) {
  const int W = (int)(blockDim.x >> 6);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (threadIdx.x < 8) cnt[threadIdx.x] = 0;
  __syncthreads();
  const int span = (int)((n - 1 + NB - 1) / NB) + 1;
  for (int64_t o = wave; o < M; o += W) {
    const int64_t m = M - 1 - o;
    LocalSync sync;
    sync.mine = cnt + wave;
    sync.before = o == 0 ? nullptr : cnt + (wave == 0 ? W - 1 : wave - 1);
    sync.base = (int)o * span;
    sync.before_base = (int)(o - 1) * span;
    sync.before_steps = o == 0 ? 0 : (int)block_steps(n, NB, K, m + 1);
    run_wyd_steps<NB, K>(P, Bt, hh, n, nev, Q, ldq, h, m, 0, block_steps(n, NB, K, m), sync,
                         lv + wave * WydGeom<NB, K>::LDS);
  }
}

template <int NB, int K>
__global__ __launch_bounds__(512, 2) void k_wyd_local(const double* __restrict__ P,
                                                      const int64_t* __restrict__ Bt,
                                                      const double* __restrict__ hh,
                                                      double* __restrict__ Q, int64_t ldq,
                                                      int64_t n, int64_t nev, int64_t M) {
  __shared__ int cnt[8];
  extern __shared__ double lv[];
  wyd_local<NB, K>(P, Bt, hh, Q, ldq, n, nev, blockIdx.x, M, cnt, lv);
}

// Batched, W > 1 waves or (ONE) a single wave, block after block with nothing
// to wait for: umap gives the unit (16 columns of a problem) of each workgroup id,
// -1 for none; units are numbered by stripes, two to a stripe.
template <int NB, int K, bool ONE>
__global__ __launch_bounds__(ONE ? 64 : 512, 2) void k_wyd_local_b(
    const ProblemDesc* __restrict__ d, int count, const int* __restrict__ umap) {
  __shared__ int cnt[8];
  extern __shared__ double lv[];
  const HalfUnit hu = half_unit((int)blockIdx.x, umap != nullptr);
  const int u = umap ? umap[hu.entry] : hu.entry;
  if (u < 0) return;
  const ProblemDesc& D = d[find_by<ProblemDesc, &ProblemDesc::unit0>(d, count, u)];
  const int64_t h = 2 * (int64_t)(u - D.unit0) + hu.half;
  if (16 * h >= D.nev) return;
  if constexpr (ONE) {
    for (int64_t m = D.M - 1; m >= 0; --m)
      run_wyd_steps<NB, K>((const double*)D.P, (const int64_t*)D.Bt, (const double*)D.hh, D.n,
                           D.nev, (double*)D.Q, D.ldq, h, m, 0, block_steps(D.n, NB, K, m),
                           NoSync{}, lv);
  } else {
    wyd_local<NB, K>((const double*)D.P, (const int64_t*)D.Bt, (const double*)D.hh, (double*)D.Q,
                     D.ldq, D.n, D.nev, h, D.M, cnt, lv);
  }
}

// Device form: units (order o, 64 columns h) by ticket, on a stripe copy.
template <int NB, int K>
__global__ __launch_bounds__(256, 2) void k_wyd_units(const double* __restrict__ P,
                                                      const int64_t* __restrict__ Bt,
                                                      const double* __restrict__ hh,
                                                      double* __restrict__ Qs, int64_t rows_pad,
                                                      int64_t n, int64_t nev, int64_t H,
                                                      int64_t M, int* __restrict__ words) {
  __shared__ double lds[2 * WydGeom<NB, K>::LDS];
  __shared__ int ticket;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0)
      ticket = __hip_atomic_fetch_add(words, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int64_t u = __builtin_amdgcn_readfirstlane(ticket);
    if (u >= M * H) return;
    const int64_t o = u / H, h = u - o * H, m = M - 1 - o, h16 = 4 * h + wave;
    const bool live = 16 * h16 < nev;
    DevSync sync;
    sync.mine = words + (u + 1) * kPipeStride;
    sync.before = o == 0 ? nullptr : words + (u - H + 1) * kPipeStride;
    sync.before_steps = o == 0 ? 0 : (int)block_steps(n, NB, K, m + 1);
    run_wyd_unit<NB, K>(P, Bt, hh, n, nev, Qs, rows_pad, live ? h16 : 0, live, m, sync, lds);
  }
}

}  // namespace ehh
