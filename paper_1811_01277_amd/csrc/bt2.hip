// Band -> full back-transformation of eigenvectors (C ABI in
// include/elpa_bt2.h; Kus et al., Sec. 2): Q <- H_0 H_1 ... H_{n-nbw-1} Q
// with the first stage's reflectors H_c = I - tau_c v_c v_c^H, v_c on rows
// [c+nbw, n).
//
// Consecutive reflectors c0 .. c0+w-1 form one compact-WY product
//   H_c0 ... H_c0+w-1 = I - V T V^H
// (V the m x w block of vectors from row c0+nbw down, unit lead on the
// diagonal and zeros above it; T the upper triangular factor of the forward
// accumulation, no division by tau: tau = 0, an identity reflector, is fine).
// The factors depend on the vectors alone, so all blocks' G = V^H V come first,
// then all T in three launches; then the blocks are applied, last block first, as
//   W = V^H Q[c0+nbw:, :],  W <- T W,  Q[c0+nbw:, :] -= V W,
// plain GEMMs on the matrix cores through rocBLAS.  Packing V (explicit zeros
// and unit lead, so the vectors may share storage with anything above them) and
// forming T are this file's kernels.  (A triangular solve per block in T's
// place, a dozen dependent launches of its own, took 1.5 of 6.6 ms at n = 6000
// with 3000 vectors, nbw = 64, fp64; the strips
// take 62 us for all sixteen blocks and the call 5.64 ms.)
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <vector>

#include "../../include/elpa_bt2.h"
#include "../../include/elpa_hh.h"
#include "wy_blas.h"

namespace ebt {

// Vp (m x wb, column major, ld m): column i = v_{c0+i} from row c0+nbw down,
// zero above row i, one at row i.
template <typename E>
__global__ __launch_bounds__(256) void k_pack(const E* __restrict__ V, int64_t ldv, int64_t nbw,
                                              int64_t c0, int64_t m, E* __restrict__ Vp) {
  const int64_t i = blockIdx.y;
  const int64_t c = c0 + i;
  E* __restrict__ dst = Vp + i * m;
  const E* __restrict__ src = V + c * ldv + c0 + nbw;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < m;
       r += (int64_t)gridDim.x * blockDim.x) {
    E v;
    if (r < i)
      v = Num<E>::zero();
    else if (r == i)
      v = Num<E>::one();
    else
      v = src[r];
    dst[r] = v;
  }
}

// G = V^H V and T share their storage: block b (w x w at F + b stride, column
// major, ld its own width) holds G, whose upper triangle becomes T.  G is
// Hermitian, so what T takes the place of is read from the lower triangle, and
// that is cleared last.  N reflectors in all, w per block; the blocks are
// numbered in the first grid dimension, as there may be as many as reflectors.

// T's diagonal blocks of 64.
template <typename E>
__global__ __launch_bounds__(256) void k_diag_factors(E* __restrict__ F, int64_t stride,
                                                      const E* __restrict__ tau, int64_t N, int w) {
  constexpr int PL = Planes<E>::PL, LD = 65;
  __shared__ double G[PL][64 * LD], T[PL][64 * LD];
  const int lane = (int)threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int per = (w + 63) / 64, o = 64 * (int)(blockIdx.x % per);
  const int64_t b = blockIdx.x / per, left = N - b * w;
  const int wb = (int)(left < w ? left : w);
  if (o >= wb) return;
  E* __restrict__ Fb = F + b * stride;
#pragma unroll
  for (int x = 0; x < 16; ++x) {
    const int c = wave + 4 * x;
    double g[2] = {0.0, 0.0};
    if (o + lane < wb && o + c < wb) split(Fb[o + lane + (int64_t)(o + c) * wb], &g[0], &g[1]);
#pragma unroll
    for (int p = 0; p < PL; ++p) {
      G[p][lane * LD + c] = g[p];
      T[p][lane * LD + c] = 0.0;
    }
  }
  double ty[2] = {0.0, 0.0};
  if (o + lane < wb) split(tau[b * w + o + lane], &ty[0], &ty[1]);
  __syncthreads();
  tri_factor64<PL>(G, T, ty, wave, lane);
#pragma unroll
  for (int x = 0; x < 16; ++x) {
    const int c = wave + 4 * x;
    double t[PL];
#pragma unroll
    for (int p = 0; p < PL; ++p) t[p] = T[p][lane * LD + c];
    if (o + lane < wb && o + c < wb) Fb[o + lane + (int64_t)(o + c) * wb] = join<E>(t);
  }
}

// The rest of T: a workgroup does the columns 16 s .. of T_b, upwards from the
// diagonal block j they lie in: T_ij = -T_ii sum_{i < l <= j} G_il T_lj, wave v
// the rows 16 v .. of each.  The strip stays in LDS; G_il = G_li^H and T_ii come
// from memory, rows of a tile together.  The columns of one block and all blocks
// run side by side: the longest strip's chain of products, sixteen per wave and
// 64 x 64 x 16 block, bounds it, with a product's operands all in flight before
// its first use.  (One wave to a strip, four times the chain: complex n = 1000
// in two blocks of up to 512 took 632 us instead of 455.)
template <typename E>
__global__ __launch_bounds__(256) void k_strip_factors(E* __restrict__ F, int64_t stride,
                                                       int64_t N, int w) {
  constexpr int PL = Planes<E>::PL, I = PL - 1;
  extern __shared__ double strip[];  // [block][plane][64 rows][16 columns]
  const int lane = (int)threadIdx.x & 63, q = lane >> 4, c16 = lane & 15;
  const int rt = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int per = (w + 15) / 16, s = (int)(blockIdx.x % per);
  const int64_t b = blockIdx.x / per, left = N - b * w;
  const int wb = (int)(left < w ? left : w), col = 16 * s + c16;
  if (16 * s >= wb) return;
  const int j = s / 4;
  E* Fb = F + b * stride;
  // (rows past the block meet zeros of the strip: any entry will do)
  auto get = [&](int r, int c) { return Fb[(r < wb ? r : wb - 1) + (int64_t)c * wb]; };
  auto at = [&](int l, int p, int row) { return ((l * PL + p) * 64 + row) * 16 + c16; };
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 16 * rt + q + 4 * r;
    double t[2] = {0.0, 0.0};
    if (64 * j + row < wb && col < wb) split(Fb[64 * j + row + (int64_t)col * wb], &t[0], &t[1]);
#pragma unroll
    for (int p = 0; p < PL; ++p) strip[at(j, p, row)] = t[p];
  }
  __syncthreads();
  for (int i = j - 1; i >= 0; --i) {
    d4 x[PL], y[PL];
#pragma unroll
    for (int p = 0; p < PL; ++p) x[p] = y[p] = d4{0, 0, 0, 0};
    E g[16], t[16];
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) g[kk] = get(64 * (i + 1) + 4 * kk + q, 64 * i + 16 * rt + c16);
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) t[kk] = get(64 * i + 16 * rt + c16, 64 * i + 4 * kk + q);
    for (int l = i + 1; l <= j; ++l) {
      E h[16];  // the next block's
      const int ln = l < j ? l + 1 : j;
#pragma unroll
      for (int kk = 0; kk < 16; ++kk) h[kk] = get(64 * ln + 4 * kk + q, 64 * i + 16 * rt + c16);
#pragma unroll
      for (int kk = 0; kk < 16; ++kk) {
        double a[2] = {0.0, 0.0};
        split(g[kk], &a[0], &a[1]);
        mac(a[0], -a[1], strip[at(l, 0, 4 * kk + q)], strip[at(l, I, 4 * kk + q)], x);
        g[kk] = h[kk];
      }
    }
    // the sum passes between the waves in the place of T_ij
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int p = 0; p < PL; ++p) strip[at(i, p, 16 * rt + q + 4 * r)] = x[p][r];
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      if (kk / 4 < rt) continue;  // T_ii is upper triangular
      double a[2] = {0.0, 0.0};
      split(t[kk], &a[0], &a[1]);
      mac(a[0], a[1], strip[at(i, 0, 4 * kk + q)], strip[at(i, I, 4 * kk + q)], y);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * rt + q + 4 * r;
      double v[PL];
#pragma unroll
      for (int p = 0; p < PL; ++p) {
        v[p] = -y[p][r];
        strip[at(i, p, row)] = v[p];
      }
      if (col < wb) Fb[64 * i + row + (int64_t)col * wb] = join<E>(v);
    }
    __syncthreads();
  }
}

// Zeros below the diagonal blocks, a wave to a column.
template <typename E>
__global__ __launch_bounds__(256) void k_lower_zeros(E* __restrict__ F, int64_t stride, int64_t N,
                                                     int w) {
  const int per = (w + 3) / 4, c = 4 * (int)(blockIdx.x % per) + (int)(threadIdx.x >> 6);
  const int64_t b = blockIdx.x / per, left = N - b * w;
  const int wb = (int)(left < w ? left : w);
  if (c >= wb) return;
  for (int r = (c / 64 + 1) * 64 + (int)(threadIdx.x & 63); r < wb; r += 64)
    F[b * stride + r + (int64_t)c * wb] = Num<E>::zero();
}

int64_t default_block(int32_t dtype) { return dtype == ELPA_C64 ? 192 : 384; }

struct Layout {
  int64_t N = 0, w = 0, mmax = 0, nev = 0;
  // packed V, one block's factor, all of them, W, partial products
  size_t vp = 0, factor = 0, factors = 0, wbuf = 0, part = 0, total = 0;
  Layout(int64_t n, int64_t nev_, int64_t nbw, int64_t block, size_t es) {
    N = n > nbw ? n - nbw : 0;
    w = std::max<int64_t>(1, std::min<int64_t>(block, std::max<int64_t>(N, 1)));
    mmax = N;  // the first block's rows
    nev = nev_;
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    vp = al((size_t)mmax * w * es);
    factor = al((size_t)w * w * es);
    factors = (size_t)((N + w - 1) / w) * factor;
    wbuf = al((size_t)w * nev * es);
    // the largest set of partial products over all blocks
    size_t pe = 0;
    for (int64_t c0 = 0; c0 < N; c0 += w) {
      const int64_t wb = std::min<int64_t>(w, N - c0), m = N - c0;
      pe = std::max(pe, (size_t)ksplit(m, wb, nev, es) * wb * nev);
      pe = std::max(pe, (size_t)ksplit(m, wb, wb, es) * wb * wb);
    }
    part = al(pe * es);
    total = vp + factors + wbuf + part;
  }
};

size_t elem_size(int32_t dtype) {
  switch (dtype) {
    case ELPA_R64: return 8;
    case ELPA_R32: return 4;
    case ELPA_C64: return 16;
    default: return 0;
  }
}

template <typename E, typename S>
int run(int64_t n, int64_t nev, int64_t nbw, const E* V, int64_t ldv, const E* tau, E* Q,
        int64_t ldq, hipStream_t st, int64_t block) {
  const Layout L(n, nev, nbw, block, sizeof(E));
  char* ws = nullptr;
  if (hipMallocAsync((void**)&ws, L.total, st) != hipSuccess) return ELPA_ERR_NOMEM;
  E* Vp = (E*)ws;
  E* F = (E*)(ws + L.vp);
  E* W = (E*)(ws + L.vp + L.factors);
  E* part = (E*)(ws + L.vp + L.factors + L.wbuf);
  const int64_t stride = (int64_t)(L.factor / sizeof(E));
  int rc = ELPA_OK;
  {
    std::lock_guard<std::mutex> lock(Handles::get().mu);
    rocblas_handle h = handle_for(st);
    if (!h) rc = ELPA_ERR_DEVICE;
    const int64_t nblk = (L.N + L.w - 1) / L.w, w = L.w;
    const auto N_ = rocblas_operation_none;
    bool ok = rc == ELPA_OK;
    auto pack = [&](int64_t c0, int64_t m, int64_t wb) {
      const unsigned gx = (unsigned)std::min<int64_t>((m + 255) / 256, 1024);
      hipLaunchKernelGGL(k_pack<E>, dim3(gx, (unsigned)wb), dim3(256), 0, st, V, ldv, nbw, c0, m,
                         Vp);
    };
    // G of every block, the first to be applied last, so that its V stays packed
    for (int64_t b = 0; ok && b < nblk; ++b) {
      const int64_t c0 = b * w, wb = std::min<int64_t>(w, L.N - c0), m = L.N - c0;
      pack(c0, m, wb);
      ok = gemm_adj_splitk<E, S>(h, wb, wb, m, Vp, m, Vp, m, ksplit(m, wb, wb, sizeof(E)), part,
                                 F + b * stride, st);
    }
    if (ok) {
      const int blocks = (int)((w + 63) / 64);
      hipLaunchKernelGGL(k_diag_factors<E>, dim3((unsigned)(nblk * blocks)), dim3(256), 0, st, F,
                         stride, tau, L.N, (int)w);
      if (blocks > 1) {
        hipLaunchKernelGGL(k_strip_factors<E>, dim3((unsigned)(nblk * ((w + 15) / 16))), dim3(256),
                           (unsigned)(blocks * Planes<E>::PL * 64 * 16 * sizeof(double)), st, F,
                           stride, L.N, (int)w);
        hipLaunchKernelGGL(k_lower_zeros<E>, dim3((unsigned)(nblk * ((w + 3) / 4))), dim3(256), 0,
                           st, F, stride, L.N, (int)w);
      }
    }
    for (int64_t b = nblk - 1; ok && b >= 0; --b) {
      const int64_t c0 = b * w, wb = std::min<int64_t>(w, L.N - c0), m = L.N - c0;
      if (b < nblk - 1) pack(c0, m, wb);
      E* Qs = Q + c0 + nbw;
      ok = gemm_adj_splitk<E, S>(h, wb, nev, m, Vp, m, Qs, ldq, ksplit(m, wb, nev, sizeof(E)),
                                 part, W, st);
      ok = ok && Blas<E>::gemm(h, N_, N_, wb, nev, wb, S(1), F + b * stride, wb, W, wb, S(0),
                               part, wb) == rocblas_status_success;  // (summed: free)
      ok = ok && Blas<E>::gemm(h, N_, N_, m, nev, wb, S(-1), Vp, m, part, wb, S(1), Qs,
                               ldq) == rocblas_status_success;
    }
    if (rc == ELPA_OK && (!ok || hipGetLastError() != hipSuccess)) rc = ELPA_ERR_DEVICE;
  }
  const hipError_t e2 = hipFreeAsync(ws, st);
  if (rc == ELPA_OK && e2 != hipSuccess) rc = ELPA_ERR_DEVICE;
  return rc;
}

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

}  // namespace ebt

extern "C" {

int64_t elpa_bt2_workspace_bytes(int64_t n, int64_t nev, int64_t nbw, int32_t dtype,
                                 int64_t block) {
  const size_t es = ebt::elem_size(dtype);
  if (n < 0 || nev < 0 || nbw < 1 || es == 0 || block < 0 || block > 512) return -1;
  if (n <= nbw || nev == 0) return 0;
  const ebt::Layout L(n, nev, nbw, block ? block : ebt::default_block(dtype), es);
  return (int64_t)L.total;
}

int elpa_bt2_trafo(int64_t n, int64_t nev, int64_t nbw, const void* V, int64_t ldv,
                   const void* tau, void* Q, int64_t ldq, int32_t dtype, void* stream,
                   int64_t block) {
  const size_t es = ebt::elem_size(dtype);
  if (es == 0) return ELPA_ERR_DTYPE;
  if (n < 0 || nev < 0 || nbw < 1 || block < 0 || block > 512) return ELPA_ERR_ARG;
  if (n <= nbw || nev == 0) return ELPA_OK;
  if (ldq < n || ldv < n || !V || !tau || !Q) return ELPA_ERR_ARG;
  if (!ebt::aligned(V, es) || !ebt::aligned(tau, es) || !ebt::aligned(Q, es))
    return ELPA_ERR_ALIGN;
  const int64_t b = block ? block : ebt::default_block(dtype);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  switch (dtype) {
    case ELPA_R64:
      return ebt::run<double, double>(n, nev, nbw, (const double*)V, ldv, (const double*)tau,
                                      (double*)Q, ldq, st, b);
    case ELPA_R32:
      return ebt::run<float, float>(n, nev, nbw, (const float*)V, ldv, (const float*)tau,
                                    (float*)Q, ldq, st, b);
    default:
      return ebt::run<ebt::zc, double>(n, nev, nbw, (const ebt::zc*)V, ldv,
                                       (const ebt::zc*)tau, (ebt::zc*)Q, ldq, st, b);
  }
}

}  // extern "C"
