// The R x R part of a CPD-ALS mode update that can run beside the MTTKRP (fp64): the Hadamard product of the other factors'
// Gram matrices and its inverse.  Shared by the ALS kernels and by the MTTKRP launch that carries it in its first block.
#ifndef HBCSF_SMALL_H_
#define HBCSF_SMALL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hbcsf_device.h"

namespace hbcsf {

// V = Hadamard product over the modes m != n of the algorithm's Gram matrices, entry (i, j)
template <int R>
__device__ __forceinline__ double v_entry(const SmallState& st, int n, int i, int j) {
  double v = 1.0;
  for (int m = 0; m < st.order; ++m)
    if (m != n) v *= st.gram[m][i * R + j] / (st.scale[m][i] * st.scale[m][j]);
  return v;
}

// d_r = product over the other modes of 1 / c_m[r]: M of the algorithm = M of the stored factors, columns times d
template <int R>
__device__ __forceinline__ double d_entry(const SmallState& st, int n, int r) {
  double d = 1.0;
  for (int m = 0; m < st.order; ++m)
    if (m != n) d /= st.scale[m][r];
  return d;
}

// p: right-hand matrix of the product kernels, P[i][j] in [R][R], or for R < 32 block-diagonal in [32][32]
template <int R>
__device__ __forceinline__ void put_p(float* __restrict__ p, int i, int j, float v) {
  if (R >= 32) {
    p[i * R + j] = v;
  } else {
    for (int b = 0; b < 32 / R; ++b) p[(b * R + i) * 32 + b * R + j] = v;
  }
}

constexpr int small_threads(int R) { return R <= 32 ? 64 : R == 64 ? 256 : 1024; }  // (R / 4)^2, at least a wavefront

// First row and column of the 4 x 4 tile of an R x R matrix that thread `tid` keeps.  Below rank 32 a wavefront has more
// threads than there are tiles: those without one are given the first (they read what it reads and store nothing).
constexpr int tile_row(int R, int tid) { return tid < (R / 4) * (R / 4) ? 4 * (tid / (R / 4)) : 0; }
constexpr int tile_column(int R, int tid) { return tid < (R / 4) * (R / 4) ? 4 * (tid % (R / 4)) : 0; }
constexpr bool tiles_inside(int R) {
  for (int tid = 0; tid < (R == 32 ? 256 : small_threads(R)); ++tid)
    if (tile_row(R, tid) + 4 > R || tile_column(R, tid) + 4 > R) return false;
  return true;
}
static_assert(tiles_inside(8) && tiles_inside(16) && tiles_inside(32) && tiles_inside(64) && tiles_inside(128),
              "every thread's tile lies in the matrix");

// 1 / x for a normal positive x: the hardware's estimate and two Newton steps (relative error near 2^-53).
__device__ __forceinline__ double reciprocal(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

// 1 / sqrt(x) for a normal positive x, in the same way.
__device__ __forceinline__ double reciprocal_root(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
  return fma(0.5 * r, fma(-x * r, r, 1.0), r);
}

// V is inverted in place by R sweep steps without pivoting,
//     d = a_kk;  a_kk <- -1 / d;  a_ik, a_ki <- a_ik / d;  a_ij <- a_ij - a_ik a_kj / d     (after all: -V^-1)
// -- for a positive definite matrix as accurate as the Cholesky route, and its pivots are the squares of the Cholesky
// factor's diagonal.  The matrix stays symmetric, so a step needs one row: each thread keeps a 4 x 4 tile in registers,
// the threads that hold row k publish it in LDS (two buffers in turn, one barrier a step; R <= 32 is one wavefront), and
// every thread reads the 4 + 4 entries its tile needs.  The chain of R steps is latency: the next pivot is formed from
// the published row by every thread, so that its reciprocal is under way while the tiles are updated (rank 32: 25 us in
// the first form, one entry per thread and a division in the chain).
// All U threads of the block call; x: the thread's tile of -V^-1.  False (for every thread) where a pivot is not safely
// positive: the eigenvalue form has to be taken.
template <int R>
struct SweepLds {
  __attribute__((aligned(16))) double row[2][R + 2];   // row k, then entry (k + 1, k + 1)
  double diag[R];
  double dmax;
  int good;
};

template <int R, int U>
__device__ __forceinline__ bool pinv_sweep(const SmallState& st, int n, SweepLds<R>& l, double (&x)[4][4]) {
  constexpr int T = small_threads(R), W = R / 4;
  static_assert(U >= T, "a thread per tile");
  const int tid = threadIdx.x;
  const bool owns = tid < W * W;
  const int i0 = tile_row(R, tid), j0 = tile_column(R, tid);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) x[i][j] = owns ? 1.0 : 0.0;
  if (owns) {
    for (int m = 0; m < st.order; ++m) {
      if (m == n) continue;
      const double* g = st.gram[m];
      double ci[4], cj[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ci[i] = 1.0 / st.scale[m][i0 + i];
        cj[i] = 1.0 / st.scale[m][j0 + i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) x[i][j] *= g[(i0 + i) * R + j0 + j] * (ci[i] * cj[j]);
    }
    if (i0 == j0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) l.diag[i0 + i] = x[i][i];
    }
  }
  __syncthreads();
  if (tid < 64) {
    double m = 0.0;
    for (int r = tid; r < R; r += 64) m = fmax(m, l.diag[r]);
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
    if (tid == 0) l.dmax = m;
  }
  __syncthreads();
  const double least = 1e-10 * l.dmax;
  double pivot = l.diag[0];
  bool good = true;
  for (int kb = 0; kb < R && good && tid < T; kb += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = kb + q;
      double* row = l.row[k & 1];
      if (owns && i0 == kb) {
#pragma unroll
        for (int j = 0; j < 4; ++j) row[j0 + j] = x[q][j];
        if (q < 3 && j0 == kb) row[R] = x[q < 3 ? q + 1 : 0][q < 3 ? q + 1 : 0];
      }
      if (q == 3 && owns && i0 == kb + 4 && j0 == kb + 4) row[R] = x[0][0];
      if (!(pivot > least)) good = false;   // the same for every thread
      const double inv = reciprocal(pivot);
      if constexpr (T == 64) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // one wavefront sweeps
      else __syncthreads();
      double ri[4], rj[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ri[i] = row[i0 + i];
        rj[i] = row[j0 + i];
      }
      const double nextRow = k + 1 < R ? row[k + 1] : 0.0;
      pivot = fma(-nextRow * inv, nextRow, row[R]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double f = ri[i] * inv;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool inRow = i == q && i0 == kb, inCol = j == q && j0 == kb;
          const double swept = fma(-f, rj[j], x[i][j]);
          if (i == q || j == q) x[i][j] = inRow ? (inCol ? -inv : rj[j] * inv) : inCol ? f : swept;
          else x[i][j] = swept;
        }
      }
    }
  }
  if constexpr (U > T) {  // the other wavefronts have waited here
    if (tid == 0) l.good = good;
    __syncthreads();
    good = l.good;
  }
  return good;
}

// ---------------------------------------------------------------------------------------------------
// Guest of an MTTKRP launch (its first block of 256 threads, rank <= 64): inverts V for the update that the MTTKRP belongs to.
// Nothing the MTTKRP reads or writes is touched, and nothing here is needed before the product that follows it, so the
// chain of R dependent steps runs beside the MTTKRP instead of before it (5 iterations, 5 M nonzeros at rank 32 1381 ->
// 1290 us, 0.8 M at rank 64 1204 -> 916).  *good = 0 leaves the update to the eigenvalue form.  (The sum of the slots would
// fit in beside it, but not for nothing: the blocks that sum have to hand over to the one that inverts, and with agent-scope
// fences for that, which write an L2 back, the MTTKRP of a small tensor took 70 instead of 28 us.)
// ---------------------------------------------------------------------------------------------------
template <int R>
constexpr uint32_t guest_lds_bytes() {
  return sizeof(SweepLds<R>);
}

template <int R>
__device__ __forceinline__ void guest_block(const GuestArgs& a, uint32_t* lds) {
  static_assert(R <= 64, "one block of 256 threads inverts V");
  const int tid = threadIdx.x;
  double x[4][4];
  const bool good = pinv_sweep<R, 256>(a.small, a.n, *reinterpret_cast<SweepLds<R>*>(lds), x);
  if (tid == 0) *a.good = good;
  const int i0 = tile_row(R, tid), j0 = tile_column(R, tid);
  if (good && tid < (R / 4) * (R / 4)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double d = d_entry<R>(a.small, a.n, i0 + i);
#pragma unroll
      for (int j = 0; j < 4; ++j) put_p<R>(a.p, i0 + i, j0 + j, (float)(-d * x[i][j]));
    }
  }
  // after the product the stored factor is the unnormalised one
  for (int r = tid; r < R; r += 256) a.small.scale[a.n][r] = 1.0;
}

}  // namespace hbcsf

#endif  // HBCSF_SMALL_H_
