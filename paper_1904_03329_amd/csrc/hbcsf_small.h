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

// The thread's number in its block; COUNTED: made of its wavefront's, `wave` (uniform), and its lane's.  Held from a kernel's
// beginning, as threadIdx is, it goes to memory and back in every wavefront of an MTTKRP that carries a guest and is held to 96
// registers (rank 16 on 5 M nonzeros, five iterations 835 -> 903 us); in other kernels the inverse is 1 us faster with threadIdx.
template <bool COUNTED>
__device__ __forceinline__ int thread_number(uint32_t wave) {
  if constexpr (COUNTED) return (int)(wave * 64u + __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)));
  else return threadIdx.x;
}

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
// All U threads of the block call (COUNTED, wave: thread_number()); x: the thread's tile of -V^-1.  False (for every thread) where a pivot is not safely
// positive: the eigenvalue form has to be taken.
template <int R>
struct SweepLds {
  __attribute__((aligned(16))) double row[2][R + 2];   // row k, then entry (k + 1, k + 1)
  double diag[R];
  double dmax;
  int good;
};

template <int R, int U, bool COUNTED = false>
__device__ __forceinline__ bool pinv_sweep(const SmallState& st, int n, SweepLds<R>& l, double (&x)[4][4], uint32_t wave = 0) {
  constexpr int T = small_threads(R), W = R / 4;
  static_assert(U >= T, "a thread per tile");
  const int tid = thread_number<COUNTED>(wave);
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

constexpr int pinv_threads(int R) { return R == 32 ? 256 : small_threads(R); }       // the eigenvalue form uses them all

// Pseudo-inverse of the symmetric matrix V by cyclic Jacobi rotations, n / 2 disjoint pairs at a time (round-robin
// pairing): only when V is not safely positive definite.  Eigenvalues below 1e-15 of the largest magnitude count as zero
// (the cut-off numpy.linalg.pinv applies to singular values).
// A round is a chain of its angles, the rotations and two barriers, some hundred rounds a matrix, so the matrix stays in
// LDS: a 2 x 2 block of row pair k and column pair l takes both its rotations from one thread, which loads all its blocks
// before it stores any.  So do the eigenvectors up to rank 64; at 128, where both do not fit, a wavefront keeps to its own
// rows of them in `qGlobal` ([R][R] scratch).  At rank 32 four wavefronts work on it, which wait while one sweeps: 1.6 ->
// 0.7 us a round.  One matrix with half the components equal takes 52 / 147 / 820 / 6200 us at ranks 16 / 32 / 64 / 128
// (150 / 1170 / 6000 / 52700 with both matrices in global memory; the host routine 23 / 180 / 1640 / 22600 and two copies).
// Two diagonal entries that would both count as zero are rotated only once the entry between them is no smaller than the
// others: rounding noise would turn them by any angle and stir what the sweep has just cleared back into their columns
// (half the components equal, rank 32: 7 sweeps instead of 12 to 17).
template <int R, int T = pinv_threads(R)>
struct JacobiLds {
  static constexpr bool kVectors = R <= 64;
  double a[R * R];
  double q[kVectors ? R * R : 1];
  double c[R / 2], s[R / 2], inv[R];
  double sums[3][T / 64];
  int2 pair[R / 2];
};

template <int R, int T = pinv_threads(R), bool COUNTED = false>
__device__ void jacobi_pinv(const SmallState& st, int n, JacobiLds<R, T>& lds, double* __restrict__ qGlobal, double* __restrict__ out,
                            uint32_t wave = 0) {
  constexpr int H = R / 2, S = T / H;   // S row pairs of a, or rows of q, at a time
  constexpr bool kVectors = JacobiLds<R, T>::kVectors;
  // blocks of a and rows of q a thread takes, and rows of q it holds at a time (with all eight at rank 128 it would spill)
  constexpr int KA = (H + S - 1) / S, KQ = (R + S - 1) / S, KB = kVectors ? KQ : 4;
  const int tid = thread_number<COUNTED>(wave);
  const int l = tid % H, first = tid / H;
  double* a = lds.a;
  double* q = kVectors ? lds.q : qGlobal;
  for (int e = tid; e < R * R; e += T) {
    a[e] = v_entry<R>(st, n, e / R, e % R);
    q[e] = e / R == e % R ? 1.0 : 0.0;
  }
  __syncthreads();
  for (int sweep = 0; sweep < 60; ++sweep) {
    double off = 0.0, diagonal = 0.0, most = 0.0;
    for (int e = tid; e < R * R; e += T) {
      const double x = a[e] * a[e];
      if (e / R == e % R) {
        diagonal += x;
        most = fmax(most, fabs(a[e]));
      } else {
        off += x;
      }
    }
    for (int o = 32; o > 0; o >>= 1) {
      off += __shfl_xor(off, o);
      diagonal += __shfl_xor(diagonal, o);
      most = fmax(most, __shfl_xor(most, o));
    }
    if ((tid & 63) == 0) {
      lds.sums[0][tid >> 6] = off;
      lds.sums[1][tid >> 6] = diagonal;
      lds.sums[2][tid >> 6] = most;
    }
    __syncthreads();
    off = diagonal = most = 0.0;
    for (int w = 0; w < T / 64; ++w) {
      off += lds.sums[0][w];
      diagonal += lds.sums[1][w];
      most = fmax(most, lds.sums[2][w]);
    }
    if (off <= 1e-30 * diagonal || off == 0.0) break;   // the same for every thread
    const double small = 1e-15 * most, least = off / (R * R);
    for (int round = 0; round < R - 1; ++round) {
      // pair k of this round: players 0 (fixed) and 1 .. R-1 (rotating)
      auto player = [&](int slot) {
        const int x = slot - 1 + round;
        return slot == 0 ? 0 : 1 + (x >= R - 1 ? x - (R - 1) : x);
      };
      if (tid < H) {
        const int x = player(tid), y = player(R - 1 - tid);
        const int p = x < y ? x : y, r = x < y ? y : x;
        const double app = a[p * R + p], arr = a[r * R + r], apr = a[p * R + r];
        // t = tan of the angle, the smaller root: tan(2 angle) = 2 apr / (arr - app)
        const double d = arr - app, h = 2.0 * apr, dh = fma(d, d, h * h);
        double c = 1.0, sn = 0.0;
        const bool skip = fabs(app) <= small && fabs(arr) <= small && apr * apr < least;
        if (apr != 0.0 && !skip && !(dh <= 1e-280)) {
          const double t = (d >= 0 ? h : -h) * reciprocal(fabs(d) + dh * reciprocal_root(dh));
          c = reciprocal_root(fma(t, t, 1.0));
          sn = t * c;
        }
        lds.c[tid] = c;
        lds.s[tid] = sn;
        lds.pair[tid] = make_int2(p, r);
      }
      __syncthreads();
      const int2 cols = lds.pair[l];
      const double cl = lds.c[l], sl = lds.s[l];
      double x[KA][4], y[KB][2];
      auto load_vectors = [&](int from) {
#pragma unroll
        for (int m = 0; m < KB; ++m) {
          const int row = first + (from + m) * S;
          if (row < R) {
            y[m][0] = q[row * R + cols.x];
            y[m][1] = q[row * R + cols.y];
          }
        }
      };
      auto turn_vectors = [&](int from) {
#pragma unroll
        for (int m = 0; m < KB; ++m) {
          const int row = first + (from + m) * S;
          if (row < R) {
            q[row * R + cols.x] = cl * y[m][0] - sl * y[m][1];
            q[row * R + cols.y] = sl * y[m][0] + cl * y[m][1];
          }
        }
      };
#pragma unroll
      for (int m = 0; m < KA; ++m) {
        const int k = first + m * S;
        if (k < H) {
          const int2 rows = lds.pair[k];
          x[m][0] = a[rows.x * R + cols.x];
          x[m][1] = a[rows.x * R + cols.y];
          x[m][2] = a[rows.y * R + cols.x];
          x[m][3] = a[rows.y * R + cols.y];
        }
      }
      if (kVectors) load_vectors(0);
#pragma unroll
      for (int m = 0; m < KA; ++m) {
        const int k = first + m * S;
        if (k < H) {
          const int2 rows = lds.pair[k];
          const double ck = lds.c[k], sk = lds.s[k];
          const double p0 = cl * x[m][0] - sl * x[m][1], p1 = sl * x[m][0] + cl * x[m][1];
          const double r0 = cl * x[m][2] - sl * x[m][3], r1 = sl * x[m][2] + cl * x[m][3];
          a[rows.x * R + cols.x] = ck * p0 - sk * r0;
          a[rows.y * R + cols.x] = sk * p0 + ck * r0;
          a[rows.x * R + cols.y] = ck * p1 - sk * r1;
          a[rows.y * R + cols.y] = sk * p1 + ck * r1;
        }
      }
      if (kVectors) {
        turn_vectors(0);
      } else {
        for (int from = 0; from < KQ; from += KB) {
          load_vectors(from);
          turn_vectors(from);
        }
      }
      __syncthreads();
    }
  }
  double wmax = 0.0;
  for (int k = 0; k < R; ++k) wmax = fmax(wmax, fabs(a[k * R + k]));
  for (int k = tid; k < R; k += T) {
    const double w = a[k * R + k];
    lds.inv[k] = fabs(w) <= 1e-15 * wmax ? 0.0 : 1.0 / w;   // (a NaN is not small)
  }
  __syncthreads();
  if constexpr (!kVectors) {
    for (int e = tid; e < R * R; e += T) a[e] = q[e];
    __syncthreads();
    q = a;
  }
  // the terms of entry (i, j) from number i + j on: neighbouring threads then read different LDS banks, and (j, i) adds
  // the same terms in the same order
  for (int e = tid; e < R * R; e += T) {
    const int i = e / R, j = e % R;
    double t = 0.0;
    for (int m = 0; m < R; ++m) {
      const int k = (i + j + m) & (R - 1);
      if (lds.inv[k] != 0.0) t += q[i * R + k] * lds.inv[k] * q[j * R + k];
    }
    out[e] = t;
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------------------------------
// Guest of an MTTKRP launch (its first block of 256 threads, rank <= 64): inverts V for the update that the MTTKRP belongs to.
// Nothing the MTTKRP reads or writes is touched, and nothing here is needed before the product that follows it, so the
// chain of R dependent steps runs beside the MTTKRP instead of before it (5 iterations, 5 M nonzeros at rank 32 1381 ->
// 1290 us, 0.8 M at rank 64 1204 -> 916).  *good = 0: the eigenvalue form is needed.  (The sum of the slots would
// fit in beside it, but not for nothing: the blocks that sum have to hand over to the one that inverts, and with agent-scope
// fences for that, which write an L2 back, the MTTKRP of a small tensor took 70 instead of 28 us.)
// ---------------------------------------------------------------------------------------------------
// Up to rank 32 the eigenvalue form follows in the same block, where its two matrices fit the LDS that four wavefronts' staging
// takes anyway: with it in a launch of its own every update waited 1.5 to 4.6 us for a kernel that nearly always has nothing to do
// (five iterations, two runs each: 50 000 nonzeros at rank 32 432, 458 -> 411, 405 us, 0.3 M of order 4 at rank 8 491, 518 -> 468,
// 459, 5 M at rank 32 1239, 1254 -> 1233, 1235).  At rank 64 its 68 KB would hold every block of the launch to two on a compute
// unit.
constexpr bool guest_finishes(int rank) { return rank <= 32; }

template <int R>
constexpr uint32_t guest_lds_bytes() {
  constexpr uint32_t sweep = sizeof(SweepLds<R>), form = guest_finishes(R) ? sizeof(JacobiLds<R, 256>) : 0;
  return sweep > form ? sweep : form;
}

template <int R, bool COUNTED>
__device__ __forceinline__ void guest_block(const GuestArgs& a, uint32_t* lds, uint32_t wave) {
  static_assert(R <= 64, "one block of 256 threads inverts V");
  const int tid = thread_number<COUNTED>(wave);
  double x[4][4];
  bool done = pinv_sweep<R, 256, COUNTED>(a.small, a.n, *reinterpret_cast<SweepLds<R>*>(lds), x, wave);
  if (tid == 0) __hip_atomic_store(a.good, (int)done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // read beside, too
  const int i0 = tile_row(R, tid), j0 = tile_column(R, tid);
  if constexpr (guest_finishes(R)) {
    if (!done) {
      if (tid == 0) a.stamp[1] = wall_clock64();
      __syncthreads();   // the sweep's part of the LDS is read no more
      jacobi_pinv<R, 256, COUNTED>(a.small, a.n, *reinterpret_cast<JacobiLds<R, 256>*>(lds), nullptr, a.vp, wave);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) x[i][j] = -a.vp[(i0 + i) * R + j0 + j];
      done = true;
    }
  }
  if (done && tid < (R / 4) * (R / 4)) {
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
