// CPD-ALS iteration around the MTTKRP kernels (Section II-B, Eq. 1-3, Algorithm "CPD-ALS"): the dense
// steps of a mode update -- Gram matrix of a tall factor, product with the R x R pseudo-inverse, the R x R algebra
// between them -- as gfx950 kernels, and the C entry points that tie them to hbcsf_mttkrp.
//
// Every mode update runs on the device from end to end; the host only enqueues, and waits once at the end of an
// iteration (or, where no iteration's fit decides anything, once at the end of the run):
//   V = Hadamard of the other factors' Gram matrices, P = V^+      (fp64, one workgroup: small_pinv_kernel, or up to rank
//                                                                   64 a block of the MTTKRP launch)
//   M = MTTKRP
//   ordinary call:   S = M^T M;  A_n^T A_n = V^+ S V^+ without another pass over the rows, and its diagonal gives the
//                    column norms, so the product A_n = M P is written normalised in the pass that computes it
//   put-off call:    A_n = M P unnormalised and G = A_n^T A_n (in the same pass for R <= 32)
// The algorithm normalises after all modes are updated; writing a factor with another column scaling scales the next
// MTTKRP's columns by a known diagonal, which is folded back into the R x R matrices (column scaling commutes with
// every step), so the result is that of the algorithm's order up to rounding.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "hbcsf.h"
#include "hbcsf_small.h"
#include "hbcsf_tensor.h"

using namespace hbcsf;

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Steps of 32 rows between two flushes of the fp32 partial sums into fp64: rank 32 sums 128 rows in fp32 (relative error
// of the matrix 1.0e-8 on 30 011 uniform rows, 1.7e-9 on 1 M), the other ranks 32 rows (2.9e-9 and 5e-10; with 128 rows
// 1.0e-8 and 1.8e-9).
constexpr int gram_flush(int R) { return R == 32 ? 4 : 1; }

// ---------------------------------------------------------------------------------------------------
// Gram matrix S = A^T A of a tall matrix in two steps, without atomics and therefore with the same bits on
// every run: each block writes the partial sums of its rows (all R x R entries, zeros included) to its own
// slot of a scratch buffer, and a second kernel adds the slots in block order.
//
// R <= 32: the 32x32x2 fp32 matrix instruction over the matrix taken as rows of 32 floats (R < 32: 32 / R rows side by
// side; their R x R Gram matrices are the diagonal blocks of the 32 x 32 product and are added when the slot is
// written).  One instruction consumes two 32-float rows: lane (h = lane / 32, c = lane % 32) supplies element c of row
// 2u + h as both operands, since the left operand is the transpose of the right one.  A wavefront walks a contiguous
// chunk of rows, sixteen coalesced 256-byte loads in flight; partial sums leave fp32 every gram_flush(R) steps of 32.
// Accumulator register v of a lane holds entry (8 (v / 4) + 4 h + v % 4, c).
// ---------------------------------------------------------------------------------------------------
// Writes a block's slot from its wavefronts' 32 x 32 sums: R x R entries, the diagonal blocks added up.
template <int R>
__device__ __forceinline__ void write_slot32(const double (*red)[1024], double* __restrict__ mine) {
  for (int e = threadIdx.x; e < R * R; e += 256) {
    double t = 0.0;
#pragma unroll
    for (int b = 0; b < 32 / R; ++b) {
      const int at = (b * R + e / R) * 32 + b * R + e % R;
      t += (red[0][at] + red[1][at]) + (red[2][at] + red[3][at]);
    }
    mine[e] = t;
  }
}

// rows: of 32 floats, the last one perhaps cut at `total` floats.
template <int R>
__global__ __launch_bounds__(256) void gram32_partial_kernel(const float* __restrict__ a, uint64_t rows, uint64_t total,
                                                             uint64_t rowsPerWave, double* __restrict__ partial,
                                                             unsigned long long* __restrict__ stamp) {
  __shared__ double red[4][1024];
  if (stamp && blockIdx.x == 0 && threadIdx.x == 0) *stamp = wall_clock64();
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int h = lane >> 5, c = lane & 31;
  const uint64_t w = (uint64_t)blockIdx.x * 4 + wave;
  uint64_t r0 = w * rowsPerWave;
  const uint64_t r1 = (r0 + rowsPerWave < rows) ? r0 + rowsPerWave : rows;
  double acc64[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc64[v] = 0.0;
  while (r0 < r1) {
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    for (int it = 0; it < gram_flush(R) && r0 < r1; ++it, r0 += 32) {
      float x[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const uint64_t r = r0 + 2 * u + h;
        x[u] = (r < r1 && (R == 32 || r * 32 + c < total)) ? __builtin_nontemporal_load(a + r * 32 + c) : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[u], x[u], acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) acc64[v] += (double)acc[v];
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) red[wave][(8 * (v / 4) + 4 * h + (v % 4)) * 32 + c] = acc64[v];
  __syncthreads();
  write_slot32<R>(red, partial + (size_t)blockIdx.x * (R * R));
}

// R = 64, 128: S is symmetric, so a block's wavefronts take one pair (i <= j) of 32-column tiles each (3 or 10 of them)
// and all walk the same rows, whose lines the first brings into the L1; a pair is accumulated as above, with tile i's
// elements as left and tile j's as right operands, and written to both its places.
constexpr int tile_pairs(int R) { return (R / 32) * (R / 32 + 1) / 2; }

template <int R>
__global__ __launch_bounds__(64 * tile_pairs(R)) void gram_tiles_partial_kernel(const float* __restrict__ a, uint64_t rows,
                                                                                uint64_t rowsPerBlock,
                                                                                double* __restrict__ partial,
                                                                                unsigned long long* __restrict__ stamp) {
  if (stamp && blockIdx.x == 0 && threadIdx.x == 0) *stamp = wall_clock64();
  const int lane = threadIdx.x & 63;
  const int h = lane >> 5, c = lane & 31;
  int i = 0, j = threadIdx.x >> 6;            // wavefront number -> tile pair
  while (j >= R / 32 - i) {
    j -= R / 32 - i;
    ++i;
  }
  j += i;
  uint64_t r0 = (uint64_t)blockIdx.x * rowsPerBlock;
  const uint64_t r1 = (r0 + rowsPerBlock < rows) ? r0 + rowsPerBlock : rows;
  double acc64[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc64[v] = 0.0;
  while (r0 < r1) {
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    for (int it = 0; it < gram_flush(R) && r0 < r1; ++it, r0 += 32) {
      float x[16], y[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const uint64_t r = r0 + 2 * u + h;
        x[u] = r < r1 ? a[r * R + 32 * i + c] : 0.f;
        y[u] = r < r1 ? a[r * R + 32 * j + c] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[u], y[u], acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) acc64[v] += (double)acc[v];
  }
  double* mine = partial + (size_t)blockIdx.x * (R * R);
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int row = 32 * i + 8 * (v / 4) + 4 * h + (v % 4), col = 32 * j + c;
    mine[row * R + col] = acc64[v];
    if (i != j) mine[col * R + row] = acc64[v];
  }
}

// s[e] = sum over the blocks' slots, in block order.  16 entries x 64 interleaved block subsets per workgroup (128
// contiguous bytes per slot and enough workgroups to spread a few MB of slots over the chip; 64 x 16 took 11.5 us for
// 780 slots of rank 32); the 64 subset sums are added in a fixed order.
__global__ __launch_bounds__(1024) void gram_reduce_kernel(const double* __restrict__ partial, uint32_t nSlots,
                                                           uint32_t rr, double* __restrict__ s) {
  __shared__ double part[64][17];
  const int el = threadIdx.x & 15, q = threadIdx.x >> 4;
  const uint32_t e = blockIdx.x * 16u + (uint32_t)el;
  double t = 0.0;
  for (uint32_t b = (uint32_t)q; b < nSlots; b += 64) t += partial[(size_t)b * rr + e];
  part[q][el] = t;
  __syncthreads();
  for (int half = 32; half > 0; half >>= 1) {
    if (q < half) part[q][el] += part[q + half][el];
    __syncthreads();
  }
  if (q == 0) s[e] = part[0][el];
}

// dots[block] = sum of v over the block's W wavefronts, in a fixed order.
template <int W>
__device__ __forceinline__ void block_dot(double v, double* __restrict__ dots) {
  __shared__ double part[W];
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = part[0];
#pragma unroll
    for (int w = 1; w < W; ++w) t += part[w];
    dots[blockIdx.x] = t;
  }
}

// 32 rows of 32 floats that a wavefront turns from the row layout of its loads into the layout of a product tile: row stride
// 36, so that whole float4s are written.  The `count` float4s x[first ..] of row c from column `from` on; then the sum of the
// products with acc.
constexpr int kTurnStride = 36;
template <int first, int count, int n>
__device__ __forceinline__ void put_rows(float* turned, int c, int from, const float4 (&x)[n]) {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int q = 0; q < count; ++q) *reinterpret_cast<float4*>(turned + c * kTurnStride + from + 4 * q) = x[first + q];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}
__device__ __forceinline__ void add_dot(const float* turned, int h, int c, const f32x16& acc, double& dot) {
#pragma unroll
  for (int v = 0; v < 16; ++v)
    dot = fma((double)turned[(8 * (v / 4) + 4 * h + (v % 4)) * kTurnStride + c], (double)acc[v], dot);
}

// R <= 32: out = M P for blocks of 32 rows of 32 floats (R < 32: P is the block-diagonal matrix of 32 / R copies).  The
// contraction index is split as k = 16 h + t so that lane (h, c) reads the 64 contiguous bytes M[row c of the
// block][16 h .. 16 h + 15] as its sixteen left operands, and holds P[16 h + t][c] as the sixteen right operands for
// the whole kernel.
// GRAM: in the same pass the Gram matrix of the rows just computed: the 32 x 32 product tile leaves the matrix unit as
// sixteen registers whose lane (h, c) entries are out[row 8 (v / 4) + 4 h + v % 4][c], i.e. for every v two different
// rows of the tile with lane c on column c -- exactly the operand shape of gram32_partial_kernel -- so sixteen more
// matrix instructions add the tile's out^T out without moving any data.  The partial Gram sums go to the block's
// scratch slot (reduced by gram_reduce_kernel), so M is read once per mode update instead of twice.
// DOTS (with GRAM): dots receives per block the sum of M[i][r] out[i][r] over its entries, i.e. <X, model> of these factors
// once the blocks' sums are added.  M's entries reach the product tile's layout through LDS, in what the end of the kernel
// sums in (five iterations whose last mode has 5 M rows of 32: 4.81 ms with M loaded a second time, 3.30 this way, 3.40
// without the sum in the code before it); an instantiation of its own, since only an iteration's last mode asks for it.
template <int R, bool GRAM, bool DOTS>
__global__ __launch_bounds__(256, DOTS ? 3 : 1) void apply32_kernel(const float* __restrict__ m, uint64_t rows, uint64_t total,
                                                      const float* __restrict__ p, float* __restrict__ out,
                                                      uint64_t blocksPerWave, double* __restrict__ partial,
                                                      double* __restrict__ dots,
                                                      unsigned long long* __restrict__ stamp) {
  if (stamp && blockIdx.x == 0 && threadIdx.x == 0) *stamp = wall_clock64();
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int h = lane >> 5, c = lane & 31;
  double dot = 0.0;
  __shared__ double red[GRAM ? 4 : 1][1024];
  float* turned = reinterpret_cast<float*>(red[GRAM ? wave : 0]);   // DOTS: a wavefront's 32 rows of M
  float pb[16];
#pragma unroll
  for (int t = 0; t < 16; ++t) pb[t] = p[(16 * h + t) * 32 + c];
  const uint64_t w = (uint64_t)blockIdx.x * 4 + wave;
  const uint64_t nBlocks = (rows + 31) / 32;
  uint64_t b = w * blocksPerWave;
  const uint64_t bEnd = (b + blocksPerWave < nBlocks) ? b + blocksPerWave : nBlocks;
  double acc64[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc64[v] = 0.0;
  // the next block's rows are in flight while the matrix unit works on this one's
  auto load = [&](float4 (&x)[4], uint64_t block) {
    const uint64_t at = (block * 32 + c) * 32 + 16 * h;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      x[q] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (at + 4 * q < total) x[q] = *reinterpret_cast<const float4*>(m + at + 4 * q);
    }
  };
  float4 next[4];
  if (b < bEnd) load(next, b);
  while (b < bEnd) {
    f32x16 gacc;
#pragma unroll
    for (int v = 0; v < 16; ++v) gacc[v] = 0.f;
    for (int it = 0; it < gram_flush(R) && b < bEnd; ++it, ++b) {
      float4 x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = next[q];
      if (b + 1 < bEnd) load(next, b + 1);
      if constexpr (DOTS) put_rows<0, 4>(turned, c, 16 * h, x);
      f32x16 acc;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[q].x, pb[4 * q + 0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[q].y, pb[4 * q + 1], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[q].z, pb[4 * q + 2], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[q].w, pb[4 * q + 3], acc, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint64_t to = (b * 32 + (uint64_t)(8 * (v / 4) + 4 * h + (v % 4))) * 32 + c;
        if (to < total) __builtin_nontemporal_store(acc[v], out + to);
      }
      if constexpr (DOTS) add_dot(turned, h, c, acc, dot);  // (a row past the end is zero)
      if (GRAM) {
        // rows past the end of the matrix were computed from zeros and add nothing
#pragma unroll
        for (int v = 0; v < 16; ++v) gacc = __builtin_amdgcn_mfma_f32_32x32x2f32(acc[v], acc[v], gacc, 0, 0, 0);
      }
    }
    if (GRAM) {
#pragma unroll
      for (int v = 0; v < 16; ++v) acc64[v] += (double)gacc[v];
    }
  }
  if constexpr (GRAM) {
    if constexpr (DOTS) __syncthreads();
#pragma unroll
    for (int v = 0; v < 16; ++v) red[wave][(8 * (v / 4) + 4 * h + (v % 4)) * 32 + c] = acc64[v];
    __syncthreads();
    write_slot32<R>(red, partial + (size_t)blockIdx.x * (R * R));
    if constexpr (DOTS) block_dot<4>(dot, dots);
  }
}

// R = 64, 128: out = M P; a wavefront takes 32 rows x 32 columns (tile column q = wavefront of the block), the block's
// wavefronts share the rows.  The contraction index is split as k = (R / 2) h + t, so a lane reads 2 R contiguous bytes
// of its row and keeps its R / 2 right operands for the whole kernel.  DOTS: as in apply32_kernel; the 32 columns of a
// wavefront's tile are in the registers of one half of its lanes.
template <int R, bool DOTS>
__global__ __launch_bounds__(2 * R) void apply_tiles_kernel(const float* __restrict__ m, uint64_t rows,
                                                            const float* __restrict__ p, float* __restrict__ out,
                                                            uint64_t rowBlocksPerBlock, double* __restrict__ dots,
                                                            unsigned long long* __restrict__ stamp) {
  if (stamp && blockIdx.x == 0 && threadIdx.x == 0) *stamp = wall_clock64();
  constexpr int K = R / 2;
  const int lane = threadIdx.x & 63;
  const int q = threadIdx.x >> 6;
  const int h = lane >> 5, c = lane & 31;
  double dot = 0.0;
  __shared__ __align__(16) float turned[DOTS ? R / 32 : 1][32 * kTurnStride];
  float pb[K];
#pragma unroll
  for (int t = 0; t < K; ++t) pb[t] = p[(K * h + t) * R + 32 * q + c];
  const uint64_t nBlocks = (rows + 31) / 32;
  uint64_t b = (uint64_t)blockIdx.x * rowBlocksPerBlock;
  const uint64_t bEnd = (b + rowBlocksPerBlock < nBlocks) ? b + rowBlocksPerBlock : nBlocks;
  for (; b < bEnd; ++b) {
    const uint64_t r = b * 32 + c;
    float4 x[K / 4];
#pragma unroll
    for (int t = 0; t < K / 4; ++t) x[t] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (r < rows) {
      const float4* src = reinterpret_cast<const float4*>(m + r * R + K * h);
#pragma unroll
      for (int t = 0; t < K / 4; ++t) x[t] = src[t];
    }
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int t = 0; t < K / 4; ++t) {
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[t].x, pb[4 * t + 0], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[t].y, pb[4 * t + 1], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[t].z, pb[4 * t + 2], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[t].w, pb[4 * t + 3], acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const uint64_t ro = b * 32 + (uint64_t)(8 * (v / 4) + 4 * h + (v % 4));
      if (ro < rows) __builtin_nontemporal_store(acc[v], out + ro * R + 32 * q + c);
    }
    if constexpr (DOTS) {
      if (h == 32 * q / K) {
        if (K == 64 && (q & 1)) put_rows<K == 64 ? 8 : 0, 8>(turned[q], c, 0, x);
        else put_rows<0, 8>(turned[q], c, 0, x);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      add_dot(turned[q], h, c, acc, dot);
    }
  }
  if constexpr (DOTS) block_dot<R / 32>(dot, dots);
}

// a[i][r] *= s[r]: the column normalisation of Algorithm "CPD-ALS" when it was put off.
__global__ __launch_bounds__(256) void scale_columns_kernel(float4* __restrict__ a, uint64_t nvec,
                                                            const float* __restrict__ s, int vecPerRow) {
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < nvec; i += (uint64_t)gridDim.x * 256) {
    const float4 sc = reinterpret_cast<const float4*>(s)[i % (uint64_t)vecPerRow];
    float4 v = a[i];
    v.x *= sc.x; v.y *= sc.y; v.z *= sc.z; v.w *= sc.w;
    a[i] = v;
  }
}

// Scratch of the Gram computation: one R x R fp64 slot per block.  At most kGramSlotsMax blocks, fewer when the
// scratch buffer is smaller; any number of blocks >= 1 gives the same sum up to fp64 rounding.
constexpr uint32_t kGramSlotsMax = 1024;
constexpr uint32_t kDotsMax = 4096;   // blocks of a product kernel that leaves <M, out> (at most kGramSlotsMax for R <= 32)
constexpr uint64_t kGramWorkspaceCap = 32ull << 20;   // hbcsf_gram_workspace_bytes never asks for more

uint32_t gram_slots_for(int rank, uint64_t scratchBytes) {
  const uint64_t fit = scratchBytes / ((uint64_t)rank * rank * 8);
  return (uint32_t)(fit < kGramSlotsMax ? fit : kGramSlotsMax);
}

// The matrix as rows of 32 floats (R < 32: 32 / R rows in each).
uint64_t rows_of_32(uint64_t rows, int rank) { return (rows * (uint64_t)rank + 31) / 32; }

void launch_reduce(const double* scratch, uint32_t used, int rank, double* s, hipStream_t st) {
  const uint32_t rr = (uint32_t)(rank * rank);
  hipLaunchKernelGGL(gram_reduce_kernel, dim3(rr / 16), dim3(1024), 0, st, scratch, used, rr, s);
}

// s (device, [R][R] fp64) = a^T a; scratch holds `slots` R x R fp64 partial sums (slots >= 1).  Nothing has to be
// cleared between calls: every launched block writes its whole slot, and only the launched blocks' slots are read.
void launch_gram(const float* a, uint64_t rows, int rank, double* scratch, uint32_t slots, double* s, int numCU,
                 hipStream_t st, unsigned long long* stamp = nullptr) {
  uint32_t used = 0;
  if (rows > 0 && rank <= 32) {
    // a wavefront takes at least four steps of 32 rows, so that the slots stay a small part of the traffic; at ranks 8 and
    // 16 (512 and 2048 bytes a slot) one, since its steps come one after the other: 1001 rows 21.5 -> 18.0 us a call
    const uint64_t n = rows_of_32(rows, rank), total = rows * (uint64_t)rank;
    const uint64_t least = rank < 32 ? 32 : 4 * 32;
    uint64_t waves = (uint64_t)numCU * 16;
    if (waves > (uint64_t)slots * 4) waves = (uint64_t)slots * 4;
    uint64_t per = (n + waves - 1) / waves;
    per = (per + 31) / 32 * 32;
    if (per < least && slots > 1) per = least;
    const uint64_t nWaves = (n + per - 1) / per;
    used = (uint32_t)((nWaves + 3) / 4);
    switch (rank) {
      case 8: hipLaunchKernelGGL(gram32_partial_kernel<8>, dim3(used), dim3(256), 0, st, a, n, total, per, scratch, stamp); break;
      case 16: hipLaunchKernelGGL(gram32_partial_kernel<16>, dim3(used), dim3(256), 0, st, a, n, total, per, scratch, stamp); break;
      default: hipLaunchKernelGGL(gram32_partial_kernel<32>, dim3(used), dim3(256), 0, st, a, n, total, per, scratch, stamp); break;
    }
  } else if (rows > 0) {
    uint64_t blocks = (uint64_t)numCU * 4;
    if (blocks > slots) blocks = slots;
    uint64_t per = (rows + blocks - 1) / blocks;
    per = (per + 31) / 32 * 32;
    if (per < 4 * 32 && slots > 1) per = 4 * 32;
    used = (uint32_t)((rows + per - 1) / per);
    if (rank == 64)
      hipLaunchKernelGGL(gram_tiles_partial_kernel<64>, dim3(used), dim3(64 * tile_pairs(64)), 0, st, a, rows, per, scratch, stamp);
    else
      hipLaunchKernelGGL(gram_tiles_partial_kernel<128>, dim3(used), dim3(64 * tile_pairs(128)), 0, st, a, rows, per, scratch, stamp);
  }
  // with no rows no slot is read and the result is all zeros
  launch_reduce(scratch, used, rank, s, st);
}

template <int R>
void launch_apply32(const float* m, uint64_t n, uint64_t total, const float* p, float* out, uint64_t per, uint32_t blocks,
                    double* scratch, double* dots, unsigned long long* stamp, hipStream_t st) {
  auto kernel = !scratch ? apply32_kernel<R, false, false> : dots ? apply32_kernel<R, true, true> : apply32_kernel<R, true, false>;
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, st, m, n, total, p, out, per, scratch, dots, stamp);
}

// out = m p, and with g: g (device, [R][R] fp64) = out^T out (in the same pass over m for R <= 32).  p: [R][R], for
// R < 32 the [32][32] block-diagonal matrix of it.  dots (with g only, [kDotsMax]): <m, out> as one sum per block; returns
// how many there are.
uint32_t launch_apply(const float* m, uint64_t rows, int rank, const float* p, float* out, double* scratch, uint32_t slots,
                      double* g, double* dots, int numCU, hipStream_t st, unsigned long long* stamp) {
  uint32_t used = 0;
  if (rank > 32) {
    if (rows > 0) {
      const uint64_t nBlocks = (rows + 31) / 32;
      uint64_t blocks = (uint64_t)numCU * 16;
      if (blocks > kDotsMax) blocks = kDotsMax;
      const uint64_t per = (nBlocks + blocks - 1) / blocks;
      used = (uint32_t)((nBlocks + per - 1) / per);
      if (rank == 64)
        hipLaunchKernelGGL((dots ? apply_tiles_kernel<64, true> : apply_tiles_kernel<64, false>), dim3(used), dim3(128), 0, st,
                           m, rows, p, out, per, dots, stamp);
      else
        hipLaunchKernelGGL((dots ? apply_tiles_kernel<128, true> : apply_tiles_kernel<128, false>), dim3(used), dim3(256), 0, st,
                           m, rows, p, out, per, dots, stamp);
    }
    if (g) launch_gram(out, rows, rank, scratch, slots, g, numCU, st);
    return used;
  }
  if (rows > 0) {
    const uint64_t n = rows_of_32(rows, rank), total = rows * (uint64_t)rank;
    const uint64_t nBlocks = (n + 31) / 32;
    uint64_t waves = (uint64_t)numCU * 32;
    if (g && waves > (uint64_t)slots * 4) waves = (uint64_t)slots * 4;
    uint64_t per = (nBlocks + waves - 1) / waves;
    if (g && per < 2) per = 2;   // fewer slots to add up
    used = (uint32_t)(((nBlocks + per - 1) / per + 3) / 4);
    double* sc = g ? scratch : nullptr;
    switch (rank) {
      case 8: launch_apply32<8>(m, n, total, p, out, per, used, sc, dots, stamp, st); break;
      case 16: launch_apply32<16>(m, n, total, p, out, per, used, sc, dots, stamp, st); break;
      default: launch_apply32<32>(m, n, total, p, out, per, used, sc, dots, stamp, st); break;
    }
  }
  if (g) launch_reduce(scratch, used, rank, g, st);
  return used;
}

void launch_scale_columns(float* a, uint64_t rows, int rank, const float* s, int numCU, hipStream_t st) {
  if (rows == 0) return;
  const uint64_t nvec = rows * (uint64_t)(rank / 4);
  uint64_t blocks = (nvec + 255) / 256;
  const uint64_t cap = (uint64_t)numCU * 32;
  if (blocks > cap) blocks = cap;
  hipLaunchKernelGGL(scale_columns_kernel, dim3((unsigned)blocks), dim3(256), 0, st, reinterpret_cast<float4*>(a),
                     nvec, s, rank / 4);
}

// ---------------------------------------------------------------------------------------------------
// R x R algebra on the device (fp64).  State per mode m, in the caller's workspace: gram[m] = Gram matrix of the stored
// factor, scale[m] = c_m (the algorithm's factor is the stored one with column r divided by c_m[r]), norm[m] = column
// norms of the last update.  These kernels are one workgroup each (the work is R^3 at most 2 M multiply-adds in a serial
// chain of R steps); what they replace is a copy to the host, a wait, and a copy back for every mode update.
// ---------------------------------------------------------------------------------------------------
constexpr int entry_threads(int R) { return R * R < 1024 ? R * R : 1024; }           // for kernels that walk R x R entries

// vp = V^+ for the update of mode n, and p = diag(d) V^+ (the right-hand matrix of a put-off update; an ordinary update
// overwrites it).  A pivot of the sweep that is not safely positive sends the whole workgroup to the eigenvalue form.
// resetScale: after the product the stored factor is the unnormalised one, so its column scale becomes 1.
// hosted: null, or the outcome of the sweep that ran beside the MTTKRP: where that was good, all is done, and where it was
// not only the eigenvalue form is left (ranks that guest_finishes() leaves to this).  stamp: when it begins and ends
// (nothing where all is done).
template <int R>
__global__ __launch_bounds__(pinv_threads(R)) void small_pinv_kernel(SmallState st, int n, double* __restrict__ vp,
                                                                      float* __restrict__ p, double* __restrict__ jq,
                                                                      int resetScale, const int* __restrict__ hosted,
                                                                      unsigned long long* __restrict__ stamp) {
  constexpr int U = pinv_threads(R), W = R / 4;
  __shared__ SweepLds<R> sweep;
  __shared__ double d[R];
  __shared__ JacobiLds<R> jl;
  const int tid = threadIdx.x;
  if (hosted && *hosted) return;
  if (tid == 0 && stamp) stamp[0] = wall_clock64();
  const bool owns = tid < W * W;
  const int i0 = tile_row(R, tid), j0 = tile_column(R, tid);
  for (int r = tid; r < R; r += U) d[r] = d_entry<R>(st, n, r);
  double x[4][4];
  const bool good = !hosted && pinv_sweep<R, U>(st, n, sweep, x);
  if (good) {
    if (owns) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          x[i][j] = -x[i][j];
          vp[(i0 + i) * R + j0 + j] = x[i][j];
        }
    }
  } else {
    __syncthreads();
    jacobi_pinv<R>(st, n, jl, jq, vp);
    if (owns) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) x[i][j] = vp[(i0 + i) * R + j0 + j];
    }
  }
  if (owns) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) put_p<R>(p, i0 + i, j0 + j, (float)(d[i0 + i] * x[i][j]));
  }
  if (resetScale)
    for (int r = tid; r < R; r += U) st.scale[n][r] = 1.0;
  if (tid == 0 && stamp) stamp[1] = wall_clock64();
}

// c = a b (fp64, [R][R]); one entry per thread.  da: null, or b's rows and columns are scaled by d first (S of the
// algorithm from S of the stored factors).
template <int R>
__global__ __launch_bounds__(256) void small_matmul_kernel(const double* __restrict__ a, const double* __restrict__ b,
                                                           double* __restrict__ c, SmallState st, int n, int scaled,
                                                            unsigned long long* __restrict__ stamp) {
  const int id = blockIdx.x * 256 + threadIdx.x;
  if (id == 0 && stamp) *stamp = wall_clock64();
  if (id >= R * R) return;
  const int i = id / R, j = id % R;
  double t = 0.0;
  for (int k = 0; k < R; ++k) {
    double bk = b[k * R + j];
    if (scaled) bk *= d_entry<R>(st, n, k);
    t = fma(a[i * R + k], bk, t);
  }
  if (scaled) t *= d_entry<R>(st, n, j);
  c[id] = t;
}

// Ordinary update of mode n: t = A_n^T A_n = V^+ S V^+.  The column norms, the matrix that writes the factor with
// unit-norm columns, the stored factor's Gram matrix and scale, and (last mode) <X, model> = trace(S V^+).
template <int R>
__global__ __launch_bounds__(entry_threads(R)) void small_update_kernel(SmallState st, int n, const double* __restrict__ t,
                                                                        const double* __restrict__ vp,
                                                                        const double* __restrict__ s, float* __restrict__ p,
                                                                        double* __restrict__ inner) {
  constexpr int T = entry_threads(R);
  __shared__ double norm[R], d[R], part[T];
  const int tid = threadIdx.x;
  for (int r = tid; r < R; r += T) {
    const double g = t[r * R + r];
    norm[r] = g > 0.0 ? sqrt(g) : 1.0;
    d[r] = d_entry<R>(st, n, r);
  }
  __syncthreads();
  double sum = 0.0;
  for (int e = tid; e < R * R; e += T) {
    const int i = e / R, j = e % R;
    put_p<R>(p, i, j, (float)(d[i] * vp[e] / norm[j]));
    st.gram[n][e] = t[e] / (norm[i] * norm[j]);
    sum += s[e] * d[i] * d[j] * vp[j * R + i];
  }
  part[tid] = sum;
  __syncthreads();
  for (int half = T / 2; half > 0; half >>= 1) {
    if (tid < half) part[tid] += part[tid + half];
    __syncthreads();
  }
  if (tid == 0) *inner = part[0];
  for (int r = tid; r < R; r += T) {
    st.norm[n][r] = norm[r];
    st.scale[n][r] = 1.0 / norm[r];
  }
}

// End of an iteration: lambda_r = product over the modes of the column norms, the model's squared norm from the Gram
// matrices of the unnormalised factors, <X, model>; then the algorithm's closing normalisation c_m <- c_m norms_m (which
// makes c_m = 1 where the factor was written normalised).  report (host memory): {<X, model>, ||model||^2}.
// <X, model> of put-off updates is <M, A_n> of the last mode n (the other factors' scales are 1 by then), from the sums the
// product's blocks left in `dots`.  For the exact solution trace(V A_n^T A_n), the same sum as ||model||^2, would do, but
// A_n carries the rounding of P and of the product, and what that adds to the trace is of first order, amplified by the
// condition of V: at rank 16 with two nearly equal columns (condition 3e6) the fit is off by 1.1e-3, with <M, A_n> by 7e-6.
template <int R>
__global__ __launch_bounds__(entry_threads(R)) void small_finish_kernel(SmallState st, int lazy, const double* __restrict__ inner,
                                                                        const double* __restrict__ dots, uint32_t nDots,
                                                                        float* __restrict__ lambda,
                                                                        double* __restrict__ report,
                                                                        unsigned long long* __restrict__ stamp) {
  constexpr int T = entry_threads(R);
  __shared__ double part[T], partInner[T];
  const int tid = threadIdx.x;
  if (tid == 0) *stamp = wall_clock64();
  double model = 0.0, sum = 0.0;
  if (lazy)
    for (uint32_t k = (uint32_t)tid; k < nDots; k += T) sum += dots[k];
  for (int e = tid; e < R * R; e += T) {
    const int i = e / R, j = e % R;
    double g = 1.0;
    for (int m = 0; m < st.order; ++m) g *= st.gram[m][e] / (st.scale[m][i] * st.scale[m][j]);
    model += g;
  }
  part[tid] = model;
  partInner[tid] = sum;
  __syncthreads();
  for (int half = T / 2; half > 0; half >>= 1) {
    if (tid < half) {
      part[tid] += part[tid + half];
      partInner[tid] += partInner[tid + half];
    }
    __syncthreads();
  }
  if (tid == 0) {
    report[0] = lazy ? partInner[0] : *inner;
    report[1] = part[0];
  }
  for (int r = tid; r < R; r += T) {
    double lam = 1.0;
    for (int m = 0; m < st.order; ++m) {
      double norm;
      if (lazy) {
        const double g = st.gram[m][r * R + r];
        norm = g > 0.0 ? sqrt(g) : 1.0;
        st.scale[m][r] = norm;
      } else {
        norm = st.norm[m][r];
        st.scale[m][r] = 1.0;
      }
      lam *= norm;
    }
    if (lambda) lambda[r] = (float)lam;
  }
}

// Column factors of the put-off normalisation of mode m, with the Gram matrix and scale that go with the scaled factor.
template <int R>
__global__ __launch_bounds__(entry_threads(R)) void small_normalise_kernel(SmallState st, int m, float* __restrict__ factor) {
  constexpr int T = entry_threads(R);
  const int tid = threadIdx.x;
  for (int e = tid; e < R * R; e += T) st.gram[m][e] /= st.scale[m][e / R] * st.scale[m][e % R];
  for (int r = tid; r < R; r += T) factor[r] = (float)(1.0 / st.scale[m][r]);
  __syncthreads();
  for (int r = tid; r < R; r += T) st.scale[m][r] = 1.0;
}

// The factors are taken as they are: every column scale 1, and p cleared (R < 32 writes only its diagonal blocks).
__global__ __launch_bounds__(256) void small_reset_kernel(SmallState st, int rank, float* __restrict__ p, int pCount) {
  for (int e = threadIdx.x; e < st.order * rank; e += 256) st.scale[e / rank][e % rank] = 1.0;
  for (int e = threadIdx.x; e < pCount; e += 256) p[e] = 0.f;
}

// calls `f` with the rank as a compile-time constant
template <typename F>
void with_rank(int rank, F&& f) {
  switch (rank) {
    case 8: f(std::integral_constant<int, 8>()); break;
    case 16: f(std::integral_constant<int, 16>()); break;
    case 32: f(std::integral_constant<int, 32>()); break;
    case 64: f(std::integral_constant<int, 64>()); break;
    default: f(std::integral_constant<int, 128>()); break;
  }
}

// ---------------------------------------------------------------------------------------------------
// Host R x R pseudo-inverse (fp64): hbcsf_sym_pinv
// ---------------------------------------------------------------------------------------------------
using Mat = std::vector<double>;

// Eigen-decomposition of a symmetric matrix by cyclic Jacobi rotations: a = q diag(w) q^T.
void jacobi_eig(Mat a, int n, Mat& q, std::vector<double>& w) {
  q.assign((size_t)n * n, 0.0);
  for (int i = 0; i < n; ++i) q[(size_t)i * n + i] = 1.0;
  for (int sweep = 0; sweep < 60; ++sweep) {
    double off = 0.0, diag = 0.0;
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < n; ++j) (i == j ? diag : off) += a[(size_t)i * n + j] * a[(size_t)i * n + j];
    if (off <= 1e-30 * diag || off == 0.0) break;
    for (int p = 0; p < n - 1; ++p) {
      for (int r = p + 1; r < n; ++r) {
        const double apr = a[(size_t)p * n + r];
        if (apr == 0.0) continue;
        const double theta = (a[(size_t)r * n + r] - a[(size_t)p * n + p]) / (2.0 * apr);
        const double t = (theta >= 0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
        const double cs = 1.0 / std::sqrt(t * t + 1.0), sn = t * cs;
        for (int k = 0; k < n; ++k) {  // columns p, r
          const double akp = a[(size_t)k * n + p], akr = a[(size_t)k * n + r];
          a[(size_t)k * n + p] = cs * akp - sn * akr;
          a[(size_t)k * n + r] = sn * akp + cs * akr;
        }
        for (int k = 0; k < n; ++k) {  // rows p, r
          const double apk = a[(size_t)p * n + k], ark = a[(size_t)r * n + k];
          a[(size_t)p * n + k] = cs * apk - sn * ark;
          a[(size_t)r * n + k] = sn * apk + cs * ark;
        }
        for (int k = 0; k < n; ++k) {
          const double qkp = q[(size_t)k * n + p], qkr = q[(size_t)k * n + r];
          q[(size_t)k * n + p] = cs * qkp - sn * qkr;
          q[(size_t)k * n + r] = sn * qkp + cs * qkr;
        }
      }
    }
  }
  w.resize(n);
  for (int i = 0; i < n; ++i) w[i] = a[(size_t)i * n + i];
}

// Moore-Penrose pseudo-inverse of a symmetric matrix: eigenvalues below 1e-15 of the largest magnitude
// count as zero (the cut-off numpy.linalg.pinv applies to singular values).
Mat sym_pinv(const Mat& v, int n) {
  Mat q;
  std::vector<double> w;
  jacobi_eig(v, n, q, w);
  double wmax = 0.0;
  for (double x : w) wmax = std::fmax(wmax, std::fabs(x));
  Mat out((size_t)n * n, 0.0);
  for (int k = 0; k < n; ++k) {
    if (std::fabs(w[k]) <= 1e-15 * wmax) continue;
    const double inv = 1.0 / w[k];
    for (int i = 0; i < n; ++i) {
      const double qi = q[(size_t)i * n + k] * inv;
      for (int j = 0; j < n; ++j) out[(size_t)i * n + j] += qi * q[(size_t)j * n + k];
    }
  }
  return out;
}

// Inverse of a symmetric positive definite matrix by Cholesky factorisation; false when a pivot is not
// safely positive (then the caller takes the eigenvalue route, which handles rank deficiency).
bool spd_inverse(const Mat& v, int n, Mat& out) {
  Mat l((size_t)n * n, 0.0);
  double dmax = 0.0;
  for (int i = 0; i < n; ++i) dmax = std::fmax(dmax, v[(size_t)i * n + i]);
  for (int j = 0; j < n; ++j) {
    double d = v[(size_t)j * n + j];
    for (int k = 0; k < j; ++k) d -= l[(size_t)j * n + k] * l[(size_t)j * n + k];
    if (!(d > 1e-10 * dmax)) return false;
    const double ljj = std::sqrt(d);
    l[(size_t)j * n + j] = ljj;
    for (int i = j + 1; i < n; ++i) {
      double x = v[(size_t)i * n + j];
      for (int k = 0; k < j; ++k) x -= l[(size_t)i * n + k] * l[(size_t)j * n + k];
      l[(size_t)i * n + j] = x / ljj;
    }
  }
  // li = l^-1 (lower triangular), then v^-1 = li^T li
  Mat li((size_t)n * n, 0.0);
  for (int c = 0; c < n; ++c) {
    li[(size_t)c * n + c] = 1.0 / l[(size_t)c * n + c];
    for (int i = c + 1; i < n; ++i) {
      double x = 0.0;
      for (int k = c; k < i; ++k) x -= l[(size_t)i * n + k] * li[(size_t)k * n + c];
      li[(size_t)i * n + c] = x / l[(size_t)i * n + i];
    }
  }
  out.assign((size_t)n * n, 0.0);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j <= i; ++j) {
      double x = 0.0;
      for (int k = i; k < n; ++k) x += li[(size_t)k * n + i] * li[(size_t)k * n + j];
      out[(size_t)i * n + j] = x;
      out[(size_t)j * n + i] = x;
    }
  return true;
}

// The pseudo-inverse the update needs: the plain inverse when the matrix is safely positive definite
// (the two coincide there), the eigenvalue form otherwise.
Mat pinv_of_gram_product(const Mat& v, int n) {
  Mat out;
  if (spd_inverse(v, n, out)) return out;
  return sym_pinv(v, n);
}

uint64_t round256(uint64_t v) { return (v + 255) / 256 * 256; }

bool rank_ok(int rank) { return rank == 8 || rank == 16 || rank == 32 || rank == 64 || rank == 128; }

}  // namespace

struct hbcsf_als {
  const hbcsf_tensor* t = nullptr;
  int rank = 0;
  // workspace (device)
  float* m = nullptr;             // MTTKRP output of the mode being updated [max dim][R]
  double* s = nullptr;            // Gram matrix of it [R][R]
  double* gramScratch = nullptr;  // per-block partial sums of the Gram kernels
  uint32_t gramSlots = 0;
  float* p = nullptr;             // right-hand matrix of the product [max(R, 32)][max(R, 32)]
  float* factor = nullptr;        // [R] column factors of the put-off normalisation
  double* vp = nullptr;           // V^+ [R][R]
  double* tmp[2] = {nullptr, nullptr};  // [R][R] each
  double* inner = nullptr;        // <X, model> of an ordinary iteration
  double* dots = nullptr;         // of a put-off one, as the blocks' sums [kDotsMax]
  SmallState small{};
  int* good = nullptr;            // outcome of the sweep a guest made
  bool pending[HBCSF_MAX_ORDER] = {};  // the stored factor's columns still carry norms (small.scale)
  bool gramsValid = false;
  // Pinned host memory the kernels of an iteration write: {<X, model>, ||model||^2}, and wall-clock stamps (taken by a
  // thread of each kernel as it begins: an event record between two kernels costs 5.6 us on the stream, as much as
  // many of the kernels).  Per mode: inverse begins, inverse ends, Gram or product begins, R x R part after the Gram
  // begins; one more at the iteration's end.  Where the inverse goes with the MTTKRP the first two are: MTTKRP begins,
  // eigenvalue form begins (0: it was not needed); the last is when the MTTKRP's last blocks end
  // (if after that, otherwise some time before).
  struct Report {
    double value[2];
    unsigned long long stamp[HBCSF_MAX_ORDER][4], end;
  };
  Report* report = nullptr;
  double msPerTick = 1e-5;
  bool hosted[HBCSF_MAX_ORDER] = {};  // the last iteration's inverse of the mode went with the MTTKRP
  bool timed = false;      // an iteration has been enqueued
  bool timedGram = false;  // ... an ordinary one: stamp[.][3] is set too

  hbcsf_als() = default;
  hbcsf_als(const hbcsf_als&) = delete;
  hbcsf_als& operator=(const hbcsf_als&) = delete;
  ~hbcsf_als() {
    if (report) (void)hipHostFree(report);
  }
};

// ---------------------------------------------------------------------------------------------------
// Scratch owned by the library, for hbcsf_gram_noalloc: callers that may not allocate device memory (code
// under graph capture, serving loops, harnesses that forbid it) get the Gram computation's partial-sum
// slots from this array instead of a workspace argument.  Every device the library runs on holds its own
// copy, at its own address, until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; the address that call returns is what kernels and copies are given.
// ---------------------------------------------------------------------------------------------------
constexpr uint64_t kStaticScratchBytes = 8ull << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
struct DeviceScratch {
  void* ptr = nullptr;  // device address of `scratch` on this device
  int numCU = 0;
};
DeviceScratch g_scratch[kMaxDevices];
std::mutex g_scratchMutex;

int gram_check(const float* a, int rank, const double* s) {
  if (!a || !s) return fail(HBCSF_EINVAL, "null argument");
  if (!rank_ok(rank)) return fail(HBCSF_EINVAL, "rank must be 8, 16, 32, 64 or 128");
  if (((uintptr_t)a & 15) != 0) return fail(HBCSF_EINVAL, "the matrix must be 16-byte aligned");
  if (((uintptr_t)s & 7) != 0) return fail(HBCSF_EINVAL, "the result must be 8-byte aligned");
  return HBCSF_OK;
}

int current_cu_count(int* cu) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  e = hipDeviceGetAttribute(cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return fail_hip(e, "hipDeviceGetAttribute");
  if (*cu <= 0) *cu = 256;
  return HBCSF_OK;
}

}  // namespace

namespace {

// Scales the columns of every stored factor whose normalisation was put off, so that the stored matrices are the
// algorithm's unit-norm factors again; the Gram matrices the state keeps are scaled with them.
int apply_pending_normalisation(hbcsf_als* a, float* const* factors, hipStream_t st) {
  const hbcsf_tensor* t = a->t;
  for (int m = 0; m < t->order; ++m) {
    if (!a->pending[m]) continue;
    with_rank(a->rank, [&](auto r) {
      constexpr int R = decltype(r)::value;
      hipLaunchKernelGGL(small_normalise_kernel<R>, dim3(1), dim3(entry_threads(R)), 0, st, a->small, m, a->factor);
    });
    launch_scale_columns(factors[m], t->dims[m], a->rank, a->factor, t->numCU, st);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail_hip(e, "column scaling kernel launch");
    a->pending[m] = false;
  }
  return HBCSF_OK;
}

// Where the parts of an ALS state's workspace lie (bytes from its start).
struct AlsLayout {
  uint64_t m, s, p, factor, vp, tmp[2], inner, dots, good, gram, scale, norm, scratch, total;
};

AlsLayout als_layout(const hbcsf_tensor* t, int rank) {
  uint64_t maxDim = 0;
  for (int m = 0; m < t->order; ++m) maxDim = t->dims[m] > maxDim ? t->dims[m] : maxDim;
  uint64_t gramBytes = 0;
  (void)hbcsf_gram_workspace_bytes(rank, &gramBytes);
  const uint64_t rr = (uint64_t)rank * rank, pr = rank < 32 ? 32 : rank;
  AlsLayout l{};
  uint64_t off = 0;
  auto take = [&off](uint64_t bytes) {
    const uint64_t at = off;
    off += round256(bytes);
    return at;
  };
  l.m = take(maxDim * (uint64_t)rank * 4);
  l.s = take(rr * 8);
  l.p = take(pr * pr * 4);
  l.factor = take((uint64_t)rank * 4);
  l.vp = take(rr * 8);
  for (int k = 0; k < 2; ++k) l.tmp[k] = take(rr * 8);
  l.inner = take(8);
  l.dots = take((uint64_t)kDotsMax * 8);
  l.good = take(4);
  l.gram = take((uint64_t)t->order * rr * 8);
  l.scale = take((uint64_t)t->order * rank * 8);
  l.norm = take((uint64_t)t->order * rank * 8);
  l.scratch = take(gramBytes);
  l.total = off;
  return l;
}

// Enqueues one iteration on st (no wait).  After it small.scale holds the norms a put-off normalisation still owes.
int enqueue_iteration(hbcsf_als* a, float* const* factors, float* lambda, int flags, hipStream_t st) {
  const hbcsf_tensor* t = a->t;
  const int order = t->order, R = a->rank;
  const bool lazy = (flags & HBCSF_ALS_LAZY_NORMALISATION) != 0;
  hipError_t e;
  // Gram matrices of the factors that are read before they are updated (all but the first mode's).  Without
  // the keep flag the caller may have replaced the factors: they are then taken as they are (scale 1).
  if (!(flags & HBCSF_ALS_KEEP_GRAMS) || !a->gramsValid) {
    const int pr = R < 32 ? 32 : R;
    hipLaunchKernelGGL(small_reset_kernel, dim3(1), dim3(256), 0, st, a->small, R, a->p, pr * pr);
    for (int m = 0; m < order; ++m) a->pending[m] = false;
    for (int m = 1; m < order; ++m)
      launch_gram(factors[m], t->dims[m], R, a->gramScratch, a->gramSlots, a->small.gram[m], t->numCU, st);
  }
  a->gramsValid = false;
  a->timed = false;
  uint32_t nDots = 0;
  for (int n = 0; n < order; ++n) {
    const float* facs[HBCSF_MAX_ORDER];
    for (int m = 0; m < order; ++m) facs[m] = factors[m];
    // a put-off update's inverse goes with the MTTKRP where it takes guests
    // (the eigenvalue form then begins at stamp 1, and its end, at stamp 2, is overwritten by the product that follows)
    const bool hosted = a->hosted[n] = lazy && mttkrp_takes_guest(t, n, R);
    auto invert = [&] {
      with_rank(R, [&](auto r) {
        constexpr int RR = decltype(r)::value;
        hipLaunchKernelGGL(small_pinv_kernel<RR>, dim3(1), dim3(pinv_threads(RR)), 0, st, a->small, n, a->vp, a->p,
                           a->tmp[0], lazy ? 1 : 0, hosted ? a->good : nullptr, a->report->stamp[n] + (hosted ? 1 : 0));
      });
    };
    int rc;
    if (hosted) {
      GuestArgs guest{};
      guest.small = a->small;
      guest.n = n;
      guest.p = a->p;
      guest.vp = a->vp;
      guest.good = a->good;
      guest.stamp = a->report->stamp[n];
      rc = mttkrp_with_guest(t, n, R, facs, a->m, guest, st);
    } else {
      invert();
      rc = hbcsf_mttkrp(t, n, R, facs, a->m, st);
    }
    if (rc != HBCSF_OK) return rc;
    if (hosted && !guest_finishes(R)) invert();   // what is left of it
    if (lazy) {
      // A_n = M V^+ written unnormalised, with its Gram matrix
      nDots = launch_apply(a->m, t->dims[n], R, a->p, factors[n], a->gramScratch, a->gramSlots, a->small.gram[n],
                           n + 1 == order ? a->dots : nullptr, t->numCU, st, &a->report->stamp[n][2]);
    } else {
      launch_gram(a->m, t->dims[n], R, a->gramScratch, a->gramSlots, a->s, t->numCU, st, &a->report->stamp[n][2]);
      with_rank(R, [&](auto r) {
        constexpr int RR = decltype(r)::value;
        const dim3 grid((RR * RR + 255) / 256);
        hipLaunchKernelGGL(small_matmul_kernel<RR>, grid, dim3(256), 0, st, a->vp, a->s, a->tmp[0], a->small, n, 1,
                           &a->report->stamp[n][3]);
        hipLaunchKernelGGL(small_matmul_kernel<RR>, grid, dim3(256), 0, st, a->tmp[0], a->vp, a->tmp[1], a->small, n, 0,
                           nullptr);
        hipLaunchKernelGGL(small_update_kernel<RR>, dim3(1), dim3(entry_threads(RR)), 0, st, a->small, n, a->tmp[1],
                           a->vp, a->s, a->p, a->inner);
      });
      launch_apply(a->m, t->dims[n], R, a->p, factors[n], nullptr, 0, nullptr, nullptr, t->numCU, st, nullptr);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return fail_hip(e, "mode update kernel launch");
  }
  with_rank(R, [&](auto r) {
    constexpr int RR = decltype(r)::value;
    hipLaunchKernelGGL(small_finish_kernel<RR>, dim3(1), dim3(entry_threads(RR)), 0, st, a->small, lazy ? 1 : 0, a->inner,
                       a->dots, nDots, lambda, a->report->value, &a->report->end);
  });
  e = hipGetLastError();
  if (e != hipSuccess) return fail_hip(e, "iteration end kernel launch");
  for (int m = 0; m < order; ++m) a->pending[m] = lazy;
  a->gramsValid = true;
  a->timed = true;
  a->timedGram = !lazy;
  return HBCSF_OK;
}

// The fit of the last finished iteration.
double als_fit(const hbcsf_als* a) {
  const double x = a->t->normSq, res = x - 2.0 * a->report->value[0] + a->report->value[1];
  return x > 0.0 ? 1.0 - std::sqrt(res > 0.0 ? res : 0.0) / std::sqrt(x) : 0.0;
}

int als_check(const hbcsf_als* a, float* const* factors) {
  if (!a || !factors) return fail(HBCSF_EINVAL, "null argument");
  for (int m = 0; m < a->t->order; ++m)
    if (!factors[m]) return fail(HBCSF_EINVAL, "a factor pointer is null");
  return HBCSF_OK;
}

}  // namespace

extern "C" {

int hbcsf_gram_workspace_bytes(int rank, uint64_t* bytes) try {
  if (!bytes) return fail(HBCSF_EINVAL, "null argument");
  if (!rank_ok(rank)) return fail(HBCSF_EINVAL, "rank must be 8, 16, 32, 64 or 128");
  *bytes = (uint64_t)gram_slots_for(rank, kGramWorkspaceCap) * (uint64_t)rank * rank * 8;
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_gram(const float* a, uint64_t rows, int rank, void* workspace, uint64_t workspace_bytes, double* s,
               void* hip_stream) try {
  const int rc = gram_check(a, rank, s);
  if (rc != HBCSF_OK) return rc;
  if (!workspace) return fail(HBCSF_EINVAL, "null argument");
  if (((uintptr_t)workspace & 255) != 0) return fail(HBCSF_EINVAL, "workspace must be 256-byte aligned");
  const uint32_t slots = gram_slots_for(rank, workspace_bytes);
  if (slots == 0) return fail(HBCSF_ENOMEM, "workspace holds less than one rank x rank fp64 matrix");
  int cu = 0;
  const int rd = current_cu_count(&cu);
  if (rd != HBCSF_OK) return rd;
  launch_gram(a, rows, rank, (double*)workspace, slots, s, cu, (hipStream_t)hip_stream);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail_hip(e, "Gram kernel launch");
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_gram_noalloc(const float* a, uint64_t rows, int rank, double* s, void* hip_stream) try {
  const int rc = gram_check(a, rank, s);
  if (rc != HBCSF_OK) return rc;
  if ((uint64_t)rank * rank * 8 > kStaticScratchBytes)
    return fail(HBCSF_EINVAL, "rank is beyond what the library's own scratch holds (one rank x rank fp64 slot)");
  int dev = 0, cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices) return fail(HBCSF_EINVAL, "device ordinal beyond the library's per-device table");
  DeviceScratch& d = g_scratch[dev];
  {
    // once per device, with that device current: the array's address on this device (each device has its own copy)
    std::lock_guard<std::mutex> lock(g_scratchMutex);
    if (!d.ptr) {
      void* p = nullptr;
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess) return fail_hip(e, "hipGetSymbolAddress");
      if (!p || ((uintptr_t)p & 255) != 0) return fail(HBCSF_EHIP, "the scratch array has no usable device address");
      e = hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev);
      if (e != hipSuccess) return fail_hip(e, "hipDeviceGetAttribute");
      d.numCU = cu > 0 ? cu : 256;
      d.ptr = p;
    }
  }
  launch_gram(a, rows, rank, (double*)d.ptr, gram_slots_for(rank, kStaticScratchBytes), s, d.numCU,
              (hipStream_t)hip_stream);
  e = hipGetLastError();
  if (e != hipSuccess) return fail_hip(e, "Gram kernel launch");
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_als_workspace_bytes(const hbcsf_tensor* t, int rank, uint64_t* bytes) try {
  if (!t || !bytes) return fail(HBCSF_EINVAL, "null argument");
  if (!rank_ok(rank)) return fail(HBCSF_EINVAL, "rank must be 8, 16, 32, 64 or 128");
  *bytes = als_layout(t, rank).total;
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_als_create(const hbcsf_tensor* t, int rank, void* workspace, uint64_t workspace_bytes,
                     hbcsf_als** out) try {
  if (!out) return fail(HBCSF_EINVAL, "out is null");
  *out = nullptr;
  if (!t || !workspace) return fail(HBCSF_EINVAL, "null argument");
  if (!t->uploaded) return fail(HBCSF_ESTATE, "hbcsf_upload has not been called");
  uint64_t need = 0;
  const int rc = hbcsf_als_workspace_bytes(t, rank, &need);
  if (rc != HBCSF_OK) return rc;
  if (workspace_bytes < need) return fail(HBCSF_ENOMEM, "workspace is smaller than hbcsf_als_workspace_bytes");
  if (((uintptr_t)workspace & 255) != 0) return fail(HBCSF_EINVAL, "workspace must be 256-byte aligned");
  std::unique_ptr<hbcsf_als> a(new (std::nothrow) hbcsf_als);
  if (!a) return fail(HBCSF_ENOMEM, "out of host memory");
  a->t = t;
  a->rank = rank;
  const AlsLayout l = als_layout(t, rank);
  uint8_t* w = (uint8_t*)workspace;
  a->m = (float*)(w + l.m);
  a->s = (double*)(w + l.s);
  a->p = (float*)(w + l.p);
  a->factor = (float*)(w + l.factor);
  a->vp = (double*)(w + l.vp);
  for (int k = 0; k < 2; ++k) a->tmp[k] = (double*)(w + l.tmp[k]);
  a->inner = (double*)(w + l.inner);
  a->dots = (double*)(w + l.dots);
  a->good = (int*)(w + l.good);
  a->small.order = t->order;
  for (int m = 0; m < t->order; ++m) {
    a->small.gram[m] = (double*)(w + l.gram) + (size_t)m * rank * rank;
    a->small.scale[m] = (double*)(w + l.scale) + (size_t)m * rank;
    a->small.norm[m] = (double*)(w + l.norm) + (size_t)m * rank;
  }
  a->gramScratch = (double*)(w + l.scratch);
  uint64_t gramBytes = 0;
  (void)hbcsf_gram_workspace_bytes(rank, &gramBytes);
  a->gramSlots = gram_slots_for(rank, gramBytes);
  hipError_t e = hipHostMalloc((void**)&a->report, sizeof(hbcsf_als::Report), hipHostMallocDefault);
  if (e != hipSuccess) return fail_hip(e, "hipHostMalloc");
  int dev = 0, kHz = 0;
  e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&kHz, hipDeviceAttributeWallClockRate, dev);
  if (e != hipSuccess) return fail_hip(e, "hipDeviceGetAttribute");
  if (kHz > 0) a->msPerTick = 1.0 / kHz;
  *out = a.release();
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_als_iteration(hbcsf_als* a, float* const* factors, float* lambda, int flags, double* fit,
                        void* hip_stream) try {
  const int rc = als_check(a, factors);
  if (rc != HBCSF_OK) return rc;
  if (flags & ~(HBCSF_ALS_KEEP_GRAMS | HBCSF_ALS_LAZY_NORMALISATION)) return fail(HBCSF_EINVAL, "unknown flag");
  hipStream_t st = (hipStream_t)hip_stream;
  const int ri = enqueue_iteration(a, factors, lambda, flags, st);
  if (ri != HBCSF_OK) return ri;
  const hipError_t e = hipStreamSynchronize(st);
  if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
  if (fit) *fit = als_fit(a);
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_als_normalise(hbcsf_als* a, float* const* factors, void* hip_stream) try {
  const int rc = als_check(a, factors);
  if (rc != HBCSF_OK) return rc;
  const int rn = apply_pending_normalisation(a, factors, (hipStream_t)hip_stream);
  if (rn != HBCSF_OK) return rn;
  const hipError_t e = hipStreamSynchronize((hipStream_t)hip_stream);
  if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_als_run(hbcsf_als* a, float* const* factors, float* lambda, int max_iterations, double tolerance,
                  int* iterations_done, double* fit, void* hip_stream) try {
  const int rc = als_check(a, factors);
  if (rc != HBCSF_OK) return rc;
  if (max_iterations < 1) return fail(HBCSF_EINVAL, "max_iterations must be at least 1");
  hipStream_t st = (hipStream_t)hip_stream;
  double prev = 0.0, cur = 0.0;
  int it = 0;
  for (; it < max_iterations; ++it) {
    const int ri = enqueue_iteration(a, factors, lambda, (it > 0 ? HBCSF_ALS_KEEP_GRAMS : 0) | HBCSF_ALS_LAZY_NORMALISATION, st);
    if (ri != HBCSF_OK) return ri;
    if (!(tolerance > 0.0)) continue;   // no fit can end the loop: the iterations follow each other without a wait
    const hipError_t e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
    cur = als_fit(a);
    if (it > 0 && std::fabs(cur - prev) < tolerance) {
      ++it;
      break;
    }
    prev = cur;
  }
  const int rn = hbcsf_als_normalise(a, factors, hip_stream);
  if (rn != HBCSF_OK) return rn;
  if (iterations_done) *iterations_done = it;
  if (fit) *fit = als_fit(a);
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_sym_pinv(const double* v, int n, double* out) try {
  if (!v || !out) return fail(HBCSF_EINVAL, "null argument");
  if (n < 1 || n > 128) return fail(HBCSF_EINVAL, "n must be in 1 .. 128");
  const Mat in(v, v + (size_t)n * n);
  const Mat r = pinv_of_gram_product(in, n);
  std::memcpy(out, r.data(), (size_t)n * n * sizeof(double));
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_als_phase_ms(const hbcsf_als* a, float ms[4]) try {
  if (!a || !ms) return fail(HBCSF_EINVAL, "null argument");
  for (int k = 0; k < 4; ++k) ms[k] = 0.f;
  if (!a->timed) return HBCSF_OK;
  const int order = a->t->order;
  auto add = [&](float& to, unsigned long long from, unsigned long long until) {
    to += (float)((double)(until - from) * a->msPerTick);
  };
  for (int n = 0; n < order; ++n) {
    const unsigned long long* at = a->report->stamp[n];
    const unsigned long long end = n + 1 < order ? a->report->stamp[n + 1][0] : a->report->end;
    if (a->hosted[n]) {
      // (the eigenvalue form may begin long before the MTTKRP ends, and end before it too)
      const unsigned long long mttkrpEnd = at[1] ? std::min(std::max(at[1], at[3]), at[2]) : at[2];
      add(ms[0], at[0], mttkrpEnd);
      add(ms[2], mttkrpEnd, at[2]);
    } else {
      add(ms[2], at[0], at[1]);
      add(ms[0], at[1], at[2]);
    }
    if (a->timedGram) add(ms[1], at[2], at[3]);
    add(ms[3], at[a->timedGram ? 3 : 2], end);
  }
  return HBCSF_OK;
} HBCSF_CATCH_ALL

void hbcsf_als_free(hbcsf_als* a) { delete a; }

}  // extern "C"
