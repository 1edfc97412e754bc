// Stable radix sort of (64-bit key, 32-bit value) pairs on chosen bits of the key, for the device builder: the common order
// straight from the COO arrays, and any number of further orders of it whose digits are counted in the same reading.
//
// A pass follows the one-sweep scheme (A. Adinets and D. Merrill, "Onesweep: A Faster Least Significant Digit Radix Sort for GPUs",
// 2022) with the decoupled look-back of D. Merrill and M. Garland ("Single-pass Parallel Prefix Scan with Decoupled Look-back",
// 2016).  What bounds it is memory: 12 bytes read and 12 written per pair, the writes in short runs.  So:
//  - a pass is one launch: a block ranks a tile of 8192 pairs, learns from the tiles before it where its digits' pairs
//    go (each tile publishes its counts, then the sum up to it: a reader adds counts backwards until it meets a sum), and
//    writes them from LDS in the order of the digits, in runs of 32 on average;
//  - all digits of all orders are counted once, by one kernel that reads the indices;
//  - the first pass packs the keys itself: they are not written and read again before it;
//  - a pass clears the words the next one publishes in, so that there is no launch between passes.
// 50 M pairs of 59 bits, four orders, us: a pass 265 to 300, 4.0 to 4.5 TB/s (a library's onesweep pass 375 to 400 and two clears
// of 5); counting 320 (150 to 175 an order); the first pass 370 (packing 390, then a pass of 395).  Altogether 7.1 -> 4.65 ms.

#ifndef HBCSF_SORT_H
#define HBCSF_SORT_H

#include <hip/hip_runtime.h>

#include <cstdint>

#include "hbcsf.h"

namespace hbcsf {
namespace {

struct IndPtrs {
  const uint32_t* p[HBCSF_MAX_ORDER];
};

// Where each mode's index lies in the key of the common order.
struct BaseKey {
  int shift[HBCSF_MAX_ORDER];       // by mode
  uint64_t mask[HBCSF_MAX_ORDER], dims[HBCSF_MAX_ORDER];
};

// A tile is 512 threads with 16 pairs each: 74 KB of LDS, two blocks on a compute unit, so that one ranks while the other waits
// for memory.  Below 1 M nonzeros tiles of 4 pairs a thread, which fill the chip sooner: a whole build of order 3 / 4 (indices by
// Zipf's law of 1.2, of 1.3 to 0.8), short -> long tiles, 50 000 nonzeros 621 -> 712 / 811 -> 950 us, 0.4 M 737 -> 783 / 939 ->
// 1027, 0.8 M 825 -> 832 / 1060 -> 1078, 1.6 M 984 -> 926 / 1274 -> 1211.
constexpr int kSortThreads = 512, kSortWaves = kSortThreads / 64, kSortLong = 16, kSortShort = 4;
constexpr size_t kSortLongMin = 1u << 20;
constexpr int kSortDigits = 256;       // digits of at most 8 bits
constexpr int kSortPasses = 32;        // of all orders: 64 bits in one, at most 64 and five modes' remainders in the others
constexpr int kCountBlocks = 512, kCountAhead = 4;
constexpr uint32_t kSortCounts = 1u << 30, kSortSum = 2u << 30, kSortValue = kSortCounts - 1u;  // a published word

struct SortPasses {
  int n = 0;
  int shift[kSortPasses];
  uint32_t mask[kSortPasses];
  // `bits` bits from `from` on, lowest first, in digits whose sizes differ by at most one
  bool add(int from, int bits) {
    const int passes = (bits + 7) / 8;
    if (n + passes > kSortPasses) return false;
    for (int k = 0; k < passes; ++k) {
      const int b = bits / passes + (k < bits % passes ? 1 : 0);
      shift[n] = from;
      mask[n++] = (1u << b) - 1u;
      from += b;
    }
    return true;
  }
};

struct SortScratch {
  uint32_t* counts;  // [passes][blocks][256], until their sums are taken: it is K's memory
  uint32_t* start;   // [passes][256] where a digit's pairs begin
  uint32_t* ticket;  // [passes] tiles given out
  uint32_t* words;   // [2][tiles][256] what the tiles of a pass publish: one array in use, one being cleared
  uint64_t* K;       // [n] a third pair of buffers, from the second order on
  uint32_t* V;
};

inline int sort_items(size_t n) { return n >= kSortLongMin ? kSortLong : kSortShort; }
inline uint32_t sort_tiles(size_t n) {
  const size_t tile = (size_t)kSortThreads * sort_items(n);
  return (uint32_t)((n + tile - 1) / tile);
}

// Blocks that count: each at least two steps, so that their counts fit where K will be.
inline uint32_t count_blocks(size_t n) {
  const size_t b = (n + 2 * 512 * kCountAhead - 1) / (2 * 512 * kCountAhead);
  return b < (size_t)kCountBlocks ? (uint32_t)b : (uint32_t)kCountBlocks;
}

// Carves the scratch out of `base` (null: only the size).
inline uint64_t sort_scratch(size_t n, uint8_t* base, SortScratch* s) {
  uint64_t off = 0;
  auto take = [&](uint64_t bytes) {
    uint8_t* p = base ? base + off : nullptr;
    off += (bytes + 255) / 256 * 256;
    return p;
  };
  const uint64_t counts = (uint64_t)kSortPasses * count_blocks(n) * kSortDigits * 4;
  s->K = (uint64_t*)take((uint64_t)n * 8 > counts ? (uint64_t)n * 8 : counts);
  s->counts = (uint32_t*)s->K;
  s->V = (uint32_t*)take((uint64_t)n * 4);
  s->words = (uint32_t*)take((uint64_t)2 * sort_tiles(n) * kSortDigits * 4);
  s->start = (uint32_t*)take((uint64_t)kSortPasses * kSortDigits * 4);
  s->ticket = (uint32_t*)take(kSortPasses * 4);
  return off;
}

// A nonzero's key.  An index that is not below its dimension sets `off` and counts as 0: the call will be refused, but the
// numbering is enqueued before the host knows; it has room for as many slices as the mode has rows, so such an index must not
// become one (nor spill into the next field).
template <typename Key>
__device__ __forceinline__ Key pack_key(const IndPtrs& inds, int N, const BaseKey& bk, size_t z, bool& off) {
  Key key = 0;
#pragma unroll
  for (int m = 0; m < HBCSF_MAX_ORDER; ++m) {
    if (m >= N) break;
    uint32_t i = inds.p[m][z];
    if ((uint64_t)i >= bk.dims[m]) {
      off = true;
      i = 0;
    }
    key |= (Key)i << bk.shift[m];
  }
  return key;
}

// The keys of nonzeros z0 + j0 + i * step, those below z0 + here (the others 0): a mode's loads are all in flight together.
template <int Items>
__device__ __forceinline__ void pack_keys(const IndPtrs& inds, int N, const BaseKey& bk, size_t z0, uint32_t j0, uint32_t step,
                                          uint32_t here, uint64_t (&key)[Items], bool& off) {
#pragma unroll
  for (int i = 0; i < Items; ++i) key[i] = 0;
  for (int m = 0; m < N; ++m) {
    const uint32_t* ind = inds.p[m] + z0;
    uint32_t x[Items];
#pragma unroll
    for (int i = 0; i < Items; ++i) x[i] = j0 + i * step < here ? ind[j0 + i * step] : 0u;
#pragma unroll
    for (int i = 0; i < Items; ++i) {
      if ((uint64_t)x[i] >= bk.dims[m]) {
        off = true;
        x[i] = 0;
      }
      key[i] |= (uint64_t)x[i] << bk.shift[m];
    }
  }
}

// How often every digit of every pass occurs, per block; the first pass's words and the tickets are cleared on the way.
// copyBits: a digit has 2^copyBits counters, which its lanes share out (a digit that many lanes have is otherwise counted one
// lane after the other): 50 M nonzeros 567 -> 319 us with four, and with a mode's loads in flight together.
__global__ __launch_bounds__(512) void sort_count_kernel(IndPtrs inds, uint32_t n, int N, BaseKey bk, SortPasses ps, SortScratch s,
                                                         uint32_t tiles, int copyBits, unsigned long long* bad) {
  extern __shared__ uint32_t seen[];  // [passes][256][copies]
  for (uint32_t i = threadIdx.x; i < (uint32_t)ps.n * kSortDigits << copyBits; i += 512) seen[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x < kSortPasses) s.ticket[threadIdx.x] = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * 512 + threadIdx.x; i < (uint64_t)tiles * kSortDigits; i += (uint64_t)gridDim.x * 512)
    s.words[i] = 0;
  __syncthreads();
  bool off = false;
  const uint32_t copy = threadIdx.x & ((1u << copyBits) - 1u);
  constexpr uint32_t kStep = 512 * kCountAhead;
  for (uint64_t z0 = (uint64_t)blockIdx.x * kStep; z0 < n; z0 += (uint64_t)gridDim.x * kStep) {
    uint64_t key[kCountAhead];
    const uint32_t here = n - z0 < kStep ? (uint32_t)(n - z0) : kStep;
    pack_keys<kCountAhead>(inds, N, bk, (size_t)z0, threadIdx.x, 512, here, key, off);
    for (int p = 0; p < ps.n; ++p)
#pragma unroll
      for (int q = 0; q < kCountAhead; ++q)
        if (q * 512 + threadIdx.x < here)
          atomicAdd(&seen[((p * kSortDigits + ((uint32_t)(key[q] >> ps.shift[p]) & ps.mask[p])) << copyBits) + copy], 1u);
  }
  if (off) atomicOr(bad, 1ull);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < (uint32_t)ps.n * kSortDigits; i += 512) {
    uint32_t sum = 0;
    for (uint32_t c = 0; c < 1u << copyBits; ++c) sum += seen[(i << copyBits) + c];
    s.counts[((size_t)(i / kSortDigits) * gridDim.x + blockIdx.x) * kSortDigits + (i % kSortDigits)] = sum;
  }
}

// One block per pass: where each digit's pairs begin.
__global__ __launch_bounds__(1024) void sort_start_kernel(SortScratch s, uint32_t blocks) {
  __shared__ uint32_t part[4][kSortDigits];
  __shared__ uint32_t wave[4];
  const uint32_t d = threadIdx.x & 255, g = threadIdx.x >> 8;
  const uint32_t* c = s.counts + (size_t)blockIdx.x * blocks * kSortDigits;
  uint32_t sum = 0;
#pragma unroll 8
  for (uint32_t b = g; b < blocks; b += 4) sum += c[(size_t)b * kSortDigits + d];
  part[g][d] = sum;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  uint32_t total = 0, upTo = 0;
  if (g == 0) {
    total = part[0][d] + part[1][d] + part[2][d] + part[3][d];
    upTo = total;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t up = __shfl_up(upTo, o);
      if (lane >= o) upTo += up;
    }
    if (lane == 63) wave[d >> 6] = upTo;
  }
  __syncthreads();
  if (g == 0) {
    for (uint32_t w = 0; w < (d >> 6); ++w) upTo += wave[w];
    s.start[(size_t)blockIdx.x * kSortDigits + d] = upTo - total;
  }
}

struct SortIn {
  const uint64_t* K;  // the pairs, or for the first pass:
  const uint32_t* V;
  IndPtrs inds;
  const float* vals;
  BaseKey bk;
  int N;
};

// One pass.  Waiting: a tile's number is taken when its block runs, and a block waits only for words of tiles with lower
// numbers, whose blocks run already and publish their counts before they wait for anything themselves.
template <bool Coo, int Items>
__global__ __launch_bounds__(kSortThreads, 4) void sort_pass_kernel(SortIn in, uint64_t* __restrict__ Ko, uint32_t* __restrict__ Vo,
                                                                    uint32_t n, int shift, uint32_t mask,
                                                                    const uint32_t* __restrict__ start, uint32_t* ticket,
                                                                    uint32_t* words, uint32_t* __restrict__ clear) {
  constexpr uint32_t kTile = kSortThreads * Items;
  __shared__ uint64_t buf[kTile];
  __shared__ uint32_t cnt[kSortWaves][kSortDigits];  // pairs of a wavefront by digit; then those of the wavefronts before it
  __shared__ uint32_t local[kSortDigits];            // where a digit's pairs begin in the tile
  __shared__ uint32_t base[kSortDigits];             // where they go, minus that
  __shared__ uint32_t wave[4], number;
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) number = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  volatile uint32_t* mine = cnt[w];
#pragma unroll
  for (int k = 0; k < kSortDigits; k += 64) mine[k + lane] = 0;
  __syncthreads();
  const uint32_t tile = number, p0 = tile * kTile;
  const uint32_t here = n - p0 < kTile ? n - p0 : kTile;
  const uint32_t j0 = w * (Items * 64) + lane;

  uint64_t key[Items];
  uint32_t val[Items], rank[Items];
#pragma unroll
  for (int i = 0; i < Items; ++i) {
    const uint32_t j = j0 + i * 64;
    if constexpr (Coo) {
      val[i] = j < here ? __float_as_uint(in.vals[(size_t)p0 + j]) : 0u;
    } else {
      key[i] = j < here ? in.K[(size_t)p0 + j] : 0ull;
      val[i] = j < here ? in.V[(size_t)p0 + j] : 0u;
    }
  }
  if constexpr (Coo) {
    bool off = false;  // (counted already)
    pack_keys<Items>(in.inds, in.N, in.bk, p0, j0, 64, here, key, off);
  }
  // a pair's rank among those of its digit in the wavefront: the ones before it, and the lanes below that have the same digit
#pragma unroll
  for (int i = 0; i < Items; ++i) {
    const uint32_t d = (uint32_t)(key[i] >> shift) & mask;
    const bool valid = j0 + i * 64 < here;
    unsigned long long same = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1u;
      const unsigned long long set = __ballot(bit);
      same &= bit ? set : ~set;
    }
    const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0));
    const uint32_t before = mine[d];
    __builtin_amdgcn_wave_barrier();
    rank[i] = before + below;
    if (valid && below == 0) mine[d] = before + (uint32_t)__popcll(same);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();

  uint32_t total = 0, upTo = 0;
  if (tid < kSortDigits) {
#pragma unroll
    for (int k = 0; k < kSortWaves; ++k) {
      const uint32_t c = cnt[k][tid];
      cnt[k][tid] = total;
      total += c;
    }
    __hip_atomic_store(&words[(size_t)tile * kSortDigits + tid], (tile == 0 ? kSortSum : kSortCounts) | total, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    clear[(size_t)tile * kSortDigits + tid] = 0;
    upTo = total;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t up = __shfl_up(upTo, o);
      if ((int)lane >= o) upTo += up;
    }
    if (lane == 63) wave[w] = upTo;
  }
  __syncthreads();
  if (tid < kSortDigits) {
    for (uint32_t k = 0; k < w; ++k) upTo += wave[k];
    local[tid] = upTo - total;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < Items; ++i) {
    const uint32_t d = (uint32_t)(key[i] >> shift) & mask;
    rank[i] += local[d] + cnt[w][d];
    if (j0 + i * 64 < here) buf[rank[i]] = key[i];
  }
  if (tid < kSortDigits) {
    uint32_t prev = 0;
    if (tile > 0) {
      constexpr int kBack = 4;  // words asked for at once
      uint32_t t = tile;        // the tiles before it are still to be added
      for (;;) {
        uint32_t word[kBack];
#pragma unroll
        for (int k = 0; k < kBack; ++k)
          word[k] = t > (uint32_t)k ? __hip_atomic_load(&words[(size_t)(t - 1 - k) * kSortDigits + tid], __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT) : kSortSum;
        bool done = false, wait = false;
#pragma unroll
        for (int k = 0; k < kBack; ++k) {
          if (done || wait) continue;
          if (word[k] < kSortCounts) {
            wait = true;
          } else {
            prev += word[k] & kSortValue;
            done = word[k] >= kSortSum;
            --t;
          }
        }
        if (done) break;
        if (wait) __builtin_amdgcn_s_sleep(1);
      }
      __hip_atomic_store(&words[(size_t)tile * kSortDigits + tid], kSortSum | (prev + total), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    base[tid] = start[tid] + prev - local[tid];
  }
  __syncthreads();
  uint32_t to[Items];
#pragma unroll
  for (int i = 0; i < Items; ++i) {
    const uint32_t j = i * kSortThreads + tid;
    to[i] = 0;
    if (j < here) {
      const uint64_t k = buf[j];
      to[i] = base[(uint32_t)(k >> shift) & mask] + j;
      Ko[to[i]] = k;
    }
  }
  __syncthreads();
  uint32_t* vbuf = reinterpret_cast<uint32_t*>(buf);
#pragma unroll
  for (int i = 0; i < Items; ++i)
    if (j0 + i * 64 < here) vbuf[rank[i]] = val[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < Items; ++i) {
    const uint32_t j = i * kSortThreads + tid;
    if (j < here) Vo[to[i]] = vbuf[j];
  }
}

// The passes of one build, in order.  Each pass's tiles publish in one array of words and clear the other.
class Sorter {
 public:
  SortPasses passes;   // all of them; filled before count()
  SortScratch s{};

  hipError_t count(const IndPtrs& inds, const float* vals, size_t n, int N, const BaseKey& bk, unsigned long long* bad,
                   hipStream_t st) {
    coo_ = SortIn{nullptr, nullptr, inds, vals, bk, N};
    n_ = (uint32_t)n;
    const int copyBits = passes.n <= 16 ? 2 : 1;  // 64 KB of LDS at most
    const size_t lds = ((size_t)passes.n * kSortDigits * 4) << copyBits;
    const uint32_t blocks = count_blocks(n);
    hipLaunchKernelGGL(sort_count_kernel, dim3(blocks), dim3(512), lds, st, inds, n_, N, bk, passes, s, sort_tiles(n), copyBits,
                       bad);
    hipLaunchKernelGGL(sort_start_kernel, dim3((unsigned)passes.n), dim3(1024), 0, st, s, blocks);
    return hipGetLastError();
  }
  // Passes `from` .. `from + many - 1`: from K / V (null: the COO arrays), which stay as they are, to Ko / Vo; Kt / Vt is a
  // buffer pair that the passes between them may use.
  hipError_t run(int from, int many, const uint64_t* K, const uint32_t* V, uint64_t* Ko, uint32_t* Vo, uint64_t* Kt, uint32_t* Vt,
                 hipStream_t st) {
    const uint32_t tiles = sort_tiles(n_);
    const size_t half = (size_t)tiles * kSortDigits;
    for (int p = 0; p < many; ++p) {
      const bool out = (many - 1 - p) % 2 == 0;
      uint64_t* k = out ? Ko : Kt;
      uint32_t* v = out ? Vo : Vt;
      const int at = from + p;
      SortIn in = coo_;
      in.K = K;
      in.V = V;
      uint32_t* words = s.words + (done_ % 2) * half;
      uint32_t* clear = s.words + (1 - done_ % 2) * half;
      ++done_;
      auto kernel = sort_items(n_) == kSortLong ? (K ? sort_pass_kernel<false, kSortLong> : sort_pass_kernel<true, kSortLong>)
                                                : (K ? sort_pass_kernel<false, kSortShort> : sort_pass_kernel<true, kSortShort>);
      hipLaunchKernelGGL(kernel, dim3(tiles), dim3(kSortThreads), 0, st, in, k, v, n_, passes.shift[at], passes.mask[at],
                         s.start + (size_t)at * kSortDigits, s.ticket + at, words, clear);
      K = k;
      V = v;
    }
    return hipGetLastError();
  }

 private:
  SortIn coo_{};
  uint32_t n_ = 0;
  unsigned done_ = 0;
};

}  // namespace
}  // namespace hbcsf

#endif
