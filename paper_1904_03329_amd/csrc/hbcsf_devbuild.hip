// Device-side format builder: COO in device memory -> per-mode HB-CSF in the caller's device arena
// (Sections III-B, IV, V; the pre-processing whose cost Section VI-E discusses).  It produces, array for
// array, what the host builder produces: sort by the packed (root, ..., leaf) key, find slices and fibers,
// put each slice into the COO / CSL / CSF group, cut fibers on the run grid (fbr-split), record which
// slices span several runs (slc-split), and write the run tables and row bitmaps.
//
// Sorting.  Every mode's levels below the root keep the order of one list of all modes, so the nonzeros are sorted once
// by that list and a mode's order is one stable sort of the result by the mode's own index alone: two or three radix
// passes instead of a whole key's eight.  The keys keep the layout of the common order in every mode: the sort looks at
// the root's bits where they lie, and "the index of some level or one above it changes" is a difference of two keys
// under that level's mask (a pass that rewrote the keys as (root, ..., leaf) first took 0.23 ms of 50 M nonzeros).
// Keys of 64 bits are sorted by hbcsf_sort.h, wider ones and tensors of 2^30 nonzeros and more by rocPRIM.
//
// Numbering.  No array is kept per nonzero but a bit a level.  A wavefront takes 1024 (or 256) sorted nonzeros, 64 at a
// time; "a slice / a fiber begins here" are ballots, kept as bits for the kernels that need no more of the keys, so what
// it needs to number them is the count before its tile (one scan over the tiles).
// Slices get their group, their place in it and the fibers before them by a scan over slices; fbr-split adds a segment
// start only where a run begins inside a fiber, which is looked up once per run (a search over the slices, a scan over
// the runs), so a segment's number is the fibers before it plus the cuts before it.  The sorted keys are read twice
// and each output is written once.
//
// The scans over tiles, slices and runs are rocPRIM device primitives; everything specific to the format
// is in the kernels below.  With the per-fiber group choice a slice's nonzeros part between two groups, and the
// numbering goes through per-nonzero scans instead (number_mode_per_fiber).

#include <hip/hip_runtime.h>

#include <cstring>  // before rocPRIM, whose texture iterator calls memset without including it

#include <rocprim/rocprim.hpp>

#include <chrono>
#include <functional>
#include <memory>
#include <new>
#include <string>

#include "hbcsf.h"
#include "hbcsf_sort.h"
#include "hbcsf_tensor.h"

using namespace hbcsf;

namespace {

typedef unsigned __int128 u128;

struct Spec {
  int N, NF;
  int shift[HBCSF_MAX_ORDER];       // by level: where its index lies in the common key
  uint64_t mask[HBCSF_MAX_ORDER];
  u128 upTo[HBCSF_MAX_ORDER];       // by level: the bits of it and of every level above, the block's among them
  uint32_t L, cooOn, cslOn, cooRowFlags;
  uint32_t byteLevels;  // bit l: level l's row map holds bytes, otherwise bits
  uint32_t marked;      // bit g: group g has row maps
  uint32_t askLeaf;     // a leaf's row is looked up before it is marked
  uint32_t perFiber;  // hybrid_granularity = 1: heavy slices are split into a CSL piece and a CSF piece
  int blockBits, blockDrop;  // level-1 blocking: (index of level 1 >> blockDrop) stands above the root
};

struct C6 {  // running slice and nonzero counts of the three groups
  uint32_t s[3], m[3];
};
struct C6Plus {
  __host__ __device__ C6 operator()(const C6& a, const C6& b) const {
    C6 r;
    for (int g = 0; g < 3; ++g) {
      r.s[g] = a.s[g] + b.s[g];
      r.m[g] = a.m[g] + b.m[g];
    }
    return r;
  }
};

constexpr uint8_t kSplit = 3;  // a slice stored as a CSL piece (its singleton-fiber nonzeros) and a CSF piece

struct Tables {
  const uint32_t* sidp;    // [M] 1 + slice number of every sorted nonzero
  const uint32_t* sStart;  // [S + 1] first nonzero of every slice
  const uint8_t* grp;      // [S] group of every slice (kSplit: both)
  const C6* c6;            // [S + 1] slices / nonzeros of each group before every slice
  // per-fiber group choice only (else nullptr):
  const uint32_t* sgScan;        // [M] singleton-fiber nonzeros at or before every sorted nonzero
  const uint32_t* nat[2];        // [M] natural fiber number (inclusive scan) at fiber levels 1 and 2, where such a
                                 // level lies above the deepest one
  const uint32_t* firstKept[2];  // by natural fiber of that level: its first nonzero that stays in the CSF group
};

// Does some index of the levels in `upTo` change at sorted nonzero p?
template <typename Key>
__device__ __forceinline__ bool fresh_at(const Key* K, size_t p, Key upTo) {
  return p == 0 || ((K[p] ^ K[p - 1]) & upTo) != 0;
}

// Is nonzero p the only one of its deepest-level fiber?  (deep: the bits down to that level)
template <typename Key>
__device__ __forceinline__ bool single_at(const Key* K, size_t p, size_t M, Key deep) {
  return fresh_at(K, p, deep) && (p + 1 == M || fresh_at(K, p + 1, deep));
}

// Group and position of sorted nonzero p.  In a split slice the singleton-fiber nonzeros go, in order, to the
// slice's CSL piece and the others to its CSF piece; sgScan counts the former.
__device__ __forceinline__ void locate(const Tables& t, size_t p, uint32_t& s, int& g, uint32_t& pos) {
  s = t.sidp[p] - 1;
  g = t.grp[s];
  const uint32_t b = t.sStart[s];
  if (g != kSplit) {
    pos = t.c6[s].m[g] + (uint32_t)(p - b);
    return;
  }
  const uint32_t before = b ? t.sgScan[b - 1] : 0u;
  const uint32_t upTo = t.sgScan[p] - before;                 // singles of the slice at or before p
  const bool single = upTo != (p > b ? t.sgScan[p - 1] - before : 0u);
  if (single) {
    g = kCsl;
    pos = t.c6[s].m[kCsl] + upTo - 1u;
  } else {
    g = kCsf;
    pos = t.c6[s].m[kCsf] + (uint32_t)(p - b) - upTo;
  }
}

template <typename Key>
struct FreshFlag {  // 1 where the index at some tree level (and everything above it) changes
  const Key* K;
  Key upTo;
  __device__ uint32_t operator()(size_t p) const { return fresh_at(K, p, upTo) ? 1u : 0u; }
};

// Does a fiber of the CSF group start at nonzero p (of that group) at the level whose bits end `upTo`?  Without
// the per-fiber choice: where the index at that level or above changes.  With it, nonzeros may have left the slice
// for the CSL piece, so: where p is the first nonzero of its natural fiber that stayed (`upper` = 0 / 1 selects the
// tables of fiber level 1 / 2; the deepest level needs none: a nonzero that left was a fiber of its own).
template <typename Key>
__device__ __forceinline__ bool fiber_starts(const Key* K, size_t p, Key upTo, const Tables& t, int upper) {
  if (upper >= 0 && t.firstKept[upper]) return t.firstKept[upper][t.nat[upper][p] - 1u] == (uint32_t)p;
  return fresh_at(K, p, upTo);
}

template <typename Key>
struct SegFlag {  // 1 where a fiber segment of the CSF group starts
  const Key* K;
  Key upTo;
  Tables t;
  uint32_t L;
  size_t M;
  int upper;  // 0 / 1: fiber level 1 / 2 lies above the deepest level (per-fiber tables apply); -1: deepest level
  __device__ uint32_t operator()(size_t p) const {
    if (p >= M) return 0u;
    uint32_t s, pos;
    int g;
    locate(t, p, s, g, pos);
    if (g != kCsf) return 0u;
    return ((pos % L) == 0 || fiber_starts(K, p, upTo, t, upper)) ? 1u : 0u;
  }
};

template <typename Key>
struct SingleFlag {  // 1 where a nonzero is the only one of its deepest-level fiber
  const Key* K;
  Key deep;
  size_t M;
  __device__ uint32_t operator()(size_t p) const { return p < M && single_at(K, p, M, deep) ? 1u : 0u; }
};

struct SliceIn {  // what a slice adds to the running group counts
  const uint8_t* grp;
  const uint32_t* sStart;
  size_t S;
  const uint32_t* sgScan;  // per-fiber choice only
  __device__ C6 operator()(size_t s) const {
    C6 r{{0, 0, 0}, {0, 0, 0}};
    if (s < S) {
      const int g = grp[s];
      const uint32_t b = sStart[s], e = sStart[s + 1];
      if (g == kSplit) {
        const uint32_t ns = sgScan[e - 1] - (b ? sgScan[b - 1] : 0u);
        r.s[kCsl] = 1;
        r.m[kCsl] = ns;
        r.s[kCsf] = 1;
        r.m[kCsf] = (e - b) - ns;
      } else {
        r.s[g] = 1;
        r.m[g] = e - b;
      }
    }
    return r;
  }
};

struct PopcIn {
  const uint32_t* bits;
  size_t words;
  __device__ uint32_t operator()(size_t w) const { return w < words ? (uint32_t)__popc(bits[w]) : 0u; }
};

struct SquareIn {
  const float* v;
  __device__ double operator()(size_t z) const { return (double)v[z] * (double)v[z]; }
};

__device__ __forceinline__ void wave_add(unsigned long long* dst, unsigned long long v) {
  for (int d = 32; d > 0; d >>= 1) v += __shfl_down(v, d, 64);
  if ((threadIdx.x & 63) == 0 && v) atomicAdd(dst, v);
}

struct Carried {  // what rides along while one 64-bit half of a wide key is being sorted
  uint64_t other;  // the half that is not the sort key of this pass
  uint32_t v, pad;
};

// Key = uint64_t: K / V receive the packed key and the value bits.  Key = u128: the key is sorted in two
// stable 64-bit passes, so the low half goes to K (as uint64_t) and the high half rides in C.
template <typename Key>
__global__ void pack_kernel(IndPtrs inds, const float* vals, size_t M, int N, BaseKey bk, uint64_t* K, uint32_t* V, Carried* C,
                            unsigned long long* bad) {
  const size_t z = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (z >= M) return;
  bool off = false;
  const Key key = pack_key<Key>(inds, N, bk, z, off);
  if (sizeof(Key) == 8) {
    K[z] = (uint64_t)key;
    V[z] = __float_as_uint(vals[z]);
  } else {
    K[z] = (uint64_t)key;
    C[z] = Carried{(uint64_t)((u128)key >> 64), __float_as_uint(vals[z]), 0u};
  }
  if (off) atomicOr(bad, 1ull);
}

// Wide keys: what is sorted is (block, root) with the place in the common order, then the rest is fetched.
__global__ void root_key_kernel(const u128* __restrict__ base, size_t M, Spec sp, int rootBits, uint64_t* __restrict__ K,
                                uint32_t* __restrict__ V) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= M) return;
  uint64_t key = (uint64_t)(base[p] >> sp.shift[0]) & sp.mask[0];
  if (sp.blockBits) key |= (((uint64_t)(base[p] >> sp.shift[1]) & sp.mask[1]) >> sp.blockDrop) << rootBits;
  K[p] = key;
  V[p] = (uint32_t)p;
}
__global__ void fetch_kernel(const u128* __restrict__ base, const uint32_t* __restrict__ baseV, const uint32_t* __restrict__ at,
                             size_t M, u128* __restrict__ K, uint32_t* __restrict__ V) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= M) return;
  const uint32_t z = at[p];
  K[p] = base[z];
  V[p] = baseV[z];
}

// between the two passes of a wide sort: the high half becomes the key, the low half rides along
__global__ void swap_halves_kernel(const uint64_t* keyIn, const Carried* carIn, size_t M, uint64_t* keyOut,
                                   Carried* carOut) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= M) return;
  const Carried c = carIn[p];
  keyOut[p] = c.other;
  carOut[p] = Carried{keyIn[p], c.v, 0u};
}

__global__ void join_halves_kernel(const uint64_t* hi, const Carried* car, size_t M, u128* K, uint32_t* V) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= M) return;
  const Carried c = car[p];
  K[p] = ((u128)hi[p] << 64) | (u128)c.other;
  V[p] = c.v;
}

// first nonzero of every slice, from the scanned slice numbers
template <typename Key>
__global__ void slice_start_kernel(const Key* K, const uint32_t* sidp, size_t M, Key upTo0, uint32_t* sStart) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= M) return;
  if (fresh_at(K, p, upTo0)) sStart[sidp[p] - 1] = (uint32_t)p;
  if (p == M - 1) sStart[sidp[p]] = (uint32_t)M;
}

// Section V / VI-D: one nonzero -> COO; every fiber a single nonzero -> CSL; otherwise CSF
__global__ void classify_kernel(const uint32_t* sStart, const uint32_t* F0, const uint32_t* F1, const uint32_t* F2,
                                size_t S, Spec sp, const uint32_t* sgScan, uint8_t* grp, unsigned long long* cnt) {
  unsigned long long c0 = 0, c1 = 0, c2 = 0;
  for (size_t s = (size_t)blockIdx.x * blockDim.x + threadIdx.x; s < S; s += (size_t)gridDim.x * blockDim.x) {
    const uint32_t b = sStart[s], e = sStart[s + 1];
    const uint32_t n = e - b;
    const uint32_t nf0 = F0[e - 1] - (b ? F0[b - 1] : 0u);
    const uint32_t nf1 = sp.NF >= 2 ? F1[e - 1] - (b ? F1[b - 1] : 0u) : 0u;
    const uint32_t nf2 = sp.NF >= 3 ? F2[e - 1] - (b ? F2[b - 1] : 0u) : 0u;
    const uint32_t deep = sp.NF == 3 ? nf2 : sp.NF == 2 ? nf1 : nf0;
    uint8_t g;
    if (n == 1 && sp.cooOn) g = kCoo;
    else if (deep == n && sp.cslOn) g = kCsl;
    else g = kCsf;
    if (sp.perFiber && g == kCsf && n >= 2u * sp.L) {
      // heavy enough to be merged with atomic adds anyway, and at least an eighth of it in singleton fibers
      const uint32_t ns = sgScan[e - 1] - (b ? sgScan[b - 1] : 0u);
      if ((unsigned long long)ns * 8ull >= (unsigned long long)n) g = kSplit;
    }
    grp[s] = g;
    if (g == kCsf && !sp.perFiber) {  // with the per-fiber choice the fibers that stay are counted after the split
      c0 += nf0;
      c1 += nf1;
      c2 += nf2;
    }
  }
  wave_add(cnt + 2, c0);
  wave_add(cnt + 3, c1);
  wave_add(cnt + 5, c2);
}

// per-fiber choice: for every natural fiber of an upper fiber level, the first of its nonzeros that stays in the
// CSF group (atomic minimum over the nonzeros of CSF and split slices)
__global__ void first_kept_kernel(size_t M, Tables t, uint32_t* first0, uint32_t* first1) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= M) return;
  uint32_t s, pos;
  int g;
  locate(t, p, s, g, pos);
  if (g != kCsf) return;
  if (first0) atomicMin(&first0[t.nat[0][p] - 1u], (uint32_t)p);
  if (first1) atomicMin(&first1[t.nat[1][p] - 1u], (uint32_t)p);
}

__global__ void fill_words_kernel(uint32_t* p, size_t n, uint32_t v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// per-fiber choice: fibers per level among the nonzeros that stay in the CSF group (statistics)
template <typename Key>
__global__ void count_kept_fibers_kernel(const Key* K, size_t M, Spec sp, Tables t, unsigned long long* cnt) {
  unsigned long long c[3] = {0, 0, 0};
  for (size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x; p < M; p += (size_t)gridDim.x * blockDim.x) {
    uint32_t s, pos;
    int g;
    locate(t, p, s, g, pos);
    if (g != kCsf) continue;
    for (int l = 1; l <= sp.NF; ++l) c[l - 1] += fiber_starts(K, p, (Key)sp.upTo[l], t, l < sp.NF ? l - 1 : -1) ? 1u : 0u;
  }
  wave_add(cnt + 2, c[0]);
  wave_add(cnt + 3, c[1]);
  wave_add(cnt + 5, c[2]);
}

struct OutArrays {
  uint32_t* cooInd[HBCSF_MAX_ORDER];
  uint32_t* cooVal;
  uint32_t* cslInd[HBCSF_MAX_ORDER];
  uint32_t* cslPtr;
  uint32_t* cslRun;
  uint32_t* cslVal;
  uint32_t* csfInd[HBCSF_MAX_ORDER];
  uint32_t* csfPtr[HBCSF_MAX_ORDER];
  uint32_t* csfRun[HBCSF_MAX_ORDER];
  uint32_t* csfVal;
  uint32_t* owned;
  uint32_t* cooBits;
  uint32_t* seen[3][HBCSF_MAX_ORDER];  // statistics: map of the factor rows each group gathers, per level (mark_row)
};

// Marks a factor row as gathered (statistics).  Up to kByteRows rows one byte each: a plain store of the same byte whoever
// writes it, nothing read first and nothing atomic (as a bitmap, tested before an atomic or, the marks took 30 % of a
// 5 M-nonzero build: copies of a word in eight L2s stay stale, and every nonzero that meets one adds an atomic).  Longer
// modes keep the bitmap, which is what still fits an L2 (40 M rows: 7 ms of a 150 M-nonzero build against 10 ms).
constexpr uint64_t kByteRows = 4ull << 20;
__device__ __forceinline__ void mark_row(const Spec& sp, int group, int level, uint32_t* map, uint32_t r) {
  if (!((sp.marked >> group) & 1u)) return;
  if ((sp.byteLevels >> level) & 1u) {
    reinterpret_cast<uint8_t*>(map)[r] = 1;
  } else {
    const uint32_t bit = 1u << (r & 31);
    if (!(map[r >> 5] & bit)) atomicOr(&map[r >> 5], bit);
  }
}

// every nonzero writes itself into its group's stream; segment starts write the fiber-level entries
template <typename Key>
__global__ void fill_nonzeros_kernel(const Key* K, const uint32_t* V, size_t M, Spec sp, Tables t,
                                     const uint32_t* seg0, const uint32_t* seg1, const uint32_t* seg2, OutArrays o) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= M) return;
  uint32_t s, pos;
  int g;
  locate(t, p, s, g, pos);
  const Key key = K[p];
  uint32_t idx[HBCSF_MAX_ORDER];
  for (int l = 0; l < sp.N; ++l) idx[l] = (uint32_t)((uint64_t)(key >> sp.shift[l]) & sp.mask[l]);
  const uint32_t v = V[p];
  if (g == kCoo) {
    for (int l = sp.cooRowFlags ? 1 : 0; l < sp.N; ++l) o.cooInd[l][pos] = idx[l];
    for (int l = 1; l < sp.N; ++l) mark_row(sp, kCoo, l, o.seen[kCoo][l], idx[l]);
    o.cooVal[pos] = v;
    atomicOr(&o.cooBits[idx[0] >> 5], 1u << (idx[0] & 31));
    atomicOr(&o.owned[idx[0] >> 5], 1u << (idx[0] & 31));
    return;
  }
  const bool cut = (pos % sp.L) == 0;
  const uint32_t ord = t.c6[s].s[g];
  if (g == kCsl) {
    for (int l = 1; l < sp.N; ++l) o.cslInd[l][pos] = idx[l];
    for (int l = 1; l < sp.N; ++l) mark_row(sp, kCsl, l, o.seen[kCsl][l], idx[l]);
    o.cslVal[pos] = v;
    if (cut) o.cslRun[pos / sp.L] = ord;
    return;
  }
  o.csfInd[sp.N - 1][pos] = idx[sp.N - 1];
  mark_row(sp, kCsf, sp.N - 1, o.seen[kCsf][sp.N - 1], idx[sp.N - 1]);
  o.csfVal[pos] = v;
  if (cut) o.csfRun[0][pos / sp.L] = ord;
  for (int l = 1; l <= sp.NF; ++l) {
    const bool fresh = fiber_starts(K, p, (Key)sp.upTo[l], t, l < sp.NF ? l - 1 : -1);
    if (cut || fresh) {
      const uint32_t id = (l == 1 ? seg0 : l == 2 ? seg1 : seg2)[p];
      o.csfInd[l][id] = idx[l];
      o.csfPtr[l][id] = pos;
      mark_row(sp, kCsf, l, o.seen[kCsf][l], idx[l]);
      if (cut) o.csfRun[l][pos / sp.L] = id;
    }
  }
}

// per-slice entries of the CSL and CSF groups; a slice inside one run owns its output row
template <typename Key>
__global__ void fill_slices_kernel(const Key* K, size_t S, Spec sp, Tables t, OutArrays o,
                                   unsigned long long* cnt) {
  unsigned long long shared = 0;
  for (size_t s = (size_t)blockIdx.x * blockDim.x + threadIdx.x; s < S; s += (size_t)gridDim.x * blockDim.x) {
    const int g = t.grp[s];
    if (g == kSplit) {  // two pieces with the same root index, neither owns the row
      const uint32_t root = (uint32_t)((uint64_t)(K[t.sStart[s]] >> sp.shift[0]) & sp.mask[0]);
      o.cslInd[0][t.c6[s].s[kCsl]] = root;
      o.cslPtr[t.c6[s].s[kCsl]] = t.c6[s].m[kCsl];
      o.csfInd[0][t.c6[s].s[kCsf]] = root;
      o.csfPtr[0][t.c6[s].s[kCsf]] = t.c6[s].m[kCsf];
      ++shared;
    } else if (g != kCoo) {
      const uint32_t b = t.sStart[s], n = t.sStart[s + 1] - b;
      const uint32_t a = t.c6[s].m[g], ord = t.c6[s].s[g];
      const uint32_t root = (uint32_t)((uint64_t)(K[b] >> sp.shift[0]) & sp.mask[0]);
      const bool own = sp.blockBits == 0 && (a / sp.L) == ((a + n - 1) / sp.L);
      if (g == kCsl) {
        o.cslInd[0][ord] = root | (own ? kOwnedBit : 0u);
        o.cslPtr[ord] = a;
      } else {
        o.csfInd[0][ord] = root | (own ? kOwnedBit : 0u);
        o.csfPtr[0][ord] = a;
      }
      if (own) atomicOr(&o.owned[root >> 5], 1u << (root & 31));
      else ++shared;
    }
  }
  wave_add(cnt + 1, shared);
}

// ---- numbering without per-nonzero arrays ----
// Sorted nonzeros a wavefront numbers, 256 at a time.  Below 2 M there are fewer tiles of 1024 than the chip holds wavefronts,
// and the four steps of a tile, each a chain of dependent loads, are the kernels' time (50 000 nonzeros of order 4, tiles
// of 1024 -> 256: filling 27 -> 11 us a mode, the slices' tables 10 -> 3.4, counting 8.7 -> 4.8; builds of 50 000 to 1.6 M
// nonzeros 3 to 10 % shorter).
inline uint32_t tile_of(size_t M) { return M < (2u << 20) ? 256u : 1024u; }
constexpr uint32_t kSliceBlock = 1024; // slices a block numbers

struct Count4 {  // v[0]: slices, v[1..3]: fibers of levels 1..3
  uint32_t v[4];
};
struct Count4Plus {
  __host__ __device__ Count4 operator()(const Count4& a, const Count4& b) const {
    Count4 r;
    for (int l = 0; l < 4; ++l) r.v[l] = a.v[l] + b.v[l];
    return r;
  }
};
struct GroupCounts {  // slices and nonzeros per group, fibers of the CSF group per level
  uint32_t s[3], m[3], f[3];
};
struct GroupCountsPlus {
  __host__ __device__ GroupCounts operator()(const GroupCounts& a, const GroupCounts& b) const {
    GroupCounts r;
    for (int g = 0; g < 3; ++g) {
      r.s[g] = a.s[g] + b.s[g];
      r.m[g] = a.m[g] + b.m[g];
      r.f[g] = a.f[g] + b.f[g];
    }
    return r;
  }
};
struct alignas(16) SliceInfo {  // one load of 16 bytes; its differences are modulo 2^32
  uint32_t shift, ord;  // place in the group's stream minus sorted place, number in the group
  uint32_t grp;
  uint32_t fib0;        // CSF: level-1 fibers before the slice in its group minus those before it at all
};
struct Totals {
  uint32_t bad, S, fibNat[3];
  GroupCounts g;
  uint32_t extra[3];  // cuts that do not fall on the begin of a fiber, per level
};

// The tables one mode's numbering fills (device memory).
struct Numbers {
  uint32_t per;          // nonzeros of a tile: tile_of()
  Count4* tile;          // [tiles + 1] counts per tile, then before each
  uint32_t* sStart;      // [S + 1] first nonzero of every slice
  uint32_t* fStart[3];   // [S + 1] fibers of each level before the slice
  GroupCounts* block;    // [slice blocks + 1] counts per block of slices, then before each
  SliceInfo* info;       // [S]
  uint32_t* fib[2];      // [S] as fib0, levels 2, 3
  uint32_t* csfOff;      // by CSF slice: its first place in the stream,
  uint32_t* csfStart;    //               its first sorted nonzero
  unsigned long long* begun;  // [levels][tiles][per / 64] bit p: a slice (level 0) or a fiber of the level begins at nonzero p
  uint8_t* inside;       // [runs + 1] bit l: the run begins inside a fiber of level l
  Count4* cutBlock;      // [blocks of runs + 1] cuts inside a fiber per kCutBlock runs, then before them
  Count4* cut;           // [runs + 1] cuts inside a fiber before each run
  uint32_t* count;       // {S}
};

// x of the lane before; lane 0: `first`
template <typename Key>
__device__ __forceinline__ Key lane_before(Key x, Key first, int lane) {
  uint32_t w[sizeof(Key) / 4];
  __builtin_memcpy(w, &x, sizeof(Key));
#pragma unroll
  for (uint32_t& k : w) k = __shfl_up(k, 1);
  __builtin_memcpy(&x, w, sizeof(Key));
  return lane == 0 ? first : x;
}

template <typename Key>
__device__ __forceinline__ Key last_lane(Key x) {
  uint32_t w[sizeof(Key) / 4];
  __builtin_memcpy(w, &x, sizeof(Key));
#pragma unroll
  for (uint32_t& k : w) k = __builtin_amdgcn_readlane(k, 63);
  __builtin_memcpy(&x, w, sizeof(Key));
  return x;
}

// Keys and begins of the kFill chunks of 64 sorted nonzeros from p0 on (a whole wavefront), zeros past M.  last: the key
// before p0, then the last one here.
constexpr int kFill = 4;
template <typename Key>
__device__ __forceinline__ void load_chunks(const Key* __restrict__ K, size_t p0, size_t M, const Spec& sp, int lane, Key& last,
                                            Key (&key)[kFill], uint32_t (&b)[kFill]) {
#pragma unroll
  for (int q = 0; q < kFill; ++q) {
    const size_t p = p0 + q * 64 + lane;
    key[q] = 0;
    if (p < M) key[q] = K[p];
  }
#pragma unroll
  for (int q = 0; q < kFill; ++q) {
    const size_t p = p0 + q * 64 + lane;
    const Key x = key[q] ^ lane_before(key[q], last, lane);
    last = last_lane(key[q]);
    b[q] = 0;
    for (int l = 0; l <= sp.NF; ++l) b[q] |= (p == 0 || (x & (Key)sp.upTo[l]) != 0 ? 1u : 0u) << l;
    if (p >= M) b[q] = 0;
  }
}

// (50 M nonzeros: 106 -> 92 us, 4.4 TB/s, with one load a nonzero and four in flight.)
template <typename Key>
__global__ __launch_bounds__(256) void count_tiles_kernel(const Key* __restrict__ K, size_t M, Spec sp, uint32_t tiles, Numbers n) {
  const int lane = threadIdx.x & 63;
  const uint32_t t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t > tiles) return;
  Count4 c{{0, 0, 0, 0}};
  if (t < tiles) {
    unsigned long long mine[4] = {0, 0, 0, 0};  // lane k: the bits of the tile's chunk k
    const size_t p0 = (size_t)t * n.per;
    Key last = p0 ? K[p0 - 1] : Key(0);
    for (uint32_t j = 0; j < n.per; j += 64 * kFill) {
      Key key[kFill];
      uint32_t b[kFill];
      load_chunks(K, p0 + j, M, sp, lane, last, key, b);
#pragma unroll
      for (int q = 0; q < kFill; ++q)
#pragma unroll
        for (int l = 0; l < 4; ++l)
          if (l <= sp.NF) {
            const unsigned long long w = __ballot((b[q] >> l) & 1u);
            c.v[l] += (uint32_t)__popcll(w);
            if (lane == (int)(j / 64) + q) mine[l] = w;
          }
    }
    for (int l = 0; l < 4; ++l)
      if (l <= sp.NF && lane < (int)(n.per / 64)) n.begun[((size_t)l * tiles + t) * (n.per / 64) + lane] = mine[l];
  }
  if (lane == 0) n.tile[t] = c;
}

// From the bits alone: 50 M nonzeros 87 (from the keys) -> 37 us.
__global__ __launch_bounds__(256) void slice_tables_kernel(size_t M, Spec sp, uint32_t tiles, Numbers n) {
  const int chunks = (int)(n.per / 64);
  const int lane = threadIdx.x & 63;
  const uint32_t t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= tiles) return;
  Count4 c = n.tile[t];
  const unsigned long long below = (1ull << lane) - 1ull;
  unsigned long long mine[4] = {0, 0, 0, 0};
#pragma unroll
  for (int l = 0; l < 4; ++l)
    if (l <= sp.NF && lane < chunks) mine[l] = n.begun[((size_t)l * tiles + t) * chunks + lane];
  for (int k = 0; k < chunks; ++k) {
    unsigned long long w[4];
#pragma unroll
    for (int l = 0; l < 4; ++l)
      w[l] = (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((uint32_t)mine[l], k) |
             (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(mine[l] >> 32), k) << 32;
    if ((w[0] >> lane) & 1ull) {
      const uint32_t s = c.v[0] + (uint32_t)__popcll(w[0] & below);
      n.sStart[s] = t * n.per + k * 64 + lane;
#pragma unroll
      for (int l = 1; l < 4; ++l)
        if (l <= sp.NF) n.fStart[l - 1][s] = c.v[l] + (uint32_t)__popcll(w[l] & below);
    }
#pragma unroll
    for (int l = 0; l < 4; ++l) c.v[l] += (uint32_t)__popcll(w[l]);
  }
  if (t == tiles - 1 && lane == 0) {  // one past the last slice
    const uint32_t S = c.v[0];
    n.sStart[S] = (uint32_t)M;
#pragma unroll
    for (int l = 1; l < 4; ++l)
      if (l <= sp.NF) n.fStart[l - 1][S] = c.v[l];
    n.count[0] = S;
  }
}

// Section V / VI-D: one nonzero -> COO; every fiber a single nonzero -> CSL; otherwise CSF
__device__ __forceinline__ GroupCounts slice_counts(const Numbers& n, const Spec& sp, uint32_t s, int& g) {
  const uint32_t m = n.sStart[s + 1] - n.sStart[s];
  uint32_t f[3] = {0, 0, 0};
  for (int l = 0; l < sp.NF; ++l) f[l] = n.fStart[l][s + 1] - n.fStart[l][s];
  if (m == 1 && sp.cooOn) g = kCoo;
  else if (f[sp.NF - 1] == m && sp.cslOn) g = kCsl;
  else g = kCsf;
  GroupCounts c{{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    c.s[k] = g == k ? 1u : 0u;
    c.m[k] = g == k ? m : 0u;
    c.f[k] = g == kCsf ? f[k] : 0u;
  }
  return c;
}

// inclusive sum over the block's threads, with the block's total in `total`
__device__ __forceinline__ GroupCounts block_sum(GroupCounts c, GroupCounts& total) {
  __shared__ GroupCounts wave[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  auto each = [](GroupCounts& x, auto&& f) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      f(x.s[k]);
      f(x.m[k]);
      f(x.f[k]);
    }
  };
#pragma unroll
  for (int o = 1; o < 64; o <<= 1)
    each(c, [&](uint32_t& v) {
      const uint32_t up = __shfl_up(v, o);
      if (lane >= o) v += up;
    });
  if (lane == 63) wave[w] = c;
  __syncthreads();
  GroupCountsPlus plus;
  for (int k = 0; k < w; ++k) c = plus(c, wave[k]);
  total = plus(plus(wave[0], wave[1]), plus(wave[2], wave[3]));
  __syncthreads();
  return c;
}

__global__ __launch_bounds__(256) void count_slices_kernel(Numbers n, Spec sp, uint32_t blocks) {
  GroupCountsPlus plus;
  GroupCounts c{{0, 0, 0}, {0, 0, 0}, {0, 0, 0}}, total;
  const uint32_t S = n.count[0];
  const uint64_t first = (uint64_t)blockIdx.x * kSliceBlock;
  if (blockIdx.x < blocks)
    for (uint32_t k = 0; k < kSliceBlock; k += 256) {
      const uint64_t s = first + k + threadIdx.x;
      int g;
      if (s < S) c = plus(c, slice_counts(n, sp, (uint32_t)s, g));
    }
  block_sum(c, total);
  if (threadIdx.x == 0) n.block[blockIdx.x] = total;
}

__global__ __launch_bounds__(256) void number_slices_kernel(Numbers n, Spec sp) {
  GroupCountsPlus plus;
  const uint32_t S = n.count[0];
  GroupCounts before = n.block[blockIdx.x];
  for (uint32_t k = 0; k < kSliceBlock; k += 256) {
    const uint64_t s = (uint64_t)blockIdx.x * kSliceBlock + k + threadIdx.x;
    if ((uint64_t)blockIdx.x * kSliceBlock + k >= S) return;  // the same for the whole block
    int g = kCoo;
    GroupCounts own{{0, 0, 0}, {0, 0, 0}, {0, 0, 0}}, total;
    if (s < S) own = slice_counts(n, sp, (uint32_t)s, g);
    const GroupCounts upTo = block_sum(own, total);
    if (s < S) {
      const uint32_t off = before.m[g] + upTo.m[g] - own.m[g], start = n.sStart[s];
      SliceInfo i;
      i.shift = off - start;
      i.ord = before.s[g] + upTo.s[g] - own.s[g];
      i.grp = (uint32_t)g;
      i.fib0 = before.f[0] + upTo.f[0] - own.f[0] - n.fStart[0][s];
      n.info[s] = i;
      for (int l = 1; l < sp.NF; ++l) n.fib[l - 1][s] = before.f[l] + upTo.f[l] - own.f[l] - n.fStart[l][s];
      if (g == kCsf) {
        n.csfOff[i.ord] = off;
        n.csfStart[i.ord] = start;
      }
    }
    before = plus(before, total);
  }
}

// Per run of the CSF stream and level: does it begin inside a fiber?  A block of runs lies between two slices, which two of its
// wavefronts look for with 64 places at a time; a run's own slice is searched between those.  The bits are an eighth of a
// byte per nonzero, where the two keys they came from are a line of memory per run.  With the two kernels below 50 M nonzeros
// 110 to 145 (a search over all slices, a library scan of 16 bytes a run) -> 30 to 34 us.
constexpr uint32_t kCutBlock = 1024;
__global__ __launch_bounds__(256) void find_cuts_kernel(Spec sp, Numbers n, uint32_t tiles, uint32_t blocks, uint32_t maxRuns) {
  __shared__ uint32_t range[2], sum[4][4];
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6, r0 = blockIdx.x * kCutBlock;
  const uint64_t end = n.block[blocks].m[kCsf];
  const uint32_t slices = n.block[blocks].s[kCsf];
  if (w < 2 && (uint64_t)r0 * sp.L < end) {
    const uint64_t far = ((uint64_t)r0 + kCutBlock - 1) * sp.L;
    const uint64_t at = w == 0 ? (uint64_t)r0 * sp.L : far < end ? far : end - 1;
    uint32_t lo = 0, hi = slices;  // the last slice that begins at or before `at`
    while (hi - lo > 1) {
      const uint64_t span = hi - lo;
      const uint32_t upTo = (uint32_t)__popcll(__ballot(n.csfOff[lo + (uint32_t)(span * (lane + 1) / 65)] <= at));
      const uint32_t from = lo;
      lo = from + (uint32_t)(span * upTo / 65);
      if (upTo < 64) hi = from + (uint32_t)(span * (upTo + 1) / 65);
    }
    if (lane == 0) range[w] = lo;
  }
  __syncthreads();
  uint32_t c[4] = {0, 0, 0, 0};
  for (uint32_t j = 0; j < kCutBlock; j += 256) {
    const uint32_t r = r0 + j + threadIdx.x;
    const uint64_t at = (uint64_t)r * sp.L;
    uint32_t in = 0;
    if (r <= maxRuns && at < end) {
      uint32_t lo = range[0], hi = range[1] + 1;
      while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (n.csfOff[mid] <= at) lo = mid;
        else hi = mid;
      }
      const uint32_t p = n.csfStart[lo] + (uint32_t)(at - n.csfOff[lo]);
      for (int l = 1; l <= sp.NF; ++l)
        in |= (uint32_t)(~n.begun[(size_t)l * tiles * (n.per / 64) + p / 64] >> (p % 64) & 1ull) << l;
    }
    if (r <= maxRuns) n.inside[r] = (uint8_t)in;
#pragma unroll
    for (int l = 1; l < 4; ++l) c[l] += (uint32_t)__popcll(__ballot((in >> l) & 1u));
  }
  if (lane == 0)
    for (int l = 1; l < 4; ++l) sum[w][l] = c[l];
  __syncthreads();
  if (threadIdx.x == 0) {
    Count4 all{{0, 0, 0, 0}};
    for (int k = 0; k < 4; ++k)
      for (int l = 1; l < 4; ++l) all.v[l] += sum[k][l];
    n.cutBlock[blockIdx.x] = all;
  }
}

// Cuts before each block of runs, and what the host waits for.  One block.
__global__ __launch_bounds__(1024) void totals_kernel(Numbers n, Spec sp, uint32_t tiles, uint32_t blocks, uint32_t cutBlocks,
                                                      const unsigned long long* bad, Totals* out) {
  __shared__ uint32_t wave[16][4];
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t before[4] = {0, 0, 0, 0};
  for (uint32_t b0 = 0; b0 < cutBlocks; b0 += 1024) {
    const uint32_t b = b0 + threadIdx.x;
    Count4 own{{0, 0, 0, 0}};
    if (b < cutBlocks) own = n.cutBlock[b];
    uint32_t upTo[4];
    for (int l = 1; l < 4; ++l) {
      upTo[l] = own.v[l];
      for (uint32_t o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_up(upTo[l], o);
        if (lane >= o) upTo[l] += up;
      }
      if (lane == 63) wave[w][l] = upTo[l];
    }
    __syncthreads();
    for (int l = 1; l < 4; ++l) {
      uint32_t all = 0;
      for (uint32_t k = 0; k < 16; ++k) {
        if (k == w) upTo[l] += all;
        all += wave[k][l];
      }
      own.v[l] = before[l] + upTo[l] - own.v[l];
      before[l] += all;
    }
    if (b < cutBlocks) n.cutBlock[b] = own;
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  Totals t{};
  t.bad = (uint32_t)*bad;
  t.S = n.count[0];
  for (int l = 0; l < sp.NF; ++l) {
    t.fibNat[l] = n.tile[tiles].v[1 + l];
    t.extra[l] = before[1 + l];
  }
  t.g = n.block[blocks];
  *out = t;
}

__global__ __launch_bounds__(256) void number_cuts_kernel(Numbers n, uint32_t maxRuns) {
  constexpr int kEach = kCutBlock / 256;
  __shared__ uint32_t count[kEach][4][4];
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long below = (1ull << lane) - 1ull;
  const Count4 first = n.cutBlock[blockIdx.x];
  uint32_t pre[kEach][4];
#pragma unroll
  for (int j = 0; j < kEach; ++j) {
    const uint32_t r = blockIdx.x * kCutBlock + j * 256 + threadIdx.x;
    const uint32_t in = r <= maxRuns ? n.inside[r] : 0u;
#pragma unroll
    for (int l = 1; l < 4; ++l) {
      const unsigned long long set = __ballot((in >> l) & 1u);
      pre[j][l] = (uint32_t)__popcll(set & below);
      if (lane == 0) count[j][w][l] = (uint32_t)__popcll(set);
    }
  }
  __syncthreads();
  uint32_t before[4] = {0, first.v[1], first.v[2], first.v[3]};
#pragma unroll
  for (int j = 0; j < kEach; ++j) {
    const uint32_t r = blockIdx.x * kCutBlock + j * 256 + threadIdx.x;
    Count4 c{{0, 0, 0, 0}};
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k)
#pragma unroll
      for (int l = 1; l < 4; ++l) {
        if (k == w) c.v[l] = before[l] + pre[j][l];
        before[l] += count[j][k][l];
      }
    if (r <= maxRuns) n.cut[r] = c;
  }
}

// Every nonzero writes itself into its group's stream; segment starts write the fiber-level entries.  A wavefront takes
// kFill chunks of 64 nonzeros at a time and issues the loads of all of them first (keys, values; then slice tables; then
// cuts), since each nonzero's chain key -> slice -> place -> cuts is four loads long and the stores between them may not be
// passed by a load.  What bounds it is the number of vector-memory instructions, hence tables of differences (one entry
// instead of two) and the key before from the lane before: order 4, 50 M nonzeros, 768 -> 634 us a mode against separate
// tables with the fiber and cut entries loaded between the stores (of that, the stores of the row marks are 130 us).
template <typename Key, int N>
__global__ __launch_bounds__(256) void fill_tiles_kernel(const Key* __restrict__ K, const uint32_t* __restrict__ V, size_t M,
                                                         Spec sp, uint32_t tiles, Numbers n, OutArrays o) {
  const int lane = threadIdx.x & 63;
  const uint32_t t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= tiles) return;
  Count4 c = n.tile[t];
  const unsigned long long below = (1ull << lane) - 1ull;
  constexpr int leaf = N - 1, NF = N - 2;
  const uint32_t ls = __builtin_ctz(sp.L);  // runs are of 8, 16, 32 or 64 nonzeros
  const size_t p0 = (size_t)t * n.per;
  Key last = p0 ? K[p0 - 1] : Key(0);
  for (uint32_t j0 = 0; j0 < n.per; j0 += 64 * kFill) {
    Key key[kFill];
    uint32_t b[kFill], v[kFill], begun[kFill][NF], fib[kFill][NF], pos[kFill], cuts[kFill][NF], leafIdx[kFill], marked[kFill];
    SliceInfo in[kFill];
#pragma unroll
    for (int q = 0; q < kFill; ++q) {
      const size_t p = p0 + j0 + q * 64 + lane;
      v[q] = 0;
      if (p < M) v[q] = V[p];
    }
    load_chunks(K, p0 + j0, M, sp, lane, last, key, b);
#pragma unroll
    for (int q = 0; q < kFill; ++q) {
      const size_t p = p0 + j0 + q * 64 + lane;
      uint32_t s = 0;
#pragma unroll
      for (int l = 0; l <= NF; ++l) {  // begun before p
        const unsigned long long w = __ballot((b[q] >> l) & 1u);
        const uint32_t before = c.v[l] + (uint32_t)__popcll(w & below);
        c.v[l] += (uint32_t)__popcll(w);
        if (l == 0) s = before + (b[q] & 1u) - 1u;
        else begun[q][l > 0 ? l - 1 : 0] = before;
      }
      if (p < M) {
        in[q] = n.info[s];
#pragma unroll
        for (int l = 2; l <= NF; ++l) fib[q][l - 1] = n.fib[l - 2][s];
      }
    }
#pragma unroll
    for (int q = 0; q < kFill; ++q) {
      const size_t p = p0 + j0 + q * 64 + lane;
      leafIdx[q] = (uint32_t)((uint64_t)(key[q] >> sp.shift[leaf]) & sp.mask[leaf]);
      marked[q] = 0;
      if (p < M) {
        // is the leaf's row marked already?  (a stale answer only marks it once more)
        const uint32_t grp = in[q].grp;
        if (sp.askLeaf && ((sp.marked >> grp) & 1u)) {
          const uint32_t* map = grp == kCsf ? o.seen[kCsf][leaf] : grp == kCsl ? o.seen[kCsl][leaf] : o.seen[kCoo][leaf];
          marked[q] = reinterpret_cast<const uint8_t*>(map)[leafIdx[q]];
        }
        pos[q] = (uint32_t)p + in[q].shift;
        fib[q][0] = in[q].fib0;
        if (in[q].grp == kCsf) {  // cuts before this place
          const Count4& at = n.cut[(pos[q] + sp.L - 1u) >> ls];
#pragma unroll
          for (int l = 1; l <= NF; ++l) cuts[q][l - 1] = at.v[l];
        }
      }
    }
#pragma unroll
    for (int q = 0; q < kFill; ++q) {
      if (p0 + j0 + q * 64 + lane >= M) continue;
      const uint32_t at = pos[q];
      auto index = [&](int l) { return (uint32_t)((uint64_t)(key[q] >> sp.shift[l]) & sp.mask[l]); };
      const bool cut = (at & (sp.L - 1u)) == 0;
      if (in[q].grp == kCsf) {
        o.csfVal[at] = v[q];
        o.csfInd[leaf][at] = leafIdx[q];
        if (!marked[q]) mark_row(sp, kCsf, leaf, o.seen[kCsf][leaf], leafIdx[q]);
        if (cut) o.csfRun[0][at >> ls] = in[q].ord;
#pragma unroll
        for (int l = 1; l <= NF; ++l) {
          if (cut || ((b[q] >> l) & 1u)) {
            // fibers before the slice and in it, cuts before this place
            const uint32_t id = fib[q][l - 1] + begun[q][l - 1] + cuts[q][l - 1];
            const uint32_t i = index(l);
            o.csfInd[l][id] = i;
            o.csfPtr[l][id] = at;
            mark_row(sp, kCsf, l, o.seen[kCsf][l], i);
            if (cut) o.csfRun[l][at >> ls] = id;
          }
        }
      } else if (in[q].grp == kCsl) {
        o.cslVal[at] = v[q];
        if (cut) o.cslRun[at >> ls] = in[q].ord;
        o.cslInd[leaf][at] = leafIdx[q];
        if (!marked[q]) mark_row(sp, kCsl, leaf, o.seen[kCsl][leaf], leafIdx[q]);
#pragma unroll
        for (int l = 1; l < leaf; ++l) {
          const uint32_t i = index(l);
          o.cslInd[l][at] = i;
          mark_row(sp, kCsl, l, o.seen[kCsl][l], i);
        }
      } else {
        o.cooVal[at] = v[q];
        o.cooInd[leaf][at] = leafIdx[q];
        if (!marked[q]) mark_row(sp, kCoo, leaf, o.seen[kCoo][leaf], leafIdx[q]);
#pragma unroll
        for (int l = 1; l < leaf; ++l) {
          const uint32_t i = index(l);
          o.cooInd[l][at] = i;
          mark_row(sp, kCoo, l, o.seen[kCoo][l], i);
        }
        const uint32_t root = index(0);
        if (!sp.cooRowFlags) o.cooInd[0][at] = root;
        atomicOr(&o.cooBits[root >> 5], 1u << (root & 31));
        atomicOr(&o.owned[root >> 5], 1u << (root & 31));
      }
    }
  }
}

struct Sentinels {
  uint64_t cslN0, cslNnz, cslRuns, csfN[HBCSF_MAX_ORDER], csfNnz, csfRuns;
};

__device__ __forceinline__ void put_sentinels(const Spec& sp, const OutArrays& o, const Sentinels& z) {
  o.cslInd[0][z.cslN0] = 0;
  o.cslPtr[z.cslN0] = (uint32_t)z.cslNnz;
  o.cslRun[z.cslRuns] = (uint32_t)z.cslN0;
  for (int l = 0; l < sp.N - 1; ++l) {
    o.csfInd[l][z.csfN[l]] = 0;
    o.csfPtr[l][z.csfN[l]] = (uint32_t)z.csfNnz;
    o.csfRun[l][z.csfRuns] = (uint32_t)z.csfN[l];
  }
}
__global__ void sentinel_kernel(Spec sp, OutArrays o, Sentinels z) {
  if (blockIdx.x == 0 && threadIdx.x == 0) put_sentinels(sp, o, z);
}

// Per-slice entries of the CSL and CSF groups; a slice inside one run owns its output row.  The arrays' sentinels are written
// beside.  The shared slices are counted per block, 512 blocks: one add a wavefront to the same word, 8192 of them, was the
// kernel's time (0.9 M slices 108 -> 21 us).
template <typename Key>
__global__ __launch_bounds__(256) void fill_slice_entries_kernel(const Key* __restrict__ K, uint32_t S, Spec sp, Numbers n,
                                                                 OutArrays o, Sentinels z, unsigned long long* cnt) {
  __shared__ uint32_t wave[4];
  if (blockIdx.x == 0 && threadIdx.x == 0) put_sentinels(sp, o, z);
  uint32_t shared = 0;
  for (uint64_t s = (uint64_t)blockIdx.x * 256 + threadIdx.x; s < S; s += (uint64_t)gridDim.x * 256) {
    const SliceInfo in = n.info[s];
    if (in.grp == kCoo) continue;
    const uint32_t b = n.sStart[s], m = n.sStart[s + 1] - b;
    const uint32_t root = (uint32_t)((uint64_t)(K[b] >> sp.shift[0]) & sp.mask[0]);
    const uint32_t off = in.shift + b;
    const bool own = sp.blockBits == 0 && (off / sp.L) == ((off + m - 1) / sp.L);
    uint32_t* ind = in.grp == kCsl ? o.cslInd[0] : o.csfInd[0];
    uint32_t* ptr = in.grp == kCsl ? o.cslPtr : o.csfPtr[0];
    ind[in.ord] = root | (own ? kOwnedBit : 0u);
    ptr[in.ord] = off;
    if (own) atomicOr(&o.owned[root >> 5], 1u << (root & 31));
    else ++shared;
  }
  for (int d = 32; d > 0; d >>= 1) shared += __shfl_down(shared, d);
  if ((threadIdx.x & 63) == 0) wave[threadIdx.x >> 6] = shared;
  __syncthreads();
  const uint32_t all = wave[0] + wave[1] + wave[2] + wave[3];
  if (threadIdx.x == 0 && all) atomicAdd(cnt + 1, (unsigned long long)all);
}

__global__ void zero_words_kernel(uint32_t* a, size_t na, uint32_t* b, size_t nb, uint32_t* c, size_t nc) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < na + nb + nc; i += (size_t)gridDim.x * blockDim.x)
    *(i < na ? a + i : i < na + nb ? b + (i - na) : c + (i - na - nb)) = 0;
}

// Bits set in several maps (bitmaps, or bytes of 0 and 1): blockIdx.y says which.
struct BitCounts {
  const uint32_t* map[1 + 3 * (HBCSF_MAX_ORDER - 1)];
  size_t words[1 + 3 * (HBCSF_MAX_ORDER - 1)];
  int to[1 + 3 * (HBCSF_MAX_ORDER - 1)];  // place in cnt
};
__global__ void count_bits_kernel(BitCounts b, unsigned long long* cnt) {
  const uint32_t* map = b.map[blockIdx.y];
  const size_t words = b.words[blockIdx.y];
  unsigned long long c = 0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (size_t)gridDim.x * blockDim.x)
    c += (unsigned long long)__popc(map[i]);
  wave_add(cnt + b.to[blockIdx.y], c);
}

// for kernels that loop over their items and end in a few same-address atomics per wavefront
inline unsigned grid_capped(size_t n) { const size_t b = (n + 255) / 256; return (unsigned)(b < 1 ? 1 : (b > 2048 ? 2048 : b)); }
inline unsigned grid_for(size_t n) { return (unsigned)((n + 255) / 256 > 0 ? (n + 255) / 256 : 1); }
inline uint64_t up256(uint64_t v) { return (v + 255) / 256 * 256; }

// Workspace carve-up for M nonzeros; `temp` is the rocPRIM scratch, sized by temp_bytes().
struct Workspace {
  uint64_t* K[3];        // 64-bit sort keys.  Up to 64 bits: [2] the common order, [0] one mode's order, [1] where the
  uint32_t* V[3];        // per-fiber choice or a blocked order by rocPRIM's sort needs it; wide keys: [0], [1] a double
                         // buffer.  V: the values (or places) riding along
  Carried* C[2];         // wide keys only: the other half + value, double buffered
  u128* K128[2];         // wide keys only: the common order, one mode's order
  Numbers n;             // numbering tables
  uint32_t* seg2;        // order 5 with the per-fiber choice: the third fiber level's scan
  uint32_t* sgScan;      // per-fiber choice only: scan of the singleton-fiber flags
  uint32_t* nat[2];      // per-fiber choice, orders 4 / 5: natural fiber numbers of the upper fiber levels
  uint32_t* firstKept[2];  // ... and the first nonzero of each such fiber that stays in the CSF group
  uint8_t* grp;          // per-fiber choice only
  C6* c6;                // per-fiber choice only
  unsigned long long* bad;  // an index is not below its dimension
  unsigned long long* cnt;  // kCounters per mode; behind them normSq
  Totals* totals;
  double* normSq;
  uint8_t* seen;         // row maps of the 3 groups and the levels below the root (statistics)
  bool ownSort;          // own_sort(): its scratch is sort.s
  Sorter sort;
  void* temp;
  size_t tempBytes;
  uint64_t total;
};

constexpr int kCounters = 32;

// Is the group chosen per fiber?  (needs the CSL group)
bool per_fiber(const hbcsf_opts& o) { return o.hybrid_granularity == 1 && (o.group_mask == 0 || (o.group_mask & 2u)); }

// Is a leaf's row looked up before it is marked?  With a few nonzeros a row it is nearly always marked already, and the load, which
// goes with the others, costs less than the store; with fewer it only adds to it.  Whole builds, marked at once -> looked up, us:
// 50 M nonzeros of order 4 over 1 M leaf rows 7824 -> 7666, 20 M over 1 M 2976 -> 2948, 20 M over 4 M 4306 -> 4216, 10 M over 2 M 3396
// -> 3402; but 8 M over 4 M 2003 -> 2114 (order 4 2545 -> 2660), 4 M over 4 M 1333 -> 1404 and 1619 -> 1766 (uniform leaf indices,
// but for the 50 M).
constexpr uint64_t kAskLeafPer = 4;   // nonzeros a row
bool asks_leaf(size_t M, uint64_t rows) { return rows <= kByteRows && M >= kAskLeafPer * rows; }

// Bytes of a mode's row map, and of one group's row maps of all modes.
uint64_t row_map_bytes(uint64_t rows) { return up256(rows <= kByteRows ? rows : (rows + 7) / 8); }
uint64_t row_maps_bytes(int order, const uint64_t* dims) {
  uint64_t sum = 0;
  for (int m = 0; m < order; ++m) sum += row_map_bytes(dims[m]);
  return sum;
}

// Entries the slice tables need: slices are at most nonzeros, and without blocking at most rows.
uint64_t slice_bound(size_t M, uint64_t maxDim, bool blocked) { return blocked || (uint64_t)M < maxDim ? (uint64_t)M : maxDim; }

// Does the pair sort of hbcsf_sort.h serve?  Keys of 64 bits, and places that fit its published words.  (A whole build by
// rocPRIM's sort -> by that one, order 3, indices by Zipf's law of 1.2, us: 20 000 nonzeros 668 -> 636, 0.2 M 745 -> 688, 0.8 M
// 1079 -> 825, 3.2 M 1271 -> 1071, 40 M 7032 -> 4853; order 4, 1.3 to 0.8: 803 -> 795, 979 -> 873, 1440 -> 1061, 1751 -> 1426,
// 10 142 -> 6974; a sixth of the last two's gain is that the arrays are not copied any more.  Of 60 builds of 3000 to 20 M
// nonzeros, uniform and skewed, orders 3 to 5 and every option, each is 3 to 80 % faster since.)
bool own_sort(size_t M, int maxBits) { return maxBits <= 64 && M > 0 && M < (size_t)kSortCounts; }

hipError_t temp_bytes(size_t M, size_t maxWords, uint64_t slices, int totalBits, size_t* out) {
  const bool wide = totalBits > 64;
  // the largest scratch any rocPRIM call below asks for
  size_t need = 0, b = 0;
  hipError_t e = hipSuccess;
  if (wide) {
    rocprim::double_buffer<uint64_t> kb((uint64_t*)nullptr, (uint64_t*)nullptr);
    rocprim::double_buffer<uint32_t> vb((uint32_t*)nullptr, (uint32_t*)nullptr);
    e = rocprim::radix_sort_pairs(nullptr, b, kb, vb, M, 0u, 64u);
    if (e != hipSuccess) return e;
    need = b > need ? b : need;
    rocprim::double_buffer<Carried> cb((Carried*)nullptr, (Carried*)nullptr);
    e = rocprim::radix_sort_pairs(nullptr, b, kb, cb, M, 0u, 64u);
  } else if (!own_sort(M, totalBits)) {
    // (the most any range of bits takes: with more than one pass the scratch holds a second copy of the pairs)
    e = rocprim::radix_sort_pairs(nullptr, b, (const uint64_t*)nullptr, (uint64_t*)nullptr, (const uint32_t*)nullptr,
                                  (uint32_t*)nullptr, M, 0u, 64u);
  }
  if (e != hipSuccess) return e;
  need = b > need ? b : need;
  const size_t tiles = M / tile_of(M) + 2;
  e = rocprim::exclusive_scan(nullptr, b, (Count4*)nullptr, (Count4*)nullptr, Count4{}, tiles, Count4Plus());
  if (e != hipSuccess) return e;
  need = b > need ? b : need;
  e = rocprim::exclusive_scan(nullptr, b, (GroupCounts*)nullptr, (GroupCounts*)nullptr, GroupCounts{},
                              (size_t)(slices / kSliceBlock + 2), GroupCountsPlus());
  if (e != hipSuccess) return e;
  need = b > need ? b : need;
  auto cnt = rocprim::counting_iterator<size_t>(0);
  e = rocprim::inclusive_scan(nullptr, b, rocprim::make_transform_iterator(cnt, FreshFlag<u128>{nullptr, 0}),
                              (uint32_t*)nullptr, M + 1, rocprim::plus<uint32_t>());
  if (e != hipSuccess) return e;
  need = b > need ? b : need;
  e = rocprim::inclusive_scan(nullptr, b, rocprim::make_transform_iterator(cnt, SingleFlag<u128>{nullptr, 0, 0}),
                              (uint32_t*)nullptr, M + 1, rocprim::plus<uint32_t>());
  if (e != hipSuccess) return e;
  need = b > need ? b : need;
  e = rocprim::exclusive_scan(nullptr, b, rocprim::make_transform_iterator(cnt, SegFlag<u128>{nullptr, 0, Tables{}, 1, 0, -1}),
                              (uint32_t*)nullptr, 0u, M + 1, rocprim::plus<uint32_t>());
  if (e != hipSuccess) return e;
  need = b > need ? b : need;
  e = rocprim::exclusive_scan(nullptr, b, rocprim::make_transform_iterator(cnt, SliceIn{nullptr, nullptr, 0, nullptr}),
                              (C6*)nullptr, C6{{0, 0, 0}, {0, 0, 0}}, M + 1, C6Plus());
  if (e != hipSuccess) return e;
  need = b > need ? b : need;
  e = rocprim::exclusive_scan(nullptr, b, rocprim::make_transform_iterator(cnt, PopcIn{nullptr, 0}),
                              (uint32_t*)nullptr, 0u, maxWords + 1, rocprim::plus<uint32_t>());
  if (e != hipSuccess) return e;
  need = b > need ? b : need;
  e = rocprim::reduce(nullptr, b, rocprim::make_transform_iterator(cnt, SquareIn{nullptr}), (double*)nullptr, 0.0,
                      M, rocprim::plus<double>());
  if (e != hipSuccess) return e;
  need = b > need ? b : need;
  *out = need + 256;
  return hipSuccess;
}

void carve(Workspace& w, uint8_t* base, int order, size_t M, uint64_t mapBytes, uint64_t slices, uint32_t L, size_t tempBytes,
           bool wide, bool perFiber, bool blocked) {
  uint64_t off = 0;
  w.ownSort = own_sort(M, wide ? 65 : 64);
  auto take = [&](uint64_t bytes) {
    uint8_t* p = base ? base + off : nullptr;
    off += up256(bytes);
    return p;
  };
  const bool second = perFiber || (blocked && !w.ownSort);   // K[1], V[1] of keys up to 64 bits
  for (int i = 0; i < 3; ++i) w.K[i] = (wide ? i < 2 : i != 1 || second) ? (uint64_t*)take((M + 1) * 8) : nullptr;
  for (int i = 0; i < 3; ++i) w.V[i] = wide || i != 1 || second ? (uint32_t*)take((M + 1) * 4) : nullptr;
  for (int i = 0; i < 2; ++i) w.C[i] = wide ? (Carried*)take((M + 1) * sizeof(Carried)) : nullptr;
  for (int i = 0; i < 2; ++i) w.K128[i] = wide ? (u128*)take((M + 1) * 16) : nullptr;
  const uint64_t tables = perFiber ? (uint64_t)M : slices;
  w.n.tile = (Count4*)take((M / tile_of(M) + 2) * sizeof(Count4));
  w.n.per = tile_of(M);
  w.n.sStart = (uint32_t*)take((tables + 2) * 4);
  for (int l = 0; l < 3; ++l) w.n.fStart[l] = l < order - 2 && !perFiber ? (uint32_t*)take((tables + 2) * 4) : nullptr;
  w.n.block = (GroupCounts*)take((tables / kSliceBlock + 2) * sizeof(GroupCounts));
  w.n.info = perFiber ? nullptr : (SliceInfo*)take((tables + 1) * sizeof(SliceInfo));
  for (int l = 0; l < 2; ++l) w.n.fib[l] = l + 1 < order - 2 && !perFiber ? (uint32_t*)take((tables + 1) * 4) : nullptr;
  w.n.csfOff = perFiber ? nullptr : (uint32_t*)take((tables + 1) * 4);
  w.n.csfStart = perFiber ? nullptr : (uint32_t*)take((tables + 1) * 4);
  w.n.cut = (Count4*)take((M / L + 2) * sizeof(Count4));
  w.n.cutBlock = (Count4*)take((M / L / kCutBlock + 2) * sizeof(Count4));
  w.n.count = (uint32_t*)take(4);
  w.seg2 = perFiber && order >= 5 ? (uint32_t*)take((M + 2) * 4) : nullptr;
  w.sgScan = perFiber ? (uint32_t*)take((M + 2) * 4) : nullptr;
  for (int f = 0; f < 2; ++f) {
    const bool upper = perFiber && f < order - 3;   // fiber level f + 1 lies above the deepest one
    w.nat[f] = upper ? (uint32_t*)take((M + 2) * 4) : nullptr;
    w.firstKept[f] = upper ? (uint32_t*)take((M + 2) * 4) : nullptr;
  }
  w.grp = perFiber ? (uint8_t*)take(M + 1) : nullptr;
  w.c6 = perFiber ? (C6*)take((M + 2) * sizeof(C6)) : nullptr;
  w.bad = (unsigned long long*)take(8);
  w.cnt = (unsigned long long*)take((HBCSF_MAX_ORDER * kCounters + 1) * 8);
  w.normSq = (double*)(w.cnt + HBCSF_MAX_ORDER * kCounters);
  w.totals = (Totals*)take(sizeof(Totals));
  w.seen = (uint8_t*)take(3 * mapBytes);
  if (w.ownSort) sort_scratch(M, take(sort_scratch(M, nullptr, &w.sort.s)), &w.sort.s);
  // between the sorts of two modes the third buffer pair of hbcsf_sort.h is free (at least 32 KB and 12 bytes a nonzero)
  const uint64_t begunBytes = (uint64_t)(order - 1) * ((M + tile_of(M) - 1) / tile_of(M)) * (tile_of(M) / 8);
  w.n.begun = perFiber ? nullptr : w.ownSort ? (unsigned long long*)w.sort.s.K : (unsigned long long*)take(begunBytes);
  w.n.inside = perFiber ? nullptr : w.ownSort ? (uint8_t*)w.sort.s.K + up256(begunBytes) : take(M / L + 2);
  w.temp = take(tempBytes);
  w.tempBytes = tempBytes;
  w.total = off;
}

uint64_t arena_bound(int N, const uint64_t* dims, uint64_t M, uint32_t L) {
  uint64_t bytes = 0;
  for (int m = 0; m < N; ++m) {
    const uint64_t words = (uint64_t)(2 * N + 1) * M + (uint64_t)3 * N * (M / L + 2) + 3 * (dims[m] / 32 + 2) + 64;
    bytes += words * 4 + 40 * kAlign + define_state_bytes(dims[m]);
  }
  return bytes;
}

// totalBits: bits of the packed (root, .., leaf) key; maxBits: the widest key of any mode, block bits included
int check_args(int order, const uint64_t* dims, uint64_t nnz, const hbcsf_opts* opts, hbcsf_opts* o, int* totalBits,
               int* maxBits) {
  if (order < 3 || order > HBCSF_MAX_ORDER) return fail(HBCSF_EINVAL, "order must be 3, 4 or 5");
  if (!dims) return fail(HBCSF_EINVAL, "dims is null");
  if (nnz >= 0xffff0000ull) return fail(HBCSF_ERANGE, "nnz must be below 2^32 - 2^16");
  int total = 0;
  for (int m = 0; m < order; ++m) {
    if (dims[m] == 0 || dims[m] > 0x7ffffffeull) return fail(HBCSF_ERANGE, "each dimension must be in 1 .. 2^31-2");
    total += bits_for(dims[m]);
  }
  *o = hbcsf_opts{};
  if (opts) *o = *opts;
  if (o->fiber_threshold == 0) o->fiber_threshold = default_fiber_threshold(order);
  const uint32_t ft = o->fiber_threshold;
  if (!(ft == 8 || ft == 16 || ft == 32 || ft == 64)) return fail(HBCSF_EINVAL, "fiber_threshold must be 8, 16, 32 or 64");
  if (o->mode_order_policy > 2) return fail(HBCSF_EINVAL, "mode_order_policy must be 0, 1 or 2");
  if (o->group_mask > 4) return fail(HBCSF_EINVAL, "group_mask must be 0..4");
  if (o->coo_row_flags > 1) return fail(HBCSF_EINVAL, "coo_row_flags must be 0 or 1");
  if (o->mid_blocking > 13) return fail(HBCSF_EINVAL, "mid_blocking must be 0 or 1 (off) or 2..13 bits");
  if (o->hybrid_granularity > 1) return fail(HBCSF_EINVAL, "hybrid_granularity must be 0 or 1");
  if (o->single_representation > 1) return fail(HBCSF_EINVAL, "single_representation must be 0 or 1");
  if (o->single_representation) {
    if ((opts->fiber_threshold && opts->fiber_threshold != default_fiber_threshold(order)) || o->group_mask ||
        o->hybrid_granularity || o->coo_row_flags || o->mid_blocking > 1)
      return fail(HBCSF_EINVAL, "single_representation goes with default options only");
    o->group_mask = 4;  // plain B-CSF: the kernel for the other modes walks one group
  }
  if (total > 128)
    return fail(HBCSF_ERANGE, "the packed coordinates exceed 128 bits");
  *totalBits = total;
  int bbMax = 0;
  for (int m = 0; m < order; ++m) {
    const int bb = mid_block_bits(order, dims, *o, m);
    bbMax = bb > bbMax ? bb : bbMax;
  }
  *maxBits = total + bbMax;
  return HBCSF_OK;
}

#define HIP_TRY(expr, what)                         \
  do {                                              \
    const hipError_t e_ = (expr);                   \
    if (e_ != hipSuccess) return fail_hip(e_, what); \
  } while (0)

// Where a mode's arrays go: memory of that many bytes, 256-byte aligned, or an error code.
using Place = std::function<int(uint64_t, uint8_t**)>;

// What one mode's build needs to know, and what it leaves for the end.
struct ModeBuild {
  Spec sp{};
  int rootBits = 0;
  uint64_t S = 0, gS[3] = {0, 0, 0}, gM[3] = {0, 0, 0};
  uint64_t nSeg[HBCSF_MAX_FIBER_LEVELS] = {0, 0, 0}, fibNat[HBCSF_MAX_FIBER_LEVELS] = {0, 0, 0};
  uint64_t fibCsf[HBCSF_MAX_FIBER_LEVELS] = {0, 0, 0};
  int sortFrom = 0, sortMany = 0;  // own_sort(): the passes of this mode's order
  bool whole[3] = {false, false, false};  // the group holds all nonzeros: its distinct rows are the other modes' slices
  unsigned long long* cnt = nullptr;  // device counters: [1] shared slices, [2], [3], [5] CSF fibers (per-fiber choice),
                                      // [4] owned rows, [8 ..] distinct rows
};

// The sorted nonzeros of one mode, and two buffers of 8 (M + 1) and 4 (M + 1) bytes free until the next mode.
template <typename Key>
struct Sorted {
  const Key* K = nullptr;
  const uint32_t* V = nullptr;
  void* freeKeys = nullptr;
  void* freeVals = nullptr;
};

// The common order of all modes: base.K / base.V (they must survive until the last mode is built).
template <typename Key>
int sort_base(int N, size_t M, const uint32_t* const* inds, const float* vals, const BaseKey& bk, int totalBits, Workspace& w,
              Sorted<Key>* base, hipStream_t st) {
  constexpr bool kWide = sizeof(Key) == 16;
  IndPtrs ip{};
  for (int m = 0; m < N; ++m) ip.p[m] = inds[m];
  if constexpr (!kWide) {
    if (w.ownSort) {
      base->K = w.K[2];
      base->V = w.V[2];
      HIP_TRY(w.sort.count(ip, vals, M, N, bk, w.bad, st), "counting of the digits");
      HIP_TRY(w.sort.run(0, (totalBits + 7) / 8, nullptr, nullptr, w.K[2], w.V[2], w.K[0], w.V[0], st), "radix sort");
      return HBCSF_OK;
    }
  }
  hipLaunchKernelGGL(pack_kernel<Key>, dim3(grid_for(M)), dim3(256), 0, st, ip, vals, M, N, bk, w.K[0], w.V[0], w.C[0], w.bad);
  size_t tb = w.tempBytes;
  if constexpr (!kWide) {
    HIP_TRY(rocprim::radix_sort_pairs(w.temp, tb, (const uint64_t*)w.K[0], w.K[2], (const uint32_t*)w.V[0], w.V[2], M, 0u,
                                      (unsigned)totalBits, st), "radix sort");
    base->K = w.K[2];
    base->V = w.V[2];
  } else {
    // two stable passes: by the low 64 bits with the high half riding along, then by the high bits
    rocprim::double_buffer<uint64_t> kb(w.K[0], w.K[1]);
    rocprim::double_buffer<Carried> cb(w.C[0], w.C[1]);
    HIP_TRY(rocprim::radix_sort_pairs(w.temp, tb, kb, cb, M, 0u, 64u, st), "radix sort");
    hipLaunchKernelGGL(swap_halves_kernel, dim3(grid_for(M)), dim3(256), 0, st, kb.current(), cb.current(), M,
                       kb.alternate(), cb.alternate());
    rocprim::double_buffer<uint64_t> kb2(kb.alternate(), kb.current());
    rocprim::double_buffer<Carried> cb2(cb.alternate(), cb.current());
    tb = w.tempBytes;
    // (a key may be wide by its block bits alone, which are not in this order)
    HIP_TRY(rocprim::radix_sort_pairs(w.temp, tb, kb2, cb2, M, 0u, (unsigned)(totalBits > 64 ? totalBits - 64 : 1), st),
            "radix sort");
    hipLaunchKernelGGL(join_halves_kernel, dim3(grid_for(M)), dim3(256), 0, st, kb2.current(), cb2.current(), M,
                       w.K128[0], w.V[2]);
    base->K = w.K128[0];
    base->V = w.V[2];
  }
  return HBCSF_OK;
}

// One mode's order: a stable sort of the common order by (block,) root.  isBase: the common order is this mode's own.
template <typename Key>
int sort_mode(size_t M, const Sorted<Key>& base, const ModeBuild& mb, bool isBase, Workspace& w, Sorted<Key>* out, hipStream_t st) {
  constexpr bool kWide = sizeof(Key) == 16;
  size_t tb = w.tempBytes;
  if constexpr (!kWide) {
    out->freeKeys = w.K[1];
    out->freeVals = w.V[1];
    out->K = base.K;
    out->V = base.V;
    if (isBase) return HBCSF_OK;
    const Spec& sp = mb.sp;
    if (w.ownSort) {
      HIP_TRY(w.sort.run(mb.sortFrom, mb.sortMany, base.K, base.V, w.K[0], w.V[0], w.sort.s.K, w.sort.s.V, st), "radix sort");
      out->K = w.K[0];
      out->V = w.V[0];
      return HBCSF_OK;
    }
    // by root, then (blocked modes) by block: the top bits of the level-1 index
    uint64_t* k = w.K[sp.blockBits ? 1 : 0];
    uint32_t* v = w.V[sp.blockBits ? 1 : 0];
    HIP_TRY(rocprim::radix_sort_pairs(w.temp, tb, base.K, k, base.V, v, M, (unsigned)sp.shift[0],
                                      (unsigned)(sp.shift[0] + mb.rootBits), st), "radix sort");
    if (sp.blockBits) {
      const unsigned from = (unsigned)(sp.shift[1] + sp.blockDrop);
      tb = w.tempBytes;
      HIP_TRY(rocprim::radix_sort_pairs(w.temp, tb, (const uint64_t*)k, w.K[0], (const uint32_t*)v, w.V[0], M, from,
                                        from + (unsigned)sp.blockBits, st), "radix sort");
    }
    out->K = w.K[0];
    out->V = w.V[0];
  } else {
    if (isBase) {
      *out = base;
      out->freeKeys = w.K[0];
      out->freeVals = w.V[0];
      return HBCSF_OK;
    }
    rocprim::double_buffer<uint64_t> kb(w.K[0], w.K[1]);
    rocprim::double_buffer<uint32_t> vb(w.V[0], w.V[1]);
    hipLaunchKernelGGL(root_key_kernel, dim3(grid_for(M)), dim3(256), 0, st, base.K, M, mb.sp, mb.rootBits, w.K[0], w.V[0]);
    HIP_TRY(rocprim::radix_sort_pairs(w.temp, tb, kb, vb, M, 0u, (unsigned)(mb.rootBits + mb.sp.blockBits), st), "radix sort");
    hipLaunchKernelGGL(fetch_kernel, dim3(grid_for(M)), dim3(256), 0, st, base.K, base.V, vb.current(), M, w.K128[1],
                       vb.alternate());
    out->K = w.K128[1];
    out->V = vb.alternate();
    out->freeKeys = kb.current();
    out->freeVals = vb.current();
  }
  return HBCSF_OK;
}

// Numbers slices, fibers and cuts of one mode and brings the group sizes to the host (one wait).
template <typename Key>
int number_mode(size_t M, uint64_t slices, const Sorted<Key>& so, ModeBuild& mb, Workspace& w, hipStream_t st) {
  const Spec& sp = mb.sp;
  const uint32_t tiles = (uint32_t)((M + w.n.per - 1) / w.n.per);
  const uint32_t blocks = (uint32_t)((slices + kSliceBlock - 1) / kSliceBlock);
  const uint32_t maxRuns = (uint32_t)((M + sp.L - 1) / sp.L);
  const dim3 tileGrid(tiles / 4 + 1);
  size_t tb = w.tempBytes;
  const uint32_t cutBlocks = maxRuns / kCutBlock + 1;
  hipLaunchKernelGGL(count_tiles_kernel<Key>, tileGrid, dim3(256), 0, st, so.K, M, sp, tiles, w.n);
  HIP_TRY(rocprim::exclusive_scan(w.temp, tb, w.n.tile, w.n.tile, Count4{}, (size_t)tiles + 1, Count4Plus(), st), "scan");
  hipLaunchKernelGGL(slice_tables_kernel, tileGrid, dim3(256), 0, st, M, sp, tiles, w.n);
  hipLaunchKernelGGL(count_slices_kernel, dim3(blocks + 1), dim3(256), 0, st, w.n, sp, blocks);
  tb = w.tempBytes;
  HIP_TRY(rocprim::exclusive_scan(w.temp, tb, w.n.block, w.n.block, GroupCounts{}, (size_t)blocks + 1, GroupCountsPlus(), st),
          "scan");
  hipLaunchKernelGGL(number_slices_kernel, dim3(blocks), dim3(256), 0, st, w.n, sp);
  hipLaunchKernelGGL(find_cuts_kernel, dim3(cutBlocks), dim3(256), 0, st, sp, w.n, tiles, blocks, maxRuns);
  hipLaunchKernelGGL(totals_kernel, dim3(1), dim3(1024), 0, st, w.n, sp, tiles, blocks, cutBlocks, w.bad, w.totals);
  Totals t{};
  HIP_TRY(hipMemcpyAsync(&t, w.totals, sizeof(Totals), hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
  HIP_TRY(hipStreamSynchronize(st), "hipStreamSynchronize");
  if (t.bad) return fail(HBCSF_ERANGE, "an index is not below its dimension");
  hipLaunchKernelGGL(number_cuts_kernel, dim3(cutBlocks), dim3(256), 0, st, w.n, maxRuns);  // (beside the caller's allocation)
  mb.S = t.S;
  for (int g = 0; g < 3; ++g) {
    mb.gS[g] = t.g.s[g];
    mb.gM[g] = t.g.m[g];
  }
  for (int f = 0; f < sp.NF; ++f) {
    mb.fibNat[f] = t.fibNat[f];
    mb.fibCsf[f] = t.g.f[f];
    mb.nSeg[f] = (uint64_t)t.g.f[f] + t.extra[f];
  }
  return HBCSF_OK;
}

// The per-fiber group choice: numbering through scans over the nonzeros (two waits).  sidp and seg[] lie in the sort's
// free buffers.
template <typename Key>
int number_mode_per_fiber(size_t M, const Sorted<Key>& so, ModeBuild& mb, Workspace& w, Tables* tables, uint32_t* (&seg)[3],
                          hipStream_t st) {
  const Spec& sp = mb.sp;
  const Key* K = so.K;
  uint32_t* sidp = (uint32_t*)so.freeKeys;
  seg[0] = sidp + (M + 1);
  seg[1] = (uint32_t*)so.freeVals;
  seg[2] = w.seg2;
  Tables& tb = *tables;
  auto cit = rocprim::counting_iterator<size_t>(0);
  // ---- slices: scan of "root index changes" ----
  size_t tb_ = w.tempBytes;
  HIP_TRY(rocprim::inclusive_scan(w.temp, tb_, rocprim::make_transform_iterator(cit, FreshFlag<Key>{K, (Key)sp.upTo[0]}),
                                  sidp, M, rocprim::plus<uint32_t>(), st), "scan");
  hipLaunchKernelGGL(slice_start_kernel<Key>, dim3(grid_for(M)), dim3(256), 0, st, K, sidp, M, (Key)sp.upTo[0], w.n.sStart);
  // natural fibers per level (the deepest level decides CSL membership)
  for (int f = 0; f < sp.NF; ++f) {
    tb_ = w.tempBytes;
    HIP_TRY(rocprim::inclusive_scan(w.temp, tb_, rocprim::make_transform_iterator(cit, FreshFlag<Key>{K, (Key)sp.upTo[1 + f]}),
                                    seg[f], M, rocprim::plus<uint32_t>(), st), "scan");
  }
  uint32_t tail[4] = {0, 0, 0, 0};
  HIP_TRY(hipMemcpyAsync(&tail[0], sidp + (M - 1), 4, hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
  for (int f = 0; f < sp.NF; ++f)
    HIP_TRY(hipMemcpyAsync(&tail[1 + f], seg[f] + (M - 1), 4, hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
  unsigned long long bad = 0;
  HIP_TRY(hipMemcpyAsync(&bad, w.bad, 8, hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
  HIP_TRY(hipStreamSynchronize(st), "hipStreamSynchronize");
  if (bad) return fail(HBCSF_ERANGE, "an index is not below its dimension");
  const size_t S = tail[0];
  mb.S = S;
  for (int f = 0; f < 3; ++f) mb.fibNat[f] = tail[1 + f];

  // ---- per-fiber group choice: which nonzeros are whole fibers of their own; the natural fiber numbers of the
  //      upper fiber levels are kept (the segment scans below overwrite seg[]) ----
  tb_ = w.tempBytes;
  HIP_TRY(rocprim::inclusive_scan(w.temp, tb_,
                                  rocprim::make_transform_iterator(cit, SingleFlag<Key>{K, (Key)sp.upTo[sp.NF], M}),
                                  w.sgScan, M, rocprim::plus<uint32_t>(), st), "scan");
  for (int f = 0; f + 1 < sp.NF; ++f)
    HIP_TRY(hipMemcpyAsync(w.nat[f], seg[f], M * 4, hipMemcpyDeviceToDevice, st), "hipMemcpyAsync");
  // ---- groups, and where every slice starts inside its group ----
  hipLaunchKernelGGL(classify_kernel, dim3(grid_capped(S)), dim3(256), 0, st, w.n.sStart, seg[0], seg[1], seg[2], S, sp,
                     w.sgScan, w.grp, mb.cnt);
  tb_ = w.tempBytes;
  HIP_TRY(rocprim::exclusive_scan(w.temp, tb_,
                                  rocprim::make_transform_iterator(cit, SliceIn{w.grp, w.n.sStart, S, w.sgScan}),
                                  w.c6, C6{{0, 0, 0}, {0, 0, 0}}, S + 1, C6Plus(), st), "scan");
  tb = Tables{sidp, w.n.sStart, w.grp, w.c6, w.sgScan, {nullptr, nullptr}, {nullptr, nullptr}};
  // the first nonzero of every upper-level fiber that stays in the CSF group, then the fibers that stay
  for (int f = 0; f + 1 < sp.NF; ++f) {
    tb.nat[f] = w.nat[f];
    hipLaunchKernelGGL(fill_words_kernel, dim3(grid_for(M + 1)), dim3(256), 0, st, w.firstKept[f], M + 1, 0xffffffffu);
  }
  if (sp.NF >= 2)
    hipLaunchKernelGGL(first_kept_kernel, dim3(grid_for(M)), dim3(256), 0, st, M, tb, w.firstKept[0],
                       sp.NF >= 3 ? w.firstKept[1] : nullptr);
  for (int f = 0; f + 1 < sp.NF; ++f) tb.firstKept[f] = w.firstKept[f];
  hipLaunchKernelGGL(count_kept_fibers_kernel<Key>, dim3(grid_capped(M)), dim3(256), 0, st, K, M, sp, tb, mb.cnt);
  // ---- fiber segments of the CSF group: numbered by a scan over the sorted order ----
  for (int f = 0; f < sp.NF; ++f) {
    tb_ = w.tempBytes;
    HIP_TRY(rocprim::exclusive_scan(w.temp, tb_,
                                    rocprim::make_transform_iterator(
                                        cit, SegFlag<Key>{K, (Key)sp.upTo[1 + f], tb, sp.L, M, f + 1 < sp.NF ? f : -1}),
                                    seg[f], 0u, M + 1, rocprim::plus<uint32_t>(), st), "scan");
  }
  C6 totals{};
  uint32_t segTotal[3] = {0, 0, 0};
  unsigned long long kept[kCounters];
  HIP_TRY(hipMemcpyAsync(&totals, w.c6 + S, sizeof(C6), hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
  for (int f = 0; f < sp.NF; ++f)
    HIP_TRY(hipMemcpyAsync(&segTotal[f], seg[f] + M, 4, hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
  HIP_TRY(hipMemcpyAsync(kept, mb.cnt, sizeof(kept), hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
  HIP_TRY(hipStreamSynchronize(st), "hipStreamSynchronize");
  for (int g = 0; g < 3; ++g) {
    mb.gS[g] = totals.s[g];
    mb.gM[g] = totals.m[g];
  }
  const int place[3] = {2, 3, 5};
  for (int f = 0; f < 3; ++f) {
    mb.nSeg[f] = segTotal[f];
    mb.fibCsf[f] = kept[place[f]];
  }
  return HBCSF_OK;
}

// Builds one mode from its sorted nonzeros: sizes, layout, fill.  The statistics that need counters are left in mb.cnt.
template <typename Key>
int build_mode_device(int N, const uint64_t* dims, size_t M, uint64_t slices, const Sorted<Key>& so, ModeBuild& mb, Workspace& w,
                      const Place& place, ModeFormat* out, bool othersCounted, hipStream_t st) {
  const Spec& sp = mb.sp;
  Tables tb{};
  uint32_t* seg[3] = {nullptr, nullptr, nullptr};
  if (M > 0) {
    const int rn = sp.perFiber ? number_mode_per_fiber(M, so, mb, w, &tb, seg, st) : number_mode(M, slices, so, mb, w, st);
    if (rn != HBCSF_OK) return rn;
  }
  // ---- layout, then fill ----
  layout_mode(out, N, mb.gS, mb.gM, mb.nSeg);
  uint8_t* base = nullptr;
  const int rp = place(out->blobBytes, &base);
  if (rp != HBCSF_OK) return rp;
  out->dev = base;
  auto U32 = [&](const ArrayRef& r) { return (uint32_t*)(base + r.off); };
  OutArrays o{};
  for (int l = 0; l < N; ++l) {
    o.cooInd[l] = U32(out->g[kCoo].ind[l]);
    o.cslInd[l] = U32(out->g[kCsl].ind[l]);
    o.csfInd[l] = U32(out->g[kCsf].ind[l]);
    o.csfPtr[l] = l < N - 1 ? U32(out->g[kCsf].ptr[l]) : nullptr;
    o.csfRun[l] = l < N - 1 ? U32(out->g[kCsf].runFirst[l]) : nullptr;
  }
  o.cooVal = U32(out->g[kCoo].val);
  o.cslVal = U32(out->g[kCsl].val);
  o.csfVal = U32(out->g[kCsf].val);
  o.cslPtr = U32(out->g[kCsl].ptr[0]);
  o.cslRun = U32(out->g[kCsl].runFirst[0]);
  o.owned = U32(out->ownedBits);
  o.cooBits = U32(out->cooBits);
  const size_t ownedWords = (out->rows + 31) / 32;
  // row maps: the groups that exist, their levels one after the other.  A group that holds all nonzeros gathers every row of a
  // mode that has a nonzero, as many as that mode has slices, and needs no map (50 M nonzeros 130 us a mode).
  for (int g = 0; g < 3; ++g) {
    mb.whole[g] = othersCounted && !sp.perFiber && M > 0 && out->g[g].nnz == M;
    if (out->g[g].nnz > 0 && !mb.whole[g]) mb.sp.marked |= 1u << g;
  }
  uint64_t mapBytes = 0;
  for (int g = 0; g < 3; ++g)
    for (int l = 1; l < N; ++l) {
      o.seen[g][l] = (uint32_t*)(w.seen + mapBytes);
      if ((sp.marked >> g) & 1u) mapBytes += row_map_bytes(dims[out->levelMode[l]]);
    }
  {
    const size_t mapWords = (size_t)(mapBytes / 4);
    hipLaunchKernelGGL(zero_words_kernel, dim3(grid_capped(mapWords + 2 * ownedWords)), dim3(256), 0, st, (uint32_t*)w.seen,
                       mapWords, o.owned, ownedWords, o.cooBits, ownedWords);
  }
  Sentinels z{};
  z.cslN0 = out->g[kCsl].n[0];
  z.cslNnz = out->g[kCsl].nnz;
  z.cslRuns = out->g[kCsl].runs;
  for (int l = 0; l < N - 1; ++l) z.csfN[l] = out->g[kCsf].n[l];
  z.csfNnz = out->g[kCsf].nnz;
  z.csfRuns = out->g[kCsf].runs;
  if (M == 0 || sp.perFiber) hipLaunchKernelGGL(sentinel_kernel, dim3(1), dim3(64), 0, st, sp, o, z);
  if (M > 0 && sp.perFiber) {
    hipLaunchKernelGGL(fill_nonzeros_kernel<Key>, dim3(grid_for(M)), dim3(256), 0, st, so.K, so.V, M, sp, tb, seg[0], seg[1],
                       seg[2], o);
    hipLaunchKernelGGL(fill_slices_kernel<Key>, dim3(grid_capped(mb.S)), dim3(256), 0, st, so.K, mb.S, sp, tb, o, mb.cnt);
  } else if (M > 0) {
    const uint32_t tiles = (uint32_t)((M + w.n.per - 1) / w.n.per);
    const dim3 grid(tiles / 4 + 1);
    if (N == 3) hipLaunchKernelGGL((fill_tiles_kernel<Key, 3>), grid, dim3(256), 0, st, so.K, so.V, M, sp, tiles, w.n, o);
    else if (N == 4) hipLaunchKernelGGL((fill_tiles_kernel<Key, 4>), grid, dim3(256), 0, st, so.K, so.V, M, sp, tiles, w.n, o);
    else hipLaunchKernelGGL((fill_tiles_kernel<Key, 5>), grid, dim3(256), 0, st, so.K, so.V, M, sp, tiles, w.n, o);
    const unsigned sliceBlocks = grid_capped(mb.S);
    hipLaunchKernelGGL(fill_slice_entries_kernel<Key>, dim3(sliceBlocks < 512 ? sliceBlocks : 512), dim3(256), 0, st, so.K,
                       (uint32_t)mb.S, sp, w.n, o, z, mb.cnt);
  }
  {
    size_t tb_ = w.tempBytes;
    auto cit = rocprim::counting_iterator<size_t>(0);
    HIP_TRY(rocprim::exclusive_scan(w.temp, tb_, rocprim::make_transform_iterator(cit, PopcIn{o.cooBits, ownedWords}),
                                    U32(out->cooPtr), 0u, ownedWords + 1, rocprim::plus<uint32_t>(), st), "scan");
  }

  // ---- statistics that need a pass: rows owned by a plain store, distinct factor rows per group and level ----
  BitCounts bc{};
  int which = 0;
  auto count = [&](const uint32_t* map, size_t words, int to) {
    bc.map[which] = map;
    bc.words[which] = words;
    bc.to[which++] = to;
  };
  count(o.owned, ownedWords, 4);
  for (int g = 0; g < 3; ++g)
    for (int l = 1; l < N; ++l)
      if ((sp.marked >> g) & 1u)
        count(o.seen[g][l], (size_t)(row_map_bytes(dims[out->levelMode[l]]) / 4), 8 + g * HBCSF_MAX_ORDER + l);
  size_t most = 0;
  for (int k = 0; k < which; ++k) most = bc.words[k] > most ? bc.words[k] : most;
  const unsigned bx = grid_capped((most + 15) / 16);
  hipLaunchKernelGGL(count_bits_kernel, dim3(bx, (unsigned)which), dim3(256), 0, st, bc, mb.cnt);
  HIP_TRY(hipGetLastError(), "format kernels");
  return HBCSF_OK;
}

// All modes of one key type.
template <typename Key>
int build_all(int N, const uint64_t* dims, size_t M, const uint32_t* const* inds, const float* vals, const hbcsf_opts& opts,
              int totalBits, Workspace& w, const Place& place, hbcsf_tensor* t, hipStream_t st) {
  const auto t_begin = std::chrono::steady_clock::now();
  const int nModes = t->single ? 1 : N;  // single representation: only mode 0's tree is stored
  // the common order: the list every mode's levels below the root follow (with one mode to build, that mode's own order)
  int order[HBCSF_MAX_ORDER];
  common_order(N, dims, opts.mode_order_policy, t->single, order);
  BaseKey bk{};
  for (int l = N - 1, at = 0; l >= 0; --l) {
    const int m = order[l], b = bits_for(dims[m]);
    bk.shift[m] = at;
    bk.mask[m] = (1ull << b) - 1;
    bk.dims[m] = dims[m];
    at += b;
  }
  const int counters = HBCSF_MAX_ORDER * kCounters + 1;
  hipLaunchKernelGGL(zero_words_kernel, dim3(1), dim3(256), 0, st, (uint32_t*)w.cnt, (size_t)counters * 2, (uint32_t*)w.bad,
                     (size_t)2, (uint32_t*)nullptr, (size_t)0);
  ModeBuild mbs[HBCSF_MAX_ORDER];
  // a mode's order: by root, then (blocked modes) by block, the top bits of the level-1 index
  for (int mode = 0; mode < nModes; ++mode) {
    Spec& sp = mbs[mode].sp;
    int lv[HBCSF_MAX_ORDER];
    level_order(N, dims, mode, opts.mode_order_policy, lv);
    sp.blockBits = mid_block_bits(N, dims, opts, mode);
    sp.blockDrop = sp.blockBits ? bits_for(dims[lv[1]]) - sp.blockBits : 0;
    mbs[mode].rootBits = bits_for(dims[mode]);
  }
  if (w.ownSort) {
    SortPasses& ps = w.sort.passes;
    bool room = ps.add(0, totalBits);
    for (int mode = 0; mode < nModes; ++mode) {
      ModeBuild& mb = mbs[mode];
      mb.sortFrom = ps.n;
      if (mode == order[0] && mb.sp.blockBits == 0) continue;
      int lv[HBCSF_MAX_ORDER];
      level_order(N, dims, mode, opts.mode_order_policy, lv);
      room = room && ps.add(bk.shift[mode], mb.rootBits);
      if (mb.sp.blockBits) room = room && ps.add(bk.shift[lv[1]] + mb.sp.blockDrop, mb.sp.blockBits);
      mb.sortMany = ps.n - mb.sortFrom;
    }
    if (!room) return fail(HBCSF_ERANGE, "too many radix passes");
  }
  Sorted<Key> base;
  if (M > 0) {
    size_t tb = w.tempBytes;
    auto cit = rocprim::counting_iterator<size_t>(0);
    HIP_TRY(rocprim::reduce(w.temp, tb, rocprim::make_transform_iterator(cit, SquareIn{vals}), w.normSq, 0.0, M,
                            rocprim::plus<double>(), st), "reduce");
    const int rs = sort_base<Key>(N, M, inds, vals, bk, totalBits, w, &base, st);
    if (rs != HBCSF_OK) return rs;
  }
  bool othersCounted = nModes == N;   // every mode's slices are its distinct indices (with blocking they are pieces)
  for (int m = 0; m < N; ++m) othersCounted = othersCounted && mid_block_bits(N, dims, opts, m) == 0;
  for (int mode = 0; mode < nModes; ++mode) {
    ModeBuild& mb = mbs[mode];
    ModeFormat* out = t->modes[mode].get();
    Spec& sp = mb.sp;
    sp.N = N;
    sp.NF = N - 2;
    sp.L = opts.fiber_threshold;
    const uint32_t gmask = opts.group_mask == 0 ? 3u : (opts.group_mask & 3u);
    sp.cooOn = (gmask & 1u) && sp.blockBits == 0 ? 1u : 0u;   // with blocking no piece owns its row
    sp.cslOn = (gmask & 2u) ? 1u : 0u;
    sp.cooRowFlags = opts.coo_row_flags == 1 ? 1u : 0u;
    sp.perFiber = per_fiber(opts) ? 1u : 0u;
    int lv[HBCSF_MAX_ORDER];
    level_order(N, dims, mode, opts.mode_order_policy, lv);
    u128 upTo = 0;
    for (int l = 0; l < N; ++l) {
      sp.shift[l] = bk.shift[lv[l]];
      sp.mask[l] = bk.mask[lv[l]];
      upTo |= (u128)sp.mask[l] << sp.shift[l];
      sp.upTo[l] = upTo;
      if (dims[lv[l]] <= kByteRows) sp.byteLevels |= 1u << l;
    }
    sp.askLeaf = asks_leaf(M, dims[lv[N - 1]]) ? 1u : 0u;
    if (sp.blockBits) sp.upTo[0] |= ((u128)((1ull << sp.blockBits) - 1)) << (bk.shift[lv[1]] + sp.blockDrop);
    mb.cnt = w.cnt + (size_t)mode * kCounters;
    out->order = N;
    out->mode = mode;
    out->L = sp.L;
    out->blockBits = sp.blockBits;
    out->cooRowFlags = sp.cooRowFlags != 0;
    out->rows = dims[mode];
    for (int l = 0; l < N; ++l) out->levelMode[l] = lv[l];
    Sorted<Key> so;
    if (M > 0) {
      const int rs = sort_mode<Key>(M, base, mb, mode == order[0] && sp.blockBits == 0, w, &so, st);
      if (rs != HBCSF_OK) return rs;
    }
    const int rb = build_mode_device<Key>(N, dims, M, slice_bound(M, dims[mode], sp.blockBits != 0), so, mb, w, place, out,
                                          othersCounted, st);
    if (rb != HBCSF_OK) return rb;
  }
  // the last wait: for the counters, the sum of squares and the words of state
  size_arena(t);
  if (t->arenaBytes > t->formatBytes) {
    uint8_t* states = nullptr;
    const int rp = place(t->arenaBytes - t->formatBytes, &states);
    if (rp != HBCSF_OK) return rp;
    HIP_TRY(clear_states(t, states, st), "launch of the zero-fill kernel");
    use_states(t, states);
  }
  unsigned long long host[HBCSF_MAX_ORDER * kCounters + 1];
  HIP_TRY(hipMemcpyAsync(host, w.cnt, sizeof(host), hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
  HIP_TRY(hipStreamSynchronize(st), "hipStreamSynchronize");
  std::memcpy(&t->normSq, host + HBCSF_MAX_ORDER * kCounters, sizeof(double));
  const double seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t_begin).count();
  for (int mode = 0; mode < nModes; ++mode) {
    const ModeBuild& mb = mbs[mode];
    const unsigned long long* c = host + (size_t)mode * kCounters;
    ModeFormat* out = t->modes[mode].get();
    fill_count_stats(out, N, M, mb.S, mb.fibNat, mb.fibCsf, mb.nSeg, mb.gS, mb.gM, c[1]);
    out->stats.owned_rows = c[4];
    for (int g = 0; g < 3; ++g)
      for (int l = 1; l < N; ++l)
        out->stats.distinct_rows[g][l] = mb.whole[g] ? mbs[out->levelMode[l]].S : c[8 + g * HBCSF_MAX_ORDER + l];
    out->stats.build_seconds = seconds / nModes;
  }
  return HBCSF_OK;
}

// hbcsf_build_format_device; place: where the modes' arrays and the words of state go.
int build_device(int order, const uint64_t* dims, uint64_t nnz, const uint32_t* const* inds, const float* vals,
                 const hbcsf_opts* opts, void* device_arena, const Place& place, void* workspace, uint64_t workspace_bytes,
                 void* hip_stream, hbcsf_tensor** out) {
  if (!out) return fail(HBCSF_EINVAL, "out is null");
  *out = nullptr;
  hbcsf_opts o;
  int totalBits = 0, maxBits = 0;
  const int rc = check_args(order, dims, nnz, opts, &o, &totalBits, &maxBits);
  if (rc != HBCSF_OK) return rc;
  if (nnz > 0 && (!inds || !vals)) return fail(HBCSF_EINVAL, "inds or vals is null");
  for (int m = 0; m < order; ++m)
    if (nnz > 0 && !inds[m]) return fail(HBCSF_EINVAL, "an index array is null");
  if (!device_arena || !workspace) return fail(HBCSF_EINVAL, "null argument");
  if ((((uintptr_t)device_arena | (uintptr_t)workspace) & (kAlign - 1)) != 0)
    return fail(HBCSF_EINVAL, "device arena and workspace must be 256-byte aligned");
  hipStream_t st = (hipStream_t)hip_stream;
  uint64_t maxDim = 0;
  for (int m = 0; m < order; ++m) maxDim = dims[m] > maxDim ? dims[m] : maxDim;
  size_t tbytes = 0;
  const uint64_t slices = slice_bound((size_t)nnz, maxDim, o.mid_blocking > 1);
  HIP_TRY(temp_bytes((size_t)nnz, (size_t)((maxDim + 31) / 32), slices, maxBits, &tbytes),
          "rocPRIM scratch query");
  Workspace w{};
  carve(w, (uint8_t*)workspace, order, (size_t)nnz, row_maps_bytes(order, dims), slices, o.fiber_threshold, tbytes, maxBits > 64,
        per_fiber(o), o.mid_blocking > 1);
  if (workspace_bytes < w.total) return fail(HBCSF_ENOMEM, "workspace is smaller than hbcsf_device_build_bytes");

  std::unique_ptr<hbcsf_tensor> t(new (std::nothrow) hbcsf_tensor);
  if (!t) return fail(HBCSF_ENOMEM, "out of host memory");
  t->order = order;
  t->nnz = nnz;
  t->opts = o;
  t->sliceThreshold = o.slice_threshold;
  for (int m = 0; m < order; ++m) t->dims[m] = dims[m];
  int dev = 0, cu = 0;
  HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
  HIP_TRY(hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev), "hipDeviceGetAttribute");
  t->numCU = cu > 0 ? cu : 256;
  t->device = dev;
  t->single = o.single_representation == 1;
  for (int m = 0; m < (t->single ? 1 : order); ++m) {
    t->modes[m].reset(new (std::nothrow) ModeFormat);
    if (!t->modes[m]) return fail(HBCSF_ENOMEM, "out of host memory");
  }
  WaitOnError wait(st);
  const int rb = maxBits > 64 ? build_all<u128>(order, dims, (size_t)nnz, inds, vals, o, totalBits, w, place, t.get(), st)
                              : build_all<uint64_t>(order, dims, (size_t)nnz, inds, vals, o, totalBits, w, place, t.get(), st);
  if (rb != HBCSF_OK) return rb;
  wait.done();
  t->uploaded = true;
  *out = t.release();
  return HBCSF_OK;
}

}  // namespace

extern "C" {

int hbcsf_device_build_bytes(int order, const uint64_t* dims, uint64_t nnz, const hbcsf_opts* opts,
                             uint64_t* arena_bytes, uint64_t* workspace_bytes) try {
  hbcsf_opts o;
  int totalBits = 0, maxBits = 0;
  const int rc = check_args(order, dims, nnz, opts, &o, &totalBits, &maxBits);
  if (rc != HBCSF_OK) return rc;
  if (!arena_bytes || !workspace_bytes) return fail(HBCSF_EINVAL, "null argument");
  uint64_t maxDim = 0;
  for (int m = 0; m < order; ++m) maxDim = dims[m] > maxDim ? dims[m] : maxDim;
  size_t tbytes = 0;
  const uint64_t slices = slice_bound((size_t)nnz, maxDim, o.mid_blocking > 1);
  HIP_TRY(temp_bytes((size_t)nnz, (size_t)((maxDim + 31) / 32), slices, maxBits, &tbytes),
          "rocPRIM scratch query");
  Workspace w{};
  carve(w, nullptr, order, (size_t)nnz, row_maps_bytes(order, dims), slices, o.fiber_threshold, tbytes, maxBits > 64, per_fiber(o),
        o.mid_blocking > 1);
  *workspace_bytes = w.total;
  *arena_bytes = arena_bound(order, dims, nnz, o.fiber_threshold);
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_build_format_device(int order, const uint64_t* dims, uint64_t nnz, const uint32_t* const* inds,
                              const float* vals, const hbcsf_opts* opts, void* device_arena, uint64_t arena_bytes,
                              void* workspace, uint64_t workspace_bytes, void* hip_stream, hbcsf_tensor** out) try {
  uint64_t used = 0;
  return build_device(order, dims, nnz, inds, vals, opts, device_arena, [&](uint64_t bytes, uint8_t** at) {
    if (used + bytes > arena_bytes) return fail(HBCSF_ENOMEM, "device arena is too small for the format");
    *at = (uint8_t*)device_arena + used;
    used += bytes;
    return (int)HBCSF_OK;
  }, workspace, workspace_bytes, hip_stream, out);
} HBCSF_CATCH_ALL

int hbcsf_build_format_device_pieces(int order, const uint64_t* dims, uint64_t nnz, const uint32_t* const* inds, const float* vals,
                                     const hbcsf_opts* opts, hbcsf_allocate allocate, void* context, void* workspace,
                                     uint64_t workspace_bytes, void* hip_stream, hbcsf_tensor** out) try {
  if (!allocate) {
    if (out) *out = nullptr;
    return fail(HBCSF_EINVAL, "null argument");
  }
  return build_device(order, dims, nnz, inds, vals, opts, workspace, [&](uint64_t bytes, uint8_t** at) {
    *at = (uint8_t*)allocate(context, bytes);
    if (!*at) return fail(HBCSF_ENOMEM, "no device memory was given for a part of the format");
    if (((uintptr_t)*at & (kAlign - 1)) != 0) return fail(HBCSF_EINVAL, "device memory must be 256-byte aligned");
    return (int)HBCSF_OK;
  }, workspace, workspace_bytes, hip_stream, out);
} HBCSF_CATCH_ALL

int hbcsf_relocate(hbcsf_tensor* t, void* new_arena, uint64_t bytes, void* hip_stream) try {
  if (!t || !new_arena) return fail(HBCSF_EINVAL, "null argument");
  if (!t->uploaded) return fail(HBCSF_ESTATE, "the tensor has no device copy");
  if (bytes < t->arenaBytes) return fail(HBCSF_ENOMEM, "the new arena is smaller than hbcsf_device_bytes");
  if (((uintptr_t)new_arena & (kAlign - 1)) != 0) return fail(HBCSF_EINVAL, "device arena must be 256-byte aligned");
  hipStream_t st = (hipStream_t)hip_stream;
  WaitOnError wait(st);
  uint8_t* at = (uint8_t*)new_arena;
  for (int m = 0; m < t->order; ++m) {
    if (!t->modes[m]) continue;
    HIP_TRY(hipMemcpyAsync(at, t->modes[m]->dev, t->modes[m]->blobBytes, hipMemcpyDeviceToDevice, st), "hipMemcpyAsync");
    at += t->modes[m]->blobBytes;
  }
  HIP_TRY(clear_states(t, at, st), "launch of the zero-fill kernel");
  HIP_TRY(hipStreamSynchronize(st), "hipStreamSynchronize");
  wait.done();
  use_arena(t, (uint8_t*)new_arena);
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_download(hbcsf_tensor* t, void* hip_stream) try {
  if (!t) return fail(HBCSF_EINVAL, "null argument");
  if (!t->uploaded) return fail(HBCSF_ESTATE, "the tensor has no device copy");
  hipStream_t st = (hipStream_t)hip_stream;
  for (int m = 0; m < t->order; ++m) {
    if (!t->modes[m]) continue;   // single representation: only mode 0 exists
    ModeFormat& f = *t->modes[m];
    if (f.blob) continue;
    void* mem = nullptr;
    if (posix_memalign(&mem, kAlign, (size_t)f.blobBytes) != 0 || !mem) return fail(HBCSF_ENOMEM, "out of host memory");
    f.blob = (uint8_t*)mem;
    HIP_TRY(hipMemcpyAsync(f.blob, f.dev, f.blobBytes, hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
  }
  HIP_TRY(hipStreamSynchronize(st), "hipStreamSynchronize");
  return HBCSF_OK;
} HBCSF_CATCH_ALL

}  // extern "C"
