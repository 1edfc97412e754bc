// HIP kernels for gfx950 (MI355X): one per HB-CSF slice group plus the output definition.
//
// Mapping (wave64).  One factor row of R = 4G floats is held by G adjacent lanes, a float4
// each, so a wavefront has NG = 64/G lane groups and a row gather is one 16-byte load per
// lane.  (Built with HBCSF_F64 the factor matrices, the partial sums and the output are fp64: a lane
// then holds two doubles, R = 2G, and every address computation stays the same; the tensor's
// values are stored as fp32 either way and widened where they are multiplied.)  The nonzero stream of a group is
// cut into runs of L nonzeros (L = fiber threshold).  A unit is NG parts of P <= L nonzeros (a whole number of
// runs), one per lane group; a lane group walks its part sequentially with its partial sums in
// registers, so every lane group has exactly the same amount of work whatever the slice and fiber
// lengths are.  A wavefront works through a contiguous span of units.
//
// B-CSF kernel (Algorithm "CSF-MTTKRP" with fbr-split / slc-split, Sections III-B and IV):
// per unit the wavefront brings the leaf indices and values straight from memory to LDS, an
// array each, and turns the compressed pointer arrays into per-nonzero end marks in further
// arrays (a lane takes four fiber segments, or one slice).  The inner loop then reads four
// nonzeros' words with one LDS load per array: tmp += v*C(k,:); at a segment end acc += tmp*B(j,:)
// (Eq. 8's factored form); at a slice end the row goes out with one plain 128-byte store if the
// slice lies in one run, else with atomic adds (Section IV-A's merge of split slices).  The first slice that
// ends in a part may have begun in the parts before it: it waits until the unit is closed, when a
// segmented sum over the lane groups completes it.  What is open at the end of a unit stays in
// registers for the next one, and what is open at the ends of a block's spans is summed over its
// wavefronts, so a heavy slice costs one atomic row per block.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hbcsf_device.h"
#ifndef HBCSF_F64
#include "hbcsf_small.h"
#endif

namespace hbcsf {

namespace {

constexpr int kDenseCache = kDenseCacheRows;  // rows of the dense variant's per-wavefront row cache
constexpr uint32_t kOwned = 0x80000000u;      // in a slice entry or mark: the slice lies inside one run


// A lane's 16 bytes of a row: four floats, or two doubles.
#ifdef HBCSF_F64
typedef double real;
struct __attribute__((aligned(16))) rowvec {
  double x, y;
};
typedef double vec16 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ rowvec rv_zero() { return rowvec{0.0, 0.0}; }
__device__ __forceinline__ rowvec rv_ones() { return rowvec{1.0, 1.0}; }
__device__ __forceinline__ vec16 to_vec16(const rowvec& a) { return vec16{a.x, a.y}; }
__device__ __forceinline__ rowvec from_vec16(const vec16& v) { return rowvec{v.x, v.y}; }
#else
typedef float real;
typedef float4 rowvec;
typedef float vec16 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ rowvec rv_zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
__device__ __forceinline__ rowvec rv_ones() { return make_float4(1.f, 1.f, 1.f, 1.f); }
__device__ __forceinline__ vec16 to_vec16(const rowvec& a) { return vec16{a.x, a.y, a.z, a.w}; }
__device__ __forceinline__ rowvec from_vec16(const vec16& v) { return make_float4(v.x, v.y, v.z, v.w); }
#endif

// Streaming 16-byte store: the data is not read again by the kernel that writes it.
__device__ __forceinline__ void store_streaming(rowvec* p, const rowvec& a) {
  __builtin_nontemporal_store(to_vec16(a), reinterpret_cast<vec16*>(p));
}

// Rows are addressed in bytes (16 G per row, 16 per lane) from a base typed `const float*` whatever the
// element type.  WIDE = false: the factor matrix is smaller than 4 GiB, so a 32-bit byte offset from a
// scalar base is enough (one VALU instruction per gather); WIDE = true: 64-bit arithmetic.
template <int G, bool WIDE>
__device__ __forceinline__ rowvec row_load(const float* __restrict__ base, uint32_t row, int c) {
  if (WIDE) {
    return *reinterpret_cast<const rowvec*>(base + ((size_t)row * (size_t)(4 * G) + (size_t)(4 * c)));
  } else {
    const uint32_t off = row * (uint32_t)(16 * G) + (uint32_t)(16 * c);
    return *reinterpret_cast<const rowvec*>(reinterpret_cast<const char*>(base) + off);
  }
}

// Streaming variant: the row is not expected to be used again while it could still be cached, so
// it should not push reusable rows out of the L2.
template <int G, bool WIDE>
__device__ __forceinline__ rowvec row_load_streaming(const float* __restrict__ base, uint32_t row, int c) {
  const vec16* p;
  if (WIDE) {
    p = reinterpret_cast<const vec16*>(base + ((size_t)row * (size_t)(4 * G) + (size_t)(4 * c)));
  } else {
    const uint32_t off = row * (uint32_t)(16 * G) + (uint32_t)(16 * c);
    p = reinterpret_cast<const vec16*>(reinterpret_cast<const char*>(base) + off);
  }
  return from_vec16(__builtin_nontemporal_load(p));
}

// A fiber level's row by its mark (index + 1, perhaps with bit 31 set, which the 32-bit offset drops by itself): `before`
// = row_before(the factor matrix), so that the mark scales to an offset as it is.  Streaming loads exist in the WIDE form only (the caller chooses it when it asks for them): a
// second load instruction per step costs the common form a branch each.
template <int G>
__device__ __forceinline__ const float* row_before(const float* fac) {
  return fac - 4 * G;  // kept a pointer all through: a round trip over an integer would make the loads flat ones
}

template <int G, bool WIDE>
__device__ __forceinline__ rowvec marked_row_load(const float* before, uint32_t mark, int c, bool streaming) {
  if (WIDE) mark &= 0x7fffffffu;
  if (WIDE && streaming) return row_load_streaming<G, WIDE>(before, mark, c);
  return row_load<G, WIDE>(before, mark, c);
}

template <int G>
__device__ __forceinline__ void row_store(float* __restrict__ out, uint32_t row, int c, rowvec a) {
  store_streaming(reinterpret_cast<rowvec*>(out + ((size_t)row * (size_t)(4 * G) + (size_t)(4 * c))), a);
}

template <int G>
__device__ __forceinline__ void row_atomic(float* __restrict__ out, uint32_t row, int c, rowvec a) {
  real* p = reinterpret_cast<real*>(out + ((size_t)row * (size_t)(4 * G) + (size_t)(4 * c)));
  unsafeAtomicAdd(p + 0, a.x);
  unsafeAtomicAdd(p + 1, a.y);
#ifndef HBCSF_F64
  unsafeAtomicAdd(p + 2, a.z);
  unsafeAtomicAdd(p + 3, a.w);
#endif
}

#ifdef HBCSF_F64
__device__ __forceinline__ void fma4(rowvec& d, float s, const rowvec& x) {
  d.x = fma((double)s, x.x, d.x);
  d.y = fma((double)s, x.y, d.y);
}

__device__ __forceinline__ void fma4(rowvec& d, const rowvec& a, const rowvec& x) {
  d.x = fma(a.x, x.x, d.x);
  d.y = fma(a.y, x.y, d.y);
}

__device__ __forceinline__ rowvec mul4(const rowvec& a, const rowvec& x) { return rowvec{a.x * x.x, a.y * x.y}; }

__device__ __forceinline__ rowvec scale4(float s, const rowvec& x) { return rowvec{(double)s * x.x, (double)s * x.y}; }

// Sum over the lanes 2^k * G apart (the same row position in every lane group).
template <int G>
__device__ __forceinline__ void sum_lane_groups(rowvec& a) {
#pragma unroll
  for (int o = G; o < 64; o <<= 1) {
    a.x += __shfl_xor(a.x, o);
    a.y += __shfl_xor(a.y, o);
  }
}
#else
__device__ __forceinline__ void fma4(rowvec& d, float s, const rowvec& x) {
  d.x = fmaf(s, x.x, d.x);
  d.y = fmaf(s, x.y, d.y);
  d.z = fmaf(s, x.z, d.z);
  d.w = fmaf(s, x.w, d.w);
}

__device__ __forceinline__ void fma4(rowvec& d, const rowvec& a, const rowvec& x) {
  d.x = fmaf(a.x, x.x, d.x);
  d.y = fmaf(a.y, x.y, d.y);
  d.z = fmaf(a.z, x.z, d.z);
  d.w = fmaf(a.w, x.w, d.w);
}

__device__ __forceinline__ rowvec mul4(const rowvec& a, const rowvec& x) {
  return make_float4(a.x * x.x, a.y * x.y, a.z * x.z, a.w * x.w);
}

__device__ __forceinline__ rowvec scale4(float s, const rowvec& x) {
  return make_float4(s * x.x, s * x.y, s * x.z, s * x.w);
}

// Sum over the lanes 2^k * G apart (the same row position in every lane group).
template <int G>
__device__ __forceinline__ void sum_lane_groups(rowvec& a) {
#pragma unroll
  for (int o = G; o < 64; o <<= 1) {
    a.x += __shfl_xor(a.x, o);
    a.y += __shfl_xor(a.y, o);
    a.z += __shfl_xor(a.z, o);
    a.w += __shfl_xor(a.w, o);
  }
}
#endif

#ifdef HBCSF_F64
__device__ __forceinline__ void add_row(rowvec& d, const rowvec& x) { d.x += x.x; d.y += x.y; }
__device__ __forceinline__ rowvec shfl_up_row(const rowvec& a, int o) { return rowvec{__shfl_up(a.x, o), __shfl_up(a.y, o)}; }
__device__ __forceinline__ rowvec shfl_row(const rowvec& a, int from) { return rowvec{__shfl(a.x, from), __shfl(a.y, from)}; }
#else
__device__ __forceinline__ void add_row(rowvec& d, const rowvec& x) { d.x += x.x; d.y += x.y; d.z += x.z; d.w += x.w; }
__device__ __forceinline__ rowvec shfl_up_row(const rowvec& a, int o) {
  return make_float4(__shfl_up(a.x, o), __shfl_up(a.y, o), __shfl_up(a.z, o), __shfl_up(a.w, o));
}
__device__ __forceinline__ rowvec shfl_row(const rowvec& a, int from) {
  return make_float4(__shfl(a.x, from), __shfl(a.y, from), __shfl(a.z, from), __shfl(a.w, from));
}
#endif

// Which spans a wavefront works through.  Blocks are dealt round-robin to the 8 XCDs and the
// grid is a multiple of 8, so XCD x = blockIdx % 8 is given the x-th eighth of the stream: one
// slice's partial rows and its factor rows then stay within one L2 where possible.
//   default      one wavefront per span (the grid has as many wavefronts as spans);
//   persistent   a grid of resident blocks only; an XCD's wavefronts take the spans of its
//                eighth round-robin, so each gets the same number of spans from all over it.
struct SpanWalk {
  uint32_t first, end, stride;
};

// block / blocks: this block's number among the blocks that work on the group, and how many they are.
__device__ __forceinline__ SpanWalk span_walk(const GroupArgs& a, uint32_t block, uint32_t blocks, int wib, int wpb) {
  const uint32_t xcd = block & 7u;
  const uint32_t local = (block >> 3) * (uint32_t)wpb + (uint32_t)wib;  // wavefront within its XCD
  const uint32_t wavesPerXcd = (blocks >> 3) * (uint32_t)wpb;
  SpanWalk w;
  if (a.persistent) {
    const uint32_t perXcd = (a.nSpans + 7u) >> 3;
    w.stride = wavesPerXcd;
    w.first = __builtin_amdgcn_readfirstlane(xcd * perXcd + local);
    w.end = min((xcd + 1u) * perXcd, a.nSpans);
  } else {
    w.stride = 1;
    w.first = __builtin_amdgcn_readfirstlane(xcd * wavesPerXcd + local);
    w.end = min(w.first + 1u, a.nSpans);
  }
  return w;
}

// Adds the row that lane group `first / G` holds (lane first + c: its 16-byte piece c) to output row `row`, the whole
// wavefront taking part (first and row wave-uniform): consecutive lanes add consecutive elements, so a row is one
// atomic instruction of whole cache lines.  Atomics on one row are served one line operation after the other, and
// row_atomic's four strided ones per row cost four times as much there (measured on one row: 12.9 ns against 50.9 ns a
// row added, however many wavefronts ask), which bounds a slice that thousands of wavefronts share.
template <int G>
__device__ __forceinline__ void row_atomic_wave(float* __restrict__ out, uint32_t row, int first, const rowvec& a, int lane) {
#ifdef HBCSF_F64
  constexpr int R = 2 * G;
#else
  constexpr int R = 4 * G;
#endif
  real* p = reinterpret_cast<real*>(out + (size_t)row * (size_t)(4 * G));
#pragma unroll
  for (int b = 0; b < R; b += 64) {
    const int e = b + lane;
#ifdef HBCSF_F64
    const int from = first + (e / 2) % G;
    const real x = __shfl(a.x, from), y = __shfl(a.y, from);
    const real v = (e & 1) ? y : x;
#else
    const int from = first + (e / 4) % G;
    const real x = __shfl(a.x, from), y = __shfl(a.y, from), z = __shfl(a.z, from), w = __shfl(a.w, from);
    const real v = (e & 2) ? ((e & 1) ? w : z) : ((e & 1) ? y : x);
#endif
    if (e < R) unsafeAtomicAdd(p + e, v);
  }
}

// A finished slice: a row that lies inside one run is written by this one store, any other is merged with atomic adds.  (A
// part lies in one run, so that a slice which begins and ends in it is merged only where it is a piece of one: never in a
// launch that defines the output itself.)
template <int G>
__device__ __forceinline__ void emit_row(float* __restrict__ out, uint32_t mark, int c, const rowvec& acc) {
  const uint32_t row = (mark & 0x7fffffffu) - 1u;
  if (mark & kOwned) row_store<G>(out, row, c, acc);
  else row_atomic<G>(out, row, c, acc);
}

// Closes a unit in which some slice ends.  The lane groups' parts are consecutive, so a slice that began before a
// lane group's part continues from the parts before it: `acc` is what a lane group holds of the slice still open at the
// end of its part, `headMark` / `head` the first slice that ended in it (mark 0: none did, zeros).  A segmented sum over the
// lane groups (a part with an end starts a new segment) gives every part what the open slice had collected before it;
// the heads go out with that added, and what is still open after the last part stays in lane group 0's accumulator.
template <int G>
__device__ __forceinline__ void close_unit(float* __restrict__ out, const rowvec& head, uint32_t headMark, rowvec& acc,
                                           int lane, int g, int c) {
  rowvec t = acc;
  uint32_t ended = headMark ? 1u : 0u;
#pragma unroll
  for (int o = G; o < 64; o <<= 1) {
    const rowvec up = shfl_up_row(t, o);
    const uint32_t eu = __shfl_up(ended, o);
    if (lane >= o) {
      if (!ended) add_row(t, up);
      ended |= eu;
    }
  }
  const rowvec before = shfl_up_row(t, G);
  rowvec h = head;
  if (headMark) {
    if (g > 0) add_row(h, before);
    if (headMark & kOwned) row_store<G>(out, (headMark & 0x7fffffffu) - 1u, c, h);
  }
  unsigned long long shared = __ballot(c == 0 && headMark != 0u && !(headMark & kOwned));
  while (shared) {
    const int first = __builtin_ctzll(shared);
    shared &= shared - 1;
    row_atomic_wave<G>(out, (uint32_t)__builtin_amdgcn_readlane((int)headMark, first) - 1u, first, h, lane);
  }
  const rowvec last = shfl_row(t, 64 - G + c);
  acc = g == 0 ? last : rv_zero();
}

// The slice still open at the end of the wavefront's span: one atomic row.
template <int G>
__device__ __forceinline__ void close_span(float* __restrict__ out, bool open, uint32_t row, rowvec acc, int lane) {
  if (!open) return;  // wave-uniform
  sum_lane_groups<G>(acc);
  row_atomic_wave<G>(out, row, 0, acc, lane);
}

// The slices still open at the ends of a block's spans (one span a wavefront, all wavefronts take part; they are
// consecutive): one atomic row for each sequence of wavefronts with the same row.  `words`: the wavefront's LDS, `stride`
// words from one wavefront's to the next.  With an atomic row per wavefront a slice of 472 000 nonzeros of a 5 M-nonzero
// tensor was added up by 1844 of them on its row, 12.9 ns after each other, while a mode takes 60 us; that is also what kept
// the spans long (all modes, with one span of 256 nonzeros and up a wavefront, per-wavefront atomics -> this: 5 M
// 189.7 -> 181 us, fp64 307 -> 288, 100 M 2188 -> 2057, 150 M hypersparse 9200 -> 9008, 50 M of order 4 no gain).
template <int G>
__device__ __forceinline__ void close_block(float* __restrict__ out, uint32_t* words, uint32_t stride, bool open,
                                            uint32_t row, rowvec acc, int lane, int wib, int wpb) {
  constexpr uint32_t kNone = 0xffffffffu;
  sum_lane_groups<G>(acc);
  rowvec* mine = reinterpret_cast<rowvec*>(words);
  if (lane < G) mine[lane] = acc;
  if (lane == 0) words[4 * G] = open ? row : kNone;
  __syncthreads();
  if (!open) return;
  if (wib > 0 && (words - stride)[4 * G] == row) return;   // the wavefront before it adds this row up
  for (int w = wib + 1; w < wpb; ++w) {
    words += stride;
    if (words[4 * G] != row) break;
    add_row(acc, reinterpret_cast<const rowvec*>(words)[lane % G]);
  }
  row_atomic_wave<G>(out, row, 0, acc, lane);
}

// One trace record per wavefront: which compute unit it ran on and when (profiling only).
__device__ __forceinline__ void trace_wave(const GroupArgs& a, int kind, unsigned long long t0, int lane) {
  if (a.trace == nullptr || lane != 0) return;
  const unsigned long long t1 = wall_clock64();
  // s_getreg_b32: HW_ID (register 4, 32 bits) = wave / SIMD / CU / SH / SE ids; XCC_ID (register 20, 4 bits)
  const uint32_t hw = __builtin_amdgcn_s_getreg((31 << 11) | (0 << 6) | 4);
  const uint32_t xcc = __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20);
  const unsigned long long slot = atomicAdd(a.trace, 1ull);
  if (slot < a.traceCapacity) {
    unsigned long long* r = a.trace + 4 + 4 * slot;
    r[0] = (unsigned long long)kind;
    r[1] = ((unsigned long long)xcc << 32) | hw;
    r[2] = t0;
    r[3] = t1;
  }
}

// GuestArgs' stamps: an MTTKRP that carries ALS work begins with this kernel.
__device__ __forceinline__ void stamp_begin(unsigned long long* __restrict__ stamp) {
  if (stamp == nullptr || blockIdx.x != 0 || threadIdx.x != 0) return;
  stamp[0] = wall_clock64();
  stamp[1] = 0;
}

__device__ __forceinline__ uint32_t mark_of_slice(uint32_t si) {
  return ((si & 0x7fffffffu) + 1u) | (si & 0x80000000u);
}


// ---------------------------------------------------------------------------------------
// Output definition in the launch that adds to the rows.  A launch of its own takes 1.4 us for 100 rows and 5 us for 100 000,
// all of it before the first wavefront of the group kernels starts; here its words are the work of the first blocks of
// their launch.  What a group kernel adds to must have been zeroed: every word is claimed by the wavefront that writes its
// zeros and marked when they are written, and whoever wants to add to a row of a word that nobody has claimed yet
// claims and zeroes it itself.  So nothing waits for a wavefront that has not started (blocks of one launch may start in any
// order, and another launch may occupy the chip): a wait is for one that is between its claim and its mark, where it waits
// for nothing but memory.  The zeros are written through the L2, which the atomic adds pass by.
// A row's state is asked for before the row is added to, behind the last gathers of a part, so that the answer costs little
// time (asked for where it is used it took 1.3 us a mode of 80 000 nonzeros, asked for while the unit is staged, before the
// rows are defined, 1.2).
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void store_zero_through(rowvec* p) {
  unsigned long long* q = reinterpret_cast<unsigned long long*>(p);
  __hip_atomic_store(q, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(q + 1, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct DefinedBefore {  // by an earlier launch
  static constexpr bool kAsks = false;
  __device__ __forceinline__ uint32_t ask(uint32_t) const { return 0; }
};

template <int G>
struct DefinedHere {
  static constexpr bool kAsks = true;
  const DefineArgs& d;
  float* out;

  // State of the row's word.
  __device__ __forceinline__ uint32_t ask(uint32_t row) const {
    return __hip_atomic_load(d.state + (row >> 5), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }

  // Zeroes the rows of word `wd` (uniform) that nothing stores, unless another wavefront has claimed it.  A whole wavefront.
  __device__ __forceinline__ bool claim(uint32_t wd, int lane) const {
    uint32_t old = 0;
    const uint32_t stored = d.ownedBits[wd];
    if (lane == 0) old = atomicMax(d.state + wd, d.claimed);
    if ((uint32_t)__builtin_amdgcn_readfirstlane((int)old) >= d.claimed) return false;
    constexpr uint32_t NG = 64 / G;
#pragma unroll 1
    for (uint32_t bit = (uint32_t)lane / G; bit < 32; bit += NG) {
      const uint32_t row = (wd << 5) + bit;
      if (row < d.rows && ((stored >> bit) & 1u) == 0u)
        store_zero_through(reinterpret_cast<rowvec*>(out + ((size_t)row * (size_t)(4 * G) + (size_t)(4 * (lane % G)))));
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the zeros have arrived, then the mark
    if (lane == 0) __hip_atomic_store(d.state + wd, d.claimed + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
  }

  // Returns when `row` (uniform) is defined.
  __device__ __forceinline__ void wait(uint32_t row, int lane) const {
    for (;;) {
      const uint32_t now = (uint32_t)__builtin_amdgcn_readfirstlane((int)ask(row));
      if (now > d.claimed || (now < d.claimed && claim(row >> 5, lane))) return;
      __builtin_amdgcn_s_sleep(4);
    }
  }
};

// Before a unit is closed: waits for the rows that are added to there, those of the heads that are shared (headMark: a lane
// group's) and of the slice left open (openRow).  headState, openState: what ask() said of them.
template <typename Defined>
__device__ __forceinline__ void wait_defined(const Defined& defined, uint32_t headMark, uint32_t headState, bool open,
                                             uint32_t openRow, uint32_t openState, int lane, int c) {
  constexpr unsigned long long kOpen = 1ull << 63;   // (lane 63 is no lane group's first)
  unsigned long long late = __ballot(c == 0 && headMark != 0u && !(headMark & kOwned) && headState <= defined.d.claimed);
  if (open && (uint32_t)__builtin_amdgcn_readfirstlane((int)openState) <= defined.d.claimed) late |= kOpen;
#pragma unroll 1
  while (late) {
    const int from = __builtin_ctzll(late);
    late &= late - 1;
    defined.wait(from == 63 ? openRow : (uint32_t)__builtin_amdgcn_readlane((int)headMark, from) - 1u, lane);
  }
}

// ---------------------------------------------------------------------------------------
// Unit staging.
//
// A unit is NG parts of 2^SS nonzeros, one per lane group, and a whole number of runs (2^a.lshift nonzeros each,
// SS <= a.lshift <= SS + log2 NG), so neither a fiber segment nor an owned slice crosses a unit's ends.
//
// All global loads a unit needs before its inner loop (stream data, fiber-segment and slice
// arrays, the row of the slice at the unit's end) are issued back to back and awaited once, and the end marks scattered
// into LDS.  The run-table entries of the next unit are fetched one unit ahead (UnitBounds), so nothing here waits on a
// chain of dependent loads.
// ---------------------------------------------------------------------------------------
struct UnitBounds {
  uint32_t rf;      // lane t <= runs per unit: slice holding the first nonzero of run r0 + t (clipped to runs)
  uint32_t fHi[3];  // fiber levels 1..3: first segment of the next unit (wave-uniform)
};

// Runs in a unit.
template <int G, int SS>
__device__ __forceinline__ uint32_t runs_per_unit(const GroupArgs& a) {
  return ((uint32_t)(64 / G) << SS) >> a.lshift;
}

template <int G, int N, int SS, bool CSF>
__device__ __forceinline__ UnitBounds load_bounds(const GroupArgs& a, uint32_t u, int lane) {
  UnitBounds b;
  const uint32_t rpu = runs_per_unit<G, SS>(a);
  const uint32_t r0 = u * rpu;
  b.rf = a.runFirst[0][min(r0 + min((uint32_t)lane, rpu), a.runs)];
  b.fHi[0] = b.fHi[1] = b.fHi[2] = 0;
  if (CSF) {
    const uint32_t rN = min(r0 + rpu, a.runs);
#pragma unroll
    for (int l = 1; l <= N - 2; ++l) b.fHi[l - 1] = a.runFirst[l][rN];
  }
  return b;
}

struct UnitEnds {
  uint32_t row;     // END marks: output row of the slice holding the next unit's first nonzero (wave-uniform)
                    // START marks: output row of the slice holding this lane group's first nonzero
  bool open;        // END marks: that slice began before the next unit (wave-uniform)
  bool ends;        // END marks: some slice ends in this unit (wave-uniform)
  uint32_t ng;      // nonzeros in this lane group's part (0 beyond the end of the stream)
  uint32_t sideAt;  // B-CSF: where the slices that end in this lane group's part start in the unit's slice list
  uint32_t slices;  // entries of that list (wave-uniform)
};

// Staging as one LDS record per nonzero, through registers: for the dense-gather variant of the B-CSF kernel and the
// single-representation kernel, whose parts are runs (SS = a.lshift).
// fLo: first segment of this unit per fiber level (wave-uniform; = previous unit's fHi).
// START = false: end marks (index + 1 at the LAST nonzero of a segment / slice; slice marks carry the owned bit).
// START = true : start marks (index + 1 at the FIRST nonzero), for the kernel that needs a level's index while
//                its segment is still open; a slice that began before the unit has no mark in it (the row tells).
template <int G, int N, int SS, bool START = false>
__device__ __forceinline__ UnitEnds stage_unit(const GroupArgs& a, uint32_t* __restrict__ rec, uint32_t u,
                                               const UnitBounds& b, const uint32_t (&fLo)[3], int lane) {
  constexpr int NG = 64 / G;
  constexpr int NF = N - 2;
  constexpr int RW = N == 3 ? 4 : 8;
  constexpr int KV = 8;  // stream loads per lane issued together (covers 512 nonzeros)
  constexpr int KF = 4;  // segment loads per lane and level issued together (256 segments)
  constexpr int KS = 2;  // slice loads per lane issued together (128 slices)
  constexpr int markWord = (N == 3) ? 3 : N;  // slice mark: after the N-2 segment marks
  constexpr uint32_t ss = SS, SUB = 1u << SS;
  constexpr uint32_t slots = (uint32_t)NG << SS;
  const uint32_t z0 = u * slots;
  const int g = lane / G;
  const uint32_t* __restrict__ valb = reinterpret_cast<const uint32_t*>(a.val);

  // -- issue: stream data
  uint32_t w0[KV], w1[KV];   // leaf index, value
  if (z0 + slots <= a.nnz) {  // wave-uniform: every slot of the unit holds a nonzero
#pragma unroll
    for (int t = 0; t < KV; ++t) {
      const uint32_t p = (uint32_t)t * 64u + lane;
      w0[t] = w1[t] = 0;
      if ((uint32_t)t * 64u < slots && (slots >= 64u || p < slots)) {
        w0[t] = __builtin_nontemporal_load(a.ind[N - 1] + z0 + p);
        w1[t] = __builtin_nontemporal_load(valb + z0 + p);
      }
    }
  } else {
#pragma unroll
    for (int t = 0; t < KV; ++t) {
      const uint32_t p = (uint32_t)t * 64u + lane;
      const uint32_t z = z0 + p;
      w0[t] = w1[t] = 0;
      if (p < slots && z < a.nnz) {
        w0[t] = __builtin_nontemporal_load(a.ind[N - 1] + z);
        w1[t] = __builtin_nontemporal_load(valb + z);
      }
    }
  }
  // -- issue: fiber-segment ends and indices
  uint32_t fe[3][KF], fi[3][KF];
#pragma unroll
  for (int l = 1; l <= NF; ++l) {
#pragma unroll
    for (int t = 0; t < KF; ++t) {
      const uint32_t f = fLo[l - 1] + (uint32_t)t * 64u + lane;
      fe[l - 1][t] = 0;
      fi[l - 1][t] = 0;
      if (f < b.fHi[l - 1]) {
        fe[l - 1][t] = __builtin_nontemporal_load(a.ptr[l] + f + (START ? 0 : 1));
        fi[l - 1][t] = __builtin_nontemporal_load(a.ind[l] + f);
      }
    }
  }
  // -- issue: slice ends and indices
  // END marks: the slices that end in this unit are those before the one holding the next unit's first nonzero.
  // START marks: that slice may itself begin in this unit, so it is looked at too (a position test decides).
  const uint32_t s0 = __builtin_amdgcn_readfirstlane(b.rf);
  const uint32_t sNext = __builtin_amdgcn_readlane(b.rf, (int)runs_per_unit<G, SS>(a));
  const uint32_t s1 = sNext + (START ? 1u : 0u);
  uint32_t rowRaw = 0, nextStart = 0;
  if (START) {
    rowRaw = a.ind[0][__shfl(b.rf, g)];
  } else {
    rowRaw = a.ind[0][sNext];
    nextStart = a.ptr[0][sNext];
  }
  uint32_t se[KS], si[KS];
#pragma unroll
  for (int t = 0; t < KS; ++t) {
    const uint32_t sl = s0 + (uint32_t)t * 64u + lane;
    se[t] = 0;
    si[t] = 0;
    if (sl < s1) {
      se[t] = a.ptr[0][sl + (START ? 0 : 1)];
      si[t] = a.ind[0][sl];
    }
  }

  // -- records: stream data in, marks cleared
#pragma unroll
  for (int t = 0; t < KV; ++t) {
    const uint32_t p = (uint32_t)t * 64u + lane;
    if (p < slots) {
      uint4* dst = reinterpret_cast<uint4*>(rec + (size_t)(p + (p >> ss)) * RW);
      dst[0] = make_uint4(w0[t], w1[t], 0u, 0u);
      if (N >= 4) dst[1] = make_uint4(0u, 0u, 0u, 0u);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");

  // -- segment end marks
#pragma unroll
  for (int l = 1; l <= NF; ++l) {
    const int word = 2 + (NF - l);
    auto mark = [&](uint32_t p, uint32_t index) { rec[(size_t)(p + (p >> ss)) * RW + word] = index + 1u; };
#pragma unroll
    for (int t = 0; t < KF; ++t) {
      const uint32_t f = fLo[l - 1] + (uint32_t)t * 64u + lane;
      if (f < b.fHi[l - 1]) mark(fe[l - 1][t] - (START ? 0u : 1u) - z0, fi[l - 1][t]);
    }
    for (uint32_t f = fLo[l - 1] + (uint32_t)KF * 64u + lane; f < b.fHi[l - 1]; f += 64)
      mark(a.ptr[l][f + (START ? 0 : 1)] - (START ? 0u : 1u) - z0, a.ind[l][f]);
  }
  // -- slice end marks
  auto mark_slice = [&](uint32_t at, uint32_t entry) {
    const uint32_t p = at - (START ? 0u : 1u) - z0;
    rec[(size_t)(p + (p >> ss)) * RW + markWord] = START ? (entry & 0x7fffffffu) + 1u : mark_of_slice(entry);
  };
#pragma unroll
  for (int t = 0; t < KS; ++t) {
    const uint32_t sl = s0 + (uint32_t)t * 64u + lane;
    if (sl < s1 && (!START || (se[t] >= z0 && se[t] < z0 + slots && se[t] < a.nnz))) mark_slice(se[t], si[t]);
  }
  for (uint32_t sl = s0 + (uint32_t)KS * 64u + lane; sl < s1; sl += 64) {
    const uint32_t at = a.ptr[0][sl + (START ? 0 : 1)];
    if (START && (at < z0 || at >= z0 + slots || at >= a.nnz)) continue;
    mark_slice(at, a.ind[0][sl]);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

  UnitEnds e;
  const uint32_t z = z0 + ((uint32_t)g << ss);
  e.row = rowRaw & 0x7fffffffu;
  e.open = nextStart < min(z0 + slots, a.nnz);
  e.ends = s1 > s0;
  e.ng = z < a.nnz ? min(SUB, a.nnz - z) : 0u;
  e.sideAt = 0;
  e.slices = 0;
  return e;
}

// ---------------------------------------------------------------------------------------
// Staging of the B-CSF and CSL kernels: arrays of one word per nonzero in LDS instead of records.
//
// A vector-memory instruction of a full wavefront occupies the compute unit's address unit for 16 cycles whatever its
// width, and that unit is what these kernels wait for, so a unit is staged with the widest loads there are: the stream
// data (leaf index and value, or the N - 1 indices and the value) goes from memory straight to LDS, 16 bytes a lane and
// without passing through registers, and a lane takes four consecutive fiber segments with one load of their ends and
// one of their indices (with dword loads through registers into records: 50 M nonzeros of order 4 2514 -> 2427 us over
// all modes, 150 M hypersparse 9290 -> 9200, rank 16 on 7.7 M 204 -> 196, fp64 on 5 M 314 -> 307, 100 M of order 3 with
// long fibers 2185 -> 2188, 5 M 190 -> 190).  A part's words are read four nonzeros at a time, so within each array the
// quads of a part are exchanged by quad_swizzle: the lane groups then read from different banks, which the padded records
// did by a pad that a direct load to LDS (lane l writes place l) cannot leave.
//
// With SS = a.lshift a part is a run.  With shorter parts several lane groups share a run: the fiber segments that cross a
// part's end get an extra end mark there (each side of the cut adds its own product with the fiber's row), and slices
// are summed over the parts when the unit is closed.  Short parts buy latency with a few more marks: a wavefront walks
// 2^SS nonzeros per lane group one block after the other.
// ---------------------------------------------------------------------------------------

// Place of quad j (of 2^(SS - 2)) of part g is j ^ quad_swizzle(g): 128 bytes of LDS, eight quads, hold one quad of each
// of eight consecutive reads.
template <int SS>
__device__ __forceinline__ uint32_t quad_swizzle(uint32_t g) {
  return SS >= 5 ? (g & 7u) : SS == 4 ? ((g >> 1) & 3u) : ((g >> 2) & 1u);
}

// Word that holds nonzero p of the unit.
template <int SS>
__device__ __forceinline__ uint32_t word_of(uint32_t p) {
  return p ^ (quad_swizzle<SS>(p >> SS) << 2);
}

typedef uint32_t quad __attribute__((ext_vector_type(4)));
typedef uint32_t quad_unaligned __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ quad load_quad_unaligned(const uint32_t* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const quad_unaligned*>(p));
}

// Words z0 .. z0 + SLOTS - 1 of the K arrays from(0 .. K - 1) to `to` (K x SLOTS words, wave-uniform), 16 bytes a lane,
// not awaited.  Quads that begin past `nnz` are left out; one that straddles it reads on inside the array's padding to
// 256 bytes.
template <uint32_t K, int SS, uint32_t SLOTS, typename From>
__device__ __forceinline__ void stream_to_lds(From from, uint32_t* to, uint32_t z0, uint32_t nnz, int lane) {
  constexpr uint32_t Q = SLOTS / 4, total = K * Q;
  constexpr int kNonTemporal = 2;
#pragma unroll
  for (uint32_t t = 0; t < (total + 63) / 64; ++t) {
    const uint32_t q = t * 64u + (uint32_t)lane;
    const uint32_t* src = from(Q % 64 == 0 ? t * 64u / Q : 0u);
    if (Q % 64 != 0) {
#pragma unroll
      for (uint32_t k = 1; k < K; ++k)
        if (q >= k * Q) src = from(k);
    }
    const uint32_t p = word_of<SS>((q % Q) * 4u);
    if (q < total && p < nnz - z0)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + z0 + p),
                                       (__attribute__((address_space(3))) void*)(to + t * 256u), 16, 0, kNonTemporal);
  }
}

// LDS of a unit, in arrays of SLOTS words.  B-CSF: leaf index, value, then the marks of the fiber levels from the deepest
// up; where a slice ends, bit 31 of the level-1 mark is set, and the marks of the unit's slices stand in `side`, one word
// per slice in slice order; `sideFirst` (NG words) says where each part's begin.  CSL: the N - 1 indices, the value, the
// slice marks.  Marks are end marks: index + 1 at the LAST nonzero of a segment / slice, else 0; a slice mark carries the
// owned bit.
// fLo: first segment of this unit per fiber level (wave-uniform; = previous unit's fHi).
template <int G, int N, int SS, bool CSF>
__device__ __forceinline__ UnitEnds stage_arrays(const GroupArgs& a, uint32_t* __restrict__ words, uint32_t u,
                                                 const UnitBounds& b, const uint32_t (&fLo)[3], int lane,
                                                 uint32_t* __restrict__ side = nullptr,
                                                 uint32_t* __restrict__ sideFirst = nullptr) {
  constexpr int NG = 64 / G;
  constexpr int NF = N - 2;
  constexpr uint32_t SUB = 1u << SS;
  constexpr uint32_t slots = (uint32_t)NG << SS;
  constexpr int KF = (slots + 255) / 256;   // a segment holds at least one nonzero
  constexpr int KS = 2;                     // slice loads per lane issued together (128 slices)
  constexpr uint32_t kData = CSF ? 2 : N;   // arrays of stream data
  constexpr uint32_t kMarks = CSF ? NF : 1;
  const uint32_t z0 = u * slots;
  const uint32_t zEnd = min(z0 + slots, a.nnz);
  const int g = lane / G;
  // parts shorter than runs (of at most 64 nonzeros): segments are cut at part ends too
  const bool cutSegments = CSF && SS < 6 && SS < a.lshift;

  // -- issue: ends and indices of the slices that end in this unit, those before the one holding the next unit's first
  // nonzero (first: the run table's entries are awaited here, and with them whatever was issued before)
  const uint32_t s0 = __builtin_amdgcn_readfirstlane(b.rf);
  const uint32_t s1 = __builtin_amdgcn_readlane(b.rf, (int)runs_per_unit<G, SS>(a));
  const uint32_t rowRaw = a.ind[0][s1];
  const uint32_t nextStart = a.ptr[0][s1];
  uint32_t se[KS], si[KS], sb[KS];
#pragma unroll
  for (int t = 0; t < KS; ++t) {
    const uint32_t sl = s0 + (uint32_t)t * 64u + lane;
    se[t] = 0;
    si[t] = 0;
    sb[t] = 0;
    if (sl < s1) {
      se[t] = a.ptr[0][sl + 1];
      si[t] = a.ind[0][sl];
      if (CSF) sb[t] = a.ptr[0][sl];
    }
  }
  // -- issue: stream data
  stream_to_lds<kData, SS, slots>(
      [&](uint32_t k) { return k == kData - 1 ? reinterpret_cast<const uint32_t*>(a.val) : a.ind[CSF ? N - 1 : k + 1]; },
      words, z0, a.nnz, lane);
  // -- issue: fiber-segment ends and indices, four segments a lane (the last lane's may reach three words past the array,
  // which the arrays that follow it in the arena cover)
  quad fe[3][KF], fi[3][KF];
  if constexpr (CSF) {
#pragma unroll
    for (int l = 1; l <= NF; ++l) {
#pragma unroll
      for (int t = 0; t < KF; ++t) {
        const uint32_t f = fLo[l - 1] + ((uint32_t)t * 64u + lane) * 4u;
        fe[l - 1][t] = fi[l - 1][t] = quad{0u, 0u, 0u, 0u};
        if (f < b.fHi[l - 1]) {
          fe[l - 1][t] = load_quad_unaligned(a.ptr[l] + f + 1);
          fi[l - 1][t] = load_quad_unaligned(a.ind[l] + f);
        }
      }
    }
  }
  // -- marks cleared
  uint32_t* __restrict__ marks = words + kData * slots;
#pragma unroll
  for (uint32_t t = 0; t < (kMarks * slots + 255) / 256; ++t) {
    const uint32_t q = t * 64u + (uint32_t)lane;
    if ((kMarks * slots) % 256 == 0 || q < kMarks * slots / 4) reinterpret_cast<quad*>(marks)[q] = quad{0u, 0u, 0u, 0u};
  }
  if (CSF && lane < NG) sideFirst[lane] = s1 - s0;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");

  // -- segment end marks
  if constexpr (CSF) {
#pragma unroll
    for (int l = 1; l <= NF; ++l) {
      uint32_t* __restrict__ at = marks + (uint32_t)(NF - l) * slots;
      auto mark = [&](uint32_t p, uint32_t index) { at[word_of<SS>(p)] = index + 1u; };
      uint32_t before = z0;   // lane 0's first segment begins with the unit
#pragma unroll
      for (int t = 0; t < KF; ++t) {
        const uint32_t f = fLo[l - 1] + ((uint32_t)t * 64u + lane) * 4u;
        uint32_t begin = 0;
        if (cutSegments) {
          begin = __shfl_up(fe[l - 1][t].w, 1);
          if (lane == 0) begin = before;
          before = __builtin_amdgcn_readlane(fe[l - 1][t].w, 63);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (f + (uint32_t)k < b.fHi[l - 1]) {
            const uint32_t p = fe[l - 1][t][k] - 1u - z0, index = fi[l - 1][t][k];
            mark(p, index);
            if (cutSegments)
              for (uint32_t q = (begin - z0) | (SUB - 1u); q < p; q += SUB) mark(q, index);
          }
          begin = fe[l - 1][t][k];
        }
      }
    }
  }
  // -- slice end marks
  auto end_slice = [&](uint32_t sl, uint32_t begin, uint32_t end, uint32_t entry) {
    const uint32_t p = end - 1u - z0;
    if constexpr (CSF) {
      atomicOr(marks + (NF - 1) * slots + word_of<SS>(p), 0x80000000u);
      side[sl - s0] = mark_of_slice(entry);
      // the parts whose first nonzero lies in this slice start with it
      for (uint32_t q = begin > z0 ? (begin - z0 + SUB - 1u) >> SS : 0u; (q << SS) <= p; ++q) sideFirst[q] = sl - s0;
    } else {
      marks[word_of<SS>(p)] = mark_of_slice(entry);
    }
  };
#pragma unroll
  for (int t = 0; t < KS; ++t) {
    const uint32_t sl = s0 + (uint32_t)t * 64u + lane;
    if (sl < s1) end_slice(sl, sb[t], se[t], si[t]);
  }
  for (uint32_t sl = s0 + (uint32_t)KS * 64u + lane; sl < s1; sl += 64)
    end_slice(sl, CSF ? a.ptr[0][sl] : 0u, a.ptr[0][sl + 1], a.ind[0][sl]);

  // -- the stream data has arrived; past the end of the stream (last unit only) zeros, which add nothing
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  if (zEnd < z0 + slots) {
    for (uint32_t p = zEnd - z0 + lane; p < slots; p += 64) {
#pragma unroll
      for (uint32_t k = 0; k < kData; ++k) words[k * slots + word_of<SS>(p)] = 0u;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }

  UnitEnds e;
  const uint32_t z = z0 + ((uint32_t)g << SS);
  e.row = rowRaw & 0x7fffffffu;
  e.open = nextStart < zEnd;
  e.ends = s1 > s0;
  e.ng = z < a.nnz ? min(SUB, a.nnz - z) : 0u;
  e.sideAt = CSF ? sideFirst[g] : 0u;
  e.slices = s1 - s0;
  return e;
}

}  // namespace

// The fp64 objects instantiate the same kernel templates with the same arguments as the fp32 ones: a namespace of
// their own keeps the two sets of kernels apart at link time.
#ifdef HBCSF_F64
namespace f64 {
#endif

// ---------------------------------------------------------------------------------------
// Output definition: rows that no plain store will write (empty slices and rows merged with
// atomic adds) are set to zero; the others are left to their single store.
// ---------------------------------------------------------------------------------------
#ifdef HBCSF_WITH_DEFINE
// One wavefront takes one bitmap word (32 rows) at a time: the word is read once through the
// scalar path and each lane then stores its share of the 32 rows' float4s.
__global__ __launch_bounds__(256) void define_rows_kernel(rowvec* __restrict__ out,
                                                          const uint32_t* __restrict__ ownedBits,
                                                          uint64_t nvec, int gshift,
                                                          unsigned long long* __restrict__ stamp) {
  stamp_begin(stamp);
  const int lane = threadIdx.x & 63;
  const uint32_t waves = (gridDim.x * blockDim.x) >> 6;
  const uint32_t wave = __builtin_amdgcn_readfirstlane((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const uint64_t perWord = (uint64_t)32 << gshift;      // float4s covered by one bitmap word
  const uint64_t words = (nvec + perWord - 1) / perWord;
  const int reps = (int)(perWord >> 6);                  // stores per lane per word (G / 2)
  // a wavefront fills kChunk consecutive words (kChunk x 32 rows) before it strides on
  constexpr uint64_t kChunk = 8;
  for (uint64_t w0 = (uint64_t)wave * kChunk; w0 < words; w0 += (uint64_t)waves * kChunk) {
    const uint64_t w1 = min(w0 + kChunk, words);
    for (uint64_t wd = w0; wd < w1; ++wd) {
      const uint32_t w = ownedBits[wd];
      const uint64_t base = wd * perWord;
      for (int q = 0; q < reps; ++q) {
        const uint32_t f = (uint32_t)q * 64u + lane;        // rowvec within the word's 32 rows
        const uint64_t t = base + f;
        if (t < nvec && !((w >> (f >> gshift)) & 1u)) store_streaming(out + t, rv_zero());
      }
    }
  }
}
#endif  // HBCSF_WITH_DEFINE

// ---------------------------------------------------------------------------------------
// Output definition fused with the COO group, 32 rows (one word of the bitmaps) a wavefront: rows of the COO group get v *
// hadamard(factor rows), rows that nothing else stores get zeros, rows owned by a CSL / CSF slice are left alone.  The rows
// of single-nonzero slices are scattered thinly over the output (about one row in five on the hypersparse workloads), and
// writing them in a pass of their own costs far more DRAM time per byte than writing them together with the zero fill of
// their neighbours.  COO nonzeros are stored in row order, so the nonzero of a row is cooPtr[word] + (number of COO rows
// before it in the word).
// ZEROS = false: the COO group's rows alone.
// ---------------------------------------------------------------------------------------
struct CooGroup {
  const uint32_t* ind[5];
  const float* val;
};

template <int G, int N, bool WIDE, bool ZEROS>
__device__ __forceinline__ void define_word(const float* const (&fac)[5], float* __restrict__ out, const CooGroup& coo, uint32_t wo,
                                            uint32_t wc, uint32_t zBase, uint64_t wd, uint64_t rows, int lane) {
  constexpr int NG = 64 / G;
  constexpr int RPG = 32 / NG;              // rows of a word per lane group (NG <= 32)
  constexpr int CH = RPG < 4 ? RPG : 4;     // rows per lane group handled together
  const int g = lane / G, c = lane % G;
  const uint32_t* __restrict__ valb = reinterpret_cast<const uint32_t*>(coo.val);
#pragma unroll (ZEROS ? 4 : 1)
  for (int qb = 0; qb < RPG; qb += CH) {
    uint32_t i1[CH], i2[CH], i3[CH], i4[CH], v[CH];
    bool isCoo[CH], fill[CH];
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      const uint32_t bit = (uint32_t)(g * RPG + qb + q);
      const uint64_t row = (wd << 5) + bit;
      isCoo[q] = ((wc >> bit) & 1u) != 0u;
      fill[q] = ZEROS && row < rows && !isCoo[q] && ((wo >> bit) & 1u) == 0u;
      i1[q] = i2[q] = i3[q] = i4[q] = v[q] = 0;
      if (isCoo[q]) {
        const uint32_t z = zBase + (uint32_t)__builtin_popcount(wc & ((1u << bit) - 1u));
        i1[q] = coo.ind[1][z];
        i2[q] = coo.ind[2][z];
        if (N >= 4) i3[q] = coo.ind[3][z];
        if (N >= 5) i4[q] = coo.ind[4][z];
        v[q] = valb[z];
      }
    }
    rowvec x1[CH], x2[CH], x3[CH], x4[CH];
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      if (isCoo[q]) {
        x1[q] = row_load<G, WIDE>(fac[1], i1[q], c);
        x2[q] = row_load<G, WIDE>(fac[2], i2[q], c);
        if (N >= 4) x3[q] = row_load<G, WIDE>(fac[3], i3[q], c);
        if (N >= 5) x4[q] = row_load<G, WIDE>(fac[4], i4[q], c);
      }
    }
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      const uint32_t bit = (uint32_t)(g * RPG + qb + q);
      rowvec* dst = reinterpret_cast<rowvec*>(out + (((wd << 5) + bit) * (uint64_t)(4 * G) + (uint64_t)(4 * c)));
      if (isCoo[q]) {
        rowvec pr = mul4(x1[q], x2[q]);
        if (N >= 4) pr = mul4(pr, x3[q]);
        if (N >= 5) pr = mul4(pr, x4[q]);
        store_streaming(dst, scale4(__uint_as_float(v[q]), pr));
      } else if (fill[q]) {
        store_streaming(dst, rv_zero());
      }
    }
  }
}

template <int G, int N, bool WIDE>
__global__ __launch_bounds__(256) void define_coo_kernel(const GroupArgs a, const uint32_t* __restrict__ ownedBits,
                                                         const uint32_t* __restrict__ cooBits,
                                                         const uint32_t* __restrict__ cooPtr, uint64_t rows,
                                                         unsigned long long* __restrict__ stamp) {
  stamp_begin(stamp);
  const int lane = threadIdx.x & 63;
  const uint32_t waves = (gridDim.x * blockDim.x) >> 6;
  const uint32_t wave = __builtin_amdgcn_readfirstlane((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const uint64_t words = (rows + 31) >> 5;
  const CooGroup coo{{a.ind[0], a.ind[1], a.ind[2], a.ind[3], a.ind[4]}, a.val};
  for (uint64_t wd = wave; wd < words; wd += waves)
    define_word<G, N, WIDE, true>(a.fac, a.out, coo, ownedBits[wd], cooBits[wd], cooPtr[wd], wd, rows, lane);
}

// ---------------------------------------------------------------------------------------
// B-CSF group.  N = tensor order (3, 4 or 5); G = lanes per factor row.
// LDS words per nonzero: leaf, val, the segment marks from the deepest level up, the last with the slice-end flag (the
// marks of the slices that end in the unit sit in a list beside them, in slice order, and a lane group takes them one
// after the other as it meets the flags).  The dense-gather variant's record is {leaf, val, seg1, slice mark} or
// {leaf, val, seg2, seg1, slice mark, -, -, -}.
// A segment mark is index+1 at the segment's last nonzero, else 0.  A slice mark is
// (row+1) | owned bit at the slice's last nonzero, else 0.
// ---------------------------------------------------------------------------------------
//
// DENSE (orders 3 and 4): the rows of the fiber levels are not gathered at the step where a segment ends (one
// load instruction per step in which ANY lane group ends a segment, most of its lanes idle) but once per block of
// kSteps steps for the whole wavefront: every lane group counts the marks in its kSteps records, a prefix sum over
// the lane groups gives each mark a slot, the row numbers go to a list in LDS, and ceil(marks / NG) load
// instructions with all lanes busy bring the rows into an LDS row cache, from which the steps then read them.
// Every vector-memory instruction keeps the CU's address unit busy for the same 16 cycles however many lanes
// are active, and that unit is what bounds this kernel when the factor matrices are cache-resident.  The cache
// holds kDenseCache rows; marks beyond it (rare when segments average a few nonzeros) load their row directly.
template <int G, int N, int SS, int kSteps, bool WIDE, bool DENSE, typename Defined = DefinedBefore>
__device__ __forceinline__ void csf_group_body(const GroupArgs& a, uint32_t block, uint32_t blocks,
                                               const Defined& defined = Defined()) {
  constexpr int NG = 64 / G;
  constexpr int NF = N - 2;
  constexpr int RW = N == 3 ? 4 : 8;   // DENSE: words of a record
  // Order 3: a lane group moves the fiber marks of every kQueue steps together, without gaps, so that its k-th fiber end
  // of them is loaded by the k-th instruction: as many load instructions as the most ends any lane group has there,
  // instead of one per step in which some lane group has an end (at one end in five nonzeros and eight lane groups 1.9
  // instead of 3.2 per four steps; the address unit takes as long for a load of one row as for one of eight).  The rows
  // are used in that order: the first is always next, and an end moves the others up.  100 M nonzeros, all modes:
  // 2302 -> 2212 us; with a third of the nonzeros ending a fiber (150 M) 9230 -> 9195 us, smaller tensors equal.  At
  // order 4 nearly every step ends a deepest fiber, and the level above it gains nothing (2504 / 2517 us on 50 M).
  constexpr bool QUEUE = N == 3 && !DENSE;
  constexpr int kQueue = 4;
  static_assert(kSteps % kQueue == 0, "whole queues");
  static_assert(!DENSE || N <= 4, "the dense fiber-row gather handles orders 3 and 4");
  extern __shared__ uint32_t lds[];
  const int lane = threadIdx.x & 63;
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wpb = blockDim.x >> 6;
  const int g = lane / G, c = lane % G;
  constexpr uint32_t SUB = 1u << SS;
  constexpr uint32_t slots = NG << SS;
  constexpr uint32_t recWords = DENSE ? NG * (SUB + 1) * RW : (2 + NF) * slots;
  uint32_t* rec = lds + (uint32_t)wib * csf_wave_words(N, G, SS, DENSE);
  // first finished slice of each part (the dense variant holds it in registers: its row cache already fills the LDS)
  rowvec* head = reinterpret_cast<rowvec*>(rec + recWords);
  uint32_t* side = rec + recWords + 256;                             // marks of the slices that end in the unit,
  uint32_t* sideFirst = side + NG * SUB;                             //       and where each part's begin
  uint32_t* list = rec + recWords;                                   // DENSE: row numbers by slot
  rowvec* cache = reinterpret_cast<rowvec*>(rec + recWords + 64);    // DENSE: rows by slot, G rowvec each

  const float* __restrict__ facLeaf = a.fac[N - 1];
  const float* __restrict__ facDeep = a.fac[N - 2];   // deepest fiber level
  const float* __restrict__ facNext = a.fac[N >= 4 ? N - 3 : 1];  // the fiber level above it (N >= 4)
  const float* __restrict__ facTop = a.fac[1];        // level 1 (N = 5: the third fiber level from the leaf)
  const float* markDeep = row_before<G>(facDeep);      // the same, addressed by marks (index + 1)
  const float* markNext = row_before<G>(facNext);
  const float* markTop = row_before<G>(facTop);

  const unsigned long long traceStart = a.trace ? wall_clock64() : 0ull;
  const SpanWalk walk = span_walk(a, block, blocks, wib, wpb);
  // acc: what this lane group has collected of the slice that is open at the end of its part.  Between units it is
  // held by lane group 0 alone, unless no slice ended since (spread): then every lane group holds a share of it.
  rowvec acc = rv_zero();
  bool open = false;
  uint32_t openRow = 0;
  for (uint32_t span = walk.first; span < walk.end; span += walk.stride) {
  uint32_t u = span * a.unitsPerWave;
  const uint32_t uEnd = min(u + a.unitsPerWave, a.nUnits);
  acc = rv_zero();
  bool spread = false;

  UnitBounds cur = load_bounds<G, N, SS, true>(a, u, lane);
  uint32_t fLo[3] = {0, 0, 0};
#pragma unroll
  for (int l = 1; l <= NF; ++l) fLo[l - 1] = a.runFirst[l][u * runs_per_unit<G, SS>(a)];

  for (; u < uEnd; ++u) {
    // run-table entries of the next unit: in flight while this unit is staged and processed
    const UnitBounds nxt = load_bounds<G, N, SS, true>(a, min(u + 1, a.nUnits - 1), lane);
    UnitEnds ends;
    if constexpr (DENSE) ends = stage_unit<G, N, SS>(a, rec, u, cur, fLo, lane);
    else ends = stage_arrays<G, N, SS, true>(a, rec, u, cur, fLo, lane, side, sideFirst);
    const uint32_t ng = ends.ng;
    uint32_t sideAt = ends.sideAt;   // the next slice of this lane group's part in the unit's slice list
    uint32_t headMark = 0;           // mark of the first slice that ends in this lane group's part
    uint32_t headState = 0;          // DefinedHere: the state of its row,
    uint32_t openState = 0;          //              and of the row of the slice open at the end of the unit
    fLo[0] = cur.fHi[0];
    fLo[1] = cur.fHi[1];
    fLo[2] = cur.fHi[2];
    cur = nxt;
    open = ends.open;
    openRow = ends.row;
    if (ends.ends && spread) {
      sum_lane_groups<G>(acc);
      if (g > 0) acc = rv_zero();
    }
    spread = !ends.ends;
    rowvec held = rv_zero();         // DENSE: that slice
    // a slice ends here: the first one of a part waits for the parts before it, the others are complete
    auto slice_end = [&](uint32_t mark) {
      if (headMark) {
        emit_row<G>(a.out, mark, c, acc);
      } else {
        headMark = mark;
        if constexpr (DENSE) held = acc;
        else head[lane] = acc;
      }
      acc = rv_zero();
    };

    // A lane group whose part lies beyond the end of the stream (ng = 0, last unit only) has all-zero records.  The
    // dense variant's block loop is collective (prefix sum over the lane groups, shared list and row cache), so
    // every lane group runs it, live or not; zero records hold no marks and so change nothing.
    {
      // tmp: sum over the leaves of the open deepest-level segment; tmp1 / tmp2: sums over the closed segments
      // of the next levels up (N >= 4 / N = 5); acc: the slice's row.  Marks are nested: a segment of a level
      // can only end where one of every deeper level ends.
      rowvec tmp = rv_zero();
      rowvec tmp1 = rv_zero();
      rowvec tmp2 = rv_zero();
      if constexpr (DENSE) {
      const uint32_t* myrec = rec + (size_t)g * (SUB + 1) * RW;
      for (uint32_t sb = 0; sb < SUB; sb += kSteps) {
        uint4 rr[kSteps];
        uint32_t mi[kSteps];   // slice mark
        uint32_t sl[kSteps];   // slot (within this lane group) of the deepest level's mark, then of the next level's
        rowvec cr[kSteps];
#pragma unroll
        for (int t = 0; t < kSteps; ++t) {
          const uint4* src = reinterpret_cast<const uint4*>(myrec + (size_t)(sb + t) * RW);
          rr[t] = src[0];
          mi[t] = (N == 3) ? rr[t].w : reinterpret_cast<const uint32_t*>(src)[4];
        }
        // marks of this block per lane group, and where its slots start
        uint32_t cnt = 0;
#pragma unroll
        for (int t = 0; t < kSteps; ++t) {
          sl[t] = cnt;
          cnt += rr[t].z ? 1u : 0u;
          if (N == 4) cnt += rr[t].w ? 1u : 0u;   // its slot is sl[t] + 1 (a level-1 mark implies a level-2 mark)
        }
        uint32_t incl = cnt;
#pragma unroll
        for (int o = G; o < 64; o <<= 1) {
          const uint32_t up = __shfl_up(incl, o);
          if (lane >= o) incl += up;
        }
        const uint32_t base = incl - cnt;
        const uint32_t total = __builtin_amdgcn_readlane(incl, 63);
#pragma unroll
        for (int t = 0; t < kSteps; ++t) {
          sl[t] += base;
          if (rr[t].z && sl[t] < (uint32_t)kDenseCache) list[sl[t]] = rr[t].z - 1u;
          if (N == 4 && rr[t].w && sl[t] + 1u < (uint32_t)kDenseCache) list[sl[t] + 1u] = (rr[t].w - 1u) | 0x80000000u;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        // the rows, NG per load instruction
        const uint32_t nq = min(total, (uint32_t)kDenseCache);
        constexpr int kRounds = kDenseCache / NG;
        rowvec mr[kRounds];
#pragma unroll
        for (int u2 = 0; u2 < kRounds; ++u2) {
          const uint32_t q = (uint32_t)u2 * NG + g;
          if ((uint32_t)u2 * NG < nq) {        // wave-uniform: rounds past the last slot issue nothing
            if (q < nq) {
              const uint32_t e = list[q];
              const uint32_t row = e & 0x7fffffffu;
              if (N == 4 && (e >> 31)) {
                mr[u2] = (a.streamLevel & 2u) ? row_load_streaming<G, WIDE>(facNext, row, c)
                                              : row_load<G, WIDE>(facNext, row, c);
              } else {
                mr[u2] = (a.streamLevel & (1u << (N - 2))) ? row_load_streaming<G, WIDE>(facDeep, row, c)
                                                           : row_load<G, WIDE>(facDeep, row, c);
              }
            }
          }
        }
#pragma unroll
        for (int t = 0; t < kSteps; ++t) cr[t] = row_load<G, WIDE>(facLeaf, rr[t].x, c);
#pragma unroll
        for (int u2 = 0; u2 < kRounds; ++u2) {
          const uint32_t q = (uint32_t)u2 * NG + g;
          if ((uint32_t)u2 * NG < nq && q < nq) cache[(size_t)q * G + c] = mr[u2];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int t = 0; t < kSteps; ++t) {
          fma4(tmp, __uint_as_float(rr[t].y), cr[t]);
          if (rr[t].z) {
            const rowvec br = sl[t] < (uint32_t)kDenseCache ? cache[(size_t)sl[t] * G + c]
                                                             : row_load<G, WIDE>(facDeep, rr[t].z - 1u, c);
            if (N == 3) {
              fma4(acc, tmp, br);
            } else {
              fma4(tmp1, tmp, br);
              if (rr[t].w) {
                const rowvec nr = sl[t] + 1u < (uint32_t)kDenseCache ? cache[(size_t)(sl[t] + 1u) * G + c]
                                                                      : row_load<G, WIDE>(facNext, rr[t].w - 1u, c);
                fma4(acc, tmp1, nr);
                tmp1 = rv_zero();
              }
            }
            tmp = rv_zero();
            if (mi[t]) slice_end(mi[t]);  // a slice can only end where a segment ends
          }
        }
        // the next block rewrites the list and the cache
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
      } else if (ng > 0) {
      const uint32_t swizzle = quad_swizzle<SS>((uint32_t)g);
#pragma unroll 1
      for (uint32_t sb = 0; sb < SUB; sb += kSteps) {
        uint32_t leaf[kSteps], val[kSteps];
        // marks of the deepest fiber level, (N >= 4) the one above it, (N = 5) fiber level 1; bit 31 of a level-1 mark:
        // the slice ends too, and its mark is the next of this part's in the slice list
        uint32_t m3[kSteps], m2[kSteps], m1[kSteps];
        uint32_t (&top)[kSteps] = N == 3 ? m3 : N == 4 ? m2 : m1;
        rowvec cr[kSteps], br[kSteps], nr[kSteps], ar[kSteps];
#pragma unroll
        for (int b = 0; b < kSteps; b += 4) {
          const quad* src = reinterpret_cast<const quad*>(rec) + (((uint32_t)g << (SS - 2)) + ((sb / 4 + b / 4) ^ swizzle));
          const quad q0 = src[0], q1 = src[slots / 4], q2 = src[2 * slots / 4];
          quad q3 = quad{0u, 0u, 0u, 0u}, q4 = q3;
          if constexpr (N >= 4) q3 = src[3 * slots / 4];
          if constexpr (N == 5) q4 = src[4 * slots / 4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            leaf[b + t] = q0[t];
            val[b + t] = q1[t];
            m3[b + t] = q2[t];
            m2[b + t] = q3[t];
            m1[b + t] = q4[t];
          }
        }
        // Conditional loads first: loads return in order, so once a leaf row has arrived every
        // load issued before it has arrived too, and the leaf rows can be awaited one by one.
        if constexpr (QUEUE) {
#pragma unroll
          for (int b = 0; b < kSteps; b += kQueue) {
            uint32_t q[kQueue] = {};
#pragma unroll
            for (int t = kQueue - 1; t >= 0; --t) {
              const bool marked = m3[b + t] != 0u;
#pragma unroll
              for (int k = kQueue - 1 - t; k > 0; --k) q[k] = marked ? q[k - 1] : q[k];
              q[0] = marked ? m3[b + t] : q[0];
            }
#pragma unroll
            for (int k = 0; k < kQueue; ++k)
              if (q[k]) br[b + k] = marked_row_load<G, WIDE>(markDeep, q[k], c, (a.streamLevel & (1u << (N - 2))) != 0u);
          }
        }
#pragma unroll
        for (int t = 0; t < kSteps; ++t) {
          if (!QUEUE && m3[t])
            br[t] = marked_row_load<G, WIDE>(markDeep, m3[t], c, (a.streamLevel & (1u << (N - 2))) != 0u);
          if (N >= 4 && m2[t])
            nr[t] = marked_row_load<G, WIDE>(markNext, m2[t], c, (a.streamLevel & (1u << (N - 3))) != 0u);
          if (N == 5 && m1[t]) ar[t] = marked_row_load<G, WIDE>(markTop, m1[t], c, (a.streamLevel & 2u) != 0u);
        }
#pragma unroll
        for (int t = 0; t < kSteps; ++t) cr[t] = row_load<G, WIDE>(facLeaf, leaf[t], c);
        if constexpr (Defined::kAsks) {
          if (sb == SUB - kSteps) {
            // the first slice that ends here or after this part (if that is not here, nothing comes of the answer)
            if (ends.sideAt < ends.slices) headState = defined.ask((side[ends.sideAt] & 0x7fffffffu) - 1u);
            openState = defined.ask(ends.row);
          }
        }
#pragma unroll
        for (int t = 0; t < kSteps; ++t) {
          fma4(tmp, __uint_as_float(val[t]), cr[t]);
          if (m3[t]) {
            if (QUEUE) {
              const int head = t / kQueue * kQueue;
              fma4(acc, tmp, br[head]);
#pragma unroll
              for (int k = 0; k < kQueue - 1 - t % kQueue; ++k) br[head + k] = br[head + k + 1];
            } else {
              fma4(tmp1, tmp, br[t]);
              if (m2[t]) {
                if (N == 4) {
                  fma4(acc, tmp1, nr[t]);
                } else {
                  fma4(tmp2, tmp1, nr[t]);
                  if (m1[t]) {
                    fma4(acc, tmp2, ar[t]);
                    tmp2 = rv_zero();
                  }
                }
                tmp1 = rv_zero();
              }
            }
            tmp = rv_zero();
            if ((int)top[t] < 0) slice_end(side[sideAt++]);   // a slice can only end where a segment ends
          }
        }
      }
      }  // classic / dense
    }
    if constexpr (Defined::kAsks) wait_defined(defined, headMark, headState, open, openRow, openState, lane, c);
    if (ends.ends) {
      if constexpr (!DENSE)
        if (headMark) held = head[lane];
      close_unit<G>(a.out, held, headMark, acc, lane, g, c);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  if (a.persistent) close_span<G>(a.out, open, openRow, acc, lane);
  }  // spans
  if (!a.persistent)
    close_block<G>(a.out, rec, csf_wave_words(N, G, SS, DENSE), open, openRow, acc, lane, wib, wpb);
  trace_wave(a, kCsfKernel, traceStart, lane);
}

template <int G, int N, int SS, int kSteps, bool WIDE>
__global__ __launch_bounds__(256) void csf_group_kernel(const GroupArgs a) {
  csf_group_body<G, N, SS, kSteps, WIDE, false>(a, blockIdx.x, gridDim.x);
}

template <int G, int N, int SS, int kSteps, bool WIDE>
__global__ __launch_bounds__(256) void csf_group_dense_kernel(const GroupArgs a) {
  csf_group_body<G, N, SS, kSteps, WIDE, true>(a, blockIdx.x, gridDim.x);
}

// With 8 gathers in flight the order-3, R = 32, 32-bit-offset instantiation needs a few more vector registers than fit
// four wavefronts per SIMD; held to 128 it gains a wavefront.  (With 4 in flight: 82 to 96 registers at order 3, five
// wavefronts, 108 to 122 at order 4.  Holding order 3 to 80 for a sixth spills and takes 206 instead of 181 us on 5 M
// nonzeros, order 4 to 96 for a fifth 2702 instead of 2420 us on 50 M.)
template <int G, int N, int SS, int kSteps>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void csf_group_kernel_occ4(const GroupArgs a) {
  csf_group_body<G, N, SS, kSteps, false, false>(a, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------------------
// Single-representation variant (Section VI-A's other setting: one representation serves every mode, at 1 / N of
// the storage).  The target mode sits at tree level T >= 1 of another mode's B-CSF representation (all slices in
// the CSF group).  A lane group walks its run with START marks and keeps the current row of every level above the
// leaf; writing i_l for the index at level l,
//     out(i_T, :) += prod_{l < T} A_l(i_l, :)  *  sum over the level-T segment of  v * prod_{l > T} A_l(i_l, :)
// is added with atomic adds at the end of each level-T segment (T = leaf: per nonzero; then no leaf row is
// gathered).  The rows of the levels above the leaf are loaded where they change; leaf rows kSteps at a time.
// Rank 32 only (G = 8).  Every output row is reached by atomics, so the caller zero-fills the output first.
// ---------------------------------------------------------------------------------------
template <int N, int LS, int T, bool WIDE>
__global__ __launch_bounds__(256) void csf_nonroot_kernel(const GroupArgs a) {
  constexpr int G = 8;
  constexpr int NG = 64 / G;
  constexpr int NF = N - 2;
  constexpr int RW = (N == 3) ? 4 : 8;
  constexpr int LEAF = N - 1;
  constexpr int kSteps = 4;
  static_assert(T >= 1 && T <= LEAF, "the target is below the root");
  extern __shared__ uint32_t lds[];
  const int lane = threadIdx.x & 63;
  const int wib = threadIdx.x >> 6;
  const int wpb = blockDim.x >> 6;
  const int g = lane / G, c = lane % G;
  constexpr uint32_t L = 1u << LS;
  uint32_t* rec = lds + (size_t)wib * (NG * (L + 1) * RW);

  const SpanWalk walk = span_walk(a, blockIdx.x, gridDim.x, wib, wpb);
  for (uint32_t span = walk.first; span < walk.end; span += walk.stride) {
    uint32_t u = span * a.unitsPerWave;
    const uint32_t uEnd = min(u + a.unitsPerWave, a.nUnits);
    UnitBounds cur = load_bounds<G, N, LS, true>(a, u, lane);
    uint32_t fLo[3] = {0, 0, 0};
#pragma unroll
    for (int l = 1; l <= NF; ++l) fLo[l - 1] = a.runFirst[l][u * NG];

    for (; u < uEnd; ++u) {
      const UnitBounds nxt = load_bounds<G, N, LS, true>(a, min(u + 1, a.nUnits - 1), lane);
      const UnitEnds ends = stage_unit<G, N, LS, true>(a, rec, u, cur, fLo, lane);
      fLo[0] = cur.fHi[0];
      fLo[1] = cur.fHi[1];
      fLo[2] = cur.fHi[2];
      cur = nxt;
      const uint32_t ng = ends.ng;
      if (ng > 0) {
        // rows of the levels above the leaf (lr[T] unused), their products above / below the target level
        rowvec lr[LEAF];
#pragma unroll
        for (int l = 0; l < LEAF; ++l) lr[l] = rv_ones();
        lr[0] = row_load<G, WIDE>(a.fac[0], ends.row, c);   // the slice may have begun in an earlier run
        rowvec up = rv_ones(), dn = rv_ones();
        rowvec acc = rv_zero();
        uint32_t curT = 0;
        bool open = false;
        const uint32_t* myrec = rec + (size_t)g * (L + 1) * RW;
        for (uint32_t sb = 0; sb < ng; sb += kSteps) {
          uint4 rr[kSteps];
          uint32_t hi0[kSteps], hi1[kSteps];   // record words 4 and 5 (N >= 4)
          rowvec cr[kSteps];
#pragma unroll
          for (int t = 0; t < kSteps; ++t) {
            const uint4* src = reinterpret_cast<const uint4*>(myrec + (size_t)(sb + t) * RW);
            rr[t] = src[0];
            hi0[t] = hi1[t] = 0;
            if (N >= 4) {
              const uint2 h2 = reinterpret_cast<const uint2*>(src)[2];
              hi0[t] = h2.x;
              hi1[t] = h2.y;
            }
          }
          if (T < LEAF) {
#pragma unroll
            for (int t = 0; t < kSteps; ++t) cr[t] = row_load<G, WIDE>(a.fac[LEAF], rr[t].x, c);
          }
#pragma unroll
          for (int t = 0; t < kSteps; ++t) {
            if (sb + (uint32_t)t < ng) {
              // start marks by level: fiber level l at record word 2 + (NF - l), the slice after them
              uint32_t mk[LEAF];
              mk[0] = (N == 3) ? rr[t].w : (N == 4 ? hi0[t] : hi1[t]);
              mk[LEAF - 1] = rr[t].z;                           // deepest fiber level
              if constexpr (N >= 4) mk[LEAF - 2] = rr[t].w;
              if constexpr (N == 5) mk[1] = hi0[t];
              bool any = false;
#pragma unroll
              for (int l = 0; l < LEAF; ++l) any = any || mk[l] != 0u;
              if (any) {
                if (T < LEAF && mk[T < LEAF ? T : 0] != 0u) {
                  if (open) {
                    row_atomic<G>(a.out, curT, c, mul4(acc, up));
                    acc = rv_zero();
                  }
                  curT = mk[T < LEAF ? T : 0] - 1u;
                  open = true;
                }
#pragma unroll
                for (int l = 0; l < LEAF; ++l)
                  if (l != T && mk[l] != 0u) lr[l] = row_load<G, WIDE>(a.fac[l], mk[l] - 1u, c);
                up = lr[0];
#pragma unroll
                for (int l = 1; l < T && l < LEAF; ++l) up = mul4(up, lr[l]);
                dn = rv_ones();
#pragma unroll
                for (int l = T + 1; l < LEAF; ++l) dn = mul4(dn, lr[l]);
              }
              const float v = __uint_as_float(rr[t].y);
              if (T == LEAF) {
                row_atomic<G>(a.out, rr[t].x, c, scale4(v, up));
              } else {
                fma4(acc, v, mul4(cr[t], dn));
              }
            }
          }
        }
        if (T < LEAF && open) row_atomic<G>(a.out, curT, c, mul4(acc, up));
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  }
}

// ---------------------------------------------------------------------------------------
// CSL group (Algorithm "CSL-MTTKRP"): every nonzero carries all its non-root indices; the
// slice pointer goes straight to the nonzeros.
// LDS of a unit: an array each for the N - 1 indices, the value and the slice mark.
// ---------------------------------------------------------------------------------------
template <int G, int N, int SS, int kSteps, bool WIDE, typename Defined = DefinedBefore>
__device__ __forceinline__ void csl_group_body(const GroupArgs& a, uint32_t block, uint32_t blocks,
                                               const Defined& defined = Defined()) {
  constexpr int NG = 64 / G;
  extern __shared__ uint32_t lds[];
  const int lane = threadIdx.x & 63;
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wpb = blockDim.x >> 6;
  const int g = lane / G, c = lane % G;
  constexpr uint32_t SUB = 1u << SS;
  constexpr uint32_t slots = NG << SS;
  uint32_t* words = lds + (uint32_t)wib * csl_wave_words(N, G, SS);
  rowvec* head = reinterpret_cast<rowvec*>(words + (N + 1) * slots);

  const unsigned long long traceStart = a.trace ? wall_clock64() : 0ull;
  const SpanWalk walk = span_walk(a, block, blocks, wib, wpb);
  rowvec acc = rv_zero();               // as in the B-CSF kernel
  bool open = false;
  uint32_t openRow = 0;
  for (uint32_t span = walk.first; span < walk.end; span += walk.stride) {
  uint32_t u = span * a.unitsPerWave;
  const uint32_t uEnd = min(u + a.unitsPerWave, a.nUnits);
  acc = rv_zero();
  bool spread = false;

  UnitBounds cur = load_bounds<G, N, SS, false>(a, u, lane);
  const uint32_t fLo[3] = {0, 0, 0};

  for (; u < uEnd; ++u) {
    const UnitBounds nxt = load_bounds<G, N, SS, false>(a, min(u + 1, a.nUnits - 1), lane);
    const UnitEnds ends = stage_arrays<G, N, SS, false>(a, words, u, cur, fLo, lane);
    uint32_t headMark = 0;
    cur = nxt;
    open = ends.open;
    openRow = ends.row;
    if (ends.ends && spread) {
      sum_lane_groups<G>(acc);
      if (g > 0) acc = rv_zero();
    }
    spread = !ends.ends;

    if (ends.ng > 0) {
      const uint32_t swizzle = quad_swizzle<SS>((uint32_t)g);
#pragma unroll 1
      for (uint32_t sb = 0; sb < SUB; sb += kSteps) {
        uint32_t ix[N - 1][kSteps];
        uint32_t vv[kSteps];   // value bits
        uint32_t mi[kSteps];   // slice mark
        rowvec x1[kSteps], x2[kSteps], x3[kSteps], x4[kSteps];
#pragma unroll
        for (int b = 0; b < kSteps; b += 4) {
          const quad* src = reinterpret_cast<const quad*>(words) + (((uint32_t)g << (SS - 2)) + ((sb / 4 + b / 4) ^ swizzle));
          quad q[N + 1];
#pragma unroll
          for (int k = 0; k <= N; ++k) q[k] = src[(uint32_t)k * slots / 4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
#pragma unroll
            for (int k = 0; k < N - 1; ++k) ix[k][b + t] = q[k][t];
            vv[b + t] = q[N - 1][t];
            mi[b + t] = q[N][t];
          }
        }
#pragma unroll
        for (int t = 0; t < kSteps; ++t) {
          x1[t] = row_load<G, WIDE>(a.fac[1], ix[0][t], c);
          x2[t] = row_load<G, WIDE>(a.fac[2], ix[1][t], c);
          if constexpr (N >= 4) x3[t] = row_load<G, WIDE>(a.fac[3], ix[2][t], c);
          if constexpr (N >= 5) x4[t] = row_load<G, WIDE>(a.fac[4], ix[3][t], c);
        }
#pragma unroll
        for (int t = 0; t < kSteps; ++t) {
          rowvec pr = mul4(x1[t], x2[t]);
          if (N >= 4) pr = mul4(pr, x3[t]);
          if (N >= 5) pr = mul4(pr, x4[t]);
          fma4(acc, __uint_as_float(vv[t]), pr);
          if (mi[t]) {
            if (headMark) {
              emit_row<G>(a.out, mi[t], c, acc);
            } else {
              headMark = mi[t];
              head[lane] = acc;
            }
            acc = rv_zero();
          }
        }
      }
    }
    if constexpr (Defined::kAsks) {
      const uint32_t headState = headMark ? defined.ask((headMark & 0x7fffffffu) - 1u) : 0u;
      wait_defined(defined, headMark, headState, open, openRow, defined.ask(openRow), lane, c);
    }
    if (ends.ends) close_unit<G>(a.out, headMark ? head[lane] : rv_zero(), headMark, acc, lane, g, c);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  if (a.persistent) close_span<G>(a.out, open, openRow, acc, lane);
  }  // spans
  if (!a.persistent) close_block<G>(a.out, words, csl_wave_words(N, G, SS), open, openRow, acc, lane, wib, wpb);
  trace_wave(a, kCslKernel, traceStart, lane);
}

template <int G, int N, int SS, int kSteps, bool WIDE>
__global__ __launch_bounds__(256) void csl_group_kernel(const GroupArgs a) {
  csl_group_body<G, N, SS, kSteps, WIDE>(a, blockIdx.x, gridDim.x);
}

// The output definition's share of one of the first blocks of a launch.
template <int G, int N>
__device__ __forceinline__ void define_block(const GroupArgs& a, const DefineArgs& d, uint32_t block) {
  const DefinedHere<G> defined{d, a.out};
  const int lane = threadIdx.x & 63;
  const uint32_t words = (d.rows + 31u) >> 5, waves = d.blocks * (blockDim.x >> 6);
  const CooGroup coo{{d.ind[0], d.ind[1], d.ind[2], d.ind[3], d.ind[4]}, d.val};
  for (uint32_t wd = __builtin_amdgcn_readfirstlane(block * (blockDim.x >> 6) + (threadIdx.x >> 6)); wd < words; wd += waves) {
    const uint32_t wc = d.cooBits[wd], zBase = d.cooPtr[wd];
    (void)defined.claim(wd, lane);
    if (wc) define_word<G, N, false, false>(a.fac, a.out, coo, 0u, wc, zBase, wd, d.rows, lane);
  }
}

// Both groups in one launch (neither reads what the other writes; rows they share are added atomically): the first
// cslBlocks blocks walk the CSL group, the others the B-CSF group, so that the tail of one is filled with work of the
// other.  On a 5 M-nonzero tensor the CSL kernel alone took 16 us for 80 000 nonzeros, nearly all of it latency.
template <int G, int N, int SS, int kSteps, bool WIDE>
__global__ __launch_bounds__(256) void csl_csf_kernel(const GroupArgs csl, const GroupArgs csf, uint32_t cslBlocks) {
  if (blockIdx.x < cslBlocks) csl_group_body<G, N, SS, kSteps, WIDE>(csl, blockIdx.x, cslBlocks);
  else csf_group_body<G, N, SS, kSteps, WIDE, false>(csf, blockIdx.x - cslBlocks, gridDim.x - cslBlocks);
}

// The same with the output definition in its first blocks.
template <int G, int N, int SS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(N == 3 ? 5 : N == 4 ? 4 : 3)))
void define_csl_csf_kernel(const GroupArgs csl, const GroupArgs csf, uint32_t cslBlocks, const DefineArgs define) {
  if (blockIdx.x < define.blocks) {
    define_block<G, N>(csf, define, blockIdx.x);
    return;
  }
  const DefinedHere<G> defined{define, csf.out};
  const uint32_t block = blockIdx.x - define.blocks, blocks = gridDim.x - define.blocks;
  if (block < cslBlocks) csl_group_body<G, N, SS, 4, false>(csl, block, cslBlocks, defined);
  else csf_group_body<G, N, SS, 4, false, false>(csf, block - cslBlocks, blocks - cslBlocks, defined);
}

#ifndef HBCSF_F64
// The same with ALS work in the launch's first block (of 8, so that the others keep their XCDs).  The inverse takes 110
// registers: where units of 256 nonzeros fill the chip, the order-3 kernels are held to the 96 that leave five wavefronts
// per SIMD.
// Two forms: with the output definition in the next blocks, and after one in a launch of its own, without the code that asks for
// rows, which costs 1 to 6 % of a launch (five iterations at rank 32, asking -> not asking: 8 M nonzeros of order 4 2870 -> 2782 us,
// 6 M of order 5 3842 -> 3564).
constexpr uint32_t kGuestBlocks = 8;
constexpr bool guest_held(int G, int N, int SS) { return N == 3 && ((64 / G) << SS) == 256; }

// Where the sweep has failed, the last blocks (a launch's very last may have no span) leave the time; who ends last stays.  (All
// updates together took 0.7 us each to write it to the host.  One whose sweep ends after them is not seen to fail here,
// but then the eigenvalue form's begin says as much.  The lane is counted: see thread_number().)
__device__ __forceinline__ void stamp_end(const GuestArgs& guest) {
  if (gridDim.x - blockIdx.x <= 64 && thread_number<true>(0) == 0 &&
      __hip_atomic_load(guest.good, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
    guest.stamp[3] = wall_clock64();
}

// (The two kernels share no function around the groups': inlined in two steps, the groups' blockDim is a load that every wavefront
// begins with by waiting for it, 1 % of the launch.)
template <int G, int N, int SS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(guest_held(G, N, SS) ? 5 : 4)))
void guest_csl_csf_kernel(const GroupArgs csl, const GroupArgs csf, uint32_t cslBlocks, const GuestArgs guest) {
  extern __shared__ uint32_t lds[];
  constexpr bool kCounted = guest_held(G, N, SS);
  const uint32_t wave = kCounted ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0u;
  if (blockIdx.x < kGuestBlocks) {
    if (blockIdx.x == 0) guest_block<4 * G, kCounted>(guest, lds, wave);
    return;
  }
  const uint32_t block = blockIdx.x - kGuestBlocks, blocks = gridDim.x - kGuestBlocks;
  if (block < cslBlocks) csl_group_body<G, N, SS, 4, false>(csl, block, cslBlocks);
  else csf_group_body<G, N, SS, 4, false, false>(csf, block - cslBlocks, blocks - cslBlocks);
  stamp_end(guest);
}

template <int G, int N, int SS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(guest_held(G, N, SS) ? 5 : 4)))
void guest_define_csl_csf_kernel(const GroupArgs csl, const GroupArgs csf, uint32_t cslBlocks, const DefineArgs define,
                                 const GuestArgs guest) {
  extern __shared__ uint32_t lds[];
  if (blockIdx.x < kGuestBlocks) {
    stamp_begin(guest.stamp);
    if (blockIdx.x == 0) guest_block<4 * G, false>(guest, lds, 0);
    return;
  }
  if (blockIdx.x < kGuestBlocks + define.blocks) {
    define_block<G, N>(csf, define, blockIdx.x - kGuestBlocks);
    return;
  }
  const DefinedHere<G> defined{define, csf.out};
  const uint32_t first = kGuestBlocks + define.blocks;
  const uint32_t block = blockIdx.x - first, blocks = gridDim.x - first;
  if (block < cslBlocks) csl_group_body<G, N, SS, 4, false>(csl, block, cslBlocks, defined);
  else csf_group_body<G, N, SS, 4, false, false>(csf, block - cslBlocks, blocks - cslBlocks, defined);
  stamp_end(guest);
}
#endif

// ---------------------------------------------------------------------------------------
// COO group (Algorithm "COO-MTTKRP" restricted to slices with one nonzero): each nonzero owns
// its output row, so the row is written with a plain store and no atomic is needed.
// Lane group g of a wavefront takes nonzero z = base + step*NG + g.
// ---------------------------------------------------------------------------------------
template <int G, int N, bool WIDE>
__global__ __launch_bounds__(256) void coo_group_kernel(const GroupArgs a) {
  constexpr int NG = 64 / G;
  constexpr int kU = G < 8 ? G : 8;  // nonzeros per lane group in flight
  const int lane = threadIdx.x & 63;
  const int g = lane / G, c = lane % G;
  const uint32_t waves = (gridDim.x * blockDim.x) >> 6;
  const uint32_t wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const uint32_t* __restrict__ valb = reinterpret_cast<const uint32_t*>(a.val);
  // 64 nonzeros per wavefront and iteration: lane l loads the coordinates of nonzero base + l
  // (coalesced), then lane group g takes nonzero base + step*NG + g from lane step*NG + g.
  for (uint64_t base = (uint64_t)wave * 64u; base < a.nnz; base += (uint64_t)waves * 64u) {
    const uint64_t z = base + lane;
    uint32_t m0 = 0, m1 = 0, m2 = 0, m3 = 0, m4 = 0, mv = 0;
    if (z < a.nnz) {
      m0 = __builtin_nontemporal_load(a.ind[0] + z);
      m1 = __builtin_nontemporal_load(a.ind[1] + z);
      m2 = __builtin_nontemporal_load(a.ind[2] + z);
      if (N >= 4) m3 = __builtin_nontemporal_load(a.ind[3] + z);
      if (N >= 5) m4 = __builtin_nontemporal_load(a.ind[4] + z);
      mv = __builtin_nontemporal_load(valb + z);
    }
    const uint32_t left = (uint32_t)min((uint64_t)64, a.nnz - base);
#pragma unroll
    for (int sb = 0; sb < G; sb += kU) {
      uint32_t i0[kU], v[kU];
      rowvec x1[kU], x2[kU], x3[kU], x4[kU];
      bool ok[kU];
#pragma unroll
      for (int t = 0; t < kU; ++t) {
        const int src = (sb + t) * NG + g;
        ok[t] = (uint32_t)src < left;
        i0[t] = __shfl(m0, src);
        v[t] = __shfl(mv, src);
        const uint32_t i1 = __shfl(m1, src), i2 = __shfl(m2, src);
        const uint32_t i3 = N >= 4 ? __shfl(m3, src) : 0u;
        const uint32_t i4 = N >= 5 ? __shfl(m4, src) : 0u;
        if (ok[t]) {
          x1[t] = row_load<G, WIDE>(a.fac[1], i1, c);
          x2[t] = row_load<G, WIDE>(a.fac[2], i2, c);
          if (N >= 4) x3[t] = row_load<G, WIDE>(a.fac[3], i3, c);
          if (N >= 5) x4[t] = row_load<G, WIDE>(a.fac[4], i4, c);
        }
      }
#pragma unroll
      for (int t = 0; t < kU; ++t) {
        if (ok[t]) {
          rowvec pr = mul4(x1[t], x2[t]);
          if (N >= 4) pr = mul4(pr, x3[t]);
          if (N >= 5) pr = mul4(pr, x4[t]);
          row_store<G>(a.out, i0[t], c, scale4(__uint_as_float(v[t]), pr));
        }
      }
    }
  }
}

#ifdef HBCSF_F64
}  // namespace f64
using namespace f64;
#endif

// ---------------------------------------------------------------------------------------
// Launch helpers (host)
// ---------------------------------------------------------------------------------------
namespace {

// Blocks of `wpb` wavefronts for a group: one wavefront per span, a multiple of 8 blocks.
uint64_t span_blocks(const GroupArgs& a, uint32_t wpb) { return (((uint64_t)a.nSpans + wpb - 1) / wpb + 7) / 8 * 8; }

// `cus`: compute units.  Default launch: one wavefront per span.  Persistent launch: (resident blocks per CU) x CUs
// blocks, capped by the spans.  Both rounded to a multiple of 8.
template <int G, int N, int SS, int S, bool WIDE>
hipError_t launch_one(int kind, const GroupArgs& a, const GroupArgs* csl, const DefineArgs* define, const GuestArgs* guest,
                      uint32_t cus, dim3 block, size_t lds, hipStream_t s) {
  constexpr bool occ4 = G == 8 && N == 3 && S == 8 && !WIDE;
  const uint32_t wpb = block.x >> 6;
  if (guest) {
#ifndef HBCSF_F64
    if constexpr (G <= 16 && S == 4 && !WIDE && (G != 8 || SS < 6)) {
      constexpr int R = 4 * G;
      if (!csl || block.x != 256) return hipErrorInvalidValue;
      if (lds < guest_lds_bytes<R>()) lds = guest_lds_bytes<R>();
      const uint32_t cslBlocks = (uint32_t)span_blocks(*csl, wpb);
      const uint32_t blocks = kGuestBlocks + cslBlocks + (uint32_t)span_blocks(a, wpb);
      if (define)
        hipLaunchKernelGGL((guest_define_csl_csf_kernel<G, N, SS>), dim3(blocks + define->blocks), block, lds, s, *csl, a, cslBlocks,
                           *define, *guest);
      else hipLaunchKernelGGL((guest_csl_csf_kernel<G, N, SS>), dim3(blocks), block, lds, s, *csl, a, cslBlocks, *guest);
      return hipGetLastError();
    }
#endif
    return hipErrorInvalidValue;
  }
  if (define) {
    if constexpr (S == 4 && !WIDE && (G != 8 || SS < 6)) {
      if (!csl) return hipErrorInvalidValue;
      const uint32_t cslBlocks = (uint32_t)span_blocks(*csl, wpb);
      hipLaunchKernelGGL((define_csl_csf_kernel<G, N, SS>), dim3(define->blocks + cslBlocks + (uint32_t)span_blocks(a, wpb)), block,
                         lds, s, *csl, a, cslBlocks, *define);
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  }
  if (csl) {
    if constexpr (S == 4) {
      const uint32_t cslBlocks = (uint32_t)span_blocks(*csl, wpb);
      hipLaunchKernelGGL((csl_csf_kernel<G, N, SS, S, WIDE>), dim3(cslBlocks + (uint32_t)span_blocks(a, wpb)), block, lds,
                         s, *csl, a, cslBlocks);
      return hipGetLastError();
    }
    return hipErrorInvalidValue;  // with 8 gathers in flight the groups are launched one by one
  }
  void (*kernel)(GroupArgs) = nullptr;
  if constexpr (G != 8 || SS < 6 || S == 8) {  // (G = 8, 4 gathers: parts of at most 32 except in the dense variant)
    kernel = csl_group_kernel<G, N, SS, S, WIDE>;
    if (kind == kCsfKernel) {
      if constexpr (occ4) kernel = csf_group_kernel_occ4<G, N, SS, S>;
      else kernel = csf_group_kernel<G, N, SS, S, WIDE>;
    }
  }
  if constexpr (G == 8 && N <= 4 && (SS == 5 || SS == 6)) {
    if (kind == kCsfKernel && a.denseMid) kernel = csf_group_dense_kernel<G, N, SS, S, WIDE>;
  }
  if (!kernel) return hipErrorInvalidValue;
  uint64_t blocks = span_blocks(a, wpb);
  if (a.persistent) {
    // resident blocks per CU of this kernel on the current device (asked per launch: the persistent launch is a
    // tuning variant, and a cached answer would be wrong for another device of the process)
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, (int)block.x, lds);
    if (e != hipSuccess) return e;
    const uint64_t resident = ((uint64_t)cus * (uint64_t)(n > 0 ? n : 1) + 7) / 8 * 8;
    if (blocks > resident) blocks = resident;
  }
  hipLaunchKernelGGL(kernel, dim3((uint32_t)blocks), block, lds, s, a);
  return hipGetLastError();
}

template <int G, int N, int SS>
hipError_t launch_ss(int kind, int steps, bool wide, const GroupArgs& a, const GroupArgs* csl, const DefineArgs* define,
                     const GuestArgs* guest, uint32_t cus, dim3 block, size_t lds, hipStream_t s) {
  if constexpr (G == 8) {
    if (steps == 8)
      return wide ? launch_one<G, N, SS, 8, true>(kind, a, csl, define, guest, cus, block, lds, s)
                  : launch_one<G, N, SS, 8, false>(kind, a, csl, define, guest, cus, block, lds, s);
  }
  if (steps != 4) return hipErrorInvalidValue;
  return wide ? launch_one<G, N, SS, 4, true>(kind, a, csl, define, guest, cus, block, lds, s)
              : launch_one<G, N, SS, 4, false>(kind, a, csl, define, guest, cus, block, lds, s);
}

// The part sizes the caller can ask for at this G: units of at most 256 nonzeros, or at G = 8 parts of 64.
template <int G, int N>
hipError_t launch_g(int kind, int steps, bool wide, const GroupArgs& a, const GroupArgs* csl, const DefineArgs* define,
                    const GuestArgs* guest, dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  if (kind == kCooKernel) {
    if (wide) hipLaunchKernelGGL((coo_group_kernel<G, N, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((coo_group_kernel<G, N, false>), grid, block, 0, s, a);
    return hipGetLastError();
  }
  switch (a.partShift) {
    case 3: return launch_ss<G, N, 3>(kind, steps, wide, a, csl, define, guest, grid.x, block, lds, s);
    case 4:
      if constexpr (G >= 4) return launch_ss<G, N, 4>(kind, steps, wide, a, csl, define, guest, grid.x, block, lds, s);
      break;
    case 5:
      if constexpr (G >= 8) return launch_ss<G, N, 5>(kind, steps, wide, a, csl, define, guest, grid.x, block, lds, s);
      break;
    case 6:
      if constexpr (G >= 8) return launch_ss<G, N, 6>(kind, steps, wide, a, csl, define, guest, grid.x, block, lds, s);
      break;
  }
  return hipErrorInvalidValue;
}

}  // namespace

// This file is compiled once per (HBCSF_G, HBCSF_N) pair so that the instantiations build in
// parallel; each object exports one launch function, and the object built with
// HBCSF_WITH_DEFINE also holds the output-definition kernel's launcher.
#ifndef HBCSF_G
#error "compile with -DHBCSF_G=<lanes per row> -DHBCSF_N=<order>"
#endif
#define HBCSF_CAT2(a, b, c, d) a##b##c##d
#define HBCSF_CAT(a, b, c, d) HBCSF_CAT2(a, b, c, d)
#ifdef HBCSF_F64
#define HBCSF_LAUNCH_DEFINE_COO launch_define_coo64_g
#define HBCSF_LAUNCH_GROUP launch_group64_g
#else
#define HBCSF_LAUNCH_DEFINE_COO launch_define_coo_g
#define HBCSF_LAUNCH_GROUP launch_group_g
#endif

hipError_t HBCSF_CAT(HBCSF_LAUNCH_DEFINE_COO, HBCSF_G, _n, HBCSF_N)(bool wide, const GroupArgs& a,
                                                               const uint32_t* ownedBits, const uint32_t* cooBits,
                                                               const uint32_t* cooPtr, uint64_t rows, uint32_t blocks,
                                                               unsigned long long* stamp, hipStream_t s) {
  if (wide)
    hipLaunchKernelGGL((define_coo_kernel<HBCSF_G, HBCSF_N, true>), dim3(blocks), dim3(256), 0, s, a, ownedBits,
                       cooBits, cooPtr, rows, stamp);
  else
    hipLaunchKernelGGL((define_coo_kernel<HBCSF_G, HBCSF_N, false>), dim3(blocks), dim3(256), 0, s, a, ownedBits,
                       cooBits, cooPtr, rows, stamp);
  return hipGetLastError();
}

hipError_t HBCSF_CAT(HBCSF_LAUNCH_GROUP, HBCSF_G, _n, HBCSF_N)(int kind, int steps, bool wide, const GroupArgs& a,
                                                          const GroupArgs* csl, const DefineArgs* define,
                                                          const GuestArgs* guest, uint32_t blocks, uint32_t threads, size_t ldsBytes, hipStream_t s) {
  return launch_g<HBCSF_G, HBCSF_N>(kind, steps, wide, a, csl, define, guest, dim3(blocks), dim3(threads), ldsBytes, s);
}

#if HBCSF_G == 8 && !defined(HBCSF_F64)
namespace {
template <int N, int LS, int T>
hipError_t launch_nonroot_t(bool wide, const GroupArgs& a, uint32_t threads, size_t lds, hipStream_t s) {
  const uint32_t wpb = threads >> 6;
  const uint64_t blocks = (((uint64_t)a.nSpans + wpb - 1) / wpb + 7) / 8 * 8;
  if (wide) hipLaunchKernelGGL((csf_nonroot_kernel<N, LS, T, true>), dim3((uint32_t)blocks), dim3(threads), lds, s, a);
  else hipLaunchKernelGGL((csf_nonroot_kernel<N, LS, T, false>), dim3((uint32_t)blocks), dim3(threads), lds, s, a);
  return hipGetLastError();
}
}  // namespace

// Single-representation kernel for this object's order: target at tree level `level` (1 .. order-1) of the
// representation in `a` (B-CSF group only, runs of the order's default length), rank 32.
hipError_t HBCSF_CAT(launch_nonroot_n, HBCSF_N, , )(int level, bool wide, const GroupArgs& a, uint32_t threads,
                                                     size_t ldsBytes, hipStream_t s) {
  constexpr int LS = HBCSF_N == 3 ? 6 : 5;
  if (a.lshift != (uint32_t)LS || a.partShift != (uint32_t)LS || a.persistent) return hipErrorInvalidValue;
  switch (level) {
    case 1: return launch_nonroot_t<HBCSF_N, LS, 1>(wide, a, threads, ldsBytes, s);
    case 2: return launch_nonroot_t<HBCSF_N, LS, 2>(wide, a, threads, ldsBytes, s);
#if HBCSF_N >= 4
    case 3: return launch_nonroot_t<HBCSF_N, LS, 3>(wide, a, threads, ldsBytes, s);
#endif
#if HBCSF_N >= 5
    case 4: return launch_nonroot_t<HBCSF_N, LS, 4>(wide, a, threads, ldsBytes, s);
#endif
    default: return hipErrorInvalidValue;
  }
}
#endif  // HBCSF_G == 8, fp32

#ifdef HBCSF_WITH_DEFINE
// Plain zero fill of an output every row of which is then reached by atomic adds (the single-representation kernel).
__global__ __launch_bounds__(256) void zero_rows_kernel(rowvec* __restrict__ out, uint64_t nvec) {
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < nvec; i += (uint64_t)gridDim.x * 256)
    store_streaming(out + i, rv_zero());
}

hipError_t launch_zero_rows(float* out, uint64_t nvec, uint32_t blocks, hipStream_t s) {
  hipLaunchKernelGGL(zero_rows_kernel, dim3(blocks), dim3(256), 0, s, reinterpret_cast<rowvec*>(out), nvec);
  return hipGetLastError();
}

hipError_t launch_define(float* out, const uint32_t* ownedBits, uint64_t rows, int G, uint32_t blocks,
                         unsigned long long* stamp, hipStream_t s) {
  int gshift = 0;
  while ((1 << gshift) < G) ++gshift;
  hipLaunchKernelGGL(define_rows_kernel, dim3(blocks), dim3(256), 0, s, reinterpret_cast<rowvec*>(out),
                     ownedBits, rows * (uint64_t)G, gshift, stamp);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Diagnostic: the row-gather rate the memory system sustains for this access shape (128-byte
// rows, 8 lanes x rowvec, 8 gathers in flight per lane group), with none of the MTTKRP work
// around it.  Used to put a measured ceiling beside the kernels' achieved rates.
// `active` (1..8): load instruction t of a block of 8 is executed by the lane groups g with
// (g - t) mod 8 < active only, the others sit it out, as the lane groups without a segment end
// do in the B-CSF kernel's fiber-row loads; every instruction is still issued by the wavefront.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void probe_gather_kernel(const uint32_t* __restrict__ idx, uint64_t n,
                                                           const float* __restrict__ table,
                                                           float* __restrict__ sink, uint32_t perWave, int active) {
  constexpr int S = 8;
  const int lane = threadIdx.x & 63;
  const int g = lane >> 3, c = lane & 7;
  const uint64_t wave = (uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const uint32_t per = perWave / 8;
  uint64_t p = wave * perWave + (uint64_t)g * per;
  const uint64_t pEnd = p + per;
  rowvec acc = rv_zero();
  for (; p + S <= pEnd && p + S <= n; p += S) {
    // one index load per block: lane c of a lane group fetches the index of step c
    const uint32_t mine = idx[p + c];
    uint32_t k[S];
    rowvec r[S];
#pragma unroll
    for (int t = 0; t < S; ++t) k[t] = __shfl(mine, (g << 3) + t);
#pragma unroll
    for (int t = 0; t < S; ++t) {
      r[t] = rv_zero();
      if (((g - t) & 7) < active) r[t] = *reinterpret_cast<const rowvec*>(table + ((size_t)k[t] * 32 + (size_t)(4 * c)));
    }
#pragma unroll
    for (int t = 0; t < S; ++t) {
      acc.x += r[t].x;
      acc.y += r[t].y;
      acc.z += r[t].z;
      acc.w += r[t].w;
    }
  }
  if (acc.x == 123.456f) sink[0] = acc.x + acc.y + acc.z + acc.w;  // keeps the loads alive
}

hipError_t launch_probe_gather(const uint32_t* idx, uint64_t n, const float* table, float* sink,
                               uint32_t waves, uint32_t perWave, int active, hipStream_t s) {
  hipLaunchKernelGGL(probe_gather_kernel, dim3(waves / 4), dim3(256), 0, s, idx, n, table, sink, perWave, active);
  return hipGetLastError();
}
#endif  // HBCSF_WITH_DEFINE

}  // namespace hbcsf
