// Kernel argument block and launch entry points shared by the kernels and the C-ABI layer.
#ifndef HBCSF_DEVICE_H_
#define HBCSF_DEVICE_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hbcsf.h"

namespace hbcsf {

enum KernelKind { kCooKernel = 0, kCslKernel = 1, kCsfKernel = 2 };

// The B-CSF kernel's dense fiber-row gather: rows its per-wavefront LDS cache holds, the instantiations that
// exist (rank 32, orders 3 and 4, runs of 32 or 64 nonzeros).
constexpr int kDenseCacheRows = 32;
inline bool dense_mid_available(int order, int G, uint32_t lshift) {
  return G == 8 && (order == 3 || order == 4) && (lshift == 5 || lshift == 6);
}

// LDS words a wavefront of the B-CSF / CSL kernel uses: an array of one word per nonzero of a unit (64 / G parts of 2^ss
// nonzeros) for each of the things it stages, one row slot per lane (the first finished slice of each part), and for the
// B-CSF kernel the list of the unit's slices with each part's place in it.  The dense variant: one record per nonzero,
// one pad record per part, its row numbers and row cache.
constexpr uint32_t csf_wave_words(int order, int G, int ss, bool dense) {
  const uint32_t parts = 64u / (uint32_t)G, slots = parts << ss;
  if (dense) return (slots + parts) * (order == 3 ? 4u : 8u) + 64u + (uint32_t)kDenseCacheRows * 4u * (uint32_t)G;
  return slots * (uint32_t)(order + 1) + (parts < 4u ? 4u : parts) + 256u;
}
constexpr uint32_t csl_wave_words(int order, int G, int ss) {
  return ((64u / (uint32_t)G) << ss) * (uint32_t)(order + 1) + 256u;
}

// What a CPD-ALS state keeps per mode m in the caller's workspace: the Gram matrix of the stored factor, c_m (the
// algorithm's factor is the stored one with column r divided by c_m[r]) and the column norms of the last update.
struct SmallState {
  double* gram[HBCSF_MAX_ORDER];
  double* scale[HBCSF_MAX_ORDER];
  double* norm[HBCSF_MAX_ORDER];
  int order;
};

// The part of a put-off ALS update that an MTTKRP launch carries in its first block (hbcsf_small.h).
struct GuestArgs {
  SmallState small;
  int n;                     // the mode being updated
  float* p;                  // right-hand matrix of the product that follows
  double* vp;                // [rank][rank], where the eigenvalue form is put
  int* good;                 // receives 1 where the sweep succeeded, else 0
  unsigned long long* stamp; // [4]: receives in [0] the time at which the MTTKRP's first kernel begins, in [1] 0 or when the
                             // eigenvalue form does; where the sweep fails while the last blocks are at work, in [3] when
                             // those end
};

// Device pointers of one slice group of one mode, by tree level (0 = root .. order-1 = leaf).
struct GroupArgs {
  const uint32_t* ind[5];       // index arrays (per slice / segment / nonzero, by group kind)
  const uint32_t* ptr[5];       // starts in the group's nonzero stream (n+1 entries)
  const uint32_t* runFirst[5];  // slice / segment holding the first nonzero of each run
  const float* val;             // values in stream order
  const float* fac[5];          // factor matrix of each tree level (fac[0] unused)
  float* out;                   // [rows][rank]
  uint32_t nnz;                 // nonzeros in the group
  uint32_t runs;                // ceil(nnz / L)
  uint32_t lshift;              // log2 L
  uint32_t partShift;           // log2 of the nonzeros a lane group takes of a unit (<= lshift)
  uint32_t nUnits;              // ceil(nnz / (lane groups per wavefront << partShift))
  uint32_t unitsPerWave;        // consecutive units in one span
  uint32_t nSpans;              // ceil(nUnits / unitsPerWave)
  uint32_t streamLevel;         // bit l: the factor rows of fiber level l are gathered with streaming loads
  uint32_t persistent;          // 1: resident wavefronts take spans round-robin; 0: one wavefront per span
  uint32_t denseMid;            // B-CSF kernel: 1 = fiber-level rows gathered once per block of steps for the whole
                                // wavefront through an LDS row cache (needs dense_mid_available and its LDS size)
  // Optional wavefront trace (profiling only, nullptr = off): trace[0] counts records; record i
  // is the four words at trace[4 + 4 i]: {kernel kind, XCC_ID << 32 | HW_ID, start, end} with
  // start / end from the constant-rate wall clock.
  unsigned long long* trace;
  uint32_t traceCapacity;       // records the buffer can hold
};

// Output definition inside an MTTKRP launch: the rows that no CSL / B-CSF slice stores by itself are written by the launch's
// first blocks, one 32-row word of the bitmaps at a time.  state[word] grows from call to call: `claimed` (2 call + 1) while a
// wavefront of this call writes the word's rows, claimed + 1 once they are written.
struct DefineArgs {
  const uint32_t* ownedBits;
  const uint32_t* cooBits;
  const uint32_t* cooPtr;
  const uint32_t* ind[5];        // the COO group, by tree level
  const float* val;
  uint32_t rows;
  uint32_t blocks;               // the launch's first blocks, a multiple of 8
  uint32_t* state;
  uint32_t claimed;
};

// Longest mode whose format has room for DefineArgs' state.
constexpr uint64_t kDefineStateRows = 1ull << 18;

// kind: KernelKind; order 3, 4 or 5; G = row bytes / 16 lanes per factor row (fp32: rank / 4 = 2, 4, 8, 16 or 32;
// fp64: rank / 2 = 8, 16 or 32, the launch functions named ...64...);
// steps = records a lane group keeps in flight (4, or at G = 8 also 8; not used for the COO group); csl = null, or with
// kind = kCsfKernel and 4 steps the CSL group's arguments: both groups in one launch (same part size), one of them perhaps
// without a nonzero; define = null, or (not wide, with csl) the output definition for the first blocks of that launch; guest
// = null, or (fp32, G <= 16, 4 steps, not wide, with csl, blocks of 256 threads) ALS work for the first block; wide = some
// gathered factor matrix is 4 GiB or larger (64-bit row addressing).  One launch function per (G, order) pair, each
// compiled in its own object file.  For the CSL and B-CSF kernels `blocks` is the number of compute
// units and the launcher sizes the grid (one wavefront per span, or persistent).
#define HBCSF_DECLARE_LAUNCH(G, N)                                                                  \
  hipError_t launch_group_g##G##_n##N(int kind, int steps, bool wide, const GroupArgs& a,          \
                                      const GroupArgs* csl, const DefineArgs* define, const GuestArgs* guest, uint32_t blocks, uint32_t threads, size_t ldsBytes, \
                                      hipStream_t s);                                                \
  hipError_t launch_define_coo_g##G##_n##N(bool wide, const GroupArgs& a, const uint32_t* ownedBits,   \
                                           const uint32_t* cooBits, const uint32_t* cooPtr, uint64_t rows, \
                                           uint32_t blocks, unsigned long long* stamp, hipStream_t s);
HBCSF_DECLARE_LAUNCH(2, 3)
HBCSF_DECLARE_LAUNCH(4, 3)
HBCSF_DECLARE_LAUNCH(8, 3)
HBCSF_DECLARE_LAUNCH(16, 3)
HBCSF_DECLARE_LAUNCH(32, 3)
HBCSF_DECLARE_LAUNCH(2, 4)
HBCSF_DECLARE_LAUNCH(4, 4)
HBCSF_DECLARE_LAUNCH(8, 4)
HBCSF_DECLARE_LAUNCH(16, 4)
HBCSF_DECLARE_LAUNCH(32, 4)
HBCSF_DECLARE_LAUNCH(2, 5)
HBCSF_DECLARE_LAUNCH(4, 5)
HBCSF_DECLARE_LAUNCH(8, 5)
HBCSF_DECLARE_LAUNCH(16, 5)
HBCSF_DECLARE_LAUNCH(32, 5)
#undef HBCSF_DECLARE_LAUNCH
#define HBCSF_DECLARE_LAUNCH64(G, N)                                                                  \
  hipError_t launch_group64_g##G##_n##N(int kind, int steps, bool wide, const GroupArgs& a,          \
                                        const GroupArgs* csl, const DefineArgs* define, const GuestArgs* guest, uint32_t blocks, uint32_t threads, size_t ldsBytes, \
                                        hipStream_t s);                                                \
  hipError_t launch_define_coo64_g##G##_n##N(bool wide, const GroupArgs& a, const uint32_t* ownedBits,   \
                                             const uint32_t* cooBits, const uint32_t* cooPtr, uint64_t rows, \
                                             uint32_t blocks, unsigned long long* stamp, hipStream_t s);
HBCSF_DECLARE_LAUNCH64(8, 3)
HBCSF_DECLARE_LAUNCH64(16, 3)
HBCSF_DECLARE_LAUNCH64(32, 3)
HBCSF_DECLARE_LAUNCH64(8, 4)
HBCSF_DECLARE_LAUNCH64(16, 4)
HBCSF_DECLARE_LAUNCH64(32, 4)
HBCSF_DECLARE_LAUNCH64(8, 5)
HBCSF_DECLARE_LAUNCH64(16, 5)
HBCSF_DECLARE_LAUNCH64(32, 5)
#undef HBCSF_DECLARE_LAUNCH64

// f64: the factor matrices and the output hold doubles (GroupArgs' float pointers then address doubles).
inline hipError_t launch_group(bool f64, int kind, int order, int G, int steps, bool wide, const GroupArgs& a,
                               const GroupArgs* csl, const DefineArgs* define, const GuestArgs* guest, uint32_t blocks, uint32_t threads, size_t ldsBytes,
                               hipStream_t s) {
#define HBCSF_CASE64(GV)                                                                              \
  case GV:                                                                                            \
    return order == 3   ? launch_group64_g##GV##_n3(kind, steps, wide, a, csl, define, guest, blocks, threads, ldsBytes, s) \
           : order == 4 ? launch_group64_g##GV##_n4(kind, steps, wide, a, csl, define, guest, blocks, threads, ldsBytes, s) \
                        : launch_group64_g##GV##_n5(kind, steps, wide, a, csl, define, guest, blocks, threads, ldsBytes, s);
  if (f64) {
    switch (G) {
      HBCSF_CASE64(8)
      HBCSF_CASE64(16)
      HBCSF_CASE64(32)
      default:
        return hipErrorInvalidValue;
    }
  }
#undef HBCSF_CASE64
#define HBCSF_CASE(GV)                                                                              \
  case GV:                                                                                          \
    return order == 3   ? launch_group_g##GV##_n3(kind, steps, wide, a, csl, define, guest, blocks, threads, ldsBytes, s) \
           : order == 4 ? launch_group_g##GV##_n4(kind, steps, wide, a, csl, define, guest, blocks, threads, ldsBytes, s) \
                        : launch_group_g##GV##_n5(kind, steps, wide, a, csl, define, guest, blocks, threads, ldsBytes, s);
  switch (G) {
    HBCSF_CASE(2)
    HBCSF_CASE(4)
    HBCSF_CASE(8)
    HBCSF_CASE(16)
    HBCSF_CASE(32)
    default:
      return hipErrorInvalidValue;
  }
#undef HBCSF_CASE
}

// Output definition fused with the COO group (a: the COO group's arguments).  stamp: null, or GuestArgs' stamps.
inline hipError_t launch_define_coo(bool f64, int order, int G, bool wide, const GroupArgs& a,
                                    const uint32_t* ownedBits, const uint32_t* cooBits, const uint32_t* cooPtr,
                                    uint64_t rows, uint32_t blocks, unsigned long long* stamp, hipStream_t s) {
#define HBCSF_CASE64(GV)                                                                                     \
  case GV:                                                                                                   \
    return order == 3   ? launch_define_coo64_g##GV##_n3(wide, a, ownedBits, cooBits, cooPtr, rows, blocks, stamp, s) \
           : order == 4 ? launch_define_coo64_g##GV##_n4(wide, a, ownedBits, cooBits, cooPtr, rows, blocks, stamp, s) \
                        : launch_define_coo64_g##GV##_n5(wide, a, ownedBits, cooBits, cooPtr, rows, blocks, stamp, s);
  if (f64) {
    switch (G) {
      HBCSF_CASE64(8)
      HBCSF_CASE64(16)
      HBCSF_CASE64(32)
      default:
        return hipErrorInvalidValue;
    }
  }
#undef HBCSF_CASE64
#define HBCSF_CASE(GV)                                                                                     \
  case GV:                                                                                                 \
    return order == 3   ? launch_define_coo_g##GV##_n3(wide, a, ownedBits, cooBits, cooPtr, rows, blocks, stamp, s) \
           : order == 4 ? launch_define_coo_g##GV##_n4(wide, a, ownedBits, cooBits, cooPtr, rows, blocks, stamp, s) \
                        : launch_define_coo_g##GV##_n5(wide, a, ownedBits, cooBits, cooPtr, rows, blocks, stamp, s);
  switch (G) {
    HBCSF_CASE(2)
    HBCSF_CASE(4)
    HBCSF_CASE(8)
    HBCSF_CASE(16)
    HBCSF_CASE(32)
    default:
      return hipErrorInvalidValue;
  }
#undef HBCSF_CASE
}

// Zero fill of the rows whose bit in ownedBits is clear; a row is G 16-byte pieces (fp32 or fp64 alike).  stamp as above.
hipError_t launch_define(float* out, const uint32_t* ownedBits, uint64_t rows, int G,
                         uint32_t blocks, unsigned long long* stamp, hipStream_t s);

// Zero fill of nvec float4s (an output that is then only reached by atomic adds).
hipError_t launch_zero_rows(float* out, uint64_t nvec, uint32_t blocks, hipStream_t s);

// Single-representation kernels (rank 32): the target mode is at tree level `level` >= 1 of the representation
// whose B-CSF group `a` describes (fac[l] set for every level but `level`, fac[0] included).
hipError_t launch_nonroot_n3(int level, bool wide, const GroupArgs& a, uint32_t threads, size_t ldsBytes, hipStream_t s);
hipError_t launch_nonroot_n4(int level, bool wide, const GroupArgs& a, uint32_t threads, size_t ldsBytes, hipStream_t s);
hipError_t launch_nonroot_n5(int level, bool wide, const GroupArgs& a, uint32_t threads, size_t ldsBytes, hipStream_t s);

// Diagnostic row-gather probe: `waves` (a multiple of 4) wavefronts, each walking `perWave`
// (a multiple of 64) entries of idx (row numbers of a table of 32-float rows); `active` (1..8) of a
// wavefront's 8 lane groups take part in each load instruction.
hipError_t launch_probe_gather(const uint32_t* idx, uint64_t n, const float* table, float* sink,
                               uint32_t waves, uint32_t perWave, int active, hipStream_t s);

}  // namespace hbcsf

#endif  // HBCSF_DEVICE_H_
