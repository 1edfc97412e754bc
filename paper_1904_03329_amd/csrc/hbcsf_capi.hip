// C-ABI layer: argument checks, device arena bookkeeping and kernel launches.

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "hbcsf.h"
#include "hbcsf_device.h"
#include "hbcsf_internal.h"
#include "hbcsf_tensor.h"

using namespace hbcsf;

namespace {

thread_local std::string g_err;

}  // namespace

namespace hbcsf {

int fail(int code, const std::string& msg) {
  g_err = msg;
  return code;
}

int fail_hip(hipError_t e, const char* what) {
  g_err = std::string(what) + ": " + hipGetErrorString(e);
  return HBCSF_EHIP;
}

int fail_exception() noexcept {
  int code = HBCSF_EINVAL;
  try {
    try {
      throw;
    } catch (const std::bad_alloc&) {
      code = HBCSF_ENOMEM;
      g_err = "out of host memory";
    } catch (const std::exception& e) {
      g_err = std::string("unexpected C++ exception: ") + e.what();
    } catch (...) {
      g_err = "unexpected C++ exception";
    }
  } catch (...) {
    g_err.clear();  // even the message could not be stored
  }
  return code;
}

uint64_t define_state_bytes(uint64_t rows) {
  return rows <= kDefineStateRows ? ((rows + 31) / 32 * 4 + kAlign - 1) / kAlign * kAlign : 0;
}

void size_arena(hbcsf_tensor* t) {
  uint64_t states = 0;
  t->formatBytes = 0;
  for (int m = 0; m < t->order; ++m) {
    if (!t->modes[m]) continue;
    ModeFormat& f = *t->modes[m];
    t->formatBytes += f.blobBytes;
    states += f.stateBytes = define_state_bytes(f.rows);
  }
  t->arenaBytes = t->formatBytes + states;
}

hipError_t clear_states(const hbcsf_tensor* t, uint8_t* at, hipStream_t s) {
  const uint64_t vecs = (t->arenaBytes - t->formatBytes) / 16;
  if (vecs == 0) return hipSuccess;
  return launch_zero_rows((float*)at, vecs, (uint32_t)(vecs < 256 * 1024 ? (vecs + 255) / 256 : 1024), s);
}

void use_states(hbcsf_tensor* t, uint8_t* at) {
  for (int m = 0; m < t->order; ++m) {
    if (!t->modes[m]) continue;
    t->modes[m]->state = at;
    at += t->modes[m]->stateBytes;
  }
}

void use_arena(hbcsf_tensor* t, uint8_t* arena) {
  uint8_t* at = arena;
  for (int m = 0; m < t->order; ++m) {
    if (!t->modes[m]) continue;
    t->modes[m]->dev = at;
    at += t->modes[m]->blobBytes;
  }
  use_states(t, at);
}

}  // namespace hbcsf

namespace {

bool pow2_in(uint32_t v, uint32_t lo, uint32_t hi) { return v >= lo && v <= hi && (v & (v - 1)) == 0; }

uint32_t round_up8(uint64_t v) { return (uint32_t)((v + 7) / 8 * 8); }

// Nonzeros a lane group takes of a unit, as a power of two: at most a run, at least what keeps a unit (NG parts) a whole
// number of runs.  Units of 256 nonzeros keep the most wavefronts resident (5 to 7 KB of LDS each) and were the
// fastest at every rank from 5 M nonzeros up (rank 8 on 42 M nonzeros 1.94 -> 1.10 ms against parts of whole runs, rank
// 16 on 7.7 M 237 -> 204 us, rank 32 on 5 M 241 -> 217 us).  Smaller tensors take 128 where there would be fewer than 16
// units of 256 per compute unit, and 64 below 3: a wavefront walks its part one dependent block after the other, so with
// the chip not full the length of that walk is the kernel's time (rank 32 on 80 000 nonzeros 67 -> 43 us, rank 8 on
// 10 000 60 -> 38 us, all modes).
uint32_t part_shift(uint64_t nnz, int NG, uint32_t lshift, int numCU) {
  uint32_t lo = 3, s = 3;
  while (((uint32_t)NG << lo) < (1u << lshift)) ++lo;
  while (((uint32_t)NG << s) < 256) ++s;
  const uint64_t units = nnz / ((uint64_t)NG << s);
  if (units < 16ull * (uint64_t)numCU) --s;
  if (units < 3ull * (uint64_t)numCU) --s;
  if (s < lo) s = lo;
  return s < lshift ? s : lshift;
}

// Single representation: mode-`mode` MTTKRP from mode 0's B-CSF tree, the target at tree level T >= 1.  The
// output is zero-filled, then every level-T segment (T = leaf: every nonzero) adds its contribution atomically.
int mttkrp_from_mode0(const hbcsf_tensor* t, int mode, int rank, const float* const* factors, float* out,
                      hipStream_t s) {
  if (rank != 32) return fail(HBCSF_EINVAL, "single representation: modes other than 0 need rank 32");
  if (!factors[0]) return fail(HBCSF_EINVAL, "a factor pointer is null");
  const ModeFormat& f = *t->modes[0];
  const int N = t->order;
  const int G = 8, NG = 8;
  int level = 0;
  for (int l = 1; l < N; ++l)
    if (f.levelMode[l] == mode) level = l;
  if (level == 0) return fail(HBCSF_EINVAL, "mode out of range");
  const uint8_t* base = f.dev;
  const GroupFormat& gf = f.g[kCsf];
  const uint64_t nvec = t->dims[mode] * (uint64_t)G;
  uint64_t zb = (nvec + 255) / 256;
  const uint64_t cap = (uint64_t)t->numCU * 32;
  if (zb > cap) zb = cap;
  if (zb == 0) zb = 1;
  hipError_t e = launch_zero_rows(out, nvec, (uint32_t)zb, s);
  if (e != hipSuccess) return fail_hip(e, "launch of the zero-fill kernel");
  if (gf.nnz == 0) return HBCSF_OK;
  GroupArgs a;
  std::memset(&a, 0, sizeof(a));
  bool wide = false;
  for (int l = 0; l < N; ++l) {
    a.ind[l] = gf.ind[l].present ? (const uint32_t*)(base + gf.ind[l].off) : nullptr;
    a.ptr[l] = gf.ptr[l].present ? (const uint32_t*)(base + gf.ptr[l].off) : nullptr;
    a.runFirst[l] = gf.runFirst[l].present ? (const uint32_t*)(base + gf.runFirst[l].off) : nullptr;
    a.fac[l] = l == level ? nullptr : factors[f.levelMode[l]];
    if (l != level) wide = wide || t->dims[f.levelMode[l]] * (uint64_t)rank * 4ull >= (1ull << 32);
  }
  uint32_t lshift = 0;
  while ((1u << lshift) < f.L) ++lshift;
  a.val = (const float*)(base + gf.val.off);
  a.out = out;
  a.nnz = (uint32_t)gf.nnz;
  a.runs = (uint32_t)gf.runs;
  a.lshift = lshift;
  a.partShift = lshift;
  a.nUnits = (uint32_t)((gf.runs + NG - 1) / NG);
  const uint64_t target = (uint64_t)t->numCU * (t->wavesPerCU ? t->wavesPerCU : 128);
  uint64_t upw = t->sliceThreshold ? t->sliceThreshold / ((uint64_t)NG * f.L) : (a.nUnits + target - 1) / target;
  if (upw == 0) upw = 1;
  a.unitsPerWave = (uint32_t)upw;
  a.nSpans = (uint32_t)((a.nUnits + upw - 1) / upw);
  const int RW = N == 3 ? 4 : 8;
  const size_t ldsWave = (size_t)NG * (f.L + 1) * RW * 4;
  int wpb = 4;
  while (wpb > 1 && ldsWave * wpb > 48 * 1024) wpb >>= 1;
  const uint32_t threads = 64 * wpb;
  e = N == 3   ? launch_nonroot_n3(level, wide, a, threads, ldsWave * wpb, s)
      : N == 4 ? launch_nonroot_n4(level, wide, a, threads, ldsWave * wpb, s)
               : launch_nonroot_n5(level, wide, a, threads, ldsWave * wpb, s);
  if (e != hipSuccess) return fail_hip(e, "launch of the single-representation kernel");
  return HBCSF_OK;
}

}  // namespace

extern "C" {

int hbcsf_build_format(int order, const uint64_t* dims, uint64_t nnz, const uint32_t* const* inds,
                       const float* vals, const hbcsf_opts* opts, hbcsf_tensor** out) try {
  if (!out) return fail(HBCSF_EINVAL, "out is null");
  *out = nullptr;
  if (order < 3 || order > HBCSF_MAX_ORDER) return fail(HBCSF_EINVAL, "order must be 3, 4 or 5");
  if (!dims) return fail(HBCSF_EINVAL, "dims is null");
  if (nnz > 0 && (!inds || !vals)) return fail(HBCSF_EINVAL, "inds or vals is null");
  if (nnz >= 0xffff0000ull) return fail(HBCSF_ERANGE, "nnz must be below 2^32 - 2^16");
  for (int m = 0; m < order; ++m) {
    if (dims[m] == 0 || dims[m] > 0x7ffffffeull) return fail(HBCSF_ERANGE, "each dimension must be in 1 .. 2^31-2");
    if (nnz > 0 && !inds[m]) return fail(HBCSF_EINVAL, "an index array is null");
  }
  hbcsf_opts o{};
  if (opts) o = *opts;
  if (o.fiber_threshold == 0) o.fiber_threshold = default_fiber_threshold(order);
  if (!pow2_in(o.fiber_threshold, 8, 64)) return fail(HBCSF_EINVAL, "fiber_threshold must be 8, 16, 32 or 64");
  if (o.mode_order_policy > 2) return fail(HBCSF_EINVAL, "mode_order_policy must be 0, 1 or 2");
  if (o.group_mask > 4) return fail(HBCSF_EINVAL, "group_mask must be 0..4");
  if (o.hybrid_granularity > 1) return fail(HBCSF_EINVAL, "hybrid_granularity must be 0 or 1");
  if (o.coo_row_flags > 1) return fail(HBCSF_EINVAL, "coo_row_flags must be 0 or 1");
  if (o.mid_blocking > 13) return fail(HBCSF_EINVAL, "mid_blocking must be 0 or 1 (off) or 2..13 bits");
  if (o.single_representation > 1) return fail(HBCSF_EINVAL, "single_representation must be 0 or 1");
  if (o.single_representation) {
    if ((opts->fiber_threshold && opts->fiber_threshold != default_fiber_threshold(order)) || o.group_mask ||
        o.hybrid_granularity || o.coo_row_flags || o.mid_blocking > 1)
      return fail(HBCSF_EINVAL, "single_representation goes with default options only");
    o.group_mask = 4;  // plain B-CSF: the kernel for the other modes walks one group
  }
  std::unique_ptr<hbcsf_tensor> t(new (std::nothrow) hbcsf_tensor);
  if (!t) return fail(HBCSF_ENOMEM, "out of host memory");
  t->order = order;
  t->nnz = nnz;
  t->opts = o;
  t->sliceThreshold = o.slice_threshold;
  for (int m = 0; m < order; ++m) t->dims[m] = dims[m];
  t->normSq = sum_of_squares(vals, nnz);
  t->single = o.single_representation == 1;
  const int nModes = t->single ? 1 : order;
  ModeFormat* formats[HBCSF_MAX_ORDER];
  for (int m = 0; m < nModes; ++m) {
    t->modes[m].reset(new (std::nothrow) ModeFormat);
    if (!t->modes[m]) return fail(HBCSF_ENOMEM, "out of host memory");
    formats[m] = t->modes[m].get();
  }
  std::string err;
  const int rc = build_modes(order, dims, nnz, inds, vals, o, nModes, formats, &err);
  if (rc != HBCSF_OK) return fail(rc, err);
  size_arena(t.get());
  *out = t.release();
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_device_bytes(const hbcsf_tensor* t, uint64_t* bytes) try {
  if (!t || !bytes) return fail(HBCSF_EINVAL, "null argument");
  *bytes = t->arenaBytes;
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_upload(hbcsf_tensor* t, void* device_arena, uint64_t bytes, void* hip_stream) try {
  if (!t || !device_arena) return fail(HBCSF_EINVAL, "null argument");
  const int nModes = t->single ? 1 : t->order;
  for (int m = 0; m < nModes; ++m)
    if (!t->modes[m]->blob) return fail(HBCSF_ESTATE, "the format was built on the device: it is already resident");
  if (bytes < t->arenaBytes) return fail(HBCSF_ENOMEM, "device arena is smaller than hbcsf_device_bytes");
  if (((uintptr_t)device_arena & (kAlign - 1)) != 0) return fail(HBCSF_EINVAL, "device arena must be 256-byte aligned");
  hipStream_t s = (hipStream_t)hip_stream;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  int cu = 0;
  e = hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return fail_hip(e, "hipDeviceGetAttribute");
  WaitOnError wait(s);
  uint8_t* at = (uint8_t*)device_arena;
  for (int m = 0; m < nModes; ++m) {
    const ModeFormat& f = *t->modes[m];
    e = hipMemcpyAsync(at, f.blob, f.blobBytes, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return fail_hip(e, "hipMemcpyAsync");
    at += f.blobBytes;
  }
  e = clear_states(t, at, s);
  if (e != hipSuccess) return fail_hip(e, "launch of the zero-fill kernel");
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
  wait.done();
  t->numCU = cu > 0 ? cu : 256;
  t->device = dev;
  use_arena(t, (uint8_t*)device_arena);
  t->uploaded = true;
  return HBCSF_OK;
} HBCSF_CATCH_ALL

}  // extern "C"

namespace {

// Some gathered factor matrix needs 64-bit row addressing (marks address one row further on, hence the + rowBytes); fiber
// levels gathered with streaming loads take the wide form too.
bool needs_wide(const hbcsf_tensor* t, const ModeFormat& f, uint64_t rowBytes) {
  for (int l = 1; l < t->order; ++l) {
    const uint64_t bytes = t->dims[f.levelMode[l]] * rowBytes;
    if (bytes + rowBytes >= (1ull << 32) || (l < t->order - 1 && bytes >= t->streamBytes)) return true;
  }
  return false;
}

// 8 gathers in flight with parts of whole runs: at order 3 and runs of 64 four wavefronts per SIMD instead of five, but
// half the staging per nonzero.  Pays there with rows of 128 bytes, narrow factor matrices and a stream that fills the
// chip many times over, 25 M nonzeros on 256 compute units (100 M nonzeros 2.15 -> 2.03 ms, 30 M 867 -> 841 us, 25 M 735 ->
// 727 and 926 -> 926, 20 M 578 -> 579 and 496 -> 480, 12 M 370 -> 381, 5 M 181 -> 221; rank 16 in fp64, medians over three
// index laws whose runs differ by 2 to 4 %: 60 M 1514 -> 1490, 1506 -> 1475 and 1407 -> 1361, 30 M 819 -> 829, 814 -> 796 and
// 768 -> 766, 25 M 709 -> 717, 693 -> 677 and 665 -> 660, 20 M 587 -> 601, 572 -> 562 and 543 -> 546); at other run lengths
// and orders only where the tuning key asks.
bool long_parts(const hbcsf_tensor* t, const ModeFormat& f, int G, uint32_t lshift, bool wide) {
  if (G != 8 || t->steps == 8) return G == 8;
  return t->steps == 0 && t->order == 3 && lshift == 6 && !wide && f.g[kCsl].nnz + f.g[kCsf].nnz >= 97656ull * (uint64_t)t->numCU;
}

// Is the output defined in the launch of the group kernels?  That saves a launch, 1.4 to 5 us, and costs the group kernels the
// code that asks for rows, 1 to 4 % of a launch.  So: at most 8192 nonzeros per compute unit (2 M on 256 of them), at order 3
// rows of up to 1 GiB together (8 M at rank 32); all modes, launch of its own -> here, rank 32: order 3 on 0.3 M 43 -> 37 us,
// 4 M 155 -> 147, 8 M 260 -> 255 (fp64 4 M 254 -> 249, 8 M 441 -> 445); order 4 on 0.3 M 57 -> 45, 1.5 M 130 -> 120, 8 M 422 ->
// 423 (rank 8 273 -> 278), 50 M 2435 -> 2485; order 5 on 1.5 M 182 -> 172, 8 M 766 -> 775.  And no more words of 32 rows than
// the first blocks have wavefronts, 16 MiB at most: the zeros go through the L2 8 bytes a lane, and who comes early waits for
// them (modes of 300 000 and 100 000 rows, rank 32 on 0.3 M 73 -> 77, rank 128 on 30 000 102 -> 114).  (Figures without a law
// are of skewed indices; uniform ones gain as much: order 3 on 0.3 M, ranks 8 / 32 / 128, 36.6 -> 27.5, 41.8 -> 31.0, 117 -> 92.5,
// by Zipf's law of 1.2 31.6 -> 25.5, 35.9 -> 26.2, 80.3 -> 56.9.)
// Those wavefronts come before the ones that walk the nonzeros.  That is no loss
//  - while they are few, up to 9 / 16 of what the chip holds of this kernel, 101 376 rows at order 3 and 82 944 at 4 and 5 (two modes of
//    65 001 rows, rank 32, indices by Zipf's law of 1.2: 0.3 M 38.4 -> 32.7, 1 M 62.2 -> 56.2),
//  - with many nonzeros a row to make up for it (131 001 rows: 2 M 94.3 -> 91.7, 3.5 M 132.8 -> 130.9),
//  - at order 3 where half of the rows or more are stored by their slices and need no zeros (uniform indices, 131 001 rows: 0.6 M
//    72.7 -> 63.8, 1 M 94.8 -> 88.7; by Zipf's law, where they are not, 0.3 M 40.5 -> 43.9, 1 M 63.6 -> 65.5; order 4, uniform,
//    rank 8 on 0.3 M 58 -> 68),
//  - where all find room at once and write 8 MiB at most (131 001 rows, rank 8: 0.3 M 34.4 -> 33.4, but 0.6 M 39.3 -> 41.9), or
//    where few of the rows are added to (110 001 rows, rank 32: 0.1 M 31.1 -> 29.6, but 0.2 M 34.5 -> 37.8).
constexpr uint64_t kDefineBlocksPerCU = 4;   // (with one the words are late: 5 M 180 -> 190 us)
bool defines_here(const hbcsf_tensor* t, const ModeFormat& f, uint64_t nnz, uint64_t rowBytes, int NG, uint32_t lshift) {
  const uint64_t cus = (uint64_t)t->numCU, all = t->nnz;
  if (f.stateBytes == 0 || nnz == 0 || f.rows > 32 * 4 * kDefineBlocksPerCU * cus || f.rows * rowBytes > (16ull << 20)) return false;
  if (nnz > 8192 * cus && (t->order != 3 || nnz * rowBytes > (4ull << 20) * cus)) return false;
  const uint64_t room = (t->order == 3 ? 22 : 18) * cus;   // wavefronts
  const uint64_t words = (f.rows + 31) / 32;
  if (16 * words <= 9 * room || all >= 15 * f.rows) return true;
  if (t->order == 3 && 2 * f.stats.owned_rows >= f.rows) return true;
  const uint64_t unit = (uint64_t)NG << part_shift(all, NG, lshift, t->numCU);
  return words + (all + unit - 1) / unit <= room && (f.rows * rowBytes <= (8ull << 20) || all <= f.rows);
}

// Takes the turn of the mode's words of state for a call on stream s, where that is the stream they serve
// (hbcsf_tensor::DefineTurn): the lock is then held, and `claimed` is what the call marks words with.
bool take_turn(const hbcsf_tensor* t, int mode, hipStream_t s, std::unique_lock<std::mutex>* held, uint32_t* claimed) {
  int device = -1;
  if (s != nullptr || hipGetDevice(&device) != hipSuccess || device != t->device) return false;
  hbcsf_tensor::DefineTurn& turn = t->turns[mode];
  std::unique_lock<std::mutex> lock(turn.lock);
  if (turn.call >= 0x7ffffff0u) return false;   // the marks would start again at 0
  *claimed = 2 * ++turn.call + 1;
  *held = std::move(lock);
  return true;
}

// The MTTKRP of both element types: `elem` = bytes per element of the factor matrices and the output (4: fp32,
// 8: fp64; the tensor's values are fp32 either way).  The kernels see a row as G = rank * elem / 16 lanes of 16 bytes
// and GroupArgs' float pointers as row addresses, so everything below the launch dispatch is shared.
int mttkrp_any(const hbcsf_tensor* t, int mode, int rank, int elem, const float* const* factors, float* out,
               void* hip_stream, const GuestArgs* guest = nullptr) {
  if (!t || !factors || !out) return fail(HBCSF_EINVAL, "null argument");
  if (mode < 0 || mode >= t->order) return fail(HBCSF_EINVAL, "mode out of range");
  const bool f64 = elem == 8;
  if (!f64 && !(rank == 8 || rank == 16 || rank == 32 || rank == 64 || rank == 128))
    return fail(HBCSF_EINVAL, "rank must be 8, 16, 32, 64 or 128");
  if (f64 && !(rank == 16 || rank == 32 || rank == 64)) return fail(HBCSF_EINVAL, "fp64: rank must be 16, 32 or 64");
  if (f64 && t->single) return fail(HBCSF_EINVAL, "fp64: the single-representation variant is fp32 only");
  if (!t->uploaded) return fail(HBCSF_ESTATE, "hbcsf_upload has not been called");
  if (((uintptr_t)out & 15) != 0) return fail(HBCSF_EINVAL, "out must be 16-byte aligned");
  for (int m = 0; m < t->order; ++m) {
    if (m == mode) continue;
    if (!factors[m]) return fail(HBCSF_EINVAL, "a factor pointer is null");
    if (((uintptr_t)factors[m] & 15) != 0) return fail(HBCSF_EINVAL, "factors must be 16-byte aligned");
  }
  if (t->single && mode != 0) return mttkrp_from_mode0(t, mode, rank, factors, out, (hipStream_t)hip_stream);
  const ModeFormat& f = *t->modes[mode];
  const int N = t->order;
  const int G = rank * elem / 16;
  const int NG = 64 / G;
  const uint32_t L = f.L;
  uint32_t lshift = 0;
  while ((1u << lshift) < L) ++lshift;
  hipStream_t s = (hipStream_t)hip_stream;
  const uint8_t* base = f.dev;
  const uint64_t rowBytes = (uint64_t)rank * (uint64_t)elem;
  hipError_t e;

  hbcsf_tensor::EventSet* es = nullptr;
  if (!t->ring.empty()) {
    es = &t->ring[t->calls % t->ring.size()];
    es->valid = false;
    e = hipEventRecord(es->ev[0], s);
    if (e != hipSuccess) return fail_hip(e, "hipEventRecord");
  }

  auto group_args = [&](int g) {
    const GroupFormat& gf = f.g[g];
    GroupArgs a;
    std::memset(&a, 0, sizeof(a));
    for (int l = 0; l < N; ++l) {
      a.ind[l] = gf.ind[l].present ? (const uint32_t*)(base + gf.ind[l].off) : nullptr;
      a.ptr[l] = gf.ptr[l].present ? (const uint32_t*)(base + gf.ptr[l].off) : nullptr;
      a.runFirst[l] = gf.runFirst[l].present ? (const uint32_t*)(base + gf.runFirst[l].off) : nullptr;
      a.fac[l] = l == 0 ? nullptr : factors[f.levelMode[l]];
    }
    return a;
  };
  const bool wide = needs_wide(t, f, rowBytes);

  const uint64_t sparseNnz = f.g[kCsl].nnz + f.g[kCsf].nnz;
  const bool dense = t->denseMid == 1 && dense_mid_available(N, G, lshift);
  const bool longParts = long_parts(t, f, G, lshift, wide);
  // 0. small outputs are defined in the launch of the group kernels, unless a kernel without that is asked for or needed,
  //    slices are stored in pieces (which add to rows in the middle of a part), or the stream is not the one that the
  //    mode's words of state serve
  std::unique_lock<std::mutex> turn;
  DefineArgs here{};
  const bool oneLaunch = defines_here(t, f, sparseNnz, rowBytes, NG, lshift) && t->fuseCoo == 2 && t->opts.hybrid_granularity == 0 &&
                         f.blockBits == 0 && t->kernelMask == 15u && !es && !dense && !longParts && !wide && !t->persistent &&
                         take_turn(t, mode, s, &turn, &here.claimed);
  if (oneLaunch) {
    const GroupArgs coo = group_args(kCoo);
    for (int l = 0; l < N; ++l) here.ind[l] = coo.ind[l];
    here.val = (const float*)(base + f.g[kCoo].val.off);
    here.ownedBits = (const uint32_t*)(base + f.ownedBits.off);
    here.cooBits = (const uint32_t*)(base + f.cooBits.off);
    here.cooPtr = (const uint32_t*)(base + f.cooPtr.off);
    here.rows = (uint32_t)f.rows;
    here.state = (uint32_t*)f.state;
    here.blocks = round_up8((f.rows + 127) / 128);   // a word a wavefront
  }

  // 1. define every output row that no plain store will write; the COO group's rows are written
  //    in the same pass
  // (measured: the fused pass saves a launch on small outputs but hides latency worse on large ones)
  // (without stored root indices only the fused pass can place the COO group's rows)
  const bool wantFuse = f.cooRowFlags || t->fuseCoo == 1 ||
                        (t->fuseCoo == 2 && f.rows * rowBytes <= (64ull << 20));
  unsigned long long* const stamp = guest ? guest->stamp : nullptr;
  const bool fuseCoo = oneLaunch || (wantFuse && (t->kernelMask & 3u) == 3u && f.g[kCoo].nnz > 0);
  if ((t->kernelMask & 1u) && !oneLaunch) {
    // one wavefront per 8 x 32 rows, capped at 64 wavefronts per compute unit
    uint64_t blocks = ((f.rows + 255) / 256 + 3) / 4;
    const uint64_t cap = (uint64_t)t->numCU * 16;
    if (blocks > cap) blocks = cap;
    if (blocks == 0) blocks = 1;
    if (fuseCoo) {
      blocks = ((f.rows + 31) / 32 + 3) / 4;  // the fused pass takes one 32-row word per wavefront iteration
      if (blocks > cap) blocks = cap;
      if (blocks == 0) blocks = 1;
      GroupArgs a = group_args(kCoo);
      a.val = (const float*)(base + f.g[kCoo].val.off);
      a.out = out;
      a.nnz = (uint32_t)f.g[kCoo].nnz;
      e = launch_define_coo(f64, N, G, wide, a, (const uint32_t*)(base + f.ownedBits.off),
                            (const uint32_t*)(base + f.cooBits.off), (const uint32_t*)(base + f.cooPtr.off),
                            f.rows, (uint32_t)blocks, stamp, s);
    } else {
      e = launch_define(out, (const uint32_t*)(base + f.ownedBits.off), f.rows, G, (uint32_t)blocks, stamp, s);
    }
    if (e != hipSuccess) return fail_hip(e, "launch of the output-definition kernel");
    if (es) es->launched[0] = true;
  } else if (es) {
    es->launched[0] = false;
  }
  if (es) (void)hipEventRecord(es->ev[1], s);

  // 2. the three group kernels (execute step of Algorithm "HB-CSF-MTTKRP")
  const bool runCsl = f.g[kCsl].nnz > 0 && (t->kernelMask & 4u), runCsf = f.g[kCsf].nnz > 0 && (t->kernelMask & 8u);
  const int denseSteps = t->steps ? t->steps : N == 3 ? 8 : 4;
  // CSL and B-CSF group in one launch, unless their times are asked for one by one (or the kernel with 8 gathers
  // is used: with both bodies in it, it no longer fits four wavefronts per SIMD)
  const bool together = guest || oneLaunch || (runCsl && runCsf && !es && !dense && !longParts && !t->persistent);
  auto sparse_args = [&](int g, uint32_t part) {
    const GroupFormat& gf = f.g[g];
    GroupArgs a = group_args(g);
    a.val = (const float*)(base + gf.val.off);
    a.out = out;
    a.nnz = (uint32_t)gf.nnz;
    a.runs = (uint32_t)gf.runs;
    a.lshift = lshift;
    a.trace = t->trace;
    a.traceCapacity = (uint32_t)t->traceCapacity;
    // B-CSF tuning variant: the fiber-level rows gathered densely through an LDS row cache (off by default:
    // it lowered the vector-memory instruction count as intended but lengthened every block's dependent chain
    // and measured 40-100 % slower on the benchmark tensors)
    a.denseMid = g == kCsf && dense ? 1u : 0u;
    a.partShift = part;
    const uint64_t unitNnz = (uint64_t)NG << part;
    a.nUnits = (uint32_t)((gf.nnz + unitNnz - 1) / unitNnz);
    // Spans: one unit while that gives at most 256 wavefronts per compute unit (6 M to 16 M nonzeros: with two 372 instead
    // of 369 us on 12 M), then two, since the run-table entries of a second unit are there when the first is done (20 M:
    // 577 instead of 584 us, 50 M of order 4 2400 instead of 2513), and more only beyond 512 wavefronts per compute unit
    // (150 M: 9050 us at 128 of them, 8959 at 256, 8822 at 512, 8791 at 1024; 100 M with parts of whole runs 2101, 2041,
    // 2032, 2079).
    const uint64_t cus = (uint64_t)t->numCU, target = cus * (t->wavesPerCU ? t->wavesPerCU : 512);
    uint64_t upw = t->sliceThreshold ? t->sliceThreshold / unitNnz : (a.nUnits + target - 1) / target;
    if (!t->sliceThreshold && !t->wavesPerCU && a.nUnits > 256 * cus && upw < 2) upw = 2;
    if (upw == 0) upw = 1;
    a.unitsPerWave = (uint32_t)upw;
    a.nSpans = (uint32_t)((a.nUnits + upw - 1) / upw);
    a.persistent = t->persistent ? 1u : 0u;
    if (g == kCsf)
      for (int l = 1; l < N - 1; ++l)
        if (t->dims[f.levelMode[l]] * rowBytes >= t->streamBytes) a.streamLevel |= 1u << l;
    return a;
  };
  for (int g = 0; g < 3; ++g) {
    const GroupFormat& gf = f.g[g];
    bool launched = false;
    if (g == kCoo) {
      if (gf.nnz > 0 && (t->kernelMask & 2u) && !fuseCoo && !f.cooRowFlags) {
        GroupArgs a = group_args(g);
        a.val = (const float*)(base + gf.val.off);
        a.out = out;
        a.nnz = (uint32_t)gf.nnz;
        const uint64_t perBlock = 64 * 4;  // 64 nonzeros per wavefront and iteration
        uint64_t b = (gf.nnz + perBlock - 1) / perBlock;
        const uint64_t cap = (uint64_t)t->numCU * 16;
        if (b > cap) b = cap;
        e = launch_group(f64, g, N, G, 4, wide, a, nullptr, nullptr, nullptr, round_up8(b), 256, 0, s);
        launched = true;
      }
    } else if (g == kCsl ? runCsl && !together : runCsf || guest || oneLaunch) {
      const uint32_t part = g == kCsf && dense ? lshift
                            : longParts ? lshift
                                        : part_shift(together ? sparseNnz : gf.nnz, NG, lshift, t->numCU);
      const GroupArgs a = sparse_args(g, part);
      GroupArgs csl;
      if (together) csl = sparse_args(kCsl, part);
      uint32_t words = g == kCsf ? csf_wave_words(N, G, (int)part, a.denseMid != 0) : 0u;
      if (g == kCsl || together) words = words > csl_wave_words(N, G, (int)part) ? words : csl_wave_words(N, G, (int)part);
      const size_t ldsWave = 4 * (size_t)words;
      int wpb = 4;
      while (wpb > 1 && ldsWave * wpb > 48 * 1024) wpb >>= 1;
      // the launcher sizes the grid
      e = launch_group(f64, g, N, G, a.denseMid ? denseSteps : longParts ? 8 : 4, wide, a, together ? &csl : nullptr,
                       oneLaunch ? &here : nullptr, guest, (uint32_t)t->numCU, 64 * wpb, ldsWave * wpb, s);
      launched = true;
    }
    if (launched && e != hipSuccess) return fail_hip(e, "launch of a group kernel");
    if (es) {
      es->launched[1 + g] = launched;
      (void)hipEventRecord(es->ev[2 + g], s);
    }
  }
  if (es) {
    es->valid = true;
    ++t->calls;
  }
  return HBCSF_OK;
}

}  // namespace

namespace hbcsf {

// The launch of the plain fp32 kernels with 4 gathers in flight takes a guest up to rank 64 (above, the inverse wants more
// threads than a block of theirs has); a tensor long enough for the other kernels hides nothing worth having.
bool mttkrp_takes_guest(const hbcsf_tensor* t, int mode, int rank) {
  if (rank > 64 || t->single || !t->ring.empty() || t->persistent || t->denseMid == 1 || t->kernelMask != 15u) return false;
  const ModeFormat& f = *t->modes[mode];
  uint32_t lshift = 0;
  while ((1u << lshift) < f.L) ++lshift;
  const bool wide = needs_wide(t, f, (uint64_t)rank * 4);
  return f.g[kCsl].nnz + f.g[kCsf].nnz > 0 && !wide && !long_parts(t, f, rank / 4, lshift, wide);
}

int mttkrp_with_guest(const hbcsf_tensor* t, int mode, int rank, const float* const* factors, float* out, const GuestArgs& guest,
                      hipStream_t s) {
  return mttkrp_any(t, mode, rank, 4, factors, out, (void*)s, &guest);
}

}  // namespace hbcsf

extern "C" {

int hbcsf_mttkrp(const hbcsf_tensor* t, int mode, int rank, const float* const* factors, float* out,
                 void* hip_stream) try {
  return mttkrp_any(t, mode, rank, 4, factors, out, hip_stream);
} HBCSF_CATCH_ALL

int hbcsf_mttkrp_f64(const hbcsf_tensor* t, int mode, int rank, const double* const* factors, double* out,
                     void* hip_stream) try {
  return mttkrp_any(t, mode, rank, 8, reinterpret_cast<const float* const*>(factors), reinterpret_cast<float*>(out),
                    hip_stream);
} HBCSF_CATCH_ALL

int hbcsf_get_stats(const hbcsf_tensor* t, int mode, hbcsf_stats* stats) try {
  if (!t || !stats) return fail(HBCSF_EINVAL, "null argument");
  if (mode < 0 || mode >= t->order) return fail(HBCSF_EINVAL, "mode out of range");
  if (t->single && mode != 0) return fail(HBCSF_ESTATE, "single representation: only mode 0 is stored");
  *stats = t->modes[mode]->stats;
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_host_array(const hbcsf_tensor* t, int mode, int group, int level, int array_id,
                     const void** ptr, uint64_t* count) try {
  if (!t || !ptr || !count) return fail(HBCSF_EINVAL, "null argument");
  if (mode < 0 || mode >= t->order) return fail(HBCSF_EINVAL, "mode out of range");
  if (t->single && mode != 0) return fail(HBCSF_ESTATE, "single representation: only mode 0 is stored");
  const ModeFormat& f = *t->modes[mode];
  const ArrayRef* r = nullptr;
  if (array_id == HBCSF_ARR_OWNED_BITS) {
    r = &f.ownedBits;
  } else if (array_id == HBCSF_ARR_COO_BITS) {
    r = &f.cooBits;
  } else if (array_id == HBCSF_ARR_COO_PTR) {
    r = &f.cooPtr;
  } else {
    if (group < 0 || group > 2 || level < 0 || level >= t->order) return fail(HBCSF_EINVAL, "group or level out of range");
    const GroupFormat& g = f.g[group];
    if (array_id == HBCSF_ARR_IND) r = &g.ind[level];
    else if (array_id == HBCSF_ARR_PTR) r = &g.ptr[level];
    else if (array_id == HBCSF_ARR_VAL) r = &g.val;
    else if (array_id == HBCSF_ARR_RUNFIRST) r = &g.runFirst[level];
  }
  if (!r || !r->present) return fail(HBCSF_EINVAL, "this group has no such array");
  if (!f.blob) return fail(HBCSF_ESTATE, "the format was built on the device: call hbcsf_download first");
  *ptr = f.blob + r->off;
  *count = r->count;
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_tune(hbcsf_tensor* t, int key, uint64_t value) try {
  if (!t) return fail(HBCSF_EINVAL, "null argument");
  if (key == HBCSF_TUNE_SLICE_THRESHOLD) {
    t->sliceThreshold = value;
    return HBCSF_OK;
  }
  if (key == HBCSF_TUNE_PROFILE) {
    if (value > 65536) return fail(HBCSF_EINVAL, "at most 65536 profiled calls are kept");
    for (auto& es : t->ring)
      for (int i = 0; i < 5; ++i) (void)hipEventDestroy(es.ev[i]);
    t->ring.clear();
    t->calls = 0;
    t->ring.resize((size_t)value);
    size_t made = 0;  // events created so far, in ring order
    for (auto& es : t->ring)
      for (int i = 0; i < 5; ++i, ++made) {
        hipError_t e = hipEventCreate(&es.ev[i]);
        if (e != hipSuccess) {
          for (size_t k = 0; k < made; ++k) (void)hipEventDestroy(t->ring[k / 5].ev[k % 5]);
          t->ring.clear();
          return fail_hip(e, "hipEventCreate");
        }
      }
    return HBCSF_OK;
  }
  if (key == HBCSF_TUNE_WAVES_PER_CU) {
    if (value > 1024) return fail(HBCSF_EINVAL, "waves per CU must be at most 1024");
    t->wavesPerCU = value;
    return HBCSF_OK;
  }
  if (key == HBCSF_TUNE_TRACE_BUFFER) {
    if (value & 7) return fail(HBCSF_EINVAL, "the trace buffer must be 8-byte aligned");
    t->trace = (unsigned long long*)(uintptr_t)value;
    if (!t->trace) t->traceCapacity = 0;
    return HBCSF_OK;
  }
  if (key == HBCSF_TUNE_TRACE_CAPACITY) {
    if (value > 0xffffffffull) return fail(HBCSF_EINVAL, "trace capacity too large");
    t->traceCapacity = value;
    return HBCSF_OK;
  }
  if (key == HBCSF_TUNE_STREAM_BYTES) {
    t->streamBytes = value ? value : ~0ull;  // 0 = never
    return HBCSF_OK;
  }
  if (key == HBCSF_TUNE_FUSE_COO) {
    if (value > 2) return fail(HBCSF_EINVAL, "fuse mode must be 0, 1 or 2");
    t->fuseCoo = (int)value;
    return HBCSF_OK;
  }
  if (key == HBCSF_TUNE_PERSISTENT) {
    t->persistent = value != 0;
    return HBCSF_OK;
  }
  if (key == HBCSF_TUNE_KERNEL_MASK) {
    if (value > 15) return fail(HBCSF_EINVAL, "kernel mask must be 0..15");
    t->kernelMask = (uint32_t)value;
    return HBCSF_OK;
  }
  if (key == HBCSF_TUNE_DENSE_MID) {
    if (value > 1) return fail(HBCSF_EINVAL, "dense-gather mode must be 0 or 1");
    t->denseMid = (int)value;
    return HBCSF_OK;
  }
  if (key == HBCSF_TUNE_STEPS) {
    if (value != 0 && value != 4 && value != 8) return fail(HBCSF_EINVAL, "steps must be 4 or 8, or 0 for the automatic choice");
    t->steps = (int)value;
    return HBCSF_OK;
  }
  return fail(HBCSF_EINVAL, "unknown tuning key");
} HBCSF_CATCH_ALL

int hbcsf_kernel_ms(hbcsf_tensor* t, uint32_t calls_back, float ms[4]) try {
  if (!t || !ms) return fail(HBCSF_EINVAL, "null argument");
  if (t->ring.empty() || calls_back >= t->ring.size() || calls_back >= t->calls)
    return fail(HBCSF_ESTATE, "no profiled hbcsf_mttkrp call that far back");
  const hbcsf_tensor::EventSet& es = t->ring[(t->calls - 1 - calls_back) % t->ring.size()];
  if (!es.valid) return fail(HBCSF_ESTATE, "that call did not complete its launches");
  hipError_t e = hipEventSynchronize(es.ev[4]);
  if (e != hipSuccess) return fail_hip(e, "hipEventSynchronize");
  for (int i = 0; i < 4; ++i) {
    ms[i] = 0.f;
    if (!es.launched[i]) continue;
    e = hipEventElapsedTime(&ms[i], es.ev[i], es.ev[i + 1]);
    if (e != hipSuccess) return fail_hip(e, "hipEventElapsedTime");
  }
  return HBCSF_OK;
} HBCSF_CATCH_ALL

int hbcsf_probe_row_gather(const uint32_t* idx, uint64_t n, const float* table, uint64_t table_rows,
                           int active_lane_groups, float* sink, void* hip_stream, uint64_t* rows_gathered,
                           uint64_t* load_instructions) try {
  if (!idx || !table || !sink || !rows_gathered) return fail(HBCSF_EINVAL, "null argument");
  if (active_lane_groups < 1 || active_lane_groups > 8) return fail(HBCSF_EINVAL, "active lane groups must be 1..8");
  if (table_rows == 0 || n < 64 * 1024) return fail(HBCSF_EINVAL, "need a table and at least 65536 indices");
  int dev = 0, cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  e = hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return fail_hip(e, "hipDeviceGetAttribute");
  uint64_t waves = (uint64_t)(cu > 0 ? cu : 256) * 64;
  uint64_t perWave = n / waves / 64 * 64;
  while (perWave == 0 && waves > 4) {
    waves /= 2;
    perWave = n / waves / 64 * 64;
  }
  waves = waves / 4 * 4;
  if (perWave == 0 || waves == 0) return fail(HBCSF_EINVAL, "too few indices");
  e = launch_probe_gather(idx, n, table, sink, (uint32_t)waves, (uint32_t)perWave, active_lane_groups,
                          (hipStream_t)hip_stream);
  if (e != hipSuccess) return fail_hip(e, "launch of the gather probe");
  *rows_gathered = waves * perWave / 8 * (uint64_t)active_lane_groups;
  if (load_instructions) *load_instructions = waves * perWave / 8;  // row loads: one per 8 index entries walked
  return HBCSF_OK;
} HBCSF_CATCH_ALL

void hbcsf_free(hbcsf_tensor* t) {
  if (!t) return;
  for (auto& es : t->ring)
    for (int i = 0; i < 5; ++i) (void)hipEventDestroy(es.ev[i]);
  delete t;
}

const char* hbcsf_strerror(int code) {
  switch (code) {
    case HBCSF_OK: return "ok";
    case HBCSF_EINVAL: return "invalid argument";
    case HBCSF_ERANGE: return "index or size out of range";
    case HBCSF_ENOMEM: return "out of memory or arena too small";
    case HBCSF_ESTATE: return "call out of order";
    case HBCSF_EHIP: return "HIP call failed";
    default: return "unknown error code";
  }
}

const char* hbcsf_last_error(void) { return g_err.c_str(); }

}  // extern "C"
