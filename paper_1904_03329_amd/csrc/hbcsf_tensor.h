// The tensor handle behind the C ABI, shared by the translation units that implement its entry points.
#pragma once

#include <hip/hip_runtime.h>

#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "hbcsf.h"
#include "hbcsf_internal.h"

struct hbcsf_tensor {
  int order = 0;
  uint64_t dims[HBCSF_MAX_ORDER] = {};
  uint64_t nnz = 0;
  double normSq = 0.0;  // sum of the squared values (for the CPD fit)
  hbcsf_opts opts{};
  std::unique_ptr<hbcsf::ModeFormat> modes[HBCSF_MAX_ORDER];
  uint64_t arenaBytes = 0;   // device memory of it all: the formats, then the launches' words of state
  uint64_t formatBytes = 0;  // of these, the formats'
  bool uploaded = false;
  bool single = false;       // only modes[0] exists; the other modes are computed from it (single representation)
  int numCU = 256;
  int device = -1;           // the device memory's
  uint64_t sliceThreshold = 0;
  uint64_t wavesPerCU = 0;   // launch sizing override, 0 = default
  int steps = 0;             // records in flight per lane group, 0 = automatic
  uint32_t kernelMask = 15;  // bit0 define, bit1 COO, bit2 CSL, bit3 CSF
  bool persistent = false;   // resident wavefronts walk the spans round-robin
  int denseMid = 0;          // B-CSF fiber-row gather through an LDS row cache (tuning variant): 0 off, 1 on
  int fuseCoo = 2;           // COO-group rows written by the output-definition pass: 0 never, 1 always, 2 small outputs
  uint64_t streamBytes = 1ull << 30;  // fiber-level factors at least this large are gathered with streaming loads
  unsigned long long* trace = nullptr;  // caller's device buffer for wavefront traces
  uint64_t traceCapacity = 0;
  // Calls that define the output in the launch that adds to it, per mode.  The words of state in the arena serve one call at a
  // time, so such calls are those on the null stream of the arena's device: there they follow each other, whichever threads
  // make them, and the stream is never destroyed nor captured.  A call on another stream defines the output in a launch of
  // its own, without state.  `lock`: a call's number and its launch go together.
  struct DefineTurn {
    std::mutex lock;
    uint32_t call = 0;
  };
  mutable DefineTurn turns[HBCSF_MAX_ORDER];
  // profiling: a ring of event sets, one per hbcsf_mttkrp call
  struct EventSet {
    hipEvent_t ev[5];
    bool launched[4] = {false, false, false, false};
    bool valid = false;
  };
  // hbcsf_mttkrp takes a const handle; recording a profiled call is bookkeeping, not state of the tensor
  mutable std::vector<EventSet> ring;
  mutable uint64_t calls = 0;  // profiled calls so far
};

namespace hbcsf {

// Records the message hbcsf_last_error returns on this thread and passes the code through.
int fail(int code, const std::string& msg);
int fail_hip(hipError_t e, const char* what);
// For the handler of an entry point's function-try-block: turns the exception in flight into an error code
// (std::bad_alloc -> HBCSF_ENOMEM, anything else -> HBCSF_EINVAL with its text) and never throws itself.
int fail_exception() noexcept;

// Waits for the stream when a call ends early, by an error or an exception: the memory that was to be written is then the
// caller's again, and what was enqueued must not reach it later.
class WaitOnError {
 public:
  explicit WaitOnError(hipStream_t s) : s_(s) {}
  WaitOnError(const WaitOnError&) = delete;
  WaitOnError& operator=(const WaitOnError&) = delete;
  ~WaitOnError() {
    if (!done_) (void)hipStreamSynchronize(s_);
  }
  void done() { done_ = true; }   // nothing is left on the stream

 private:
  hipStream_t s_;
  bool done_ = false;
};

// Bytes of the words of state (DefineArgs) of a mode with that many rows.
uint64_t define_state_bytes(uint64_t rows);
// Sets the sizes of the words of state and of the whole, once the formats' are known.
void size_arena(hbcsf_tensor* t);
// Clears words of state at `at` (one mode's behind the other's), which the tensor does not use yet.
hipError_t clear_states(const hbcsf_tensor* t, uint8_t* at, hipStream_t s);
// Makes the tensor use them, or an arena that holds the formats, one mode's behind the other's, and then them: only once all of
// that memory is written, so that a call which fails before leaves the tensor where it was.
void use_states(hbcsf_tensor* t, uint8_t* at);
void use_arena(hbcsf_tensor* t, uint8_t* arena);

// hbcsf_mttkrp with ALS work in the same launch, for calls that take it (fp32).
struct GuestArgs;
bool mttkrp_takes_guest(const hbcsf_tensor* t, int mode, int rank);
int mttkrp_with_guest(const hbcsf_tensor* t, int mode, int rank, const float* const* factors, float* out, const GuestArgs& guest,
                      hipStream_t s);

}  // namespace hbcsf

// Every entry point that returns an error code is a function-try-block closed by this handler, so that no C++
// exception (a failed allocation in a container, above all) crosses the C boundary.
#define HBCSF_CATCH_ALL catch (...) { return hbcsf::fail_exception(); }
