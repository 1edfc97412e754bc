// Stand-in for the HIP runtime calls that the library's host code makes, on host memory: copies are carried out at once, kernels are
// not run.  A chosen copy, launch or wait fails, and what the calls did is counted.  Loaded before the library, it takes the
// place of the runtime's functions of these names.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstring>

namespace {
long copies, waits, pending, into;
long failCopy, failWait;          // the how-manieth fails; 0: none
uintptr_t range[2];
void fillProperties(hipDeviceProp_t* p) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950");
  p->warpSize = 64;
  p->multiProcessorCount = 256;
  p->maxThreadsPerBlock = 1024;
}
}  // namespace

extern "C" {

// Counts from now on; the failCopy_-th copy and the failWait_-th wait fail.
void fake_start(long failCopy_, long failWait_) {
  copies = waits = pending = 0;
  failCopy = failCopy_;
  failWait = failWait_;
}
// Launches and copies enqueued since the last wait.
long fake_pending() { return pending; }// Counts pointers into [from, until) that the launches from now on are given: in the first 96 bytes of their arguments 0, 1 and 3,
// structures of pointers all of them (the launch that defines an MTTKRP's output itself).
void fake_range(const void* from, const void* until) {
  range[0] = (uintptr_t)from;
  range[1] = (uintptr_t)until;
  into = 0;
}
long fake_into() { return into; }

hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t* p, int) { fillProperties(p); return hipSuccess; }
int hipGetStreamDeviceId(hipStream_t) { return 0; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t) {
  if (++copies == failCopy) return hipErrorInvalidValue;
  ++pending;
  std::memcpy(to, from, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* to, int v, size_t n, hipStream_t) {
  ++pending;
  std::memset(to, v, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  pending = 0;
  return ++waits == failWait ? hipErrorUnknown : hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = *block = dim3(1, 1, 1);
  *lds = 0;
  *s = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void** args, size_t, hipStream_t) {
  ++pending;
  if (range[1] > range[0])
    for (int k : {0, 1, 3})
      for (int w = 0; w < 12; ++w) {
        uintptr_t p;
        std::memcpy(&p, (const char*)args[k] + 8 * w, 8);
        into += p >= range[0] && p < range[1];
      }
  return hipSuccess;
}

}  // extern "C"
