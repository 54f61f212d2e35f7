// The active flags of a CG iteration, read by the host while the iteration's last
// pass runs.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>

namespace dsl {

// The flags are in host memory that the device writes (CgScalars::flags); the host
// waits for an event behind the launch that writes them, and the next iteration is
// queued before the last pass ends.  Allocated per solve; not used (host == nullptr)
// where the solve may not allocate or the allocation fails: the flags are then copied
// behind the last pass, and the device idles from its end until the host has seen
// them (even-odd solve, FP16 inner, 16^3 x 32, N_v = 12: 71.2 ms so, 63.6 with the event).
//
// An event can only be recorded on a stream of the device that it was made on, so
// memory and event are made with the stream's device current, which need not be the
// caller's.  The memory is freed after the stream has drained: a solve that fails
// between the launch and the event leaves a kernel behind that still writes to it.
struct FlagPoll {
  double* host = nullptr;
  hipEvent_t ev = nullptr;
  hipStream_t st;
  bool marked = false;
  FlagPoll(int nv, bool may_allocate, hipStream_t stream) : st(stream) {
    if (!may_allocate) return;
    int cur = -1, dev = -1;
    if (hipGetDevice(&cur) != hipSuccess || (st ? hipStreamGetDevice(st, &dev) : hipGetDevice(&dev)) != hipSuccess ||
        (cur != dev && hipSetDevice(dev) != hipSuccess)) {
      (void)hipGetLastError();
      return;
    }
    void* p = nullptr;
    if (hipHostMalloc(&p, size_t(nv) * sizeof(double), hipHostMallocDefault) == hipSuccess) {
      if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) == hipSuccess) {
        host = static_cast<double*>(p);
      } else {
        (void)hipGetLastError();
        (void)hipHostFree(p);
      }
    } else {
      (void)hipGetLastError();
    }
    if (cur != dev) (void)hipSetDevice(cur);
  }
  ~FlagPoll() {
    if (!host) return;
    (void)hipStreamSynchronize(st);
    (void)hipEventDestroy(ev);
    (void)hipHostFree(host);
  }
  FlagPoll(const FlagPoll&) = delete;
  FlagPoll& operator=(const FlagPoll&) = delete;
  // after the launch that writes the flags
  void mark() {
    marked = host && hipEventRecord(ev, st) == hipSuccess;
    if (host && !marked) (void)hipGetLastError();
  }
  // the flags in hact
  hipError_t read(const double* active, double* hact, int nv) {
    if (marked) {
      const hipError_t e = hipEventSynchronize(ev);
      if (e != hipSuccess) return e;
      for (int v = 0; v < nv; ++v) hact[v] = host[v];
      return hipSuccess;
    }
    const hipError_t e = hipMemcpyAsync(hact, active, size_t(nv) * sizeof(double), hipMemcpyDeviceToHost, st);
    return e != hipSuccess ? e : hipStreamSynchronize(st);
  }
};

}  // namespace dsl
