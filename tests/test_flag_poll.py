"""The solver's flags in host memory (csrc/flag_poll.hpp) against a small stand-in for
the HIP runtime with two devices: the event belongs to the stream's device, memory is
freed behind the stream's work, and every failure falls back to the copy."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")

SOURCE = r"""
#include "flag_poll.hpp"
#include <stdio.h>
#include <string.h>

// A stream is a device number; an event remembers the device it was made on.
static int current = 0, stream_dev = 0, event_dev = -1, alloc_dev = -1;
static int launched = 0, recorded = 0, done = 0;  // launches: all, in front of the event, finished
static bool freed_early = false, fail_alloc = false, fail_event = false, fail_record = false;
static int live = 0, events = 0, copies = 0;
static double memory[4];

extern "C" {
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipSetDevice(int d) { current = d; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { *d = stream_dev; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t, unsigned) {
  if (fail_alloc) return hipErrorOutOfMemory;
  ++live; alloc_dev = current; *p = memory; return hipSuccess;
}
hipError_t hipHostFree(void*) { freed_early = freed_early || done < launched; --live; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  if (fail_event) return hipErrorOutOfMemory;
  ++events; event_dev = current; *e = reinterpret_cast<hipEvent_t>(&event_dev); return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { --events; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) {
  if (fail_record || event_dev != stream_dev) return hipErrorInvalidHandle;
  recorded = launched; return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { if (done < recorded) done = recorded; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { done = launched; return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  ++copies; memcpy(d, s, n); return hipSuccess;
}
}

int main() {
  int bad = 0;
  const auto check = [&](bool ok, const char* what) { if (!ok) { printf("wrong: %s\n", what); ++bad; } };
  for (int where = 0; where < 2; ++where)
    for (int fail = 0; fail < 5; ++fail) {
      current = 0; stream_dev = where; freed_early = false; copies = launched = recorded = done = 0;
      fail_alloc = fail == 1; fail_event = fail == 2; fail_record = fail == 3;
      {
        dsl::FlagPoll poll(4, fail != 4, reinterpret_cast<hipStream_t>(&stream_dev));
        check(current == 0, "the caller's device is current again");
        if (fail == 0) check(alloc_dev == where && event_dev == where, "memory and event on the stream's device");
        double active[4] = {1, 0, 1, 1}, got[4] = {9, 9, 9, 9};
        memcpy(memory, active, sizeof active);  // the launch
        ++launched;
        poll.mark();
        check(poll.read(active, got, 4) == hipSuccess, "flags read");
        check(!memcmp(active, got, sizeof got), "the launch's flags");
        check(copies == (fail ? 1 : 0), "copied only where the event cannot be had");
        ++launched;  // a launch behind which the solve fails, no mark
      }
      check(!freed_early, "freed while a kernel still writes");
      check(live == 0 && events == 0, "given back");
    }
  return bad != 0;
}
"""


def test_flag_poll(tmp_path):
    src, exe = tmp_path / "poll.cpp", tmp_path / "poll"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_1808_05506_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True, timeout=120)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout
