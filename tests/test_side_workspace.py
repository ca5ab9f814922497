"""The workspace of disc_backproject and disc_voxel_overlap (csrc/side_ws.h)
against a HIP runtime that only writes down its calls (CPU only): which
streams get a buffer, that uses of one are ordered on the device, and that
nothing waits, frees or allocates in a way that another stream or another
thread's graph capture would notice."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2603_03935_amd", "csrc", "side_ws.h")

HIP = r"""
#pragma once
#include <cstddef>
#include <atomic>
#include <string>
#include <mutex>
#include <thread>
#include <vector>
typedef struct Stream* hipStream_t;
typedef struct Event* hipEvent_t;
enum hipError_t { hipSuccess, hipErrorUnknown };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeThreadLocal, hipStreamCaptureModeRelaxed };
#define hipStreamPerThread ((hipStream_t)2)
#define hipEventDisableTiming 2
#define hipEventDisableSystemFence 4
inline std::mutex log_mu;
inline std::vector<std::string> calls;
inline void say(const std::string& s) { std::lock_guard<std::mutex> lk(log_mu); calls.push_back(s); }
inline std::string n(const void* p) { return std::to_string((size_t)p); }
inline thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
inline std::atomic<bool> capturing{false}, no_memory{false}, no_record{false}, malloc_waits{false}, in_malloc{false};
inline size_t next_id = 100, last_bytes = 0;
inline hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipMalloc(void** p, size_t b) {
  in_malloc = true;
  while (malloc_waits) std::this_thread::yield();
  if (no_memory) return hipErrorUnknown;
  *p = (void*)(next_id++);
  last_bytes = b;
  say(std::string(mode == hipStreamCaptureModeRelaxed ? "relaxed" : "strict") + " malloc " + n(*p));
  return hipSuccess;
}
inline hipError_t hipFree(void* p) { say("free " + n(p)); return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t s) { say("sync " + n(s)); return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { say("sync all"); return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)(next_id++); return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t s) {
  if (no_record) return hipErrorUnknown;
  say("record " + n(s));
  return hipSuccess;
}
inline hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) { say("wait " + n(s)); return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) { std::swap(*m, mode); return hipSuccess; }
"""

PROGRAM = r"""
#include "side_ws.h"
#include <cstdio>
#include <cstring>
using namespace disc::host;
static const hipStream_t A = (hipStream_t)10, B = (hipStream_t)11;
static int count(const char* what) {
  int c = 0;
  for (auto& s : calls) c += s.find(what) != std::string::npos;
  return c;
}
#define CHECK(x) do { if (!(x)) { std::printf("%s: %s\n", argv[1], #x); return 1; } } while (0)
int main(int argc, char** argv) {
  const std::string t = argv[1];
  auto use = [](hipStream_t s, size_t b) { SideLease l(s, b); if (l.ptr) say("kernels " + n(s)); return (void*)l.ptr; };
  if (t == "per_thread") {  // unordered streams under one handle
    CHECK(!use(hipStreamPerThread, 1000) && calls.empty());
    CHECK(use(A, 1000) && use(B, 1000) && use(A, 1000) != use(B, 1000));
  } else if (t == "reused_handle") {  // two uses of one handle, perhaps of two streams: device order by an event
    void* p = use(A, 1000);
    CHECK(p && use(A, 500) == p);
    const std::vector<std::string> want = {"kernels 10", "record 10", "wait 10", "kernels 10", "record 10"};
    calls.erase(calls.begin());
    CHECK(calls == want);
  } else if (t == "null_stream") {  // the one stream of its handle, never destroyed: its own order is enough
    void* p = use(nullptr, 1000);
    CHECK(p && use(nullptr, 500) == p && count("wait") == 0 && count("record") == 0 && count("sync") == 0);
  } else if (t == "growth") {  // a larger buffer while kernels use the smaller one
    void* p = use(A, 1000);
    const size_t first = last_bytes;
    void* q = use(A, first + 1);
    CHECK(p && q && p != q && last_bytes >= 2 * first);
    CHECK(use(A, 10) == q);
    CHECK(count("free") == 0 && count("sync") == 0);
    CHECK(count("wait 10") == 2 && count("record 10") == 3);
    release_side_ws();
    CHECK(count("free") == 2 && count("sync") == 1);
    CHECK(calls[calls.size() - 3] == "sync all");
    CHECK(use(A, 1000) != nullptr);
  } else if (t == "capture_elsewhere") {
    CHECK(use(A, 1000) && count("relaxed malloc") == 1 && mode == hipStreamCaptureModeGlobal);
  } else if (t == "no_buffer") {
    CHECK(!use(A, 0) && !use(A, ((size_t)128 << 20) + 1));
    capturing = true;
    CHECK(!use(A, 1000));
    capturing = false;
    no_memory = true;
    CHECK(!use(A, 1000));
    no_memory = false;
    CHECK(calls.empty() && use(A, 1000));
  } else if (t == "no_mark") {  // the end of a use cannot be marked: the next must not overtake it
    no_record = true;
    CHECK(use(A, 1000) && count("sync 10") == 1);
  } else if (t == "other_streams") {  // one stream's buffer grows while another's call goes on
    CHECK(use(B, 1000));
    malloc_waits = true;
    in_malloc = false;
    std::thread g([&] { use(A, 1000); });
    while (!in_malloc) std::this_thread::yield();
    std::atomic<bool> done{false};
    std::thread b([&] { use(B, 1000); done = true; });
    for (int i = 0; i < 2000 && !done; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    const bool went = done;
    malloc_waits = false;
    g.join();
    b.join();
    CHECK(went);
  } else {
    return 2;
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("side_ws")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime_api.h").write_text(HIP)
    (d / "side_ws.h").write_text(open(HEADER).read())
    (d / "t.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", "-I", str(d), str(d / "t.cpp"), "-o", str(d / "t")])
    return str(d / "t")


@pytest.mark.parametrize("what", ["per_thread", "reused_handle", "null_stream", "growth", "capture_elsewhere", "no_buffer", "no_mark",
                                  "other_streams"])
def test_side_workspace(program, what):
    r = subprocess.run([program, what], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
