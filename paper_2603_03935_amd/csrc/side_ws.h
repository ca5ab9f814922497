// Workspace for the faster form of a call that can do without any
// (disc_backproject, disc_voxel_overlap): a buffer per (device, stream), apart
// from the workspaces of the other calls, because these calls may be made from
// several threads on one stream.
#pragma once

#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <utility>

namespace disc {
namespace host {

constexpr size_t kSideMax = (size_t)128 << 20;  // a call that asks for more does without
constexpr int kSideOld = 16;                    // outgrown buffers: doublings from 64 KB to beyond kSideMax

struct SideWs {
  std::mutex mu;  // held while a call takes the buffer and enqueues its kernels
  void* dev = nullptr;
  size_t bytes = 0;
  hipEvent_t used = nullptr;  // after the last call's kernels (not on the null stream)
  bool recorded = false;
  void* old[kSideOld];  // outgrown buffers: kernels in flight may still use them
  int n_old = 0;
};
// Entries are never erased, so a reference to one stays valid.
inline std::mutex g_side_mu;
inline std::map<std::pair<int, hipStream_t>, SideWs> g_side;

// The buffer of a call that enqueues its kernels while the lease lives; ptr is
// null when the call has to do without: no bytes asked for or more than
// kSideMax, a stream that is being captured (or cannot say), no memory, or
// hipStreamPerThread, one handle for as many streams as there are threads.
//
// Two streams that are not ordered never use a buffer at the same time: a handle
// can come back for another stream while the destroyed one's kernels still run,
// so each call waits, on the device, for the event that the one before recorded
// (about 2 us a call).  The null stream's handle is never another's, so there
// stream order is enough.  Nothing here waits on the host or frees memory, and
// only calls on one stream share a mutex beyond the table's look-up: a buffer
// that grows at least doubles, and the outgrown ones (together smaller than it)
// are kept until release_side_ws.  Memory is allocated in the relaxed capture
// mode, so that a graph which another thread captures meanwhile is not broken.
class SideLease {
 public:
  SideLease(hipStream_t st, size_t bytes) : st_(st) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    int dev = 0;
    if (bytes == 0 || bytes > kSideMax || st == hipStreamPerThread) return;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess || hipGetDevice(&dev) != hipSuccess) {
      (void)hipGetLastError();
      return;
    }
    if (cs != hipStreamCaptureStatusNone) return;
    {
      std::lock_guard<std::mutex> lk(g_side_mu);
      ws_ = &g_side[{dev, st}];
    }
    ws_->mu.lock();
    if (!take(bytes)) {
      (void)hipGetLastError();
      ws_->mu.unlock();
      ws_ = nullptr;
      return;
    }
    ptr = static_cast<char*>(ws_->dev);
  }
  ~SideLease() {
    if (!ws_) return;
    if (st_) {
      ws_->recorded = hipEventRecord(ws_->used, st_) == hipSuccess;
      if (!ws_->recorded) {  // no mark: wait here
        (void)hipGetLastError();
        (void)hipStreamSynchronize(st_);
      }
    }
    ws_->mu.unlock();
  }
  SideLease(const SideLease&) = delete;
  SideLease& operator=(const SideLease&) = delete;

  char* ptr = nullptr;

 private:
  bool take(size_t bytes) {
    // (one device's streams: no fence to the host)
    if (st_ && !ws_->used &&
        hipEventCreateWithFlags(&ws_->used, hipEventDisableTiming | hipEventDisableSystemFence) != hipSuccess) {
      ws_->used = nullptr;
      return false;
    }
    if (ws_->recorded && hipStreamWaitEvent(st_, ws_->used, 0) != hipSuccess) return false;
    if (ws_->bytes >= bytes) return true;
    if (ws_->n_old == kSideOld) return false;
    const size_t want = (std::max(bytes + bytes / 4, 2 * ws_->bytes) + 0xFFFF) & ~(size_t)0xFFFF;
    void* p = nullptr;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    const hipError_t e = hipMalloc(&p, want);
    if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e != hipSuccess) return false;
    if (ws_->dev) ws_->old[ws_->n_old++] = ws_->dev;
    ws_->dev = p;
    ws_->bytes = want;
    return true;
  }

  hipStream_t st_;
  SideWs* ws_ = nullptr;
};

// Frees every buffer once the calls that use it have run.
inline void release_side_ws() {
  std::lock_guard<std::mutex> lk(g_side_mu);
  int dev = 0;
  (void)hipGetDevice(&dev);
  for (auto& kv : g_side) {
    SideWs& w = kv.second;
    std::lock_guard<std::mutex> one(w.mu);
    if (!w.dev) continue;
    (void)hipSetDevice(kv.first.first);
    (void)hipDeviceSynchronize();
    if (w.used) (void)hipEventDestroy(w.used);
    w.used = nullptr;
    w.recorded = false;
    for (int i = 0; i < w.n_old; ++i) (void)hipFree(w.old[i]);
    w.n_old = 0;
    (void)hipFree(w.dev);
    w.dev = nullptr;
    w.bytes = 0;
  }
  (void)hipSetDevice(dev);
}

}  // namespace host
}  // namespace disc
