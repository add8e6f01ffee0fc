// The side stream of each device, for launches that run beside the caller's.
#include <hip/hip_runtime.h>

#include <mutex>

#include "internal.h"

namespace mcmc {

namespace {

// Per device: the side stream and the events that fork it from and join it to
// a caller's stream.  Created on first use outside a stream capture (or by
// prepare_side_stream) and kept until the process ends; the mutex orders
// concurrent callers' fork-launch-join sequences.
struct Entry {
  hipStream_t side = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
};
constexpr int kDevices = 64;
std::mutex g_mu;
Entry g_entry[kDevices];

// the current device's entry, created if `create`; null if it does not exist
// (or cannot be made)
Entry* entry(bool create) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return nullptr;
  Entry& o = g_entry[dev];
  if (o.side || !create) return o.side ? &o : nullptr;
  Entry n;
  if (hipStreamCreateWithFlags(&n.side, hipStreamNonBlocking) != hipSuccess) return nullptr;
  if (hipEventCreateWithFlags(&n.fork, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&n.join, hipEventDisableTiming) != hipSuccess) {
    if (n.fork) (void)hipEventDestroy(n.fork);
    (void)hipStreamDestroy(n.side);
    return nullptr;
  }
  o = n;
  return &o;
}

bool capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(s, &st) == hipSuccess && st != hipStreamCaptureStatusNone;
}

}  // namespace

hipError_t prepare_side_stream() {
  std::lock_guard<std::mutex> lock(g_mu);
  return entry(true) ? hipSuccess : hipErrorOutOfMemory;
}

SideStream::SideStream(hipStream_t s, bool may_create, bool in_capture) : s_(s) {
  g_mu.lock();
  const bool cap = capturing(s);
  if (cap && !in_capture) return;
  const Entry* o = entry(may_create && !cap);
  // not while another caller's capture holds it
  if (!o || (!cap && capturing(o->side))) return;
  side_ = o->side;
  fork_ = o->fork;
  join_ = o->join;
}

SideStream::~SideStream() { g_mu.unlock(); }

hipError_t SideStream::fork() {
  const hipError_t e = hipEventRecord(fork_, s_);
  return e != hipSuccess ? e : hipStreamWaitEvent(side_, fork_, 0);
}

hipError_t SideStream::join() {
  const hipError_t e = hipEventRecord(join_, side_);
  return e != hipSuccess ? e : hipStreamWaitEvent(s_, join_, 0);
}

}  // namespace mcmc
