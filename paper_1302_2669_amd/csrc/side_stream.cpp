// The side streams of each device, for launches that run beside the caller's.
//
// Callers do not wait for each other through them: a side stream holds work of
// one caller's stream at a time, and goes to another's only once it is idle.  (As
// one stream per device for everybody, a decode on one stream waited at its join
// for whatever another stream's decode had forked before it, and for all that
// stream was itself waiting for.)
#include <hip/hip_runtime.h>

#include <mutex>

#include "../../include/mcmcdec.h"
#include "internal.h"

namespace mcmc {

namespace {

// A side stream, the events that fork it from and join it to a caller's stream,
// and that stream.  Created when a caller outside a stream capture finds none free
// (or by prepare_side_streams), at most kSides per device, and kept until the
// process ends; the mutex orders concurrent callers' fork-launch-join sequences.
struct Side {
  hipStream_t side = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  bool used = false, taken = false;   // taken: by a living SideStream
  hipStream_t user = nullptr;         // of the last use outside a capture
};
constexpr int kDevices = 64, kSides = 4;
std::recursive_mutex g_mu;   // a caller may hold two at once
Side g_sides[kDevices][kSides];
int g_count[kDevices];

// the current device's index, -1 if there is none
int device() {
  int dev = 0;
  return hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kDevices ? dev : -1;
}

// Queries and creations are no part of any capture that another thread has open.
struct RelaxedCapture {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  bool changed;
  RelaxedCapture() { changed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess; }
  ~RelaxedCapture() {
    if (changed) (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
};

Side* create(int dev) {
  if (g_count[dev] == kSides) return nullptr;
  RelaxedCapture relaxed;
  Side n;
  if (hipStreamCreateWithFlags(&n.side, hipStreamNonBlocking) != hipSuccess) return nullptr;
  if (hipEventCreateWithFlags(&n.fork, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&n.join, hipEventDisableTiming) != hipSuccess) {
    if (n.fork) (void)hipEventDestroy(n.fork);
    (void)hipStreamDestroy(n.side);
    return nullptr;
  }
  g_sides[dev][g_count[dev]] = n;
  return &g_sides[dev][g_count[dev]++];
}

// whether s is being captured, and into which capture
bool capturing(hipStream_t s, unsigned long long* id) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess || st == hipStreamCaptureStatusNone) return false;
  *id = 0;
  (void)hipStreamGetCaptureInfo(s, &st, id);
  return true;
}

bool idle(hipStream_t s) {
  RelaxedCapture relaxed;
  const hipError_t e = hipStreamQuery(s);
  // not ready is an answer, not an error for the next launch to report
  if (e == hipErrorNotReady && hipPeekAtLastError() == hipErrorNotReady) (void)hipGetLastError();
  return e == hipSuccess;
}

}  // namespace

hipError_t prepare_side_streams(int count) {
  std::lock_guard<std::recursive_mutex> lock(g_mu);
  const int dev = device();
  if (dev < 0) return hipErrorInvalidDevice;
  while (g_count[dev] < count)
    if (!create(dev)) return hipErrorOutOfMemory;
  return hipSuccess;
}

SideStream::SideStream(hipStream_t s, bool may_create, bool in_capture) : s_(s) {
  g_mu.lock();
  const int dev = device();
  if (dev < 0) return;
  unsigned long long id = 0, other = 0;
  const bool cap = capturing(s, &id);
  if (cap && !in_capture) return;
  Side* take = nullptr;
  bool own = false;
  for (int k = 0; k < g_count[dev] && !own; ++k) {
    Side& o = g_sides[dev][k];
    if (o.taken) continue;
    const bool held = capturing(o.side, &other);
    if (cap) {
      // what a free stream still runs is no part of this capture; one that this
      // capture has forked before follows what it holds
      own = held && other == id;
      if (own || (!held && !take)) take = &o;
    } else if (!held) {
      // s's own work on it precedes s's next anyway.  (The handle that every
      // thread's default stream shares does not name one stream.)
      own = o.used && o.user == s && s != hipStreamPerThread;
      if (own || (!take && idle(o.side))) take = &o;
    }
  }
  if (!take && may_create && !cap) take = create(dev);
  if (!take) return;
  take->taken = true;
  taken_ = &take->taken;
  if (!cap) {
    take->used = true;
    take->user = s;
  }
  side_ = take->side;
  fork_ = take->fork;
  join_ = take->join;
}

SideStream::~SideStream() {
  if (forked_) (void)join();
  if (taken_) *taken_ = false;
  g_mu.unlock();
}

hipError_t SideStream::fork() {
  hipError_t e = hipEventRecord(fork_, s_);
  if (e == hipSuccess) e = hipStreamWaitEvent(side_, fork_, 0);
  forked_ = e == hipSuccess;
  return e;
}

hipError_t SideStream::join() {
  forked_ = false;
  const hipError_t e = hipEventRecord(join_, side_);
  return e != hipSuccess ? e : hipStreamWaitEvent(s_, join_, 0);
}

}  // namespace mcmc

// The side stream that a caller on `stream` would get now, forked from and joined
// to it, or null: what the tests of the choice call.
extern "C" int mcmc_side_stream_of(void* stream, int may_create, int in_capture, void** side) {
  mcmc::SideStream s((hipStream_t)stream, may_create != 0, in_capture != 0);
  *side = s.stream();
  if (!s.stream()) return MCMC_OK;
  const bool ok = s.fork() == hipSuccess && s.join() == hipSuccess;
  return ok ? MCMC_OK : MCMC_EDEVICE;
}
