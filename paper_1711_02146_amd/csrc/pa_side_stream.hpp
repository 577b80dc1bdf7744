// pa_side_stream.hpp -- the second stream of a set of populations, and the sweep
// launches of a set on both.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

namespace pa_host {

// The device of a stream made current for a scope (streams, events and code objects
// are made on the current device, which need not be the one a caller's stream is
// on).  ok(): the device is known and current.
class DeviceOf {
 public:
  explicit DeviceOf(hipStream_t stream) {
    int dev = -1;
    if (hipStreamGetDevice(stream, &dev) != hipSuccess || hipGetDevice(&was_) != hipSuccess) {
      (void)hipGetLastError();
      return;
    }
    ok_ = dev == was_;
    if (ok_) return;
    moved_ = ok_ = hipSetDevice(dev) == hipSuccess;
  }
  ~DeviceOf() {
    if (moved_) (void)hipSetDevice(was_);
  }
  DeviceOf(const DeviceOf&) = delete;
  DeviceOf& operator=(const DeviceOf&) = delete;
  bool ok() const { return ok_; }

 private:
  int was_ = -1;
  bool ok_ = false, moved_ = false;
};

// A second stream beside a set's own, on the same device, for the sweep launches of
// its lattice sizes (one launch each): alone, the last workgroups of a launch leave
// most of the chip idle until they end (a loop of eight requests 229 -> 222 ms, a
// batch of 12 pairs 341 -> 334).  Without it (creation failed) the launches follow
// each other.
struct SideStream {
  hipStream_t s = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;

  void create(hipStream_t beside) {
    const DeviceOf dev(beside);
    if (!dev.ok()) return;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) s = nullptr;
    if (!s || hipEventCreateWithFlags(&fork, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&join, hipEventDisableTiming) != hipSuccess) {
      destroy();
      (void)hipGetLastError();  // not an error of the launches that follow
    }
  }
  void destroy() {
    if (fork) (void)hipEventDestroy(fork);
    if (join) (void)hipEventDestroy(join);
    if (s) (void)hipStreamDestroy(s);
    s = nullptr;
    fork = join = nullptr;
  }
};

// The launches of a set's sweep groups (launch(group, stream)) on `stream` and the
// side stream, the largest first (the groups are put in that order), each on the one
// with less work so far; what follows on `stream` waits for both.
template <typename SweepGroup, typename Launch>
hipError_t launch_sweeps(std::vector<SweepGroup>& groups, const SideStream& side,
                         hipStream_t stream, Launch launch) {
  const bool two = side.s && groups.size() > 1;
  // (in place: nothing here allocates, so nothing can throw between fork and join)
  std::sort(groups.begin(), groups.end(),
            [](const SweepGroup& a, const SweepGroup& b) { return a.work > b.work; });
  hipError_t e = hipSuccess;
  if (two) {
    e = hipEventRecord(side.fork, stream);
    if (e == hipSuccess) e = hipStreamWaitEvent(side.s, side.fork, 0);
    if (e != hipSuccess) return e;
  }
  uint64_t mine = 0, other = 0;
  for (const SweepGroup& g : groups) {
    const bool here = !two || mine <= other;
    (here ? mine : other) += g.work;
    const hipError_t l = launch(g, here ? stream : side.s);
    if (e == hipSuccess) e = l;
  }
  if (two) {
    const hipError_t r = hipEventRecord(side.join, side.s);
    const hipError_t w = r == hipSuccess ? hipStreamWaitEvent(stream, side.join, 0) : r;
    if (e == hipSuccess) e = w;
  }
  return e;
}

}  // namespace pa_host
