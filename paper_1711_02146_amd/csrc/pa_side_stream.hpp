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

// What a second stream can hide of a set's sweep launches, in microseconds: all but the
// longest, each about 5 and, per sweep, 2 and its attempts (work: sites x tiles) at
// 1e12/s.
template <typename SweepGroup>
double beside_us(const std::vector<SweepGroup>& groups, uint32_t n_sweeps) {
  double sum = 0.0, most = 0.0;
  for (const SweepGroup& g : groups) {
    const double us = 5.0 + n_sweeps * (2.0 + 64e-6 * (double)g.work);
    sum += us;
    most = std::max(most, us);
  }
  return sum - most;
}
// Below these the launches stay on one stream.  A stepper's step: fork and join take the
// host about 15 us (us a step on one stream / on two, 1 sweep: L = 4 and 6, R = 500 85 /
// 103, with three lattice sizes 128 / 126; 3 sweeps 99 / 105 and L = 4 and 8 109 / 103; 10
// sweeps 146 / 134).  A batch's graph: about 7 of these us a step (1 sweep 44 / 49, 2
// sweeps 51 / 51, 5 sweeps 71 / 62), and 100 to 250 once, to make the stream and a graph
// of two branches.
constexpr double kStepBesideUs = 12.0;
inline bool batch_beside(double us, uint32_t n_steps) { return n_steps * (us - 7.0) > 200.0; }

// The launches of a set's sweep groups (launch(group, stream)) on `stream` and, with
// `beside`, the side stream, the largest first (the groups are put in that order), each
// on the one with less work so far; what follows on `stream` waits for both.
template <typename SweepGroup, typename Launch>
hipError_t launch_sweeps(std::vector<SweepGroup>& groups, const SideStream& side, bool beside,
                         hipStream_t stream, Launch launch) {
  const bool two = beside && side.s && groups.size() > 1;
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
