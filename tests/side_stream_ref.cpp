// The sweep launches of a set on two streams (pa_side_stream.hpp), compiled for the
// CPU against the few HIP calls it makes, here on a machine of two devices with
// HIP's rules: streams and events are made on the current device, and an event is
// recorded only in a stream of its own device.  argv: the current device, the device of
// the set's stream and, for the rules of when the second stream is used, the sweeps of a
// step, the steps of a batch (0: a stepper) and the work (sites x tiles) of each launch.
// Prints the result of the launches, how many went to the set's stream, to a second
// stream of the same device and to anything else, whether they came largest first, and
// the current device afterwards.
#include <cstdint>
#include <cstdio>
#include <cstdlib>

enum hipError_t { hipSuccess = 0, hipErrorInvalidDevice = 101, hipErrorInvalidHandle = 400 };
struct Stream { int dev; };
struct Event { int dev; const Stream* in; };
typedef Stream* hipStream_t;
typedef Event* hipEvent_t;
constexpr unsigned hipStreamNonBlocking = 1, hipEventDisableTiming = 2;

static int g_dev = 0;
hipError_t hipGetDevice(int* d) { *d = g_dev; return hipSuccess; }
hipError_t hipSetDevice(int d) {
  if (d < 0 || d > 1) return hipErrorInvalidDevice;
  g_dev = d;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, int* d) { *d = s ? s->dev : g_dev; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = new Stream{g_dev};
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { delete s; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = new Event{g_dev, nullptr};
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (e->dev != s->dev) return hipErrorInvalidHandle;
  e->in = s;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t e, unsigned) {
  return e->in ? hipSuccess : hipErrorInvalidHandle;
}

#include "pa_side_stream.hpp"

struct Group {
  uint64_t work;
};

int main(int argc, char** argv) {
  const int dev = std::atoi(argv[2]);
  hipSetDevice(std::atoi(argv[1]));
  Stream set{dev};
  pa_host::SideStream side;
  side.create(&set);
  std::vector<Group> groups = {{3}, {10}, {5}};
  bool second = true;
  if (argc > 4) {
    groups.clear();
    for (int i = 5; i < argc; ++i) groups.push_back({std::strtoull(argv[i], nullptr, 10)});
    const int n_steps = std::atoi(argv[4]);
    const double us = pa_host::beside_us(groups, (uint32_t)std::atoi(argv[3]));
    second = n_steps ? pa_host::batch_beside(us, (uint32_t)n_steps) : us >= pa_host::kStepBesideUs;
  }
  int own = 0, beside = 0, elsewhere = 0;
  uint64_t last = ~0ull;
  bool ordered = true;
  const hipError_t e = pa_host::launch_sweeps(groups, side, second, &set, [&](const Group& g, hipStream_t s) {
    ordered = ordered && g.work <= last;
    last = g.work;
    ++(s == &set ? own : s->dev == dev ? beside : elsewhere);
    return hipSuccess;
  });
  side.destroy();
  std::printf("%d %d %d %d %d %d\n", (int)e, own, beside, elsewhere, (int)ordered, g_dev);
  return 0;
}
