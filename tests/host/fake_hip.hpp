// A HIP runtime in host memory, linked into a test program ahead of the real one: the library's
// own host code then runs on the CPU, its calls in order on one worker thread per stream.  Every
// thread has a per-thread stream (hipStreamPerThread) of its own, kernels of a stream refuse
// another current device, and a capturing stream keeps what it is given.  Of the kernels, the
// initial state, the update (f + 1, W + 1 in rho and rho E), the host images and the moments do
// their work; the others do nothing.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstddef>
#include <set>
#include <string>

namespace fake {

struct Knobs {
  std::atomic<int> step_us{0};           // time an update takes
  std::atomic<int> image_us{0};          // time the copy of one image piece takes
  std::atomic<int> pinned_left{1 << 30};  // pinned allocations that can be live besides those now
  std::atomic<int> events_left{1 << 30};  // events, likewise
  std::atomic<int> images_left{1 << 30};  // launches of the image kernel that still succeed
};
extern Knobs knobs;

struct Counts {
  std::atomic<int> pinned_allocs{0}, pinned_live{0};
  std::atomic<int> idle_workgroups{0};  // of the moment and update kernels' grids
  std::atomic<int> misuse{0};  // pinned memory freed or given out while queued work used it
};
extern Counts counts;

hipStream_t make_stream(int device);
// The (mangled) names of the kernels launched so far.
std::set<std::string> launched();
void begin_capture(hipStream_t s);
// Ends the capture; the number of operations the stream was given since.
int end_capture(hipStream_t s);

}  // namespace fake
