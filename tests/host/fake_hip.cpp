#include "fake_hip.hpp"

#include <chrono>
#include <condition_variable>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "ugks_internal.hpp"

namespace fake {
Knobs knobs;
Counts counts;
}  // namespace fake

namespace {

using namespace ugks;
typedef std::function<void()> Op;

struct Stream {
  int device = 0;
  bool capturing = false;
  std::vector<Op> captured;
  std::mutex m;
  std::condition_variable cv;
  std::deque<Op> ops;
  unsigned long long given = 0, done = 0;
  explicit Stream(int d) : device(d) {
    std::thread([this] {
      std::unique_lock<std::mutex> lock(m);
      for (;;) {
        cv.wait(lock, [this] { return !ops.empty(); });
        Op op = std::move(ops.front());
        ops.pop_front();
        lock.unlock();
        op();
        lock.lock();
        ++done;
        cv.notify_all();
      }
    }).detach();
  }
  void put(Op op) {
    if (capturing) {
      captured.push_back(std::move(op));
      return;
    }
    std::lock_guard<std::mutex> lock(m);
    ops.push_back(std::move(op));
    ++given;
    cv.notify_all();
  }
  void wait(unsigned long long n) {
    std::unique_lock<std::mutex> lock(m);
    cv.wait(lock, [&] { return done >= n; });
  }
  unsigned long long now() {
    std::lock_guard<std::mutex> lock(m);
    return given;
  }
};
struct Event {
  Stream* s = nullptr;
  unsigned long long n = 0;
};

thread_local int t_device = 0;
thread_local hipError_t t_last = hipSuccess;
thread_local hipStreamCaptureMode t_mode = hipStreamCaptureModeGlobal;
thread_local struct {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
} t_call;

std::mutex g_m;

hipError_t ret(hipError_t e) {
  if (e != hipSuccess) t_last = e;
  return e;
}

Stream& at(hipStream_t s) {
  if (s != nullptr && s != hipStreamPerThread) return *reinterpret_cast<Stream*>(s);
  std::lock_guard<std::mutex> lock(g_m);
  static std::map<std::pair<std::thread::id, int>, Stream*> streams;
  Stream*& p = streams[{s ? std::this_thread::get_id() : std::thread::id(), t_device}];
  if (!p) p = new Stream(t_device);
  return *p;
}

// pinned blocks and the queued operations that use each
std::map<const char*, std::pair<size_t, int>>& pinned() {
  static auto* p = new std::map<const char*, std::pair<size_t, int>>;
  return *p;
}
bool use_pinned(const void* ptr, int change) {
  std::lock_guard<std::mutex> lock(g_m);
  const char* c = static_cast<const char*>(ptr);
  auto it = pinned().upper_bound(c);
  if (it == pinned().begin()) return false;
  --it;
  if (c >= it->first + it->second.first) return false;
  it->second.second += change;
  return true;
}

std::map<const void*, std::string>& kernels() {
  static auto* k = new std::map<const void*, std::string>;
  return *k;
}

std::set<std::string>& names() {
  static auto* n = new std::set<std::string>;
  return *n;
}

void pause_us(int us) {
  if (us > 0) std::this_thread::sleep_for(std::chrono::microseconds(us));
}
template <typename T>
T arg(void** args, int n) {
  T v;
  std::memcpy(&v, args[n], sizeof v);
  return v;
}
size_t place(const KParams& P, long long c) {
  return (size_t)((c / P.nx + kHalo) * P.Lx + c % P.nx + kHalo);
}

template <typename S>
void init(const Inst& I) {
  S* f = (S*)I.f[I.cur];
  const KParams& P = I.P;
  for (int v = 0; v < P.NV * P.NC; ++v)
    for (long long c = 0; c < (long long)P.nx * P.ny; ++c)
      f[(size_t)v * P.PS + place(P, c)] = (S)(c % 1000 + 0.125 * (v % 64));
}
template <typename S>
void update(const Inst& I, int step) {
  const int p = (I.cur + step) & 1;
  const S* f = (const S*)I.f[p];
  S* g = (S*)I.f[p ^ 1];
  const KParams& P = I.P;
  for (int v = 0; v < P.NV * P.NC; ++v)
    for (int j = 0; j < P.ny; ++j)
      for (int i = 0; i < P.nx; ++i) {
        const size_t x = (size_t)v * P.PS + (size_t)(j + kHalo) * P.Lx + i + kHalo;
        g[x] = f[x] + S(1);
      }
  const double* W = (const double*)I.W[p];
  double* X = (double*)I.W[p ^ 1];
  for (long long e = 0; e < 4LL * P.nx * P.ny; ++e) X[e] = W[e] + (e % 4 % 3 == 0 ? 1.0 : 0.0);
}
template <typename S>
void image(bool out, S* f, const KParams& P, long long c0, int ncell, int v0, int nvel,
           double* img) {
  pause_us(fake::knobs.image_us);
  for (int c = 0; c < ncell; ++c)
    for (int v = 0; v < nvel; ++v) {
      S& x = f[(size_t)(v0 + v) * P.PS + place(P, c0 + c)];
      double& y = img[(size_t)c * nvel + v];
      if (out)
        y = x;
      else
        x = (S)y;
    }
}
void moments(const double* W, int n, double lam_c, const int* flag, double* out, int* bad) {
  if (*flag) *bad = 1;
  for (int c = 0; c < n; ++c, W += 4, out += 4) {
    const double rho = W[0], U = W[1] / rho, V = W[2] / rho;
    out[0] = rho;
    out[1] = U;
    out[2] = V;
    out[3] = (W[3] - 0.5 * rho * (U * U + V * V)) / (lam_c * rho);
    if (!(rho > 0) || !(out[3] > 0)) *bad = 1;
  }
}

}  // namespace

namespace fake {
hipStream_t make_stream(int device) { return reinterpret_cast<hipStream_t>(new Stream(device)); }
std::set<std::string> launched() {
  std::lock_guard<std::mutex> lock(g_m);
  return names();
}
void begin_capture(hipStream_t s) { at(s).capturing = true; }
int end_capture(hipStream_t s) {
  Stream& st = at(s);
  const int n = (int)st.captured.size();
  st.capturing = false;
  st.captured.clear();
  return n;
}
}  // namespace fake

extern "C" {

void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  kernels()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
  t_call = {grid, block, shared, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared,
                                     hipStream_t* stream) {
  *grid = t_call.grid;
  *block = t_call.block;
  *shared = t_call.shared;
  *stream = t_call.stream;
  return hipSuccess;
}

hipError_t hipLaunchKernel(const void* func, dim3 grid, dim3, void** args, size_t,
                           hipStream_t stream) {
  Stream& s = at(stream);
  if (s.device != t_device) return ret(hipErrorInvalidHandle);
  const std::string& name = kernels()[func];
  auto is = [&](const char* part) { return name.find(part) != std::string::npos; };
  const bool f32 = is("If");
  {
    std::lock_guard<std::mutex> lock(g_m);
    names().insert(name);
  }
  if (is("sums_kernel") || is("update_kernel")) {
    // a workgroup for each segment of 62 (update: 60) cells of a row (of two) and each chunk
    const bool sums = is("sums_kernel");
    const Inst* in = arg<const Inst*>(args, 0);
    const int n = arg<int>(args, 2);
    s.put([=] {
      long long work = 0;
      for (int q = 0; q < n; ++q) {
        const KParams& P = in[q].P;
        const int tile = sums ? 62 : 60, rows = sums ? P.ny : (P.ny + 1) / 2;
        work += (long long)((P.nx + tile - 1) / tile) * rows * P.NC *
                (sums ? in[q].gsplit : in[q].usplit * P.vsplit);
      }
      fake::counts.idle_workgroups += (int)(grid.x - work);
    });
  }
  if (is("init_kernel")) {
    const PlanView pv = arg<PlanView>(args, 0);
    s.put([=] { f32 ? init<float>(pv.inst[0]) : init<double>(pv.inst[0]); });
  } else if (is("update_kernel")) {
    const Inst* in = arg<const Inst*>(args, 0);
    const int n = arg<int>(args, 2), step = arg<int>(args, 3);
    s.put([=] {
      pause_us(fake::knobs.step_us);
      for (int q = 0; q < n; ++q) f32 ? update<float>(in[q], step) : update<double>(in[q], step);
    });
  } else if (is("state_kernel")) {
    if (fake::knobs.images_left.fetch_sub(1) <= 0) return ret(hipErrorLaunchFailure);
    void* f = arg<void*>(args, 0);
    const KParams P = arg<KParams>(args, 1);
    const long long c0 = arg<long long>(args, 2);
    const int ncell = arg<int>(args, 3), v0 = arg<int>(args, 4), nvel = arg<int>(args, 5);
    double* img = arg<double*>(args, 6);
    const bool out = is("Lb1");
    if (!use_pinned(img, 1)) return ret(hipErrorInvalidValue);
    s.put([=] {
      if (f32)
        image(out, (float*)f, P, c0, ncell, v0, nvel, img);
      else
        image(out, (double*)f, P, c0, ncell, v0, nvel, img);
      use_pinned(img, -1);
    });
  } else if (is("moments_kernel")) {
    const double* W = arg<const double*>(args, 0);
    const int n = arg<int>(args, 1);
    const double lam_c = arg<double>(args, 2);
    const int* flag = arg<const int*>(args, 3);
    double* out = arg<double*>(args, 4);
    int* bad = arg<int*>(args, 5);
    if (!use_pinned(out, 1)) return ret(hipErrorInvalidValue);
    s.put([=] {
      moments(W, n, lam_c, flag, out, bad);
      use_pinned(out, -1);
    });
  } else {
    s.put([] {});
  }
  return hipSuccess;
}

hipError_t hipGetDevice(int* d) {
  *d = t_device;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  t_device = d;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = t_last;
  t_last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "an error of the host runtime"; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* scratch = std::aligned_alloc(256, UGKS_STATIC_SCRATCH_BYTES);
  *p = scratch;
  return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n) {
  *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
  return *p ? hipSuccess : ret(hipErrorOutOfMemory);
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (fake::knobs.pinned_left.fetch_sub(1) <= 0) return ret(hipErrorOutOfMemory);
  *p = std::aligned_alloc(4096, (n + 4095) / 4096 * 4096);
  ++fake::counts.pinned_allocs;
  ++fake::counts.pinned_live;
  std::lock_guard<std::mutex> lock(g_m);
  pinned()[static_cast<const char*>(*p)] = {n, 0};
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  {
    std::lock_guard<std::mutex> lock(g_m);
    auto it = pinned().find(static_cast<const char*>(p));
    if (it == pinned().end() || it->second.second != 0) {
      ++fake::counts.misuse;
      return hipErrorInvalidValue;
    }
    pinned().erase(it);
  }
  --fake::counts.pinned_live;
  ++fake::knobs.pinned_left;
  std::free(p);
  return hipSuccess;
}

static hipError_t copy(Stream& s, Op op, const void* a, const void* b) {
  const bool async = use_pinned(a, 0) || use_pinned(b, 0);
  s.put(std::move(op));
  if (!async && !s.capturing) s.wait(s.now());
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  return copy(at(st), [=] { std::memcpy(d, s, n); }, d, s);
}
hipError_t hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h,
                            hipMemcpyKind, hipStream_t st) {
  return copy(at(st), [=] {
    for (size_t r = 0; r < h; ++r) std::memcpy((char*)d + r * dp, (const char*)s + r * sp, w);
  }, d, s);
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
  at(st).put([=] { std::memset(d, v, n); });
  return hipSuccess;
}

hipError_t hipStreamSynchronize(hipStream_t st) {
  Stream& s = at(st);
  if (s.capturing) return ret(hipErrorStreamCaptureUnsupported);
  s.wait(s.now());
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t st, hipStreamCaptureStatus* status) {
  *status = at(st).capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* mode) {
  std::swap(t_mode, *mode);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned) {
  Event ev = *reinterpret_cast<Event*>(e);
  at(st).put([ev] { if (ev.s) ev.s->wait(ev.n); });
  return hipSuccess;
}

hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  if (fake::knobs.events_left.fetch_sub(1) <= 0) return ret(hipErrorOutOfMemory);
  *e = reinterpret_cast<hipEvent_t>(new Event);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete reinterpret_cast<Event*>(e);
  ++fake::knobs.events_left;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
  Stream& s = at(st);
  *reinterpret_cast<Event*>(e) = {&s, s.now()};
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  Event* ev = reinterpret_cast<Event*>(e);
  if (ev->s) ev->s->wait(ev->n);
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}

}  // extern "C"
