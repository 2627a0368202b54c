// Cases of the library's host code over the runtime of fake_hip.hpp, one per run (argument 1).
// Exit status 0 when the case holds.
#include <dlfcn.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "fake_hip.hpp"
#include "ugks.h"

namespace {

int failures = 0;
void check(bool ok, const char* what) {
  if (ok) return;
  std::fprintf(stderr, "failed: %s\n", what);
  ++failures;
}

struct Problem {
  ugks_mesh mesh{43, 31, 2.0, 1.0};
  ugks_vgrid vg{64, 61, 5.0, 5.0, 0};  // 41.6 MB of f: 20 pieces
  ugks_bc bc{UGKS_BC_CHANNEL, 0, 2.0, 1.0, 1.0, 0.0, 0.0};
  ugks_opts o{};
  Problem(int nx = 43, int ny = 31, int nu = 64, int nv = 61) {
    mesh.nx = nx;
    mesh.ny = ny;
    vg.nu = nu;
    vg.nv = nv;
    o.cfl = 0.8;
    o.rho0 = o.T0 = 1.0;
    o.noise = 0.01;
    o.seed = 1;
  }
  size_t cells() const { return (size_t)mesh.nx * mesh.ny; }
  size_t values() const {
    return cells() * vg.nu * vg.nv * (vg.internal_dof > 0 ? 2 : 1);
  }
  ugks_handle* create(void* stream = nullptr) {
    o.stream = stream;
    ugks_handle* h = nullptr;
    check(ugks_create(&mesh, &vg, 0.1, &bc, &o, &h) == UGKS_OK, ugks_last_error(nullptr));
    return h;
  }
};

bool shifted(const std::vector<double>& a, const std::vector<double>& b, double by) {
  for (size_t k = 0; k < a.size(); ++k)
    if (b[k] != a[k] + by) return false;
  return true;
}

// Images of many pieces on a stream that every host thread reads as its own: they are taken
// after the steps enqueued before, and the next step runs on what was set.
void per_thread_stream() {
  Problem p;
  ugks_handle* h = p.create(hipStreamPerThread);
  std::vector<double> f0(p.values()), f(p.values());
  check(ugks_get_state(h, f0.data(), nullptr) == UGKS_OK, "get");
  fake::knobs.step_us = 100000;
  check(ugks_step(h, 2) == UGKS_OK, "step");
  check(ugks_get_state(h, f.data(), nullptr) == UGKS_OK, "get after steps");
  check(shifted(f0, f, 2.0), "the state after both steps");
  for (double& x : f0) x = 3.0 * x + 1.0;
  check(ugks_step(h, 1) == UGKS_OK, "step");
  check(ugks_set_state(h, f0.data(), nullptr) == UGKS_OK, "set under a step");
  check(ugks_step(h, 1) == UGKS_OK, "step");
  check(ugks_get_state(h, f.data(), nullptr) == UGKS_OK, "get");
  check(shifted(f0, f, 1.0), "the state set, one step on");
  ugks_destroy(h);
}

// A handle of another GPU than the caller's current one, which stays current.
void other_device() {
  Problem p;
  (void)hipSetDevice(1);
  ugks_handle* h = p.create(fake::make_stream(1));
  (void)hipSetDevice(0);
  auto same = [](const char* what) {
    int d = -1;
    (void)hipGetDevice(&d);
    check(d == 0, what);
  };
  std::vector<double> f(p.values()), g(p.values()), m(4 * p.cells());
  check(ugks_moments(h, m.data()) == UGKS_OK, "moments");
  same("the current device after ugks_moments");
  check(ugks_get_state(h, f.data(), nullptr) == UGKS_OK, "get");
  same("the current device after ugks_get_state");
  for (double& x : f) x += 1.0;
  check(ugks_set_state(h, f.data(), nullptr) == UGKS_OK, "set");
  same("the current device after ugks_set_state");
  check(ugks_get_state(h, g.data(), nullptr) == UGKS_OK && f == g, "the state set");
  ugks_destroy(h);
}

// Setting a state is whole or an error.  Too little pinned memory or too few events for every
// block: fewer serve.  A launch that fails: nothing was written before the first, and after it the
// handle is marked failed, as after a step that failed part-way.
void set_is_whole() {
  Problem p;
  std::vector<double> f0(p.values()), f(p.values()), g(p.values()), m(4 * p.cells());
  const int plenty = 1 << 30;
  ugks_handle* h = p.create();
  check(ugks_get_state(h, f0.data(), nullptr) == UGKS_OK, "get");
  for (int n = 1; n <= 5; n += 2) {
    for (double& x : f0) x += 1.0;
    ugks_destroy(h);  // the pool's blocks go with the last handle
    h = p.create();
    (n == 3 ? fake::knobs.events_left : fake::knobs.pinned_left) = n;
    check(ugks_set_state(h, f0.data(), nullptr) == UGKS_OK, "set with few blocks");
    check(ugks_get_state(h, g.data(), nullptr) == UGKS_OK && f0 == g, "the state set");
    fake::knobs.pinned_left = plenty;
    fake::knobs.events_left = plenty;
  }
  for (size_t k = 0; k < f.size(); ++k) f[k] = f0[k] + 5.0;
  fake::knobs.images_left = 0;
  check(ugks_set_state(h, f.data(), nullptr) == UGKS_E_DEVICE, "set without a launch");
  fake::knobs.images_left = 5;
  check(ugks_get_state(h, g.data(), nullptr) == UGKS_E_DEVICE, "get that fails part-way");
  fake::knobs.images_left = plenty;
  check(ugks_get_state(h, g.data(), nullptr) == UGKS_OK && f0 == g, "the state before");
  fake::knobs.images_left = 5;
  check(ugks_set_state(h, f.data(), nullptr) == UGKS_E_DEVICE, "set that fails part-way");
  fake::knobs.images_left = plenty;
  check(ugks_step(h, 1) == UGKS_E_DEVICE, "step after a state set in part");
  check(ugks_moments(h, m.data()) == UGKS_E_DEVICE, "moments after a state set in part");
  ugks_destroy(h);
  check(fake::counts.misuse == 0, "no block given back early");
}

// No pinned memory at all: everything that needs none of its own still works.
void no_pinned_memory() {
  fake::knobs.pinned_left = 0;
  for (int form = 0; form < 3; ++form) {
    Problem p(43, 31, 24, 25);
    p.o.precision = form == 1 ? UGKS_FP32_STORE : UGKS_FP64;
    p.vg.internal_dof = form == 2 ? 1 : 0;
    p.bc.kind = form == 2 ? UGKS_BC_PERIODIC : UGKS_BC_CHANNEL;
    ugks_handle* h = p.create();
    std::vector<double> f0(p.values()), f(p.values()), W(4 * p.cells()), m(4 * p.cells());
    check(ugks_get_state(h, f0.data(), nullptr) == UGKS_OK, "get");
    for (size_t k = 0; k < f0.size(); ++k) f0[k] = (double)(k % 4099) + 0.5;
    check(ugks_set_state(h, f0.data(), nullptr) == UGKS_OK, "set");
    check(ugks_step(h, 1) == UGKS_OK, "step");
    check(ugks_get_state(h, f.data(), W.data()) == UGKS_OK, "get");
    check(shifted(f0, f, 1.0), "the state set, one step on");
    check(ugks_moments(h, m.data()) == UGKS_OK, "moments");
    const double lam_c = 0.25 * (2 + p.vg.internal_dof);
    bool same = true;
    for (size_t c = 0; c < p.cells(); ++c) {
      const double* w = &W[4 * c];
      const double U = w[1] / w[0], V = w[2] / w[0];
      const double T = (w[3] - 0.5 * w[0] * (U * U + V * V)) / (lam_c * w[0]);
      same = same && m[4 * c] == w[0] && m[4 * c + 1] == U && m[4 * c + 2] == V && m[4 * c + 3] == T;
    }
    check(same, "the moments of W");
    W[4 * p.cells() - 1] = -1.0;
    check(ugks_set_state(h, nullptr, W.data()) == UGKS_OK, "set W");
    check(ugks_moments(h, m.data()) == UGKS_E_STATE && m[0] == W[0], "moments of an invalid state");
    ugks_destroy(h);
  }
}

// Calls that wait for their stream are refused while it is captured, and leave nothing in the
// capture that would read or write their memory when the graph is launched.
void under_capture() {
  Problem p;
  hipStream_t stream = fake::make_stream(0);
  ugks_handle* h = p.create(stream);
  std::vector<double> f0(p.values()), f(p.values()), W(4 * p.cells()), m(4 * p.cells());
  check(ugks_get_state(h, f0.data(), W.data()) == UGKS_OK, "get");
  auto refused = [&](const char* what, auto call) {
    fake::begin_capture(stream);
    const int rc = call();
    check(fake::end_capture(stream) == 0, what);
    check(rc == UGKS_E_DEVICE, what);
  };
  refused("moments", [&] { return ugks_moments(h, m.data()); });
  refused("get f", [&] { return ugks_get_state(h, f.data(), nullptr); });
  refused("get W", [&] { return ugks_get_state(h, nullptr, W.data()); });
  refused("set f", [&] { return ugks_set_state(h, f0.data(), nullptr); });
  refused("set W", [&] { return ugks_set_state(h, nullptr, W.data()); });
  refused("time", [&] { return ugks_get_time(h, &m[0], &m[1]); });
  refused("face flux", [&] { return ugks_get_face_flux(h, f.data(), nullptr); });
  refused("create", [&] {
    ugks_handle* other = nullptr;
    p.o.stream = stream;
    return ugks_create(&p.mesh, &p.vg, 0.1, &p.bc, &p.o, &other);
  });
  check(ugks_step(h, 1) == UGKS_OK && ugks_get_state(h, f.data(), nullptr) == UGKS_OK, "step");
  check(shifted(f0, f, 1.0), "the state after the step");
  ugks_destroy(h);
  check(fake::counts.misuse == 0, "no block given back early");
}

// One solver at a time: the pool keeps a block from one to the next, and no more than that once a
// solver that needed many is closed.
void one_solver_at_a_time() {
  Problem small(40, 10, 24, 24), large;
  std::vector<double> m(4 * small.cells()), f(large.values());
  for (int n = 0; n < 3; ++n) {
    ugks_handle* h = small.create();
    check(ugks_moments(h, m.data()) == UGKS_OK, "moments");
    ugks_destroy(h);
    check(fake::counts.pinned_allocs == 1, "one allocation serves every solver");
  }
  ugks_handle* h = large.create();
  check(ugks_get_state(h, f.data(), nullptr) == UGKS_OK, "get");
  check(fake::counts.pinned_live > 1 && fake::counts.pinned_live <= 8, "blocks of a live solver");
  ugks_destroy(h);
  check(fake::counts.pinned_live == 1, "blocks kept without a solver");
}

// Every workgroup of a batch's launches has work, however small its members are.
void batch_workgroups() {
  std::vector<ugks_handle*> hs;
  std::vector<Problem> ps;
  for (int k = 0; k < 9; ++k) ps.emplace_back(3 + 20 * k, 1 + k % 5, 8 + k, 8);
  for (Problem& p : ps) hs.push_back(p.create());
  ugks_batch* b = nullptr;
  check(ugks_batch_create(nullptr, 9, &b) == UGKS_OK, "batch");
  check(ugks_step_batch(b, hs.data(), 9, 2) == UGKS_OK, "batch step");
  for (ugks_handle* h : hs) check(ugks_step(h, 1) == UGKS_OK, "step alone");
  std::vector<double> m(4 * ps[0].cells());
  check(ugks_moments(hs[0], m.data()) == UGKS_OK, "moments");
  check(fake::counts.idle_workgroups == 0, "no workgroup without work");
  for (ugks_handle* h : hs) ugks_destroy(h);
  ugks_batch_destroy(b);
}

// The transient buffers of 4 x 10000 cells, 46.6 MB with 17 sums for each ghost cell, fit the static
// scratch.
void static_scratch() {
  Problem p(4, 10000, 2, 2);
  ugks_handle* h = p.create();
  check(ugks_step_static(h, 1) == UGKS_OK, ugks_last_error(h));
  ugks_destroy(h);
}

// Host threads with a solver and a stream each go through the shared pool: every image and every set
// of moments is the caller's own.
void threads_share_the_pool() {
  fake::knobs.image_us = 200;
  std::atomic<int> wrong{0};
  auto work = [&wrong](int t) {
    for (int round = 0; round < 3; ++round) {
      Problem p = t % 2 ? Problem(43, 31, 40, 41) : Problem(40, 10, 24, 24);
      ugks_handle* h = p.create(fake::make_stream(0));
      std::vector<double> f(p.values()), g(p.values()), W(4 * p.cells()), m(4 * p.cells());
      for (size_t k = 0; k < f.size(); ++k) f[k] = 1e6 * (t + 1) + (double)(k % 100003);
      for (int n = 0; n < 3; ++n) {
        if (ugks_set_state(h, f.data(), nullptr) != UGKS_OK || ugks_step(h, 1) != UGKS_OK ||
            ugks_moments(h, m.data()) != UGKS_OK ||
            ugks_get_state(h, g.data(), W.data()) != UGKS_OK || !shifted(f, g, 1.0))
          ++wrong;
        for (size_t c = 0; c < p.cells(); ++c)
          if (m[4 * c] != W[4 * c]) ++wrong;
      }
      ugks_destroy(h);
    }
  };
  std::vector<std::thread> th;
  for (int t = 0; t < 4; ++t) th.emplace_back(work, t);
  for (auto& t : th) t.join();
  check(wrong == 0, "images and moments of several threads");
  check(fake::counts.misuse == 0, "no block given back early");
  check(fake::counts.pinned_live <= 1, "blocks kept without a solver");
}

// Prints the kernels of one step: nx ny nu nv fp32 dof prandtl bc.
void kernels(char** argv) {
  Problem p(std::atoi(argv[0]), std::atoi(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]));
  p.o.precision = std::atoi(argv[4]) ? UGKS_FP32_STORE : UGKS_FP64;
  p.vg.internal_dof = std::atoi(argv[5]);
  p.o.prandtl = std::atof(argv[6]);
  p.bc.kind = std::atoi(argv[7]);
  ugks_handle* h = p.create();
  check(ugks_step(h, 1) == UGKS_OK, "step");
  for (const std::string& name : fake::launched()) std::printf("%s\n", name.c_str());
  ugks_destroy(h);
}

// Host memory runs out while the copying threads start: the images are moved all the same.
std::atomic<int> allocations_left{1 << 30};  // of the library that still succeed
void threads_that_do_not_start() {
  Problem p;
  ugks_handle* h = p.create();
  std::vector<double> f0(p.values()), f(p.values());
  check(ugks_get_state(h, f0.data(), nullptr) == UGKS_OK, "get");
  for (int n = 0; n < 4; ++n) {
    for (double& x : f0) x += 1.0;
    allocations_left = n;
    check(ugks_set_state(h, f0.data(), nullptr) == UGKS_OK, "set");
    allocations_left = n;
    check(ugks_get_state(h, f.data(), nullptr) == UGKS_OK, "get");
    allocations_left = 1 << 30;
    check(f0 == f, "the state set");
  }
  ugks_destroy(h);
}

}  // namespace

void* operator new(size_t n) {
  Dl_info at;
  if (allocations_left < (1 << 20) && dladdr(__builtin_return_address(0), &at) &&
      std::strstr(at.dli_fname, "libugks") && allocations_left.fetch_sub(1) <= 0)
    throw std::bad_alloc();
  void* p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

int main(int argc, char** argv) {
  const std::map<std::string, void (*)()> cases = {
      {"per_thread_stream", per_thread_stream},
      {"other_device", other_device},
      {"set_is_whole", set_is_whole},
      {"no_pinned_memory", no_pinned_memory},
      {"under_capture", under_capture},
      {"one_solver_at_a_time", one_solver_at_a_time},
      {"batch_workgroups", batch_workgroups},
      {"static_scratch", static_scratch},
      {"threads_share_the_pool", threads_share_the_pool},
      {"threads_that_do_not_start", threads_that_do_not_start},
  };
  const auto it = cases.find(argc > 1 ? argv[1] : "");
  if (it != cases.end())
    it->second();
  else if (argc == 10 && std::strcmp(argv[1], "kernels") == 0)
    kernels(argv + 2);
  else
    return 2;
  std::printf("%s: %s\n", argv[1], failures ? "FAILED" : "ok");
  std::fflush(stdout);
  std::_Exit(failures ? 1 : 0);  // the streams' threads never end
}
