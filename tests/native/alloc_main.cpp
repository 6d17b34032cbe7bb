// Set-ups and server admissions on the host HIP runtime (fake_hip.cpp): one
// scenario per run, results as "key value" lines.
#include <dlfcn.h>
#include <pthread.h>

#include <cerrno>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <thread>
#include <vector>

#include "../../include/dcg.h"
#include "../../paper_2606_13429_amd/csrc/kernels.hpp"
#include "fake_hip.hpp"

namespace {
std::atomic<int> g_threads{1 << 30};   // threads that can still be started
}

// in the place of the C library's, for the whole process
extern "C" int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*f)(void*), void* arg) {
  static auto real = reinterpret_cast<decltype(&pthread_create)>(dlsym(RTLD_NEXT, "pthread_create"));
  return g_threads-- > 0 ? real(t, a, f, arg) : EAGAIN;
}

namespace {

constexpr size_t kMatrix = size_t(4096) * 4096 * 8;   // a dense map of the coarse cycles

void put(const char* key, int64_t v) { std::printf("%s %lld\n", key, (long long)v); }

void put_left_over() {   // after everything was destroyed
  put("left_bytes", fake::live_bytes());
  put("left_objects", fake::state().objects);
  put("bad_frees", fake::state().bad_frees);
  put("device", fake::state().device);
}

// ---- set-up of one handle
struct Handle {
  dcg_handle h2 = nullptr;
  dcg3d_handle h3 = nullptr;
  dcg_status create(const std::string& what, int n) {
    dcg_mesh mesh{};
    dcg_options opt{};
    dcg_defaults(&mesh, &opt);
    mesh.n = n;
    if (what == "3d") {
      opt.prec = DCG_FP64;
      return dcg3d_setup(n, 40.0, 1e-3, 1.0, DCG3D_INNER_MG, &opt, &h3);
    }
    if (what == "omg") {
      opt.outer = DCG_OUTER_FCG;
      opt.outer_mg = 2;
      opt.inner = DCG_INNER_EXACT;
    }
    if (what == "fp64") opt.prec = DCG_FP64;
    return dcg_setup(&mesh, 1e-3, 1.0, &opt, &h2);
  }
  void destroy() {
    if (h2) dcg_destroy(h2);
    if (h3) dcg3d_destroy(h3);
    h2 = nullptr;
    h3 = nullptr;
    dcg_clear_cache();
  }
};

// What a set-up with all the memory it wants takes.
int64_t clean(const std::string& what, int n) {
  fake::State& s = fake::state();
  Handle h;
  put("clean_status", h.create(what, n));
  const int64_t bytes = fake::live_bytes();
  put("clean_bytes", bytes);
  put("clean_matrices", fake::live_blocks(kMatrix));
  put("clean_calls", s.malloc_calls);
  h.destroy();
  put("clean_left", fake::live_bytes());
  return bytes;
}

// room WHAT N BYTES: a device with BYTES less than the set-up's peak.
int room(const std::string& what, int n, int64_t less) {
  fake::State& s = fake::state();
  clean(what, n);
  Handle h;
  s.capacity = s.peak - less;
  put("status", h.create(what, n));
  put("bytes", fake::live_bytes());
  put("matrices", fake::live_blocks(kMatrix));
  put("last_error", hipGetLastError());
  h.destroy();
  put_left_over();
  return 0;
}

// fail WHAT N CALL...: a set-up whose allocation CALL fails, then one without a
// failure on what the first left in the cache.
int fail(const std::string& what, int n, const std::vector<std::string>& calls) {
  fake::State& s = fake::state();
  const int64_t bytes = clean(what, n);
  int64_t refused = 0, again_ok = 0, again_equal = 0;
  for (const std::string& c : calls) {
    Handle h, again;
    s.fail_call = s.malloc_calls + std::atoll(c.c_str());
    refused += h.create(what, n) == DCG_ENOMEM;
    s.fail_call = -1;
    again_ok += again.create(what, n) == DCG_OK;
    again_equal += fake::live_bytes() == bytes;
    h.destroy();
    again.destroy();
  }
  put("refused", refused);
  put("again_ok", again_ok);
  put("again_equal", again_equal);
  put_left_over();
  return 0;
}

// ---- the server
struct Server {
  dcg_server s = nullptr;
  dcg_options opt{};
  std::vector<std::vector<double>> b, x;
  Server(int64_t budget, bool fp32) {
    dcg_defaults(nullptr, &opt);
    opt.prec = fp32 ? DCG_MIXED : DCG_FP64;
    opt.hbm_budget_bytes = budget;
    opt.max_inner = 1 << 30;   // a request whose residual never falls stays in its first inner solve
    dcg_server_create(&opt, &s);
  }
  ~Server() {
    dcg_server_destroy(s);
    dcg_clear_cache();
  }
  uint64_t submit(int n, int pre = 2) {
    uint64_t t = 0;
    dcg_mesh m = mesh(n);
    m.pre = pre;
    b.emplace_back(size_t(16) * n * n);
    x.emplace_back(size_t(16) * n * n);
    if (dcg_submit(s, &m, 1e-3, 1.0, b.back().data(), x.back().data(), 1e-8, &t) != DCG_OK) std::abort();
    return t;
  }
  dcg_status wait(uint64_t t) {
    for (int i = 0; i < 60000; ++i) {
      const dcg_status st = dcg_poll(s, t, nullptr);
      if (st != DCG_PENDING) return st;
      std::this_thread::sleep_for(std::chrono::milliseconds(1));
    }
    return DCG_PENDING;
  }
  static dcg_mesh mesh(int n) {
    dcg_mesh m{};
    dcg_defaults(&m, nullptr);
    m.n = n;
    return m;
  }
};

int64_t group_bytes(int n, bool fp32) {
  const dcg_mesh m = Server::mesh(n);
  return dcg_server_group_bytes(&m, fp32 ? DCG_MIXED : DCG_FP64);
}

// The scalars the scheduler reads from a device that is busy: residuals that never fall.
void keep_busy(void* dst, size_t bytes) {
  if (bytes != sizeof(dcg::Scalars) * dcg::kBatch) return;
  for (int i = 0; i < dcg::kBatch; ++i) {
    dcg::Scalars& s = static_cast<dcg::Scalars*>(dst)[i];
    s.b2 = s.rho = s.s2 = s.r2 = 1.0;
  }
  std::this_thread::sleep_for(std::chrono::microseconds(50));
}

bool eventually(const std::function<bool()>& f) {
  for (int i = 0; i < 10000; ++i) {
    if (f()) return true;
    std::this_thread::sleep_for(std::chrono::milliseconds(1));
  }
  return false;
}

// budget N FP32 BYTES: one request on a server of that budget (0: what
// dcg_server_group_bytes says).
int budget(int n, bool fp32, int64_t bytes) {
  const int64_t group = group_bytes(n, fp32);
  put("group", group);
  {
    Server s(bytes ? bytes : group, fp32);
    put("status", s.wait(s.submit(n)));
    put("matrices", fake::live_blocks(kMatrix));
    put("products", fake::launched("k_fold_b"));
  }
  put_left_over();
  return 0;
}

// shared BYTES: two long requests whose groups take the matrix, and a third whose
// group has room beside theirs only without.
int shared(int64_t bytes) {
  {
    Server s(bytes, false);
    fake::state().on_read = keep_busy;
    const uint64_t a = s.submit(64), c = s.submit(128);
    put("taken", eventually([] { return fake::live_blocks(kMatrix) == 2; }));
    const uint64_t d = s.submit(256);
    const int64_t groups = group_bytes(64, false) + group_bytes(128, false) + group_bytes(256, false);
    put("admitted", eventually([&] { return fake::live_bytes() >= groups; }));
    put("running", (dcg_poll(s.s, a, nullptr) == DCG_PENDING) + (dcg_poll(s.s, c, nullptr) == DCG_PENDING));
    put("over_budget", fake::live_bytes() - bytes);
    fake::state().on_read = nullptr;
    put("status_64", s.wait(a));
    put("status_128", s.wait(c));
    put("status_256", s.wait(d));
  }
  put_left_over();
  return 0;
}

// evicted BYTES: the group of a mesh that a handle holds too is freed for another.
// The seven vectors of a group of n = 256 are as large as a matrix.
int evicted(int64_t bytes) {
  {
    Server s(bytes, false);
    dcg_options o{};
    const dcg_mesh m = Server::mesh(64);
    dcg_defaults(nullptr, &o);
    o.prec = DCG_FP64;
    o.levels = 1;
    dcg_handle h = nullptr;
    put("handle", dcg_setup(&m, 1e-3, 1.0, &o, &h));
    put("status", s.wait(s.submit(64)));
    put("with_64", fake::live_blocks(kMatrix));
    put("status_256", s.wait(s.submit(256)));
    put("with_256", fake::live_blocks(kMatrix));
    put("status_again", s.wait(s.submit(256, 3)));
    put("after", fake::live_blocks(kMatrix));
    dcg_destroy(h);
  }
  put_left_over();
  return 0;
}

// prepared BYTES: a mesh prepared on a server that has no room for its matrix any
// more when the group comes.
int prepared(int64_t bytes) {
  {
    Server s(bytes, false);
    const dcg_mesh m = Server::mesh(64);
    put("status_256", s.wait(s.submit(256)));
    put("status_128", s.wait(s.submit(128)));
    put("before", fake::live_blocks(kMatrix));
    put("prepare", dcg_server_prepare(s.s, &m));
    put("prepared", fake::live_blocks(kMatrix));
    put("status", s.wait(s.submit(64)));
    put("after", fake::live_blocks(kMatrix));
    put("over_budget", fake::live_bytes() - bytes);
  }
  put_left_over();
  return 0;
}

// threads STARTED: the outer multigrid's tables where only that many threads can be
// started.
int threads(int started) {
  std::vector<double> want(1024 * 1024), got(want.size());
  put("clean_status", dcg_host_outer_mg(16, 10.0, 1e-3, 1.0, 1, 2, want.data(), int64_t(want.size())));
  g_threads = started;
  put("status", dcg_host_outer_mg(16, 10.0, 1e-3, 1.0, 1, 2, got.data(), int64_t(got.size())));
  put("equal", std::memcmp(want.data(), got.data(), got.size() * sizeof(double)) == 0);
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  const std::vector<std::string> a(argv + 1, argv + argc);
  if (a.size() == 4 && a[0] == "room") return room(a[1], std::atoi(a[2].c_str()), std::atoll(a[3].c_str()));
  if (a.size() > 3 && a[0] == "fail")
    return fail(a[1], std::atoi(a[2].c_str()), std::vector<std::string>(a.begin() + 3, a.end()));
  if (a.size() == 4 && a[0] == "budget")
    return budget(std::atoi(a[1].c_str()), a[2] == "1", std::atoll(a[3].c_str()));
  if (a.size() == 2 && a[0] == "shared") return shared(std::atoll(a[1].c_str()));
  if (a.size() == 2 && a[0] == "evicted") return evicted(std::atoll(a[1].c_str()));
  if (a.size() == 2 && a[0] == "prepared") return prepared(std::atoll(a[1].c_str()));
  if (a.size() == 2 && a[0] == "threads") return threads(std::atoi(a[1].c_str()));
  std::fprintf(stderr, "unknown scenario\n");
  return 2;
}
