// Set-ups and server admissions on the host HIP runtime (fake_hip.cpp): one
// scenario per run, results as "key value" lines.
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <thread>
#include <vector>

#include "../../include/dcg.h"
#include "fake_hip.hpp"

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

}  // namespace

int main(int argc, char** argv) {
  const std::vector<std::string> a(argv + 1, argv + argc);
  if (a.size() == 4 && a[0] == "room") return room(a[1], std::atoi(a[2].c_str()), std::atoll(a[3].c_str()));
  if (a.size() > 3 && a[0] == "fail")
    return fail(a[1], std::atoi(a[2].c_str()), std::vector<std::string>(a.begin() + 3, a.end()));
  std::fprintf(stderr, "unknown scenario\n");
  return 2;
}
