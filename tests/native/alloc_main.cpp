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

// setup WHAT N fail CALL: that allocation fails; then again without a failure.
// setup WHAT N room BYTES: BYTES less than the set-up's peak.
int setup(const std::string& what, int n, const std::string& how, int64_t v) {
  fake::State& s = fake::state();
  {
    Handle h;
    put("clean_status", h.create(what, n));
    put("clean_calls", s.malloc_calls);
    put("clean_peak", s.peak);
    put("clean_bytes", fake::live_bytes());
    put("clean_matrices", fake::live_blocks(kMatrix));
    h.destroy();
    put("clean_left", fake::live_bytes());
  }
  const int64_t peak = s.peak, full = s.capacity;
  Handle h;
  if (how == "fail") s.fail_call = s.malloc_calls + v;
  if (how == "room") s.capacity = peak - v;
  put("status", h.create(what, n));
  put("bytes", fake::live_bytes());
  put("matrices", fake::live_blocks(kMatrix));
  if (h.h2 || h.h3) {   // a set-up that succeeded leaves no error behind
    put("last_error", hipGetLastError());
  }
  s.fail_call = -1;
  s.capacity = full;
  if (how == "fail") {   // the next set-up, on what the failed one left in the cache
    Handle again;
    put("again_status", again.create(what, n));
    h.destroy();
    put("again_bytes", fake::live_bytes());
    again.destroy();
  }
  h.destroy();
  put_left_over();
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  const std::vector<std::string> a(argv + 1, argv + argc);
  if (a.size() == 5 && a[0] == "setup") return setup(a[1], std::atoi(a[2].c_str()), a[3], std::atoll(a[4].c_str()));
  std::fprintf(stderr, "unknown scenario\n");
  return 2;
}
