// Controls and counters of the host HIP runtime in fake_hip.cpp.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <map>
#include <string>

namespace fake {

struct State {
  std::atomic<int64_t> capacity{int64_t(288) << 30};   // bytes of the device
  std::atomic<int64_t> fail_call{-1};                  // this hipMalloc fails
  std::atomic<int64_t> malloc_calls{0}, peak{0}, bad_frees{0};
  std::atomic<int64_t> objects{0};                     // streams, events, graphs, pinned blocks
  std::atomic<int> device{0};
  std::atomic<void (*)(void*, size_t)> on_read{nullptr};   // sees every asynchronous copy to the host
};

State& state();
int64_t live_bytes();
int64_t live_blocks(size_t size);                  // live allocations of that size (0: all)
int64_t launched(const std::string& kernel);       // launches of kernels with this in their name

}  // namespace fake
