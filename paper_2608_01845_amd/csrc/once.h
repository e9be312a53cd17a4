// One-time work per device (kernel attributes such as the dynamic LDS limit are
// set per device), safe with several host threads. Host code only.
#pragma once

#include <atomic>
#include <mutex>

namespace wdc {

struct DeviceOnce {
  static constexpr int kDevices = 64;
  std::mutex mu;
  std::atomic<bool> done[kDevices] = {};
};

// Runs fn for device dev unless a call before has succeeded there; a call that
// finds another one at it waits for it. fn returns an error code, 0 (R{}) for
// success; after a failure the next call tries again. A device id outside the
// array (a failed query) always runs fn.
template <class F>
auto once_per_device(DeviceOnce &o, int dev, F &&fn) -> decltype(fn()) {
  using R = decltype(fn());
  if (dev < 0 || dev >= DeviceOnce::kDevices) return fn();
  if (o.done[dev].load(std::memory_order_acquire)) return R{};
  std::lock_guard<std::mutex> lock(o.mu);
  if (o.done[dev].load(std::memory_order_relaxed)) return R{};
  const R r = fn();
  if (r == R{}) o.done[dev].store(true, std::memory_order_release);
  return r;
}

}  // namespace wdc
