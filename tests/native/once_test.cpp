// once_per_device (csrc/once.h) with several threads: no caller returns before
// the one-time work is done, it is done once per device, and tried again after
// a failure.
#include "../../paper_2608_01845_amd/csrc/once.h"

#include <chrono>
#include <cstdio>
#include <thread>
#include <vector>

static int fail(const char *what) {
  std::fprintf(stderr, "FAIL: %s\n", what);
  return 1;
}

int main() {
  static wdc::DeviceOnce once;
  std::atomic<int> runs{0}, ready{0}, early{0};
  std::vector<std::thread> ts;
  for (int i = 0; i < 8; ++i)
    ts.emplace_back([&] {
      const int e = wdc::once_per_device(once, 0, [&] {
        ++runs;
        std::this_thread::sleep_for(std::chrono::milliseconds(100));
        ready = 1;
        return 0;
      });
      if (e != 0 || !ready) ++early;
    });
  for (auto &t : ts) t.join();
  if (early) return fail("a thread went on before the work was done");
  if (runs != 1) return fail("not done once");
  int n = 0;
  auto fails_first = [&] { return ++n == 1 ? 7 : 0; };
  if (wdc::once_per_device(once, 3, fails_first) != 7 || wdc::once_per_device(once, 3, fails_first) != 0 ||
      wdc::once_per_device(once, 3, fails_first) != 0 || n != 2)
    return fail("a failure is returned, the work tried again, then kept");
  n = 1;
  for (int dev : {-1, 64, 1 << 20}) wdc::once_per_device(once, dev, fails_first);
  if (n != 4) return fail("devices outside the array always run it");
  std::puts("once_test: ok");
  return 0;
}
