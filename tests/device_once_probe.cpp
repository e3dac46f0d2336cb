// Host build of the once-per-device flag for tests/test_device_once_cpu.py.
#include <thread>
#include <vector>

#include "../paper_2406_17404_amd/csrc/device_once.h"

// how often the work was done in `n` calls for the given devices; the first `fail` of them fail
extern "C" int trj_test_once(const int* device, int n, int fail) {
  trj::DeviceOnce once;
  int calls = 0;
  for (int i = 0; i < n; ++i) once.run(device[i], [&] { return ++calls <= fail ? 1 : 0; });
  return calls;
}
// devices (of 64) for which no thread of eight did the work before it came back
extern "C" int trj_test_once_threads() {
  trj::DeviceOnce once;
  std::atomic<int> done[64]{}, missed{0};
  std::vector<std::thread> all;
  for (int t = 0; t < 8; ++t)
    all.emplace_back([&] {
      for (int d = 0; d < 64; ++d) {
        once.run(d, [&] { return done[d].fetch_add(1), 0; });
        if (done[d].load() == 0) ++missed;
      }
    });
  for (auto& t : all) t.join();
  return missed;
}
