// once_per_device: set-up on every device, once each, again after a failure.
#include <cstdio>

#include "../../paper_1306_2461_amd/csrc/device_once.h"

int main() {
  std::atomic<uint64_t> done{0};
  int calls = 0, fail = 0, bad = 0;
  auto run = [&](int device) {
    return ofmi::once_per_device(done, device, 0, [&] {
      ++calls;
      return fail;
    });
  };
  auto expect = [&](int device, int want, int error) {
    calls = 0;
    const int e = run(device);
    if (calls != want || e != error) ++bad, std::printf("device %d: %d calls, error %d\n", device, calls, e);
  };
  expect(0, 1, 0), expect(0, 0, 0);
  expect(1, 1, 0), expect(0, 0, 0), expect(1, 0, 0);   // the second device is set up too
  fail = 7;
  expect(0, 0, 0), expect(63, 1, 7);
  fail = 0;
  expect(63, 1, 0), expect(63, 0, 0);                  // a failure is not kept
  expect(64, 1, 0), expect(64, 1, 0);
  return bad;
}
