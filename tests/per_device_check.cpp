// Two threads set the limit of one kernel: with launches of different sizes, each
// between the other's reading and setting (built with g++ by test_per_device.py).
#include <condition_variable>
#include <cstdio>
#include <mutex>
#include <thread>

#include "per_device.h"

using namespace shot;

int main() {
  std::atomic<unsigned long long> done{0};
  std::mutex m;
  std::condition_variable cv;
  int in = 0, limit = 0, calls = 0;
  // every launch, whatever its size, sets the whole of it, after both are inside
  auto launch = [&](int size) {
    const int st = once_per_device(done, 3, [&]() -> int {
      std::unique_lock<std::mutex> l(m);
      ++in;
      cv.notify_all();
      cv.wait(l, [&] { return in == 2; });
      limit = 160;
      ++calls;
      return 0;
    });
    std::lock_guard<std::mutex> l(m);
    return st == 0 && size <= limit;
  };
  bool a = false, b = false;
  std::thread t([&] { a = launch(150); });
  b = launch(100);
  t.join();
  if (!a || !b || calls != 2) return std::printf("FAIL two threads (%d %d %d)\n", a, b, calls), 1;
  if (!launch(150) || calls != 2) return std::printf("FAIL set again\n"), 1;
  // each device by itself; a failure is not remembered; devices beyond 63 are set every time
  int n = 0;
  auto count = [&] { return ++n, 0; };
  if (once_per_device(done, 4, [&] { return ++n, 7; }) != 7 || once_per_device(done, 4, count) != 0 || n != 2)
    return std::printf("FAIL status\n"), 1;
  for (int k = 0; k < 3; ++k) once_per_device(done, 64, count);
  if (n != 5 || once_per_device(done, 4, count) != 0 || n != 5) return std::printf("FAIL devices (%d)\n", n), 1;
  std::printf("OK\n");
  return 0;
}
