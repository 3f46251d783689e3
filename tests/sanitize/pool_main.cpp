// IdlePool (gp_pool.h): by device, bounded, every resource with one holder at a time.
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>

#include "../../paper_2407_03608_amd/csrc/gp_pool.h"

static int failures = 0;
#define CHECK(c)                                                \
  do {                                                          \
    if (!(c)) {                                                 \
      ++failures;                                               \
      std::printf("line %d: %s\n", __LINE__, #c);               \
    }                                                           \
  } while (0)

int main() {
  {
    gp::IdlePool<int> p(2);
    int r = -1;
    CHECK(!p.take(0, &r));
    CHECK(p.put(0, 10) && p.put(1, 11) && !p.put(0, 12));  // bounded over all devices
    CHECK(p.take(1, &r) && r == 11);
    CHECK(!p.take(1, &r));
    CHECK(p.take(0, &r) && r == 10 && !p.take(0, &r));
  }
  // threads that take, or make what they do not get, and give back
  gp::IdlePool<int> pool(4);
  std::atomic<int> made{0}, live{0};
  std::vector<std::atomic<int>> held(4096);
  std::atomic<int> clashes{0};
  std::vector<std::thread> ts;
  for (int t = 0; t < 8; ++t)
    ts.emplace_back([&, t] {
      for (int i = 0; i < 400; ++i) {
        int r;
        if (!pool.take(t % 2, &r)) {
          r = made++;
          ++live;
        }
        if (held[r].exchange(1)) ++clashes;
        std::this_thread::yield();
        held[r] = 0;
        if (!pool.put(t % 2, r)) --live;
      }
    });
  for (auto& t : ts) t.join();
  CHECK(clashes == 0);
  CHECK(live <= 4);
  std::printf("%d failures\n", failures);
  return failures != 0;
}
