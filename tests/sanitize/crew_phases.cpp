// Phases of two callers on one crew: short ones must not wait for the other caller's long ones.
#include <algorithm>

#include "common.h"

using namespace hgnn;

int main() {
  Crew &crew = Crew::get();
  crew.join(6, true);
  std::atomic<bool> stop{false};
  std::thread other([&] {   // each of its phases keeps the threads that join it for 60 ms
    while (!stop) crew.parallel_for(3, 6, [](int) { std::this_thread::sleep_for(std::chrono::milliseconds(60)); });
  });
  // a phase of 20 us that helpers take part in; the lists of two callers meet in the same slots
  double worst = 0;
  int late = 0;
  const auto end = std::chrono::steady_clock::now() + std::chrono::seconds(4);
  std::vector<std::thread> callers;
  std::mutex m;
  for (int t = 0; t < 2; ++t)
    callers.emplace_back([&] {
      while (std::chrono::steady_clock::now() < end) {
        const auto a = std::chrono::steady_clock::now();
        crew.parallel_for(4, 6, [](int) {
          const auto t0 = std::chrono::steady_clock::now();
          while (std::chrono::steady_clock::now() - t0 < std::chrono::microseconds(5)) {}
        });
        const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - a).count();
        std::lock_guard<std::mutex> lk(m);
        worst = std::max(worst, ms);
        late += ms > 40;
      }
    });
  for (auto &t : callers) t.join();
  stop = true;
  other.join();
  crew.leave(6, true);
  printf("worst short phase %.2f ms, %d beyond 40 ms\n", worst, late);
  if (late < 2) printf("crew phases ok\n");   // a loaded machine may hold a thread back now and then
  return 0;
}
