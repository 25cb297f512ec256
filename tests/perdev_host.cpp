// c3::PerDevice on the host: once per device, a failure is tried again, threads
// that come together run it once.
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>

#include "../paper_2201_03509_amd/csrc/perdev.h"

int main() {
    c3::PerDevice p;
    int runs[3] = {0, 0, 0};
    auto go = [&](int dev, int status) {
        return p.once<int>(dev, [&] {
            ++runs[dev];
            return status;
        });
    };
    if (go(0, 0) != 0 || go(0, 7) != 0 || runs[0] != 1) return 1;  // done: not run again
    if (go(1, 5) != 5 || go(1, 0) != 0 || go(1, 5) != 0 || runs[1] != 2) return 2;  // its own, and after a failure
    if (go(0, 0) != 0 || runs[0] != 1) return 3;
    std::atomic<int> n{0};
    std::vector<std::thread> th;
    for (int i = 0; i < 8; ++i)
        th.emplace_back([&] {
            for (int d = 10; d < 20; ++d) p.once<int>(d, [&] { return ++n, 0; });
        });
    for (auto &t : th) t.join();
    if (n != 10) return 4;
    puts("per device ok");
    return 0;
}
