// Threads count themselves in at one count (csrc/arrival.h), as workgroups of several launches would.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

#include "arrival.h"

struct HostCount {
    std::atomic<uint32_t>* x;
    uint32_t next(uint32_t limit) {
        uint32_t v = x->load();
        while (!x->compare_exchange_weak(v, v >= limit ? 0 : v + 1)) {}
        return v;
    }
};

int main(int argc, char** argv) {
    const int launches = argc > 1 ? std::atoi(argv[1]) : 1, parts = argc > 2 ? std::atoi(argv[2]) : 3, rounds = 20000;
    std::atomic<uint32_t> count{0};
    std::atomic<int> started{0}, done{0}, lasts{0};
    int bad = 0;
    std::vector<std::thread> pool;
    const int n = launches * parts;
    for (int t = 0; t < n; ++t)
        pool.emplace_back([&] {
            for (int r = 0; r < rounds; ++r) {
                ++started;
                while (started.load() < n * (r + 1)) std::this_thread::yield();
                if (pk::arrives_last(HostCount{&count}, static_cast<uint32_t>(parts))) ++lasts;
                if (done.fetch_add(1) == n * (r + 1) - 1) {            // the others wait for this thread to start the next round
                    if (count.load() != 0 || lasts.load() != launches) ++bad;
                    count = 0;
                    lasts = 0;
                }
            }
        });
    for (auto& t : pool) t.join();
    std::printf("%d launches of %d parts: %d bad rounds\n", launches, parts, bad);
    return bad != 0;
}
