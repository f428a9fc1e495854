// Host-only probe of the planners' worker pool, built and run by
// test_host_pool.py: results of loops opened by several threads at once, and
// whether two loops can make progress at the same time.
#include "qs_pool.h"

#include <chrono>
#include <cstdio>
#include <cstdlib>

using qs::HostPool;

// Every index exactly once, for loops of every shape from six threads.
static long wrong_entries() {
    std::atomic<long> wrong{0};
    std::vector<std::thread> callers;
    for (unsigned k = 0; k < 6; ++k)
        callers.emplace_back([&wrong, k] {
            unsigned r = 77 * k + 1;
            for (int it = 0; it < 500; ++it) {
                r = r * 1664525u + 1013904223u;
                const size_t n = (r >> 20) % 40, chunk = (r >> 8) % 5;
                std::vector<int> seen(n, 0);
                HostPool::get().run(n, chunk, (r >> 4) % 18, [&](size_t lo, size_t hi) {
                    for (size_t i = lo; i < hi; ++i) ++seen[i];
                });
                for (int x : seen) wrong += x != 1;
            }
        });
    for (auto &c : callers) c.join();
    return wrong;
}

// A loop whose pieces wait until a second caller's loop has begun: true if it
// began within two seconds.
static bool loops_overlap() {
    std::atomic<bool> begun{false}, first_in{false}, met{false};
    std::thread first([&] {
        HostPool::get().run(2, 1, 2, [&](size_t, size_t) {
            first_in = true;
            for (int i = 0; i < 2000 && !begun; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(1));
            if (begun) met = true;
        });
    });
    while (!first_in) std::this_thread::yield();
    HostPool::get().run(2, 1, 2, [&](size_t, size_t) { begun = true; });
    first.join();
    return met;
}

int main() {
    const long wrong = wrong_entries();
    const bool overlap = loops_overlap();
    std::printf("wrong %ld overlap %d\n", wrong, int(overlap));
    std::fflush(stdout);
    std::_Exit(0);  // the workers are detached
}
