// Launch shapes of one kernel asked for in turn, by several threads: each is
// queried once (a shape may be asked again by a thread that lost a race, and
// where more shapes are in use than the cache holds).  Prints "ok".
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

#include "occupancy_cache.hpp"

static int expected(uint32_t lds, uint32_t threads) { return 1 + int((lds / 16 + threads / 64) % 200); }

int main() {
    nbb::OccupancyCache one;
    int asked = 0;
    for (int i = 0; i < 1000; ++i) {
        const uint32_t lds = i % 2 ? 9744 : 20304, threads = i % 3 ? 128 : 256;
        int got = 0;
        if (one.get(lds, threads, &got, [&](int *v) {
                ++asked;
                *v = expected(lds, threads);
                return 0;
            }) != 0 || got != expected(lds, threads))
            std::abort();
    }
    if (asked != 4) {
        std::printf("%d queries for 4 shapes\n", asked);
        return 1;
    }
    int got = 7;
    if (one.get(1, 64, &got, [](int *) { return 5; }) != 5) return 1;  // an error is not kept
    if (one.get(1, 64, &got, [](int *v) { return *v = 0; }) != 0 || got != 1) return 1;
    if (one.get(2, 64, &got, [](int *v) { *v = 400; return 0; }) != 0 || got != 255) return 1;
    nbb::OccupancyCache shared;
    std::vector<std::thread> pool;
    for (int t = 0; t < 4; ++t)
        pool.emplace_back([&shared, t] {
            for (uint32_t i = 0; i < 20000; ++i) {
                const uint32_t lds = 16 * ((i * 7 + uint32_t(t)) % 24), threads = 64;
                int v = 0;
                shared.get(lds, threads, &v, [&](int *n) {
                    *n = expected(lds, threads);
                    return 0;
                });
                if (v != expected(lds, threads)) std::abort();
            }
        });
    for (std::thread &t : pool) t.join();
    std::printf("ok\n");
    return 0;
}
