// The matrix-core plans of sparse fractals up to the largest level that a
// descriptor may have: what nbb_create works out for each, within an address
// space of 1 GiB.  Prints the number of descriptors and the longest time.
#include <sys/resource.h>

#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "plan.hpp"
using namespace nbb;

int main() {
    const rlimit lim{1u << 30, 1u << 30};
    if (setrlimit(RLIMIT_AS, &lim) != 0) return 2;
    const std::vector<std::pair<uint32_t, std::vector<int32_t>>> sparse = {
        {2, {0, 0, 1, 1}}, {3, {0, 0, 2, 0}}, {3, {0, 0, 2, 2}},       {4, {0, 0, 3, 0}},
        {4, {0, 0, 1, 1}}, {4, {2, 1, 2, 2}}, {4, {0, 0, 3, 0, 1, 3}}, {4, {0, 0, 3, 0, 0, 3, 3, 3}}};
    int made = 0;
    double longest = 0.0;
    for (const auto &n : sparse)
        for (uint32_t r = 1;; ++r) {
            Fractal f;
            std::string msg;
            if (validate_fractal(uint32_t(n.second.size() / 2), n.first, n.second.data(), r, &f, &msg)) break;
            const auto t0 = std::chrono::steady_clock::now();
            const std::vector<MatDims> md = mat_dims(f);
            const std::vector<HoldDims> hd = hold_dims(f);
            uint32_t gpw = 0;
            HoldDims d{};
            MatPlan p;
            HoldPlan h;
            const uint32_t m = pick_mat_level(md, f.k, {r}, 256, &gpw);
            if (m && !build_mat_plan(f, m, gpw, &p, &msg, false)) std::abort();
            if (pick_hold(hd, f.k, {r}, 256, &d, &gpw) && !build_hold_plan(f, d.m, d.rings, gpw, &h, &msg)) std::abort();
            const std::chrono::duration<double> t = std::chrono::steady_clock::now() - t0;
            longest = t.count() > longest ? t.count() : longest;
            ++made;
        }
    std::printf("%d %.3f\n", made, longest);
    return 0;
}
