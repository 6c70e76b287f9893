// Host check of what the step's front blocks of long rows are reckoned to
// cost (against a direct count), and of the rule on it: hubs whose chain would
// outlast the step and matrices of mostly long rows keep the launch behind,
// preferential attachment and a few moderate hubs do not.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "internal.h"

using namespace vne;

static std::vector<int32_t> row_ptr(const std::vector<int32_t> &deg) {
    std::vector<int32_t> rp(1, 0);
    for (int32_t d : deg) rp.push_back(rp.back() + d);
    return rp;
}

static Schedule make(const std::vector<int32_t> &deg) {
    const std::vector<int32_t> rp = row_ptr(deg);
    const int64_t n = (int64_t)deg.size(), cost = rp.back() + 4 * n;
    return build_schedule(rp.data(), n, 64, std::max<int64_t>(256, (cost + 1023) / 1024), 1024);
}

static bool rule(const std::vector<int32_t> &deg, int m, int tile, bool fp64) {
    return long_rows_first(make(deg), row_ptr(deg).back(), m, tile, fp64);
}

int main() {
    std::mt19937_64 rng(5);
    for (int rep = 0; rep < 20; ++rep) {
        std::vector<int32_t> deg(300 + rng() % 700);
        for (int32_t &d : deg) d = (int32_t)(rng() % 40 == 0 ? 1 + rng() % 5000 : 1 + rng() % 70);
        const Schedule s = make(deg);
        std::vector<int32_t> big;
        for (int32_t d : deg)
            if (d > 64) big.push_back(d);
        if ((int)big.size() != s.n_long) return std::puts("FAIL long rows"), 1;
        for (int i = 0; i < kLaneClasses; ++i) {
            const int per = i <= 2 ? 4 : i == 3 ? 2 : 1;
            double most = 0.0, idle = 0.0;
            for (size_t a = 0; a < big.size(); a += per) {
                double r = 0.0;
                for (size_t q = a; q < std::min(big.size(), a + per); ++q) r += big[q];
                r /= 64.0 * (256 / (1 << i));
                most = std::max({most, r, 1.0});
                idle += std::max(0.0, 1.0 - r);
            }
            if (std::fabs(most - s.front[i].most) > 1e-5 * most || std::fabs(idle - s.front[i].idle) > 1e-4 * (1 + idle))
                return std::printf("FAIL costs of class %d\n", i), 1;
        }
    }
    if (rule(std::vector<int32_t>(5000, 8), 64, 64, false)) return std::puts("FAIL no long rows"), 1;
    std::vector<int32_t> star(20000, 2), hub(200000, 7), dense(50000, 100), few(20000, 7), pa(50000);
    star[0] = 20000;
    hub[1234] = 80000;
    for (int q = 0; q < 20; ++q) few[100 * q] = 500;
    for (size_t i = 0; i < pa.size(); ++i) pa[i] = 4 + (int32_t)(3 * (std::sqrt(50000.0 / (i + 1.0)) - 1.0));
    for (int fp64 = 0; fp64 < 2; ++fp64)
        for (int tile : {16, 32, 64}) {
            if (rule(star, tile, tile, fp64) || rule(hub, tile, tile, fp64)) return std::puts("FAIL hub at the front"), 1;
            if (rule(dense, tile, tile, fp64)) return std::puts("FAIL long rows throughout"), 1;
            if (!rule(few, tile, tile, fp64) || !rule(pa, tile, tile, fp64)) return std::puts("FAIL few hubs"), 1;
        }
    std::puts("ok");
    return 0;
}
