// Host check that the shape of an on-chip layout, which the rule for these runs
// goes by, is the one that is built, and that longer rows are reckoned dearer.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "resident_layout.h"

using namespace vne;

int main() {
    std::mt19937_64 rng(3);
    for (int rep = 0; rep < 60; ++rep) {
        const int n = 1 + (int)(rng() % 3000), deg = 1 + (int)(rng() % 90);
        const bool unit = rng() & 1, fp64 = rng() & 1;
        std::vector<int32_t> rp(1, 0), ci;
        std::vector<double> va;
        for (int i = 0; i < n; ++i) {
            const int len = std::min(n, (int)(rng() % 97 == 0 ? rng() % (n + 1) : rng() % (deg + 1)));
            const int from = (int)(rng() % n);
            std::vector<int32_t> row;
            for (int q = 0; q < len; ++q) row.push_back((from + q) % n);
            std::sort(row.begin(), row.end());
            for (int32_t c : row) {
                ci.push_back(c);
                va.push_back(unit ? -1.0 : 1.0 + (double)(rng() % 5));
            }
            rp.push_back((int32_t)ci.size());
        }
        for (int waves : {1, 4, 16}) {
            ResidentLayout L;
            ResidentShape s;
            ResidentRows rows;
            const bool built = build_resident_layout(rp.data(), ci.data(), va.data(), n, waves, 19, &L, fp64);
            if (built != resident_shape(rp.data(), ci.data(), va.data(), n, waves, 19, fp64, &s, &rows))
                return std::puts("FAIL one fits"), 1;
            if (!built) continue;
            int64_t most_rows = 0, most_tail = 0;
            for (int w = 0; w < waves; ++w) {
                int64_t rows = 0, tail = 0;
                for (int r = 0; r < L.rounds; ++r) {
                    const int32_t *sl = &L.slices[4 * (w * L.rounds + r)];
                    if (sl[0] != 2) continue;
                    rows += sl[3];
                    for (int l = 0; l < sl[3]; ++l) tail += L.spans[2 * (sl[1] + l) + 1] - 1;
                }
                most_rows = std::max(most_rows, rows);
                most_tail = std::max(most_tail, tail);
            }
            if (s.waves != waves || s.rounds != L.rounds || s.unit != L.unit || s.off_value != L.off_value ||
                s.word_rows * 64 != (int64_t)L.words.size() || s.wave_long != most_rows || s.wave_tail != most_tail)
                return std::printf("FAIL shape n=%d waves=%d\n", n, waves), 1;
        }
    }
    ResidentShape a, b;
    a.waves = b.waves = 16;
    a.rounds = b.rounds = 30;
    a.unit = b.unit = true;
    a.word_rows = b.word_rows = 1200;
    b.wave_long = 1;
    b.wave_tail = 234;           // one row of 30 000 entries
    if (resident_step_us(b, 1, false) < resident_step_us(a, 1, false) + 50.0) return std::puts("FAIL hub"), 1;
    std::puts("ok");
    return 0;
}
