// Host check of the on-chip layout's limit on word rows: the kernel's byte
// offsets are 32-bit, so a matrix whose words or values would reach past 2^32
// bytes is refused, before any of its entries is laid out (only the first few
// exist here).
#include <cstdio>
#include <vector>

#include "resident_layout.h"

using vne::resident_max_word_rows;

// n rows of `row` entries each, of which the first eight are there
static bool built(int64_t n, int64_t row, double second, bool fp64, int rounds) {
    std::vector<int32_t> rp(n + 1), ci = {1, 2, 3, 4, 5, 6, 7, 8};
    for (int64_t i = 0; i <= n; ++i) rp[i] = (int32_t)(i * row);
    std::vector<double> va(8, 1.0);
    va[1] = second;
    vne::ResidentLayout L;
    return vne::build_resident_layout(rp.data(), ci.data(), va.data(), n, 16, rounds, &L, fp64);
}

int main() {
    for (int fp64 = 0; fp64 < 2; ++fp64) {
        const int64_t pair = fp64 ? 16 : 8;
        // the last byte of the last row, and no row left out
        if (resident_max_word_rows(false, fp64) * 64 * pair != int64_t(1) << 32) return std::puts("FAIL values"), 1;
        if (resident_max_word_rows(true, fp64) * 256 != int64_t(1) << 32) return std::puts("FAIL words"), 1;
    }
    // unequal values, FP32: 33 000 rows of 33 000 entries (1.09e9) need 8.5e6 word rows
    if (built(33000, 33000, 2.0, false, 39)) return std::puts("FAIL FP32 matrix past the limit"), 1;
    // FP64, 19 000 rows of 32 000 entries (duplicates or not, the count is what matters): 4.7e6
    if (built(19000, 32000, 2.0, true, 19)) return std::puts("FAIL FP64 matrix past the limit"), 1;
    std::puts("ok");
    return 0;
}
