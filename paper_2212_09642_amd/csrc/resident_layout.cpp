// Builds the row layout of the on-chip Lanczos kernel (see resident_layout.h).
#include "resident_layout.h"

#include <algorithm>
#include <numeric>

namespace vne {

bool build_resident_layout(const int32_t *row_ptr, const int32_t *col, const double *val, int64_t n, int32_t waves,
                           int32_t max_rounds, ResidentLayout *out, bool fp64) {
    if (n < 1 || waves < 1 || waves > 16 || n > (int64_t)waves * max_rounds * 64) return false;
    ResidentLayout L;
    L.waves = waves;
    // one value for every off-diagonal entry?
    L.unit = true;
    bool seen = false;
    for (int64_t i = 0; i < n && L.unit; ++i)
        for (int32_t p = row_ptr[i]; p < row_ptr[i + 1]; ++p) {
            if (col[p] == i) continue;
            if (!seen) {
                L.off_value = val[p];
                seen = true;
            } else if (val[p] != L.off_value) {
                L.unit = false;
                break;
            }
        }
    // entries of a row in words (its own entry is not among them when unit)
    std::vector<int32_t> len(n);
    int64_t total = 0;
    for (int64_t i = 0; i < n; ++i) {
        int32_t c = row_ptr[i + 1] - row_ptr[i];
        if (L.unit)
            for (int32_t p = row_ptr[i]; p < row_ptr[i + 1]; ++p) c -= col[p] == i;
        len[i] = c;
        total += c;
    }
    // rows by falling length; the ones above half a wave's share are long
    std::vector<int32_t> order(n);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return len[a] > len[b]; });
    const int64_t long_min = std::max<int64_t>(32, total / 64 / waves / 2);
    int64_t n_long = 0;
    while (n_long < n && len[order[n_long]] > long_min) ++n_long;
    n_long = std::min<int64_t>(n_long, 64 * (int64_t)waves);
    const int64_t n_short = (n - n_long + 63) / 64;
    L.rounds = (int32_t)((n_long > 0 ? 1 : 0) + (n_short + waves - 1) / waves);
    if (L.rounds > max_rounds || L.positions() > kResidentMaxPositions) return false;
    int64_t word_rows = kResidentSpareRows;
    for (int64_t q = 0; q < n_long; ++q) word_rows += (len[order[q]] + 127) / 128;
    for (int64_t a = n_long; a < n; a += 64) word_rows += (len[order[a]] + 3) / 4 * 2;
    if (word_rows > resident_max_word_rows(L.unit, fp64)) return false;
    // slices to waves: long rows in turn, then the short slices, longest
    // first, to the wave with the least work that has room
    std::vector<std::vector<std::pair<int64_t, int64_t>>> of_wave(waves);   // {first in order, rows}, -1 - w: long
    std::vector<int64_t> cost(waves, 0);
    std::vector<std::vector<int32_t>> long_rows(waves);
    for (int64_t q = 0; q < n_long; ++q) {
        const int w = (int)(q % waves);
        long_rows[w].push_back(order[q]);
        cost[w] += 2 * ((len[order[q]] + 127) / 128) + 8;
    }
    const int32_t cap = L.rounds - (n_long > 0 ? 1 : 0);
    for (int64_t s = 0; s < n_short; ++s) {
        const int64_t a = n_long + 64 * s;
        int best = -1;
        for (int w = 0; w < waves; ++w)
            if ((int32_t)of_wave[w].size() < cap && (best < 0 || cost[w] < cost[best])) best = w;
        of_wave[best].push_back({a, std::min<int64_t>(64, n - a)});
        cost[best] += len[order[a]] + 6;
    }
    L.slices.assign((size_t)waves * L.rounds * 4, 0);
    L.row_of.assign(L.positions(), -1);
    std::vector<int32_t> pos(n);
    auto place = [&](int w, int r, int lane, int32_t row) {
        const int32_t p = (w * L.rounds + r) * 64 + lane;
        L.row_of[p] = row;
        pos[row] = p;
    };
    const int r0 = n_long > 0 ? 1 : 0;
    for (int w = 0; w < waves; ++w) {
        for (size_t q = 0; q < long_rows[w].size(); ++q) place(w, 0, (int)q, long_rows[w][q]);
        for (size_t r = 0; r < of_wave[w].size(); ++r)
            for (int64_t q = 0; q < of_wave[w][r].second; ++q)
                place(w, r0 + (int)r, (int)q, order[of_wave[w][r].first + q]);
    }
    const uint32_t zero = (uint32_t)L.positions();
    const uint32_t pad = zero | (zero << 16);
    auto put = [&](size_t word, int half, uint32_t position, double v) {
        L.words[word] = half ? (L.words[word] & 0xffffu) | (position << 16) : (L.words[word] & 0xffff0000u) | position;
        if (!L.unit) L.vals[2 * word + half] = v;
    };
    auto grow = [&](size_t rows64) {
        const size_t first = L.words.size() / 64;
        L.words.resize(L.words.size() + rows64 * 64, pad);
        if (!L.unit) L.vals.resize(2 * L.words.size(), 0.0);
        return first;
    };
    for (int w = 0; w < waves; ++w)
        for (int r = 0; r < L.rounds; ++r) {
            int32_t *sl = &L.slices[4 * ((size_t)w * L.rounds + r)];
            const int32_t *rows = &L.row_of[((size_t)w * L.rounds + r) * 64];
            int count = 0, most = 0;
            for (int l = 0; l < 64; ++l)
                if (rows[l] >= 0) {
                    ++count;
                    most = std::max(most, len[rows[l]]);
                }
            if (count == 0) continue;
            const bool is_long = n_long > 0 && r == 0;
            sl[3] = count;
            if (!is_long) {
                const int words = (most + 3) / 4 * 2;
                const size_t first = grow(words);
                sl[0] = 1;
                sl[1] = (int32_t)first;
                sl[2] = words;
                L.gathers += 2 * words;
                for (int l = 0; l < 64; ++l) {
                    if (rows[l] < 0) continue;
                    int e = 0;
                    for (int32_t p = row_ptr[rows[l]]; p < row_ptr[rows[l] + 1]; ++p) {
                        if (L.unit && col[p] == rows[l]) continue;
                        put((first + e / 2) * 64 + l, e & 1, (uint32_t)pos[col[p]], val[p]);
                        ++e;
                    }
                }
            } else {
                sl[0] = 2;
                sl[1] = (int32_t)(L.spans.size() / 2);
                for (int l = 0; l < count; ++l) {
                    const int words = (len[rows[l]] + 127) / 128;
                    const size_t first = grow(words);
                    L.spans.push_back((int32_t)first);
                    L.spans.push_back(words);
                    L.gathers += 2 * words;
                    int e = 0;
                    for (int32_t p = row_ptr[rows[l]]; p < row_ptr[rows[l] + 1]; ++p) {
                        if (L.unit && col[p] == rows[l]) continue;
                        put((first + e / 128) * 64 + (e % 128) / 2, e & 1, (uint32_t)pos[col[p]], val[p]);
                        ++e;
                    }
                }
            }
        }
    grow(kResidentSpareRows);
    if (L.unit) {
        L.diag.assign(L.positions(), 0.0);
        for (int64_t i = 0; i < n; ++i)
            for (int32_t p = row_ptr[i]; p < row_ptr[i + 1]; ++p)
                if (col[p] == i) L.diag[pos[i]] = val[p];
    }
    *out = std::move(L);
    return true;
}

}  // namespace vne
