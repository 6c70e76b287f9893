// Builds the row layout of the on-chip Lanczos kernel (see resident_layout.h).
#include "resident_layout.h"

#include <algorithm>

namespace vne {

namespace {

// a row's entries in words (its own entry is not among them when unit)
std::vector<int32_t> row_lengths(const int32_t *row_ptr, const int32_t *col, int64_t n, bool unit) {
    std::vector<int32_t> len(n);
    for (int64_t i = 0; i < n; ++i) {
        int32_t c = row_ptr[i + 1] - row_ptr[i];
        if (unit)
            for (int32_t p = row_ptr[i]; p < row_ptr[i + 1]; ++p) c -= col[p] == i;
        len[i] = c;
    }
    return len;
}

}  // namespace

bool resident_shape(const int32_t *row_ptr, const int32_t *col, const double *val, int64_t n, int32_t waves,
                    int32_t max_rounds, bool fp64, ResidentShape *s, ResidentRows *rows) {
    if (n < 1 || waves < 1 || waves > 16 || n > (int64_t)waves * max_rounds * 64) return false;
    *s = ResidentShape();
    s->waves = waves;
    // one value for every off-diagonal entry?
    s->unit = true;
    bool seen = false;
    for (int64_t i = 0; i < n && s->unit; ++i)
        for (int32_t p = row_ptr[i]; p < row_ptr[i + 1]; ++p) {
            if (col[p] == i) continue;
            if (!seen) {
                s->off_value = val[p];
                seen = true;
            } else if (val[p] != s->off_value) {
                s->unit = false;
                break;
            }
        }
    rows->len = row_lengths(row_ptr, col, n, s->unit);
    const std::vector<int32_t> &len = rows->len;
    int64_t total = 0;
    int32_t longest = 0;
    for (int32_t c : len) {
        total += c;
        longest = std::max(longest, c);
    }
    // rows by falling length (counted, not compared: the first call on a graph
    // waits for this); the ones above half a wave's share are long
    std::vector<int32_t> &order = rows->order;
    order.resize(n);
    std::vector<int32_t> place((size_t)longest + 2, 0);
    for (int32_t c : len) ++place[longest - c + 1];
    for (int32_t q = 0; q <= longest; ++q) place[q + 1] += place[q];
    for (int64_t i = 0; i < n; ++i) order[place[longest - len[i]]++] = (int32_t)i;
    const int64_t long_min = std::max<int64_t>(32, total / 64 / waves / 2);
    int64_t n_long = 0;
    while (n_long < n && len[order[n_long]] > long_min) ++n_long;
    n_long = std::min<int64_t>(n_long, 64 * (int64_t)waves);
    const int64_t n_short = (n - n_long + 63) / 64;
    s->rounds = (int32_t)((n_long > 0 ? 1 : 0) + (n_short + waves - 1) / waves);
    if (s->rounds > max_rounds || s->positions() > kResidentMaxPositions) return false;
    // (long rows are dealt to the waves in turn)
    s->wave_long = (int32_t)((n_long + waves - 1) / waves);
    std::vector<int64_t> tail(waves, 0);
    s->word_rows = kResidentSpareRows;
    for (int64_t q = 0; q < n_long; ++q) {
        const int64_t words = (len[order[q]] + 127) / 128;
        s->word_rows += words;
        tail[q % waves] += words - 1;
    }
    s->wave_tail = *std::max_element(tail.begin(), tail.end());
    for (int64_t a = n_long; a < n; a += 64) s->word_rows += (len[order[a]] + 3) / 4 * 2;
    rows->n_long = n_long;
    return s->word_rows <= resident_max_word_rows(s->unit, fp64);
}

double resident_step_us(const ResidentShape &s, int cols, bool fp64) {
    // Fitted to 1224 measured steps (ER, weighted ER, preferential attachment
    // and rings with hubs, 500 to 39 000 rows, degrees 4 to 200, 1 to 600
    // columns; within a quarter but for a few): the step's two barriers and
    // serial scalars, a pass over a wave's rows, the reads of v_j, and in the
    // slowest wave a sum over the lanes per long row and a dependent load per
    // further word of one.
    const bool wide = cols * (fp64 ? 8 : 4) > 8;
    const double word = s.unit ? (wide ? 12.0 : 5.7) : fp64 ? 12.0 : wide ? 20.0 : cols == 2 ? 13.0 : 9.5;
    const double row = 0.2 * cols * (s.unit ? 1.0 : 2.0);
    return 1.8 + 0.6 * s.rounds + word * (double)s.word_rows / 1000.0 + row * s.wave_long + 0.27 * (double)s.wave_tail;
}

bool build_resident_layout(const int32_t *row_ptr, const int32_t *col, const double *val, int64_t n, int32_t waves,
                           int32_t max_rounds, ResidentLayout *out, bool fp64) {
    ResidentShape shape;
    ResidentRows rows;
    if (!resident_shape(row_ptr, col, val, n, waves, max_rounds, fp64, &shape, &rows)) return false;
    lay_out(row_ptr, col, val, n, shape, rows, out);
    return true;
}

void lay_out(const int32_t *row_ptr, const int32_t *col, const double *val, int64_t n, const ResidentShape &shape,
             const ResidentRows &rows_of, ResidentLayout *out) {
    ResidentLayout L;
    static_cast<ResidentShape &>(L) = shape;
    const std::vector<int32_t> &len = rows_of.len, &order = rows_of.order;
    const int64_t n_long = rows_of.n_long, n_short = (n - n_long + 63) / 64;
    const int32_t waves = L.waves;
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
    L.words.assign((size_t)L.word_rows * 64, pad);
    if (!L.unit) L.vals.assign(2 * L.words.size(), 0.0);
    size_t used = 0;                     // word rows; the spare ones stay behind the last
    auto grow = [&](size_t rows64) {
        used += rows64;
        return used - rows64;
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
                        int e = 0;
                    for (int32_t p = row_ptr[rows[l]]; p < row_ptr[rows[l] + 1]; ++p) {
                        if (L.unit && col[p] == rows[l]) continue;
                        put((first + e / 128) * 64 + (e % 128) / 2, e & 1, (uint32_t)pos[col[p]], val[p]);
                        ++e;
                    }
                }
            }
        }
    if (L.unit) {
        L.diag.assign(L.positions(), 0.0);
        for (int64_t i = 0; i < n; ++i)
            for (int32_t p = row_ptr[i]; p < row_ptr[i + 1]; ++p)
                if (col[p] == i) L.diag[pos[i]] = val[p];
    }
    *out = std::move(L);
}

}  // namespace vne
