// Host check of the on-chip kernel's row layout, read as the kernel reads
// it: every row has one position, every word lies inside the array, padding
// reads the zero behind the last position, and A x computed from the layout
// (integers, so exact in any order) equals A x from the CSR.
#include <cstdio>
#include <random>
#include <set>
#include <vector>

#include "resident_layout.h"

using vne::ResidentLayout;

struct Csr {
    std::vector<int32_t> rp, ci;
    std::vector<double> va;
};

// a symmetric pattern with hubs; unit: Laplacian, else integer weights with
// some rows without a diagonal entry and some empty rows
static Csr make(std::mt19937_64 &rng, int n, int deg, int hubs, bool unit) {
    std::vector<std::set<int32_t>> adj(n);
    auto join = [&](int a, int b) {
        if (a == b) return;
        adj[a].insert(b);
        adj[b].insert(a);
    };
    for (int64_t e = 0; e < (int64_t)n * deg / 2; ++e) join((int)(rng() % n), (int)(rng() % n));
    for (int h = 0; h < hubs; ++h)
        for (int e = 0; e < n / 3; ++e) join(h, (int)(rng() % n));
    Csr m;
    m.rp.push_back(0);
    for (int i = 0; i < n; ++i) {
        const bool diag = unit || rng() % 4 != 0;
        std::set<int32_t> cols = adj[i];
        if (diag) cols.insert(i);
        for (int32_t c : cols) {
            m.ci.push_back(c);
            m.va.push_back(c == i ? (double)adj[i].size() : unit ? -1.0 : (double)(1 + rng() % 7));
        }
        m.rp.push_back((int32_t)m.ci.size());
    }
    return m;
}

static const char *check(const Csr &m, int n, int waves, int max_rounds, bool unit) {
    ResidentLayout L;
    const bool ok = vne::build_resident_layout(m.rp.data(), m.ci.data(), m.va.data(), n, waves, max_rounds, &L);
    if (!ok) return (n + 63) / 64 + waves <= waves * max_rounds ? "refused although it fits" : nullptr;
    const int P = L.positions();
    if (L.waves != waves || L.rounds > max_rounds || P > vne::kResidentMaxPositions) return "shape";
    if (unit && !L.unit) return "unit not seen";
    if ((int)L.row_of.size() != P || (int)L.slices.size() != 4 * waves * L.rounds) return "sizes";
    if (L.words.size() % 64 || L.vals.size() != (L.unit ? 0 : 2 * L.words.size())) return "word sizes";
    if (L.unit && (int)L.diag.size() != P) return "diag size";
    std::vector<double> x(n), V(P + 1, 0.0), got(n, 0.0);
    std::vector<int> seen(n, 0);
    for (int i = 0; i < n; ++i) x[i] = (i * 37) % 101 - 50;
    for (int p = 0; p < P; ++p)
        if (L.row_of[p] >= 0) {
            if (L.row_of[p] >= n || seen[L.row_of[p]]++) return "row_of";
            V[p] = x[L.row_of[p]];
        }
    for (int i = 0; i < n; ++i)
        if (!seen[i]) return "row without a position";
    const char *bad = nullptr;
    auto word = [&](int64_t o) {
        double s = 0.0;
        if (o < 0 || o >= (int64_t)L.words.size()) {
            bad = "word out of range";
            return s;
        }
        for (int h = 0; h < 2; ++h) {
            const int p = h ? L.words[o] >> 16 : L.words[o] & 0xffff;
            if (p > P) bad = "position out of range";
            else s += (L.unit ? L.off_value : L.vals[2 * o + h]) * V[p];
        }
        return s;
    };
    for (int w = 0; w < waves; ++w)
        for (int r = 0; r < L.rounds; ++r) {
            const int32_t *sl = &L.slices[4 * (w * L.rounds + r)];
            if (sl[0] == 1 && (sl[2] % 2 || ((int64_t)sl[1] + sl[2] + vne::kResidentSpareRows) * 64 > (int64_t)L.words.size()))
                return "slice length";
            for (int l = 0; l < 64; ++l) {
                const int p = (w * L.rounds + r) * 64 + l;
                const int row = L.row_of[p];
                double acc = 0.0;
                if (sl[0] == 1) {
                    for (int t = 0; t < sl[2]; ++t) acc += word(((int64_t)sl[1] + t) * 64 + l);
                } else if (sl[0] == 2 && l < sl[3]) {
                    const size_t s = 2 * ((size_t)sl[1] + l);
                    if (s + 1 >= L.spans.size()) return "span out of range";
                    for (int t = 0; t < L.spans[s + 1]; ++t)
                        for (int q = 0; q < 64; ++q) acc += word(((int64_t)L.spans[s] + t) * 64 + q);
                }
                if (bad) return bad;
                if (row < 0) {
                    if (acc != 0.0) return "entries of no row";
                    continue;
                }
                if (sl[0] == 0 || l >= sl[3]) return "row outside its slice";
                got[row] = acc + (L.unit ? L.diag[p] * V[p] : 0.0);
            }
        }
    for (int i = 0; i < n; ++i) {
        double want = 0.0;
        for (int32_t p = m.rp[i]; p < m.rp[i + 1]; ++p) want += m.va[p] * x[m.ci[p]];
        if (want != got[i]) return "product";
    }
    return nullptr;
}

int main() {
    std::mt19937_64 rng(11);
    int cases = 0;
    const int sizes[] = {1, 2, 63, 64, 65, 130, 500, 1023, 1024, 1025, 2000, 4999, 16384};
    for (int n : sizes)
        for (int unit = 0; unit < 2; ++unit)
            for (int hubs = 0; hubs < 3; ++hubs) {
                const Csr m = make(rng, n, 1 + (int)(rng() % 12), n > 200 ? hubs * hubs * 4 : 0, unit);
                for (int waves : {1, 4, 7, 8, 16})
                    for (int rounds : {19, 39}) {
                        if (const char *e = check(m, n, waves, rounds, unit)) {
                            std::printf("FAIL n=%d unit=%d hubs=%d waves=%d rounds=%d: %s\n", n, unit, hubs, waves,
                                        rounds, e);
                            return 1;
                        }
                        ++cases;
                    }
            }
    std::printf("ok %d cases\n", cases);
    return 0;
}
