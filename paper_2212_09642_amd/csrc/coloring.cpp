// Greedy distance-d colouring (Section 3.1, Algorithm 1) on the host.
//
// Visiting order: descending degree (number of off-diagonal entries), ties
// by increasing row index.  Each node takes the smallest colour, counting
// from 0, that no already coloured node within distance d carries (distance
// in the graph of the off-diagonal pattern; the paper forms the same
// neighbourhoods from the pattern of A^d).
//
// Two routes give this colouring exactly.
//
// Half-depth balls (first choice): the colours within distance d of node i
// are the union, over the nodes y within distance a of i, of the colours
// within distance b of y, for any a + b = d: a shortest path from i to a
// node z at distance t <= d passes through a node y at distance min(a, t)
// from i, which is within distance t - min(a, t) <= b of z.  Each distance
// keeps, per node y, a bitset of the colours found within distance b of y
// among the nodes coloured so far (b = floor(d / 2), a = d - b).  Node i
// takes the first colour missing from the union over its distance-a ball,
// then sets that colour's bit in the sets of its distance-b ball.  The
// bitsets take n * ceil(colours / 64) words; a distance whose colours
// outgrow 256 (or a memory cap of 256 MB per distance; scale-free graphs
// can need colours in the order of n) is coloured again by the second
// route, which is faster there.
//
// Earlier neighbours (fallback): each node lists the nodes within distance
// d that come earlier in the visiting order, and the first-fit scan marks
// their colours in a per-colour stamp array.
//
// Either way the lists do not depend on the colours: worker threads list the
// balls of the coming nodes of the visiting order, in blocks, while one thread
// per distance runs its first-fit scan behind them.  Distances whose ball is a
// row of the matrix (a = 1: d = 1 and 2) scan the rows and need no lists.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdint>
#include <cstdlib>
#include <functional>
#include <memory>
#include <string>
#include <thread>
#include <vector>

#include "internal.h"

using namespace vne;

namespace {

// Past 4 words per node (256 colours) the unions cost more than the
// earlier-neighbour route's stamps (measured: BA graphs with n = 2e5 need
// 1259 colours at d = 2 and 3975 at d = 3, and take 3.5x as long with
// bitsets; a ring lattice at d = 16 with 136 colours is faster with them).
constexpr int kMaxWords = 4;

// bitset memory per distance before the earlier-neighbour route takes over
// (VNE_COLOR_BITSET_BYTES overrides it)
int64_t bitset_cap() {
    if (const char *e = std::getenv("VNE_COLOR_BITSET_BYTES")) return std::max<int64_t>(8, std::atoll(e));
    return int64_t(256) << 20;
}

// Lists of a block of the visiting order: position t lists its nodes in
// items[begin[t - t0] .. begin[t - t0 + 1]), by nondecreasing distance.
struct BlockLists {
    int64_t t0 = 0, t1 = 0;
    std::vector<int32_t> items;
    std::vector<uint8_t> depth;                  // distance of each listed node
    std::vector<int64_t> begin;
    std::atomic<int64_t> ready{-1};              // the block that is listed here
};

// one per worker thread, on cache lines of its own (the frontier vectors
// change size on every push)
class alignas(128) Searcher {
public:
    // pos == nullptr: list the whole ball (the node itself first, at
    // distance 0); else only the nodes earlier than the node in the order
    Searcher(int64_t n, const int32_t *rp, const int32_t *ci, int32_t depth, const int32_t *pos)
        : rp_(rp), ci_(ci), d_(depth), pos_(pos), seen_(n, -1) {}

    // the nodes within distance d_ of node i, breadth first, with their distance
    void list(int32_t i, int32_t stamp, std::vector<int32_t> *out, std::vector<uint8_t> *dist) {
        frontier_.clear();
        frontier_.push_back(i);
        seen_[i] = stamp;
        const int32_t pi = pos_ ? pos_[i] : 0;
        if (!pos_) {
            out->push_back(i);
            dist->push_back(0);
        }
        for (int32_t depth = 0; depth < d_ && !frontier_.empty(); ++depth) {
            next_.clear();
            const bool last = depth + 1 == d_;     // the last level is not expanded
            const uint8_t dd = (uint8_t)(depth + 1);
            for (int32_t x : frontier_) {
                for (int32_t p = rp_[x]; p < rp_[x + 1]; ++p) {
                    const int32_t y = ci_[p];
                    if (seen_[y] == stamp) continue;
                    seen_[y] = stamp;
                    if (!last) next_.push_back(y);
                    if (!pos_ || pos_[y] < pi) {
                        out->push_back(y);
                        dist->push_back(dd);
                    }
                }
            }
            frontier_.swap(next_);
        }
    }

private:
    const int32_t *rp_, *ci_;
    int32_t d_;
    const int32_t *pos_;
    std::vector<int32_t> seen_;
    std::vector<int32_t> frontier_, next_;
};

void build_lists(BlockLists *bl, Searcher *srch, const std::vector<int32_t> &order) {
    // (local while they grow: the vectors of neighbouring blocks share lines)
    std::vector<int32_t> it;
    std::vector<uint8_t> dp;
    std::vector<int64_t> bg;
    it.swap(bl->items);
    dp.swap(bl->depth);
    bg.swap(bl->begin);
    it.clear();
    dp.clear();
    bg.assign(1, 0);
    for (int64_t t = bl->t0; t < bl->t1; ++t) {
        srch->list(order[t], (int32_t)t, &it, &dp);
        bg.push_back((int64_t)it.size());
    }
    bl->items.swap(it);
    bl->depth.swap(dp);
    bl->begin.swap(bg);
}

// The nodes within a distance of the node at position t: from the lists ...
struct ListedBalls {
    const BlockLists &bl;
    int64_t t0() const { return bl.t0; }
    int64_t t1() const { return bl.t1; }
    template <class F>
    void each(int64_t t, int32_t, int32_t dist, const F &f) const {
        for (int64_t q = bl.begin[t - bl.t0]; q < bl.begin[t - bl.t0 + 1] && bl.depth[q] <= dist; ++q) f(bl.items[q]);
    }
};

// ... or, for distances up to 1, the node and its row
struct RowBalls {
    int64_t n;
    const int32_t *rp, *ci;
    int64_t t0() const { return 0; }
    int64_t t1() const { return n; }
    template <class F>
    void each(int64_t, int32_t i, int32_t dist, const F &f) const {
        f(i);
        if (dist == 0) return;
        for (int32_t p = rp[i]; p < rp[i + 1]; ++p) f(ci[p]);
    }
};

// First-fit state of one distance d, half-depth route: per node, the
// colours within distance b of it among the coloured nodes, as W 64-bit words.
struct BallFit {
    int32_t d = 1, a = 1, b = 0;
    int64_t n = 0;
    int W = 1;
    int64_t cap = 0;                             // bytes allowed for bits
    bool overflow = false;                       // colours outgrew cap
    std::vector<uint64_t> bits;                  // [n][W]
    std::vector<int32_t> color;
    int32_t ncol = 0;

    void init(int64_t nn, int32_t dist) {
        n = nn;
        d = dist;
        b = d / 2;
        a = d - b;
        W = 1;
        cap = bitset_cap();
        overflow = (int64_t)n * 8 > cap;
        if (!overflow) bits.assign((size_t)n * W, 0);
        color.assign((size_t)n, -1);
        ncol = 0;
    }

    // one more word per node; false (and overflow) past kMaxWords or the
    // memory cap
    bool widen() {
        if (W + 1 > kMaxWords || (int64_t)n * (W + 1) * 8 > cap) {
            overflow = true;
            std::vector<uint64_t>().swap(bits);
            return false;
        }
        std::vector<uint64_t> nb((size_t)n * (W + 1), 0);
        for (int64_t y = 0; y < n; ++y)
            for (int w = 0; w < W; ++w) nb[(size_t)y * (W + 1) + w] = bits[(size_t)y * W + w];
        bits.swap(nb);
        W++;
        return true;
    }

    // WW: the word count W as a compile-time constant
    template <int WW, class Balls>
    void scan_w(const Balls &balls, const std::vector<int32_t> &order, int64_t *t_next) {
        constexpr int Wn = WW;
        uint64_t forb[kMaxWords];
        uint64_t *const sets = bits.data();
        for (int64_t t = *t_next; t < balls.t1(); ++t) {
            const int32_t i = order[t];
            // union over the distance-a ball
            for (int w = 0; w < Wn; ++w) forb[w] = 0;
            balls.each(t, i, a, [&](int32_t y) {
                const uint64_t *src = sets + (size_t)y * Wn;
                for (int w = 0; w < Wn; ++w) forb[w] |= src[w];
            });
            int w = 0;
            while (w < Wn && forb[w] == ~0ull) ++w;
            const int32_t c = w * 64 + (w < Wn ? __builtin_ctzll(~forb[w]) : 0);
            if (c >= 64 * Wn) {
                // every colour of the W words is taken: one more word, and
                // the rest with the new width
                *t_next = widen() ? t : balls.t1();
                return;
            }
            color[i] = c;
            ncol = std::max(ncol, c + 1);
            // mark c in the sets of the distance-b ball
            const uint64_t m = 1ull << (c & 63);
            balls.each(t, i, b, [&](int32_t y) { sets[(size_t)y * Wn + w] |= m; });
        }
        *t_next = balls.t1();
    }

    bool finished() const { return overflow; }

    template <class Balls>
    void scan(const Balls &balls, const std::vector<int32_t> &order) {
        int64_t t = balls.t0();
        while (t < balls.t1() && !overflow) {
            switch (W) {
                case 1: scan_w<1>(balls, order, &t); break;
                case 2: scan_w<2>(balls, order, &t); break;
                case 3: scan_w<3>(balls, order, &t); break;
                default: scan_w<4>(balls, order, &t); break;
            }
        }
    }
};

// First-fit state of one distance d, earlier-neighbour route.
struct DirectFit {
    int32_t d = 1;
    std::vector<int32_t> color;
    std::vector<int64_t> banned;                 // stamp per colour
    int32_t ncol = 0;

    void init(int64_t n, int32_t dist) {
        d = dist;
        color.assign((size_t)n, -1);
        banned.clear();
        ncol = 0;
    }

    bool finished() const { return false; }

    template <class Balls>
    void scan(const Balls &balls, const std::vector<int32_t> &order) {
        for (int64_t t = balls.t0(); t < balls.t1(); ++t) {
            balls.each(t, order[t], d, [&](int32_t y) { banned[color[y]] = t; });
            int32_t c = 0;
            while (c < ncol && banned[c] == t) ++c;
            if (c == ncol) {
                ncol++;
                banned.push_back(-1);
            }
            color[order[t]] = c;
        }
    }
};

int color_threads(int64_t n) {
    int nw = (int)std::thread::hardware_concurrency();
    if (const char *e = std::getenv("VNE_COLOR_THREADS")) nw = std::atoi(e);
    nw = std::max(1, std::min(nw, 16));
    // (a thread costs the time of some hundred short lists)
    return (int)std::min<int64_t>(nw, 1 + n / 512);
}

// Lists to `depth` (whole balls, or earlier nodes when pos is given) in
// blocks of the visiting order; every fit of `fits` scans them in order, a
// thread per fit, behind the threads that list.  Ends early once every fit
// has given up.
constexpr int64_t kBlockNodes = 64;
constexpr int64_t kPendingNodes = int64_t(1) << 25;    // listed nodes that wait for a scan

template <class Fit>
void run_pipeline(int64_t n, const int32_t *rp, const int32_t *ci, const std::vector<int32_t> &order,
                  int32_t depth, const int32_t *pos, std::vector<Fit *> &fits) {
    const int nf = (int)fits.size(), nw = color_threads(n);
    const int64_t nblk = (n + kBlockNodes - 1) / kBlockNodes;
    auto place = [&](BlockLists *bl, int64_t k) {
        bl->t0 = k * kBlockNodes;
        bl->t1 = std::min<int64_t>(n, bl->t0 + kBlockNodes);
    };
    auto finished = [&]() {
        for (Fit *f : fits)
            if (!f->finished()) return false;
        return true;
    };
    if (nw == 1) {
        Searcher srch(n, rp, ci, depth, pos);
        BlockLists bl;
        for (int64_t k = 0; k < nblk && !finished(); ++k) {
            place(&bl, k);
            build_lists(&bl, &srch, order);
            for (Fit *f : fits) f->scan(ListedBalls{bl}, order);
        }
        return;
    }
    // block k is listed into ring[k mod R] once every fit is past block k - R
    const int64_t R = 8 * nw;
    std::vector<BlockLists> ring(R);
    std::vector<std::atomic<int64_t>> at(nf);          // blocks that fit q is past
    for (auto &x : at) x.store(0);
    std::atomic<int64_t> next{0}, longest{1};          // longest: most nodes listed in a block
    auto behind = [&]() {
        int64_t lo = nblk;
        for (auto &x : at) lo = std::min(lo, x.load(std::memory_order_acquire));
        return lo;
    };
    auto pause = [](int *spins) {
        if (++*spins < 256) std::this_thread::yield();
        else std::this_thread::sleep_for(std::chrono::microseconds(20));
    };
    auto lister = [&]() {
        Searcher srch(n, rp, ci, depth, pos);
        for (int64_t k = next.fetch_add(1); k < nblk; k = next.fetch_add(1)) {
            BlockLists &bl = ring[k % R];
            int spins = 0;
            while (behind() + std::min(R, std::max<int64_t>(1, kPendingNodes / longest.load())) <= k) pause(&spins);
            if (behind() >= nblk) return;              // every fit has given up
            place(&bl, k);
            build_lists(&bl, &srch, order);
            const int64_t len = (int64_t)bl.items.size();
            for (int64_t was = longest.load(); was < len && !longest.compare_exchange_weak(was, len);) {
            }
            bl.ready.store(k, std::memory_order_release);
        }
    };
    auto scanner = [&](int q) {
        for (int64_t k = 0; k < nblk; ++k) {
            BlockLists &bl = ring[k % R];
            int spins = 0;
            while (bl.ready.load(std::memory_order_acquire) != k) pause(&spins);
            fits[q]->scan(ListedBalls{bl}, order);
            if (fits[q]->finished()) break;
            at[q].store(k + 1, std::memory_order_release);
        }
        at[q].store(nblk, std::memory_order_release);
    };
    std::vector<std::thread> th;
    for (int w = 0; w < nw; ++w) th.emplace_back(lister);
    for (int q = 1; q < nf; ++q) th.emplace_back(scanner, q);
    scanner(0);
    for (auto &x : th) x.join();
}

}  // namespace

void vne::greedy_color_multi(int64_t n, const int32_t *rp, const int32_t *ci, const int32_t *ds, int nd,
                             int32_t *const *colors_out, int32_t *n_colors,
                             const std::function<void(int)> &done) {
    auto deliver = [&](int q, const std::vector<int32_t> &color, int32_t ncol) {
        std::copy(color.begin(), color.end(), colors_out[q]);
        n_colors[q] = ncol;
        if (done) done(q);
    };
    // visiting order by counting the degrees
    std::vector<int32_t> deg(n), order(n);
    int32_t dmost = 0;
    for (int64_t i = 0; i < n; ++i) {
        int32_t c = 0;
        for (int32_t p = rp[i]; p < rp[i + 1]; ++p) c += (ci[p] != i);
        deg[i] = c;
        dmost = std::max(dmost, c);
    }
    std::vector<int64_t> place((size_t)dmost + 2, 0);
    for (int64_t i = 0; i < n; ++i) place[dmost - deg[i] + 1]++;
    for (int32_t q = 0; q <= dmost; ++q) place[q + 1] += place[q];
    for (int64_t i = 0; i < n; ++i) order[place[dmost - deg[i]]++] = (int32_t)i;

    // half-depth balls for every distance; those whose balls are rows scan
    // them beside the listing of the others
    std::vector<BallFit> ball(nd);
    std::vector<BallFit *> listed;
    std::vector<std::thread> beside;
    int32_t depth = 1;                         // the deepest ball any distance needs
    for (int q = 0; q < nd; ++q) {
        ball[q].init(n, ds[q]);
        if (ball[q].a > 1) {
            listed.push_back(&ball[q]);
            depth = std::max(depth, ball[q].a);
        }
    }
    const RowBalls rows{n, rp, ci};
    for (int q = 0; q < nd; ++q) {
        if (ball[q].a > 1) continue;
        auto work = [&, q]() {
            ball[q].scan(rows, order);
            if (!ball[q].overflow) deliver(q, ball[q].color, ball[q].ncol);
        };
        if (nd > 1 && color_threads(n) > 1) beside.emplace_back(work);
        else work();
    }
    if (!listed.empty()) run_pipeline(n, rp, ci, order, depth, nullptr, listed);
    for (int q = 0; q < nd; ++q)
        if (ball[q].a > 1 && !ball[q].overflow) deliver(q, ball[q].color, ball[q].ncol);
    for (auto &x : beside) x.join();

    // distances whose colours outgrew the bitsets: earlier neighbours
    std::vector<DirectFit> direct;
    std::vector<int> redo;
    int32_t dmax = 1;
    for (int q = 0; q < nd; ++q)
        if (ball[q].overflow) {
            redo.push_back(q);
            dmax = std::max(dmax, ds[q]);
        }
    if (!redo.empty()) {
        std::vector<int32_t> pos(n);
        for (int64_t t = 0; t < n; ++t) pos[order[t]] = (int32_t)t;
        direct.resize(redo.size());
        std::vector<DirectFit *> dp;
        for (size_t r = 0; r < redo.size(); ++r) {
            direct[r].init(n, ds[redo[r]]);
            dp.push_back(&direct[r]);
        }
        run_pipeline(n, rp, ci, order, dmax, pos.data(), dp);
    }
    for (size_t r = 0; r < redo.size(); ++r) deliver(redo[r], direct[r].color, direct[r].ncol);
}

int32_t vne::greedy_color(int64_t n, const int32_t *rp, const int32_t *ci, int32_t d, int32_t *colors_out) {
    int32_t ncol = 0;
    int32_t *out[1] = {colors_out};
    greedy_color_multi(n, rp, ci, &d, 1, out, &ncol, nullptr);
    return ncol;
}

extern "C" vne_status vne_color_greedy(const vne_csr *csr, int32_t d, int32_t *colors_out,
                                       int32_t *n_colors, char *msg, int64_t msg_len) {
    if (!csr || csr->location != VNE_HOST) {
        set_msg(msg, msg_len, "vne_color_greedy needs a host CSR");
        return VNE_EINVAL;
    }
    // distances are kept in one byte per listed node
    if (d < 1 || d > 254) { set_msg(msg, msg_len, "distance d must be in [1, 254]"); return VNE_EINVAL; }
    if (!colors_out || !n_colors) { set_msg(msg, msg_len, "NULL output"); return VNE_EINVAL; }
    std::string m;
    vne_status st = validate_host_csr(csr, 0, &m);
    if (st != VNE_OK) { set_msg(msg, msg_len, m); return st; }
    *n_colors = greedy_color(csr->n, csr->row_ptr, csr->col_idx, d, colors_out);
    set_msg(msg, msg_len, "");
    return VNE_OK;
}
