// Host side of the on-chip Lanczos runs: which graphs take them, their
// device layouts, and batches that mix them with the stacked launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "ctx_internal.h"
#include "internal.h"
#include "kernels.h"
#include "resident.h"

using namespace vne;

namespace vne {
namespace rt {

namespace {

// most elements of v_j that a CU's LDS holds (with room for the reduction)
int lds_elements(bool fp64) { return fp64 ? 64 * 16 * kResidentSlots64 : 64 * 16 * kResidentSlots32; }

// VNE_RESIDENT: 0 never, 1 wherever the rows fit, else by the rule.  A
// forced tile or schedule, or the autotuner off, asks for the launched steps.
int chip_mode() {
    if (env_int("VNE_TILE", 0) > 0 || env_int("VNE_AUTOTUNE", 1) == 0 || getenv("VNE_SCHED")) return 0;
    return env_int("VNE_RESIDENT", 2);
}

template <typename T>
bool put(vne_ctx *c, DevBuf *b, const std::vector<T> &h) {
    if (dev_alloc(c, b, std::max<size_t>(h.size(), 1) * sizeof(T)) != VNE_OK) return false;
    return h.empty() || hipMemcpy(b->p, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice) == hipSuccess;
}

int slots(bool fp64) { return fp64 ? kResidentSlots64 : kResidentSlots32; }

// The shape of graph gid's layout for a workgroup of `waves`; null: does not fit.
const ResidentShape *shape_of(vne_ctx *c, int32_t gid, int waves, bool fp64) {
    Graph *g = get_graph(c, gid);
    const auto key = std::make_pair(waves, (int)fp64);
    auto it = g->shapes.find(key);
    if (it == g->shapes.end()) {
        ResidentShape s;
        ResidentRows rows;
        if (resident_shape(g->h_row_ptr.data(), g->h_col.data(), g->h_val.data(), g->n, waves, slots(fp64), fp64, &s,
                           &rows) &&
            resident_lds(s.positions(), 1, fp64) <= kResidentLds)
            g->shape_rows[key] = std::move(rows);
        else
            s = ResidentShape();
        it = g->shapes.emplace(key, s).first;
    }
    return it->second.waves > 0 ? &it->second : nullptr;
}

// The layout itself, for a run that takes it; null: does not fit, or no room.
DevLayout *layout_of(vne_ctx *c, int32_t gid, int waves, bool fp64) {
    const ResidentShape *s = shape_of(c, gid, waves, fp64);
    if (!s) return nullptr;
    Graph *g = get_graph(c, gid);
    const auto key = std::make_pair(waves, (int)fp64);
    auto it = g->layouts.find(key);
    if (it != g->layouts.end()) return it->second.get();
    ResidentLayout h;
    auto rows = g->shape_rows.find(key);
    if (rows != g->shape_rows.end())
        lay_out(g->h_row_ptr.data(), g->h_col.data(), g->h_val.data(), g->n, *s, rows->second, &h);
    else if (!build_resident_layout(g->h_row_ptr.data(), g->h_col.data(), g->h_val.data(), g->n, waves, slots(fp64), &h,
                                    fp64))
        return nullptr;
    g->shape_rows.clear();
    auto d = std::make_unique<DevLayout>();
    d->waves = waves;
    d->rounds = h.rounds;
    d->positions = h.positions();
    d->unit = h.unit;
    d->off_value = h.off_value;
    const std::string err = c->err;
    bool ok = put(c, &d->slices, h.slices) && put(c, &d->words, h.words) && put(c, &d->spans, h.spans) &&
              put(c, &d->row_of, h.row_of) && put(c, &d->diag, h.diag);
    if (ok && !h.unit)
        ok = fp64 ? put(c, &d->vals, h.vals) : put(c, &d->vals, std::vector<float>(h.vals.begin(), h.vals.end()));
    if (!ok) {
        // no room: the launched steps run, and a later call may try again
        for (DevBuf *b : {&d->slices, &d->words, &d->vals, &d->spans, &d->row_of, &d->diag}) dev_free(c, b);
        c->err = err;
        return nullptr;
    }
    return (g->layouts[key] = std::move(d)).get();
}

// the widest column group (at most cap) that the layout has room for (two FP64
// columns of unequal values spill: 5000 rows of 10, 600 columns, us a step: 55
// against 3 x 10)
int widest(const ResidentShape &s, bool fp64, int cap) {
    int cols = fp64 && !s.unit ? 1 : cap;
    while (cols > 1 && (s.rounds * cols > slots(fp64) || resident_lds(s.positions(), cols, fp64) > kResidentLds))
        cols /= 2;
    return cols;
}

// us of a launched step of one matrix or of a stack of them, by sizes alone,
// fitted to the launched times of the pairs that resident_step_us was fitted to
// (mean deviation 12%): its launches and dependent reductions (base), the
// streams, the gathers (of blocks that caches hold), more of both for long
// rows, and the rows' share of the reductions.
double launched_us(double base, int64_t n, int64_t nnz, int64_t long_entries, int m, bool fp64) {
    const int mt = choose_plan_tile(m, fp64, n, nnz);
    double gather = 0.0;
    const double streams = step_bytes_us(n, nnz, pad_columns(m, mt), mt, fp64, &gather) - gather;
    const double share = (double)long_entries / (double)std::max<int64_t>(1, nnz);
    return base + 1.1 * streams + (0.45 + 0.65 * share) * gather + (long_entries > 0 ? 3.5 : 0.0) + 0.8e-4 * (double)n;
}
constexpr double kLaunchUs = 16.0, kStackLaunchUs = 20.0;

ResidentJob job_of(const GraphSet *one, const DevLayout *L, const Graph *g, bool fp64) {
    ResidentJob j{};
    j.slices = (const int4 *)L->slices.p;
    j.words = (const uint32_t *)L->words.p;
    j.vals = L->vals.p;
    j.spans = (const int2 *)L->spans.p;
    j.row_of = (const int32_t *)L->row_of.p;
    j.diag = (const double *)L->diag.p;
    j.keys = (const int64_t *)one->keys.p;
    j.scale = g->scale;
    j.off_value = L->off_value;
    j.tau = fp64 ? std::ldexp(1.0, -23) : std::ldexp(1.0, -18);
    j.n = (int32_t)g->n;
    j.rounds = L->rounds;
    j.positions = L->positions;
    return j;
}

vne_status side_lanes(vne_ctx *c, size_t count) {
    while (c->side_streams.size() < count) {
        hipStream_t s = nullptr;
        HIP_TRY(c, hipStreamCreate(&s));
        c->side_streams.push_back(s);
    }
    while (c->side_events.size() < count + 1) {
        hipEvent_t e = nullptr;
        HIP_TRY(c, hipEventCreateWithFlags(&e, hipEventDisableTiming));
        c->side_events.push_back(e);
    }
    return VNE_OK;
}

vne_status loop_events(vne_ctx *c, Plan *p) {
    while (p->ev.size() < 2) {
        hipEvent_t e;
        HIP_TRY(c, hipEventCreate(&e));
        p->ev.push_back(e);
    }
    return VNE_OK;
}

vne_status upload_widths(vne_ctx *c, Plan *p) {
    if (p->up_graph_m != p->h_graph_m) {
        HIP_TRY(c, hipMemcpyAsync(p->graph_m.p, p->h_graph_m.data(), p->G * 4, hipMemcpyHostToDevice, c->stream));
        p->up_graph_m = p->h_graph_m;
    }
    return VNE_OK;
}

}  // namespace

DevLayout *chip_choice(vne_ctx *c, GraphSet *set, const Plan *p, int *cols) {
    const int mode = chip_mode();
    // (with a memory budget the launched steps, whose allocations do not
    // depend on the matrix's size or the rule)
    if (mode == 0 || c->budget != 0 || set->G != 1 || set->n > lds_elements(p->fp64)) return nullptr;
    const bool fp64 = p->fp64;
    const int waves = (int)std::min<int64_t>(16, (set->n + 63) / 64);
    // one column per workgroup while a CU each is left, then as many as fit
    int cap = 1;
    while (cap < (fp64 ? 2 : 4) && (p->m + cap - 1) / cap > 256) cap *= 2;
    // A step on the chip, per round of 256 workgroups, against a launched
    // one; the sizes alone decide, never a tile that was tuned, so that every
    // call of a shape runs the same way.  Few columns of a large matrix, which
    // leave most CUs idle on the chip, are launched.  Measured (us a step,
    // launched / chip): ER n = 2000, 30 columns FP64 14.7 / 3.5; BA n = 12000,
    // 300 columns 74 / 26; WS n = 12000, 21 columns FP64 19.8 / 15.1; ER n =
    // 39000, 8 columns 18 / 40, 64 columns 32 / 40, 256 columns 81 / 39; a ring
    // of 30000 rows with one of 15000 entries, 8 columns 29 / 83.  Over 1224
    // such pairs the rule is 0.8% from the faster way; in five of them the
    // chip is taken where it is 11 to 22% slower.
    const double launched =
        launched_us(kLaunchUs, set->n, set->nnz, set->sched.long_entries, p->m, fp64);
    auto slower = [&](const ResidentShape &s, int columns) {
        const double rounds = std::ceil(std::ceil((double)p->m / columns) / 256.0);
        return mode != 1 && rounds * resident_step_us(s, columns, fp64) > launched;
    };
    // (the shape is not looked for where even full slices would be slower)
    ResidentShape full;
    full.unit = true;
    full.rounds = (int32_t)((set->n + 64 * waves - 1) / (64 * waves));
    full.word_rows = (set->nnz - set->n) / 128;
    if (slower(full, cap)) return nullptr;
    const ResidentShape *s = shape_of(c, set->ids[0], waves, fp64);
    if (!s) return nullptr;
    *cols = widest(*s, fp64, cap);
    if (!slower(*s, *cols)) return layout_of(c, set->ids[0], waves, fp64);
    get_graph(c, set->ids[0])->shape_rows.clear();
    return nullptr;
}

DevLayout *chip_layout(vne_ctx *c, int32_t gid, int max_rounds) {
    const Graph *g = get_graph(c, gid);
    if (chip_mode() == 0 || c->budget != 0 || g->n > (int64_t)1024 * max_rounds) return nullptr;
    const int waves = (int)std::min<int64_t>(16, (g->n + 63) / 64);
    const ResidentShape *s = shape_of(c, gid, waves, true);
    if (s && s->rounds <= max_rounds) return layout_of(c, gid, waves, true);
    get_graph(c, gid)->shape_rows.clear();
    return nullptr;
}

vne_status run_chip(vne_ctx *c, GraphSet *set, Plan *p, const ProbeSpec &ps, bool desing, const DevLayout *L,
                    int cols) {
    c->last_tile = cols;
    c->last_m_pad = pad_columns(p->m, cols);
    VNE_TRY(upload_widths(c, p));
    HIP_TRY(c, hipMemsetAsync(p->flags.p, 0, 4, c->stream));
    ResidentJob j = job_of(set, L, get_graph(c, set->ids[0]), p->fp64);
    j.colors = ps.colors;
    j.dense = ps.dense;
    j.ld_dense = ps.ld_dense;
    j.gen = ps.gen;
    j.seed = ps.seeds.empty() ? 0 : ps.seeds[0];
    j.col_offset = ps.col_offset;
    j.desing = desing ? 1 : 0;
    j.alpha = (double *)p->alpha.p;
    j.beta = (double *)p->beta.p;
    j.norm2 = (double *)p->norm2.p;
    j.k_eff = (int32_t *)p->k_eff.p;
    j.flags = (int32_t *)p->flags.p;
    j.m = p->m;
    j.k = j.ld_k = p->k;
    if (c->timing) {
        VNE_TRY(loop_events(c, p));
        HIP_TRY(c, hipEventRecord(p->ev[0], c->stream));
    }
    HIP_TRY(c, launch_resident_one(j, L->waves, resident_kind(L->rounds, cols, L->unit, p->fp64),
                                   c->stream));
    if (c->timing) {
        HIP_TRY(c, hipEventRecord(p->ev[1], c->stream));
        c->pending.push_back({p, step_bytes(set, p), p->k, true});
    }
    HIP_TRY(c, launch_quadrature((const double *)p->alpha.p, (const double *)p->beta.p, (const int32_t *)p->k_eff.p,
                                 (const double *)p->norm2.p, p->k, p->k, p->m, (double *)p->psi.p,
                                 (int32_t *)p->flags.p, c->stream, p->fp64));
    return VNE_OK;
}

namespace {

// The on-chip graphs of a batch: row ranges and result buffers (kept per id
// sequence, as the stacked sets are), and each query's layout.
struct ChipBatch {
    GraphSet *set = nullptr;
    Plan *p = nullptr;
    ProbeSpec ps;
    int combine = 0;
    std::vector<DevLayout *> layout;
    std::vector<int> cols;
    std::vector<double> step_us;
    struct Class {
        int waves;
        ResidentKind kind;
        size_t lds;
        std::vector<int2> map;
        size_t map_at;
    };
    std::vector<Class> classes;
};

vne_status chip_set(vne_ctx *c, const std::vector<int32_t> &ids, GraphSet **out) {
    auto it = c->chip_sets.find(ids);
    if (it != c->chip_sets.end()) {
        it->second->last_use = ++c->tick;
        *out = it->second.get();
        return VNE_OK;
    }
    const size_t cap = (size_t)std::max(1, env_int("VNE_MAX_SETS", 4));
    while (c->chip_sets.size() >= cap) {
        auto victim = c->chip_sets.begin();
        for (auto jt = c->chip_sets.begin(); jt != c->chip_sets.end(); ++jt)
            if (jt->second->last_use < victim->second->last_use) victim = jt;
        HIP_TRY(c, hipStreamSynchronize(c->stream));
        free_set(c, victim->second.get());
        c->chip_sets.erase(victim);
    }
    auto s = std::make_unique<GraphSet>();
    s->last_use = ++c->tick;
    s->ids = ids;
    s->G = (int)ids.size();
    s->h_row_begin.assign(1, 0);
    for (int32_t id : ids) {
        const Graph *g = get_graph(c, id);
        s->h_row_begin.push_back(s->h_row_begin.back() + g->n);
        s->nnz += g->nnz;
    }
    s->n = s->h_row_begin.back();
    *out = s.get();
    c->chip_sets[ids] = std::move(s);
    return VNE_OK;
}

vne_status chip_plan(vne_ctx *c, GraphSet *set, int m, int k, bool fp64, Plan **out) {
    const auto key = std::make_tuple(m, k, (int)fp64, 0, 3);
    auto it = set->plans.find(key);
    if (it != set->plans.end()) {
        *out = it->second.get();
        return VNE_OK;
    }
    auto p = std::make_unique<Plan>();
    p->fp64 = fp64;
    p->G = set->G;
    p->m = m;
    p->k = k;
    p->mt = 4;
    p->m_pad = pad_columns(m, 4);
    const size_t cols = (size_t)p->G * p->m_pad;
    vne_status st = VNE_OK;
    auto take = [&](DevBuf *b, size_t bytes) {
        if (st == VNE_OK) st = dev_alloc(c, b, bytes);
    };
    take(&p->alpha, cols * k * 8);
    take(&p->beta, cols * k * 8);
    take(&p->k_eff, cols * 4);
    take(&p->norm2, cols * 8);
    take(&p->psi, cols * 8);
    take(&p->estimate, (size_t)p->G * 8);
    take(&p->flags, 4);
    take(&p->graph_m, (size_t)p->G * 4);
    if (st != VNE_OK) {
        free_plan(c, p.get());
        return st;
    }
    *out = p.get();
    set->plans[key] = std::move(p);
    return VNE_OK;
}

// Workgroup classes and maps, and the kernel arguments on the device.
// Workgroups reach the XCDs round robin, so entry 8 i + x of a map goes to
// XCD x: a graph's workgroups are kept on one XCD in runs, whose L2 then
// reads the matrix once, and the runs are dealt by falling cost.
vne_status chip_args(vne_ctx *c, ChipBatch *b, bool desing) {
    Plan *p = b->p;
    const int G = p->G;
    std::vector<ResidentJob> jobs(G);
    b->classes.clear();
    std::vector<std::vector<int>> members;
    for (int q = 0; q < G; ++q) {
        const DevLayout *L = b->layout[q];
        const Graph *g = get_graph(c, b->set->ids[q]);
        GraphSet *one = nullptr;
        VNE_TRY(get_set(c, {b->set->ids[q]}, &one));
        ResidentJob j = job_of(one, L, g, p->fp64);
        const int64_t r0 = b->set->h_row_begin[q];
        const size_t c0 = (size_t)q * p->m_pad;
        j.gen = b->ps.gen;
        j.seed = b->ps.seeds.empty() ? 0 : b->ps.seeds[q];
        j.colors = b->ps.colors ? b->ps.colors + r0 : nullptr;
        j.ld_dense = b->ps.ld_dense;
        j.dense = b->ps.dense ? (const char *)b->ps.dense + (size_t)r0 * b->ps.ld_dense * (p->fp64 ? 8 : 4) : nullptr;
        j.desing = desing ? 1 : 0;
        j.alpha = (double *)p->alpha.p + c0 * p->k;
        j.beta = (double *)p->beta.p + c0 * p->k;
        j.norm2 = (double *)p->norm2.p + c0;
        j.k_eff = (int32_t *)p->k_eff.p + c0;
        j.flags = (int32_t *)p->flags.p;
        j.m = p->h_graph_m[q];
        j.k = p->h_graph_k[q];
        j.ld_k = p->k;
        jobs[q] = j;
        const ResidentKind kind = resident_kind(L->rounds, b->cols[q], L->unit, p->fp64);
        size_t k = 0;
        while (k < b->classes.size() && !(b->classes[k].waves == L->waves && b->classes[k].kind == kind)) ++k;
        if (k == b->classes.size()) {
            b->classes.push_back({L->waves, kind, 0, {}, 0});
            members.emplace_back();
        }
        members[k].push_back(q);
        b->classes[k].lds = std::max(b->classes[k].lds, resident_lds(L->positions, b->cols[q], p->fp64));
    }
    size_t at = (jobs.size() * sizeof(ResidentJob) + 15) & ~(size_t)15;
    for (size_t k = 0; k < b->classes.size(); ++k) {
        ChipBatch::Class &cl = b->classes[k];
        struct Run {
            double cost;
            int q, first, count;
        };
        std::vector<Run> runs;
        int64_t total = 0;
        for (int q : members[k]) total += (jobs[q].m + cl.kind.cols - 1) / cl.kind.cols;
        const int chunk = (int)std::max<int64_t>(1, std::min<int64_t>(32, total / 64));
        for (int q : members[k]) {
            const int groups = (jobs[q].m + cl.kind.cols - 1) / cl.kind.cols;
            const double each = b->step_us[q] * jobs[q].k;
            for (int f = 0; f < groups; f += chunk)
                runs.push_back({each * std::min(chunk, groups - f), q, f, std::min(chunk, groups - f)});
        }
        std::stable_sort(runs.begin(), runs.end(),
                         [](const Run &x, const Run &y) { return x.cost / x.count > y.cost / y.count; });
        std::vector<int2> list[8];
        double load[8] = {0};
        for (const Run &r : runs) {
            int x = 0;
            for (int y = 1; y < 8; ++y)
                if (load[y] < load[x]) x = y;
            load[x] += r.cost;
            for (int i = 0; i < r.count; ++i) list[x].push_back(make_int2(r.q, (r.first + i) * cl.kind.cols));
        }
        size_t most = 0;
        for (const auto &l : list) most = std::max(most, l.size());
        cl.map.clear();
        for (size_t i = 0; i < most; ++i)
            for (const auto &l : list) cl.map.push_back(i < l.size() ? l[i] : make_int2(-1, 0));
        cl.map_at = at;
        at += cl.map.size() * sizeof(int2);
    }
    std::vector<char> args(at, 0);
    std::memcpy(args.data(), jobs.data(), jobs.size() * sizeof(ResidentJob));
    for (const ChipBatch::Class &cl : b->classes)
        std::memcpy(args.data() + cl.map_at, cl.map.data(), cl.map.size() * sizeof(int2));
    if (args != p->up_res_args) {
        if (p->res_args.bytes < at) {
            dev_free(c, &p->res_args);
            VNE_TRY(dev_alloc(c, &p->res_args, at));
        }
        p->up_res_args.clear();
        HIP_TRY(c, hipMemcpyAsync(p->res_args.p, args.data(), at, hipMemcpyHostToDevice, c->stream));
        HIP_TRY(c, hipStreamSynchronize(c->stream));   // args leaves scope
        p->up_res_args = std::move(args);
    }
    return VNE_OK;
}

}  // namespace

vne_status estimate_many(vne_ctx *c, const std::vector<int32_t> &ids, const vne_probes *pr, const int32_t *k_steps,
                         bool fp64, bool desing, vne_result *out) {
    const int n_queries = (int)ids.size();
    // The graphs that go on the chip, their layouts and column groups.  With
    // a memory budget every graph is stacked, so that what a budget admits
    // does not depend on the matrices' sizes.
    std::vector<int> small, large;
    ChipBatch b;
    int m_max = 0, k_max = 0;
    if (n_queries > 1 && chip_mode() != 0 && c->budget == 0) {
        int64_t n = 0, nnz = 0;
        for (int32_t id : ids) {
            const Graph *g = get_graph(c, id);
            n += g->n;
            nnz += g->nnz;
            if (desing && !g->zero_rowsum)
                return fail(c, VNE_EINVAL, "VNE_MODE_DESING needs matrices whose rows sum to zero (A 1 = 0)");
        }
        if (n > INT32_MAX - 1 || nnz > INT32_MAX) return fail(c, VNE_ENOTSUP, "batch too large for int32 indices");
        VNE_TRY(check_queries(c, n_queries, pr, k_steps, &m_max, &k_max));
        for (int q = 0; q < n_queries; ++q)
            if ((pr[q].kind == VNE_PROBE_COLORING || pr[q].kind == VNE_PROBE_DENSE) && pr[q].location != VNE_HOST)
                return fail(c, VNE_EINVAL, pr[q].kind == VNE_PROBE_COLORING
                                               ? "colors must be host arrays in a batch"
                                               : "dense blocks must be host arrays in a batch");
        const int64_t room = lds_elements(fp64);
        int64_t columns = 0;
        for (int q = 0; q < n_queries; ++q)
            if (get_graph(c, ids[q])->n <= room) columns += pr[q].m;
        // columns per workgroup: a read of the matrix serves them all, but
        // every CU wants two workgroups to go to
        int cap = fp64 ? 2 : 4;
        while (cap > 1 && columns / cap < 512) cap /= 2;
        // the smallest workgroup whose registers hold a graph's share: several
        // then share a CU and hide each other's barriers
        struct Fit {
            int q, waves, cols, groups;
            double us;                   // of a step of one workgroup
            double share;                // of a CU's time that the workgroup takes
        };
        std::vector<Fit> fits;
        for (int q = 0; q < n_queries; ++q) {
            const int64_t gn = get_graph(c, ids[q])->n;
            bool found = false;
            for (int cols = cap; gn <= room && !found && cols >= 1; cols /= 2)
                for (int waves = 4; waves <= 16 && !found; waves *= 2) {
                    if (gn * cols * 16 > room * waves) continue;
                    const int w = (int)std::min<int64_t>(waves, (gn + 63) / 64);
                    const ResidentShape *s = shape_of(c, ids[q], w, fp64);
                    if (!s || widest(*s, fp64, cols) < cols) continue;
                    // (two or more on a CU overlap: 0.55 of the lone time each)
                    const bool alone = 2 * resident_lds(s->positions(), cols, fp64) > kResidentLds;
                    fits.push_back({q, w, cols, (pr[q].m + cols - 1) / cols, resident_step_us(*s, cols, fp64),
                                    alone ? 1.0 : 0.55});
                    found = true;
                }
            if (!found) large.push_back(q);
        }
        // Which of them run on the chip: the ones whose workgroups are slowest
        // go to the stack first, as many as make the call shortest.  The chip
        // runs behind the stacked steps, so that a stack that is there anyway
        // takes small graphs of few columns almost for nothing (8 graphs of 1000 to
        // 50 000 rows, FP64, 4 columns: us a step all that fit on the chip 58,
        // all stacked 44), and a batch without one is fastest on the chip
        // (128 graphs of 1000 rows, 16 columns: 42 stacked, 8.8).
        std::stable_sort(fits.begin(), fits.end(),
                         [&](const Fit &x, const Fit &y) { return x.us * k_steps[x.q] > y.us * k_steps[y.q]; });
        size_t first = 0;                // fits[first ..] on the chip
        if (chip_mode() != 1) {
            int64_t sn = 0, snnz = 0, slong = 0;
            int sm = 0, sk = 0, sg = 0;
            auto stack = [&](int q) {
                const Graph *g = get_graph(c, ids[q]);
                sn += g->n;
                snnz += g->nnz;
                slong += g->sched.long_entries;
                sm = std::max(sm, (int)pr[q].m);
                sk = std::max(sk, (int)k_steps[q]);
                ++sg;
            };
            for (int q : large) stack(q);
            double work = 0.0;
            for (const Fit &f : fits) work += f.us * f.share * f.groups * k_steps[f.q];
            // (only for a good eighth: the models are no better, and a first
            // call pays for the larger stack and the trials of its tiles)
            double best = 0.0;
            for (size_t i = 0; i <= fits.size(); ++i) {
                double us = sg == 0 ? 0.0 : sk * launched_us(sg == 1 ? kLaunchUs : kStackLaunchUs, sn, snnz, slong, sm, fp64);
                if (i < fits.size()) us += std::max(fits[i].us * k_steps[fits[i].q], work / 256.0);
                if (i == 0) best = 0.88 * us;
                else if (us < best) {
                    best = us;
                    first = i;
                }
                if (i == fits.size()) break;
                work -= fits[i].us * fits[i].share * fits[i].groups * k_steps[fits[i].q];
                stack(fits[i].q);
            }
        }
        std::vector<const Fit *> of(n_queries, nullptr);
        for (size_t i = first; i < fits.size(); ++i) of[fits[i].q] = &fits[i];
        large.clear();
        for (int q = 0; q < n_queries; ++q) {
            DevLayout *L = of[q] ? layout_of(c, ids[q], of[q]->waves, fp64) : nullptr;
            get_graph(c, ids[q])->shape_rows.clear();
            if (!L) {
                large.push_back(q);
                continue;
            }
            small.push_back(q);
            b.layout.push_back(L);
            b.cols.push_back(of[q]->cols);
            b.step_us.push_back(of[q]->us);
        }
    }
    if (small.empty()) {
        GraphSet *set = nullptr;
        VNE_TRY(get_set(c, ids, &set));
        if (desing && !set->zero_rowsum)
            return fail(c, VNE_EINVAL, "VNE_MODE_DESING needs matrices whose rows sum to zero (A 1 = 0)");
        return estimate_set(c, set, pr, k_steps, fp64, desing, out);
    }
    // a query list of its own for either part
    struct Part {
        std::vector<int32_t> ids, ks, ms;
        std::vector<vne_probes> pr;
        std::vector<vne_result> out;
    };
    auto part_of = [&](const std::vector<int> &qs) {
        Part t;
        for (int q : qs) {
            t.ids.push_back(ids[q]);
            t.ks.push_back(k_steps[q]);
            t.ms.push_back(pr[q].m);
            t.pr.push_back(pr[q]);
            t.out.push_back(out[q]);
        }
        return t;
    };
    Part ts = part_of(small), tl = part_of(large);
    int ms = 0, ks = 0;
    VNE_TRY(check_queries(c, (int)ts.ids.size(), ts.pr.data(), ts.ks.data(), &ms, &ks));
    VNE_TRY(chip_set(c, ts.ids, &b.set));
    VNE_TRY(chip_plan(c, b.set, ms, ks, fp64, &b.p));
    b.p->h_graph_k = ts.ks;
    b.p->h_graph_m = ts.ms;
    VNE_TRY(make_probe_spec(c, b.set, b.p, ts.pr.data(), ms, fp64, &b.ps, &b.combine));
    // the stacked part's set, plan and column tile, before anything runs
    // beside them
    GraphSet *ls = nullptr;
    Plan *lp = nullptr;
    ProbeSpec lspec;
    int lcombine = 0;
    if (!large.empty()) {
        int ml = 0, kl = 0;
        VNE_TRY(check_queries(c, (int)tl.ids.size(), tl.pr.data(), tl.ks.data(), &ml, &kl));
        VNE_TRY(get_set(c, tl.ids, &ls));
        VNE_TRY(get_plan(c, ls, ml, kl, fp64, false, 0, &lp));
        lp->h_graph_k = tl.ks;
        lp->h_graph_m = tl.ms;
        VNE_TRY(make_probe_spec(c, ls, lp, tl.pr.data(), ml, fp64, &lspec, &lcombine));
        VNE_TRY(autotune(c, ls, lp, lspec, desing));
    }
    VNE_TRY(chip_args(c, &b, desing));
    VNE_TRY(side_lanes(c, b.classes.size()));
    Plan *p = b.p;
    VNE_TRY(upload_widths(c, p));
    HIP_TRY(c, hipMemsetAsync(p->flags.p, 0, 4, c->stream));
    HIP_TRY(c, hipMemsetAsync(p->k_eff.p, 0, p->k_eff.bytes, c->stream));   // columns past a query's width
    if (c->timing) {
        VNE_TRY(loop_events(c, p));
        HIP_TRY(c, hipEventRecord(p->ev[0], c->stream));
    }
    if (lp) {
        // the stacked steps first: beside workgroups that hold a CU's whole
        // LDS for milliseconds, each of their launches would wait for room.
        // (The call's span is timed as one.)
        const bool timing = c->timing;
        c->timing = false;
        const vne_status st = run_lanczos(c, ls, lp, lspec, desing);
        c->timing = timing;
        VNE_TRY(st);
    }
    HIP_TRY(c, hipEventRecord(c->side_events[0], c->stream));
    // (the classes that run are joined to the call's stream also where a later
    // one fails; only after the last launch, since a wait on the null stream
    // holds back what follows on the others: 64 graphs of 1000 to 10 000 rows, 8
    // columns, 20 steps 1.50 ms with a wait between launches, 1.08 behind them)
    hipError_t launched = hipSuccess;
    size_t running = 0;
    for (; running < b.classes.size() && launched == hipSuccess; ++running) {
        const ChipBatch::Class &cl = b.classes[running];
        hipStream_t s = c->side_streams[running];
        launched = hipStreamWaitEvent(s, c->side_events[0], 0);
        if (launched == hipSuccess)
            launched = launch_resident_many((const ResidentJob *)p->res_args.p,
                                            (const int2 *)((const char *)p->res_args.p + cl.map_at), (int)cl.map.size(),
                                            cl.waves, cl.kind, cl.lds, s);
        const hipError_t e = hipEventRecord(c->side_events[1 + running], s);
        if (launched == hipSuccess) launched = e;
    }
    for (size_t k = 0; k < running; ++k) {
        const hipError_t e = hipStreamWaitEvent(c->stream, c->side_events[1 + k], 0);
        if (launched == hipSuccess) launched = e;
    }
    HIP_TRY(c, launched);
    if (c->timing) {
        HIP_TRY(c, hipEventRecord(p->ev[1], c->stream));
        // one span: the bytes of either part's own steps, over the longer one's
        const int steps = std::max(p->k, lp ? lp->k : 0);
        const double bytes = step_bytes(b.set, p) * p->k + (lp ? step_bytes(ls, lp) * lp->k : 0.0);
        c->pending.push_back({p, bytes / steps, steps, true});
    }
    HIP_TRY(c, launch_quadrature((const double *)p->alpha.p, (const double *)p->beta.p, (const int32_t *)p->k_eff.p,
                                 (const double *)p->norm2.p, p->k, p->k, p->G * p->m_pad, (double *)p->psi.p,
                                 (int32_t *)p->flags.p, c->stream, fp64));
    if (!lp) {
        c->last_tile = b.cols[0];
        c->last_m_pad = p->m_pad;
    }
    const vne_status st = copy_out(c, p, ts.ms.data(), ts.ks.data(), ts.out.data(), nullptr, b.combine);
    const vne_status sl = lp ? copy_out(c, lp, tl.ms.data(), tl.ks.data(), tl.out.data(), nullptr, lcombine) : VNE_OK;
    for (size_t i = 0; i < small.size(); ++i) out[small[i]].estimate = ts.out[i].estimate;
    for (size_t i = 0; i < large.size(); ++i) out[large[i]].estimate = tl.out[i].estimate;
    VNE_TRY(st);
    return sl;
}

}  // namespace rt
}  // namespace vne
