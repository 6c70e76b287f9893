"""Whole Lanczos runs inside workgroups (matrices whose v_j column fits in
LDS): the sizes where the row layout changes shape (one wave, partly filled
slices, one round and several, the second register vector, long rows), column
groups of one, two and four, both probe sources that are read per row,
matrices with and without equal off-diagonal values, and batches in which
such graphs meet larger ones.  Each against the oracle at the usual bar."""
import numpy as np
import pytest

import oracle
import synth
import paper_2212_09642_amd as vne
from gpu_common import ctx, _say, _setup, _check_quad, _order_sensitivity  # noqa: F401

pytestmark = pytest.mark.gpu


def _mode(fp64):
    return vne.MODE_DESING | (vne.MODE_F64 if fp64 else 0)


def _rademacher(ctx, gid, ref, m, k, fp64, seed):
    out = ctx.estimate(gid, vne.PROBE_RADEMACHER, m, k, _mode(fp64), seed=seed)
    B = oracle.rademacher_block(seed, ref.node_ids, np.arange(m))
    A = ref.scipy()
    want = oracle.quadforms(A, B, k, oracle.breakdown_tau(fp64))
    _check_quad(out, want, fp64, sens=_order_sensitivity(A, B, k, fp64), n=ref.n)
    return out


# n: one row pair, a slice short of, at and past 64 rows, one round of 16
# waves and past it, many rounds; the last two sizes per type reach the
# second register vector (more than 32 FP32 or 16 FP64 slots a lane)
@pytest.mark.parametrize("fp64,n", [(f, n) for f in (False, True) for n in (2, 63, 64, 65, 1023, 1024, 1025, 5000)]
                         + [(True, 16300), (True, 18300), (False, 32700), (False, 36800)])
def test_sizes(ctx, fp64, n, monkeypatch):
    monkeypatch.setenv("VNE_RESIDENT", "1")       # wherever the rows fit, whatever the speed
    _say("case on chip n=%d fp64=%s" % (n, fp64))
    nn, e = synth.cycle_graph(n) if 2 < n < 100 else synth.path_graph(2) if n == 2 else synth.watts_strogatz(n, 6, 0.1, 3)
    gid, ref = _setup(ctx, nn, e, fp64)
    if n == 2:
        # eigenvalues 0 and 1, f(0) = f(1) = 0: every form is zero, which has
        # no relative error
        out = ctx.estimate(gid, vne.PROBE_RADEMACHER, 3, 12, _mode(fp64), seed=52)
        assert np.all(np.abs(out["quad"]) < 1e-12), out["quad"]
    else:
        _rademacher(ctx, gid, ref, 3, 12, fp64, 50 + n % 7)
    assert ctx.last_plan() == dict(tile=1, m_pad=3)
    ctx.release(gid)


# column groups: a CU each up to 256 columns, then two and four per workgroup
@pytest.mark.parametrize("fp64,m,cols", [(False, 256, 1), (False, 257, 2), (False, 515, 4), (True, 259, 2)])
def test_column_groups_and_hubs(ctx, fp64, m, cols, monkeypatch):
    monkeypatch.setenv("VNE_RESIDENT", "1")
    _say("case on chip hubs m=%d fp64=%s" % (m, fp64))
    n, e = synth.barabasi_albert(2500, 4, 17)     # rows of up to some hundred entries
    gid, ref = _setup(ctx, n, e, fp64)
    _rademacher(ctx, gid, ref, m, 10, fp64, 7)
    assert ctx.last_plan()["tile"] == cols
    ctx.release(gid)


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("m", [5, 300, 600])
def test_weighted_dense_and_colouring(ctx, fp64, m, monkeypatch):
    """Unequal off-diagonal values (a weighted Laplacian with hub rows), from
    a caller's block on the device, and colour indicators."""
    import torch
    monkeypatch.setenv("VNE_RESIDENT", "1")
    _say("case on chip weighted m=%d fp64=%s" % (m, fp64))
    n, e = synth.barabasi_albert(1500, 3, 23)
    ref = oracle.laplacian_from_edges(n, e)
    L = ref.scipy().tocoo()
    w = 1.0 + (np.minimum(L.row, L.col) * 31 + np.maximum(L.row, L.col) * 17) % 5
    import scipy.sparse as sp
    W = sp.csr_matrix((np.where(L.row != L.col, -w, 0.0), (L.row, L.col)), shape=L.shape)
    W = (W + sp.diags(-np.asarray(W.sum(1)).ravel())).tocsr()
    W.sort_indices()
    scale = 1.0 / W.diagonal().sum()
    gid = ctx.register(W.indptr, W.indices, W.data.astype(np.float64 if fp64 else np.float32), scale)
    B = np.random.default_rng(4).standard_normal((n, m))
    B = B if fp64 else B.astype(np.float32).astype(np.float64)
    out = ctx.estimate(gid, vne.PROBE_DENSE, m, 10, _mode(fp64),
                       dense=torch.from_numpy(B).to("cuda", torch.float64 if fp64 else torch.float32))
    A = W * scale
    want = oracle.quadforms(A, B, 10, oracle.breakdown_tau(fp64))
    _check_quad(out, want, fp64, sens=_order_sensitivity(A, B, 10, fp64), n=n)
    col = (np.arange(n) % m).astype(np.int32)
    out = ctx.estimate(gid, vne.PROBE_COLORING, m, 10, _mode(fp64), colors=col)
    P = oracle.indicator_block(col, m)
    want = oracle.quadforms(A, P, 10, oracle.breakdown_tau(fp64))
    _check_quad(out, want, fp64, sens=_order_sensitivity(A, P, 10, fp64), n=n)
    ctx.release(gid)


@pytest.mark.parametrize("fp64", [False, True])
def test_batch_of_chip_and_stacked_graphs(ctx, fp64):
    """Graphs that fit on the chip in workgroups of several shapes beside one
    that does not, widths and step counts of their own; a second call on other
    seeds, then the first again bit for bit."""
    _say("case batch on chip and stacked fp64=%s" % fp64)
    graphs = [synth.erdos_renyi(300, 6.0, 1), synth.barabasi_albert(1200, 4, 2), synth.complete_graph(70),
              synth.watts_strogatz(3000, 8, 0.1, 3), synth.barabasi_albert(9000, 3, 4),
              synth.watts_strogatz(20100 if fp64 else 41000, 6, 0.1, 5), synth.star_graph(600)]
    regs = [_setup(ctx, n, e, fp64) for n, e in graphs]
    def queries(s):
        return [dict(gid=gid, kind=vne.PROBE_RADEMACHER, m=1 + 9 * i, k=9 + i, seed=s + i)
                for i, (gid, _) in enumerate(regs)]
    first = ctx.estimate_batch(queries(70), _mode(fp64), want_coeffs=True)
    for i, ((gid, ref), out) in enumerate(zip(regs, first)):
        _say("  query %d n=%d" % (i, ref.n))
        B = oracle.rademacher_block(70 + i, ref.node_ids, np.arange(1 + 9 * i))
        A = ref.scipy()
        want = oracle.quadforms(A, B, 9 + i, oracle.breakdown_tau(fp64))
        _check_quad(out, want, fp64, sens=_order_sensitivity(A, B, 9 + i, fp64), n=ref.n)
        assert abs(out["estimate"] - out["quad"].mean()) <= 1e-13 * abs(out["estimate"])
    ctx.estimate_batch(queries(900), _mode(fp64))
    again = ctx.estimate_batch(queries(70), _mode(fp64), want_coeffs=True)
    for a, b in zip(first, again):
        for key in ("quad", "alpha", "beta", "k_eff", "norm2"):
            assert np.array_equal(a[key], b[key]), key
    for gid, _ in regs:
        ctx.release(gid)
