"""Batches on either way: the stacked launches of several graphs (per-graph
sums, long rows of several graphs, the tuner's choice of a tile for a stack)
and the on-chip workgroups of one, two and four columns, in both types and for
every probe kind of a batch, each query against the oracle."""
import numpy as np
import pytest

import oracle
import synth
import paper_2212_09642_amd as vne
from gpu_common import ctx, _say, _setup, _check_quad, _order_sensitivity  # noqa: F401
from test_gpu_batch import _graphs, _register_all

pytestmark = pytest.mark.gpu

WAYS = ["0", "1", None]        # stacked, on the chip wherever the rows fit, by the rule


def _way(monkeypatch, way):
    if way is None:
        monkeypatch.delenv("VNE_RESIDENT", raising=False)
    else:
        monkeypatch.setenv("VNE_RESIDENT", way)


def _mode(fp64):
    return vne.MODE_DESING | (vne.MODE_F64 if fp64 else 0)


def _against(ref, out, B, k, fp64, desing=True):
    A = ref.scipy()
    _check_quad(out, oracle.quadforms(A, B, k, oracle.breakdown_tau(fp64), desing=desing), fp64,
                sens=_order_sensitivity(A, B, k, fp64, desing=desing), n=ref.n)


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("way", WAYS)
def test_rademacher(ctx, fp64, way, monkeypatch):
    """Widths and step counts per graph, the tile picked by the tuner."""
    _way(monkeypatch, way)
    regs = _register_all(ctx, _graphs(), fp64)
    outs = ctx.estimate_batch([dict(gid=gid, kind=vne.PROBE_RADEMACHER, m=m, k=k, seed=300 + i)
                               for i, (_, gid, _, m, k) in enumerate(regs)], _mode(fp64), want_coeffs=True)
    for i, ((name, gid, ref, m, k), out) in enumerate(zip(regs, outs)):
        _say("case stack way=%s fp64=%s %s" % (way, fp64, name))
        _against(ref, out, oracle.rademacher_block(300 + i, ref.node_ids, np.arange(m)), k, fp64)
        assert abs(out["estimate"] - out["quad"].mean()) <= 1e-13 * abs(out["estimate"])
        ctx.release(gid)


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("way", WAYS)
def test_colouring_and_dense(ctx, fp64, way, monkeypatch):
    _way(monkeypatch, way)
    graphs = [synth.watts_strogatz(1500, 8, 0.1, 31), synth.barabasi_albert(900, 5, 32), synth.grid2d_graph(25, 17)]
    regs = [_setup(ctx, n, e, fp64) for n, e in graphs]
    _say("case stack colouring way=%s fp64=%s" % (way, fp64))
    qs, cols = [], []
    for gid, ref in regs:
        col, s = oracle.greedy_distance_coloring(ref.row_ptr, ref.col_idx, ref.n, 2)
        cols.append((col, s))
        qs.append(dict(gid=gid, kind=vne.PROBE_COLORING, m=s, k=12, colors=np.asarray(col, np.int32)))
    for (gid, ref), (col, s), out in zip(regs, cols, ctx.estimate_batch(qs, _mode(fp64))):
        _against(ref, out, oracle.indicator_block(col, s), 12, fp64)
        assert abs(out["estimate"] - out["quad"].sum()) <= 1e-13 * abs(out["estimate"])
    _say("case stack dense way=%s fp64=%s" % (way, fp64))
    rng = np.random.default_rng(7)
    ty = np.float64 if fp64 else np.float32
    blocks = [rng.standard_normal((ref.n, m)).astype(ty) for (_, ref), m in zip(regs, (3, 17, 9))]
    outs = ctx.estimate_batch([dict(gid=gid, kind=vne.PROBE_DENSE, m=B.shape[1], k=12, dense=B)
                               for (gid, _), B in zip(regs, blocks)], vne.MODE_F64 if fp64 else 0)
    for (gid, ref), B, out in zip(regs, blocks, outs):
        _against(ref, out, B.astype(np.float64), 12, fp64, desing=False)
        ctx.release(gid)


@pytest.mark.parametrize("fp64", [False, True])
def test_two_graphs_past_the_chip(ctx, fp64):
    """The stack of a mixed batch holds two graphs (one with hubs): its sums
    are per graph, beside workgroups on the chip."""
    big = 20000 if fp64 else 40500
    graphs = [synth.erdos_renyi(500, 6.0, 1), synth.barabasi_albert(big, 3, 2), synth.watts_strogatz(2500, 8, 0.1, 3),
              synth.watts_strogatz(big, 6, 0.1, 4), synth.barabasi_albert(1800, 4, 5)]
    regs = [_setup(ctx, n, e, fp64) for n, e in graphs]
    _say("case stack of two beside the chip fp64=%s" % fp64)
    outs = ctx.estimate_batch([dict(gid=gid, kind=vne.PROBE_RADEMACHER, m=5 + 3 * i, k=8 + i, seed=40 + i)
                               for i, (gid, _) in enumerate(regs)], _mode(fp64), want_coeffs=True)
    for i, ((gid, ref), out) in enumerate(zip(regs, outs)):
        _against(ref, out, oracle.rademacher_block(40 + i, ref.node_ids, np.arange(5 + 3 * i)), 8 + i, fp64)
        ctx.release(gid)


# enough columns in all for two (1024) and four (2048) in a workgroup
@pytest.mark.parametrize("fp64,m,cols", [(False, 350, 2), (False, 690, 4), (True, 350, 2)])
def test_column_groups_of_a_batch(ctx, fp64, m, cols, monkeypatch):
    _way(monkeypatch, "1")
    regs = [_setup(ctx, *synth.barabasi_albert(700 + 400 * i, 4, i), fp64) for i in range(3)]
    _say("case batch of %d columns fp64=%s" % (3 * m, fp64))
    outs = ctx.estimate_batch([dict(gid=gid, kind=vne.PROBE_RADEMACHER, m=m, k=7, seed=80 + i)
                               for i, (gid, _) in enumerate(regs)], _mode(fp64))
    assert ctx.last_plan()["tile"] == cols
    for i, ((gid, ref), out) in enumerate(zip(regs, outs)):
        _against(ref, out, oracle.rademacher_block(80 + i, ref.node_ids, np.arange(m)), 7, fp64)
        ctx.release(gid)
