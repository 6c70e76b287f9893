"""The rule for on-chip runs: matrices whose slowest wave or spilled columns
would be slower than launched steps stay there, and a batch weighs the stack
that is there anyway; every way against the oracle."""
import numpy as np
import pytest

import oracle
import synth
import paper_2212_09642_amd as vne
from gpu_common import ctx, _say, _setup, _check_quad, _order_sensitivity  # noqa: F401

pytestmark = pytest.mark.gpu


def _mode(fp64):
    return vne.MODE_DESING | (vne.MODE_F64 if fp64 else 0)


def test_lone_estimates(ctx):
    """(graph, columns, FP64): launched where the chip measured slower, on the
    chip where the launches did."""
    hub = synth.watts_strogatz(30000, 6, 0.1, 3)
    far = np.random.default_rng(1).choice(np.arange(1, 30000), 25000, replace=False)
    hub = (hub[0], np.concatenate([np.asarray(hub[1]), np.stack([np.zeros_like(far), far], 1)]))
    for name, (n, e), m, fp64, chip in (
            ("one row of 25 000", hub, 64, False, False),
            ("small", synth.erdos_renyi(2000, 8.0, 3), 30, True, True),
            ("few columns, many rows", synth.erdos_renyi(39000, 8.0, 3), 8, False, False),
            ("many columns", synth.erdos_renyi(30000, 8.0, 3), 256, False, True)):
        _say("case rule: %s m=%d fp64=%s" % (name, m, fp64))
        gid, ref = _setup(ctx, n, e, fp64)
        ctx.estimate(gid, vne.PROBE_RADEMACHER, m, 4, _mode(fp64), seed=1)
        plan = ctx.last_plan()
        assert (plan["tile"] <= 2) == chip, plan
        ctx.release(gid)


def test_two_fp64_columns_of_unequal_values_are_not_taken(ctx, monkeypatch):
    """600 columns: one a workgroup, in three rounds (two would spill)."""
    _say("case rule: unequal values, FP64, 600 columns")
    monkeypatch.setenv("VNE_RESIDENT", "1")
    n, e = synth.erdos_renyi(900, 8.0, 5)
    ref = oracle.laplacian_from_edges(n, e)
    A = ref.scipy().tocsr().copy()
    w = 1.0 + (np.arange(A.nnz) % 3)
    A.data = A.data * w
    A = (A + A.T).tocsr()
    A.sort_indices()
    gid = ctx.register(A.indptr, A.indices, A.data, 1.0)
    out = ctx.estimate(gid, vne.PROBE_RADEMACHER, 600, 8, vne.MODE_F64, seed=3)
    assert ctx.last_plan()["tile"] == 1
    B = oracle.rademacher_block(3, np.arange(ref.n), np.arange(600))
    want = oracle.quadforms(A, B, 8, oracle.breakdown_tau(True), desing=False)
    _check_quad(out, want, True, sens=_order_sensitivity(A, B, 8, True, desing=False), n=ref.n)
    ctx.release(gid)


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("m", [3, 40])
def test_batches_of_few_and_many_columns(ctx, fp64, m):
    """Small graphs beside two that do not fit: with few columns some of the
    small ones join the stack."""
    graphs = [synth.watts_strogatz(n, 6, 0.1, n) for n in (700, 2100, 6000, 15000, 41000, 42000)]
    regs = [_setup(ctx, n, e, fp64) for n, e in graphs]
    _say("case rule: batch m=%d fp64=%s" % (m, fp64))
    q = [dict(gid=gid, kind=vne.PROBE_RADEMACHER, m=m, k=8, seed=90 + i) for i, (gid, _) in enumerate(regs)]
    outs = ctx.estimate_batch(q, _mode(fp64), want_coeffs=True)
    for i, ((gid, ref), out) in enumerate(zip(regs, outs)):
        B = oracle.rademacher_block(90 + i, ref.node_ids, np.arange(m))
        want = oracle.quadforms(ref.scipy(), B, 8, oracle.breakdown_tau(fp64))
        _check_quad(out, want, fp64, sens=_order_sensitivity(ref.scipy(), B, 8, fp64), n=ref.n)
    again = ctx.estimate_batch(q, _mode(fp64), want_coeffs=True)
    for a, b in zip(outs, again):
        for key in ("quad", "alpha", "beta", "k_eff", "norm2"):
            assert np.array_equal(a[key], b[key]), key
    for gid, _ in regs:
        ctx.release(gid)


def test_timed_bytes_are_each_parts_own(ctx):
    """A batch on the chip and stacked, of different step counts: each part's
    bytes a step over its own steps."""
    _say("case timed bytes of a mixed batch")
    regs = [_setup(ctx, *synth.watts_strogatz(n, 6, 0.1, n), False) for n in (1500, 3000, 41000)]
    q = [dict(gid=gid, kind=vne.PROBE_RADEMACHER, m=64, k=k, seed=1) for (gid, _), k in zip(regs, (30, 30, 5))]
    ctx.estimate_batch(q, _mode(False))
    ctx.enable_kernel_timing(True)
    ctx.kernel_timing(reset=True)
    ctx.estimate_batch(q, _mode(False))
    got = ctx.kernel_timing(reset=True)
    ctx.enable_kernel_timing(False)

    def step(parts):
        n, nnz = sum(ref.n for _, ref in parts), sum(ref.col_idx.size for _, ref in parts)
        return 4.0 * (n + 1) + 8.0 * nnz + 3.0 * 4.0 * 64 * n

    want = 30 * step(regs[:2]) + 5 * step(regs[2:])
    assert got["launches"] == 30 and abs(got["bytes"] - want) <= 1e-9 * want, (got, want)
    for gid, _ in regs:
        ctx.release(gid)
