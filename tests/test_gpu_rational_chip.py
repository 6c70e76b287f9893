"""Rational Arnoldi steps with a workgroup per column (small matrices) against
the launched path (VNE_RESIDENT=0), which the oracle checks at the same bar:
sizes at the edges of a wave, a round of 1024 rows and the largest one, long
rows, equal and unequal off-diagonal values, one column and a padded block.

Bar: 1e-10 relative per form and step, the bar against the oracle; both sides
solve to the same relative residual of 1e-12 and differ in summation order
only.  Basis sizes and switch steps are equal."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import synth
import paper_2212_09642_amd as vne
from gpu_common import ctx, _say, _setup  # noqa: F401

pytestmark = pytest.mark.gpu

RTOL = 1e-10
MODE = vne.MODE_F64 | vne.MODE_DESING


def _both(ctx, monkeypatch, gid, m, steps, **kw):
    out = []
    for mode in ("0", None):
        if mode is None:
            monkeypatch.delenv("VNE_RESIDENT", raising=False)
        else:
            monkeypatch.setenv("VNE_RESIDENT", mode)
        out.append(ctx.rational(gid, vne.PROBE_RADEMACHER, m, MODE, steps, cg_tol=1e-12, seed=9, **kw))
    want, got = out
    err = np.abs(got["psi_steps"] - want["psi_steps"]) / np.abs(want["psi_steps"])
    _say("  worst rel err %.2e, %d and %d CG iterations" % (err.max(), want["cg_iterations"], got["cg_iterations"]))
    assert err.max() <= RTOL
    assert np.array_equal(got["basis"], want["basis"])
    assert np.array_equal(got["switch_step"], want["switch_step"])
    assert np.array_equal(got["norm2"], want["norm2"])
    # every finite pole counts its iterations once, in both totals
    assert int((got["apps_steps"][:, -1] - steps).sum()) == got["cg_iterations"]


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n,m", [(63, 3), (64, 1), (65, 17), (1023, 3), (1025, 5), (4900, 2), (5200, 2)])
def test_against_the_launched_path(ctx, n, m, weighted, monkeypatch):
    _say("case rational on chip n=%d m=%d weighted=%s" % (n, m, weighted))
    # (the Laplacian's smallest eigenvalues are far from the poles, so that
    # the solves take some tens of iterations)
    nn, e = synth.barabasi_albert(n, 3, 5)
    if weighted:
        ref = oracle.laplacian_from_edges(nn, e)
        L = ref.scipy().tocoo()
        w = 1.0 + (np.minimum(L.row, L.col) * 31 + np.maximum(L.row, L.col) * 17) % 5
        W = sp.csr_matrix((np.where(L.row != L.col, -w, 0.0), (L.row, L.col)), shape=L.shape)
        W = (W + sp.diags(-np.asarray(W.sum(1)).ravel())).tocsr()
        W.sort_indices()
        tr = W.diagonal().sum()
        lam_max = 2.0 * W.diagonal().max() / tr
        gid = ctx.register(W.indptr, W.indices, W.data.astype(np.float64), 1.0 / tr)
    else:
        gid, ref = _setup(ctx, nn, e)
        lam_max = 2.0 * ref.scipy().diagonal().max()
    steps = 11                                   # a full turn of eight basis vectors and a part of one
    poles = [np.inf] * 2 + list(-np.geomspace(lam_max, 1e-3 * lam_max, steps - 3))
    _both(ctx, monkeypatch, gid, m, steps, poles=poles)
    ctx.release(gid)


def test_switch_rule(ctx, monkeypatch):
    n, e = synth.path_graph(300)
    _say("case rational on chip switch rule path n=300 m=3")
    gid, ref = _setup(ctx, n, e)
    lam = np.linalg.eigvalsh(ref.scipy().toarray())
    _both(ctx, monkeypatch, gid, 3, 20, finite_poles=list(-np.geomspace(lam[-1], lam[1], 10)), ell=3, c=0.75,
          lam_lo=0.999 * lam[1], lam_hi=1.001 * lam[-1])
    ctx.release(gid)
