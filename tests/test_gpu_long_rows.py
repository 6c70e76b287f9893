"""Launched steps of matrices with long rows, on either side of the rule that
puts these at the front of the step's grid: hubs whose segments stay in the
ordinary blocks, matrices of mostly long rows, preferential attachment; alone
and stacked, against the oracle at the usual bar."""
import numpy as np
import pytest

import oracle
import synth
import paper_2212_09642_amd as vne
from gpu_common import ctx, _say, _setup, _check_quad, _order_sensitivity  # noqa: F401

pytestmark = pytest.mark.gpu


def _hub(n, size, seed):
    """A ring lattice with one row of about `size` entries."""
    n, e = synth.watts_strogatz(n, 6, 0.1, seed)
    far = np.random.default_rng(seed).choice(np.arange(1, n), size, replace=False)
    return n, np.concatenate([np.asarray(e), np.stack([np.zeros_like(far), far], 1)])


GRAPHS = [("hub", lambda: _hub(6000, 4500, 3)), ("dense rows", lambda: synth.erdos_renyi(1500, 100.0, 4)),
          ("attachment", lambda: synth.barabasi_albert(5000, 4, 5)), ("star", lambda: synth.star_graph(4000))]


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("m", [16, 33, 64])
def test_alone_and_stacked(ctx, fp64, m, monkeypatch):
    monkeypatch.setenv("VNE_RESIDENT", "0")
    mode = vne.MODE_DESING | (vne.MODE_F64 if fp64 else 0)
    regs = [_setup(ctx, *make(), fp64) for _, make in GRAPHS]
    want = []
    for i, ((name, _), (gid, ref)) in enumerate(zip(GRAPHS, regs)):
        _say("case long rows: %s m=%d fp64=%s" % (name, m, fp64))
        B = oracle.rademacher_block(60 + i, ref.node_ids, np.arange(m))
        want.append((oracle.quadforms(ref.scipy(), B, 9, oracle.breakdown_tau(fp64)),
                     _order_sensitivity(ref.scipy(), B, 9, fp64)))
        out = ctx.estimate(gid, vne.PROBE_RADEMACHER, m, 9, mode, seed=60 + i)
        _check_quad(out, want[i][0], fp64, sens=want[i][1], n=ref.n)
    _say("case long rows: stacked m=%d fp64=%s" % (m, fp64))
    outs = ctx.estimate_batch([dict(gid=gid, kind=vne.PROBE_RADEMACHER, m=m, k=9, seed=60 + i)
                               for i, (gid, _) in enumerate(regs)], mode, want_coeffs=True)
    for (gid, ref), (w, sens), out in zip(regs, want, outs):
        _check_quad(out, w, fp64, sens=sens, n=ref.n)
        ctx.release(gid)
