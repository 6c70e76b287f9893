"""Tasks that start and end together in the serving loop: more of them in one
tick than one launch of quadratures or results takes (32), more slots of one
width than lanes that look for one (64), group slots whose
members start at once, and a query far wider than a task.  Every query has the
bits that it has alone."""
import numpy as np
import pytest

import synth
import paper_2212_09642_amd as vne
from gpu_common import ctx, _say, _setup  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("queries", [32, 33, 300])
def test_bits_of_a_burst(ctx, fp64, queries):
    _say("case serving burst of %d fp64=%s" % (queries, fp64))
    mode = vne.MODE_DESING | (vne.MODE_F64 if fp64 else 0)
    graphs = [_setup(ctx, *g, fp64)[0] for g in (synth.barabasi_albert(900, 6, 1), synth.watts_strogatz(1500, 6, 0.1, 2))]
    # (16 columns: grouped in FP32; the last query has several tasks)
    specs = [dict(gid=graphs[i % 2], m=(1, 16, 16, 37)[i % 4], k=7, seed=i) for i in range(queries)]
    specs[-1]["m"] = 1000
    with vne.Server(ctx, mode, arena_bytes=1 << 30) as srv:
        tickets = [srv.submit(s["gid"], m=s["m"], k=s["k"], seed=s["seed"]) for s in specs]
        got = [srv.poll(t, want_quad=True) for t in tickets]
        for s, r in zip(specs, got):
            assert r["status"] == 0, r["message"]
            assert r["probes"] == s["m"] and r["steps"] == s["k"]
            alone = srv.poll(srv.submit(s["gid"], m=s["m"], k=s["k"], seed=s["seed"]), want_quad=True)
            assert np.array_equal(alone["quad"], r["quad"]) and alone["estimate"] == r["estimate"]
            assert abs(r["estimate"] - r["quad"].mean()) <= 1e-13 * abs(r["estimate"])
    for g in graphs:
        ctx.release(g)
