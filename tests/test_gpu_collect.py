"""Results of a call through one launch into pinned memory, and through copies
past 4 MiB: the arrays that both calls return are equal bit for bit (the second
call asks for the coefficients as well, which takes it past the size), and the
estimate is the mean of the forms, whose sum the two sides order differently
(n eps relative, 1e-13)."""
import numpy as np
import pytest

import synth
import paper_2212_09642_amd as vne
from gpu_common import ctx, _say, _setup  # noqa: F401

pytestmark = pytest.mark.gpu


# m * 100 steps * 16 bytes of coefficients: below, just below and past 4 MiB
@pytest.mark.parametrize("m", [1, 2500, 2700])
@pytest.mark.parametrize("n", [900, 42000])
def test_small_and_large_results(ctx, n, m):
    _say("case results n=%d m=%d" % (n, m))
    nn, e = synth.watts_strogatz(n, 4, 0.1, 3)
    gid, ref = _setup(ctx, nn, e, False)
    few = ctx.estimate(gid, vne.PROBE_RADEMACHER, m, 100, vne.MODE_DESING, seed=5, want_coeffs=False)
    all_ = ctx.estimate(gid, vne.PROBE_RADEMACHER, m, 100, vne.MODE_DESING, seed=5, want_coeffs=True)
    for f in ("quad", "norm2", "k_eff"):
        if f in few and few[f] is not None:
            assert np.array_equal(few[f], all_[f]), f
    assert few["estimate"] == all_["estimate"]
    assert abs(all_["estimate"] - np.mean(all_["quad"])) <= 1e-13 * abs(all_["estimate"])
    ke = all_["k_eff"]
    assert all_["alpha"].shape[0] == m and np.all(ke > 0)
    for c in (0, m // 2, m - 1):                  # every step's coefficients arrived
        assert np.all(all_["alpha"][c, :ke[c]] != 0.0) and np.all(all_["beta"][c, :ke[c] - 1] > 0.0)
    ctx.release(gid)
