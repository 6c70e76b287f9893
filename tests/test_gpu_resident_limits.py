"""Limits of the on-chip runs: contexts with a memory budget keep the launched
steps and their allocations; a failed allocation leaves no error for the
launches after it; whether a lone estimate runs on the chip depends on sizes
alone, and one that does not holds no layout."""
import numpy as np
import pytest

import synth
import paper_2212_09642_amd as vne
from gpu_common import _say

pytestmark = pytest.mark.gpu


def _register(c, n, e, fp64=False):
    g = vne.laplacian_from_edges(n, e, np.float64 if fp64 else np.float32)
    return c.register(g["row_ptr"], g["col_idx"], g["values"], g["scale"], node_keys=g["node_ids"])


@pytest.mark.parametrize("fp64", [False, True])
def test_budget_keeps_the_launched_allocations(fp64, monkeypatch):
    mode = vne.MODE_DESING | (vne.MODE_F64 if fp64 else 0)

    def used(budget):
        """Bytes after registration and after each of three calls."""
        with vne.Context(0, hbm_budget_bytes=budget) as c:
            gid = _register(c, *synth.erdos_renyi(3000, 8.0, 5), fp64)
            out = [c.memory()]
            for m in (16, 300):
                c.estimate(gid, vne.PROBE_RADEMACHER, m, 8, mode, seed=1)
                out.append(c.memory())
            c.estimate_batch([dict(gid=gid, kind=vne.PROBE_RADEMACHER, m=8, k=8, seed=1)], mode)
            return out + [c.memory()]

    _say("case budget fp64=%s" % fp64)
    monkeypatch.setenv("VNE_RESIDENT", "0")
    want = used(0)
    monkeypatch.delenv("VNE_RESIDENT")
    assert used(1 << 30) == want
    # what just fits without the chip fits
    assert used(want[-1]) == want


def test_failed_allocation_is_reported_once():
    _say("case call after a failed allocation")
    with vne.Context(0) as c:
        gid = _register(c, *synth.watts_strogatz(50000, 6, 0.1, 3))
        before = c.estimate(gid, vne.PROBE_RADEMACHER, 8, 4, vne.MODE_DESING, seed=1)
        held = c.memory()
        with pytest.raises(vne.VneError) as ei:      # blocks of 420 GB each
            c.estimate(gid, vne.PROBE_RADEMACHER, 1 << 20, 4, vne.MODE_DESING | vne.MODE_F64, want_coeffs=False)
        assert ei.value.status == -2 and c.memory() == held
        after = c.estimate(gid, vne.PROBE_RADEMACHER, 8, 4, vne.MODE_DESING, seed=1)
        assert np.array_equal(before["quad"], after["quad"])


def test_choice_does_not_depend_on_a_tuned_tile(tmp_path, monkeypatch):
    """A graph near the line between the two ways, with the tuner's choice
    fixed in its cache file at each tile in turn: every call runs the same
    way as the first, and a repeated call gives the same bits."""
    _say("case tuned tiles near the rule's line")
    cache = tmp_path / "tiles"
    monkeypatch.setenv("VNE_AUTOTUNE_CACHE", str(cache))
    n, e = synth.erdos_renyi(16500, 8.0, 5)
    ways = set()
    for tile in (None, 16, 32, 64):
        if tile is not None:
            lines = cache.read_text().split() if cache.exists() else []
            if not lines:
                break                        # every width went on the chip
            cache.write_text("".join("%s %d\n" % (sig, tile) for sig in lines[::2]))
        with vne.Context(0) as c:
            gid = _register(c, n, e)
            for m in (24, 32, 40, 48, 64, 80, 96):
                got = []
                for _ in range(3):
                    out = c.estimate(gid, vne.PROBE_RADEMACHER, m, 6, vne.MODE_DESING, seed=2)
                    got.append((c.last_plan(), out["quad"]))
                assert got[0][0] == got[1][0] == got[2][0], (tile, m, got)
                assert np.array_equal(got[0][1], got[1][1]) and np.array_equal(got[0][1], got[2][1])
                ways.add((m, got[0][0]["tile"] == 1))
    assert len(ways) == 7, ways


def test_a_launched_estimate_holds_no_layout(monkeypatch):
    """Widths around the rule's line on a matrix of unequal values, a fresh
    context each: a launched call holds what it holds without the chip."""
    _say("case no layout held by launched estimates")
    n, e = synth.erdos_renyi(15000, 10.0, 3)
    g = vne.laplacian_from_edges(n, e, np.float32)
    val = np.where(g["values"] < 0, -1.0 - (np.arange(g["values"].size) % 5), g["values"]).astype(np.float32)
    launched = 0
    for m in range(12, 72, 4):
        held = []
        for env in ("0", None):
            monkeypatch.setenv("VNE_RESIDENT", env) if env else monkeypatch.delenv("VNE_RESIDENT")
            with vne.Context(0) as c:
                gid = c.register(g["row_ptr"], g["col_idx"], val, g["scale"])
                c.estimate(gid, vne.PROBE_RADEMACHER, m, 4, 0, seed=1)
                held.append((c.memory(), c.last_plan()["tile"]))
        if held[1][1] >= 4:
            launched += 1
            assert held[0][0] == held[1][0], (m, held)
    assert launched > 0
