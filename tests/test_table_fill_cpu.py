"""Look-up tables against their rule, entry by entry: entry j covers
[j, j + 1) / scale; it holds the code -2 - k of the first band k that meets it,
else the bin below the band ends at or below it, else -1."""
import numpy as np
import pytest

from paper_2301_12557_amd import fcfc
from test_bands_cpu import _tables

EDGES = {
    "uniform": np.linspace(0, 150, 31),
    "from above zero": np.linspace(7, 90, 12),
    "one bin": np.array([0.0, 30.0]),
    "one bin, no zero": np.array([29.9, 30.0]),
    "logarithmic": np.concatenate([[0.0], np.geomspace(1e-3, 200, 40)]),
    "many edges in one entry": np.concatenate([np.linspace(0.0, 0.5, 40), [100.0, 200.0]]),
    "narrow": 50.0 + np.arange(6) * 1e-2,
}


@pytest.mark.parametrize("name", sorted(EDGES))
@pytest.mark.parametrize("lut_log2", [0, 8, 14])
def test_entries_follow_the_rule(name, lut_log2):
    e = EDGES[name]
    p = fcfc.Plan("s", e, box=1000.0, n_hint=10000, lut_log2=lut_log2)
    seen = 0
    for _, t, _ in _tables(p):
        lo, hi = t["lo"].astype(np.float64), t["hi"].astype(np.float64)
        a = np.arange(len(t["tab"])) / float(t["scale"])
        b = (np.arange(len(t["tab"])) + 1) / float(t["scale"])
        want = np.full(len(a), -1, dtype=np.int64)
        below = (hi[None, :] <= a[:, None]).sum(axis=1)  # band ends never decrease
        want[(below >= 1) & (below < len(e))] = below[(below >= 1) & (below < len(e))] - 1
        meets = (lo[None, :] < b[:, None]) & (hi[None, :] > a[:, None]) & (hi > lo)[None, :]
        hot = meets.any(axis=1)
        want[hot] = -2 - meets.argmax(axis=1)[hot]
        assert np.array_equal(t["tab"], want)
        seen += 1
    assert seen >= 1
    p.close()
