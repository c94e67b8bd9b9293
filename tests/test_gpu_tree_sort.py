"""The tree's radix sort and its scans where a tile or a level ends."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 65, 2047, 2048, 2049, 131072, 131073, 300001])
def test_sort_is_stable_and_complete(n):
    """Keys ascend, equal keys keep the input order, every particle appears
    once, and every key is its particle's (equal positions have equal keys)."""
    from paper_1304_4235_amd import Solver
    rng = np.random.default_rng(n)
    wl = W.isothermal_halo(n=n, n_bins=1, seed=2)
    cells = rng.integers(0, 40, (n, 3))                       # many equal positions
    wl.pos = cells.astype(np.float32)
    wl.h = np.full(n, 0.4, np.float32)
    s = Solver.from_workload(wl, record_paths=0)
    t = s.tree()
    code, perm = np.asarray(t["codes"], np.uint64), np.asarray(t["perm"])
    s.close()
    np.testing.assert_array_equal(np.sort(perm), np.arange(n))
    assert np.all(code[1:] >= code[:-1])
    same = code[1:] == code[:-1]
    assert np.all(perm[1:][same] > perm[:-1][same])
    cell = (cells[:, 0] * 40 + cells[:, 1]) * 40 + cells[:, 2]
    first = np.concatenate([[True], ~same])
    assert first.sum() == np.unique(cell).size
    assert np.all(cell[perm][1:][same] == cell[perm][:-1][same])
