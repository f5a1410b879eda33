"""Left-hand sides of Eq. 5 above the FP64 range, which tie at infinity, and
exponents at which a component's last bits decide whether a magnet can flip, on
every path of the relax: flips, spins and fields bit for bit those of the max
tree, and the oracle's."""
import dataclasses

import numpy as np
import pytest

from paper_2002_11401_amd import workloads as W
from test_relax_lds import LDS_MAX_N, assert_oracle, assert_same, line, result
from test_relax_many import SMALL_TILES_MAX_N, spec_and_tree

pytestmark = pytest.mark.gpu


# keys in LDS, batches by tiles with tiles of 64 (from LDS keys and without)
# and of 128, the window's batches, the max tree with a wide row
@pytest.mark.parametrize("n,distance", [(5000, 10.0), (LDS_MAX_N + 300, 10.0), (SMALL_TILES_MAX_N + 300, 10.0),
                                        (LDS_MAX_N + 300, 2.0), (5000, 70.0)])
@pytest.mark.parametrize("case", ["soft", "field"])
def test_infinite_keys(n, distance, case):
    """Two soft magnets in every second tile of 128 (one in 64 tiles of the
    largest size), not each other's neighbours, among magnets with finite keys;
    a field in which every key is infinite."""
    w = dataclasses.replace(line(n, steps=3), neighbor_distance=distance, beta=1.5, gamma=1.5)
    w.H = np.array([[0.2, 0.0], [0.1, 0.0], [-0.27, 0.0]])
    if case == "soft":
        tiles = np.arange(0, n - 128, 256 if n < SMALL_TILES_MAX_N else 8192)
        w.hk[np.concatenate([tiles + 5, tiles + 40])] = 1e-300
    else:
        w.H[:, 0] = 0.0, 0.0, -1e240
        w.spin0[:-20000] = -1  # at most 20,000 of them can flip
    r, tree = spec_and_tree(w)
    assert r["flips"] > 1000
    if case == "soft":  # the infinite keys first, by index
        k = int((w.hk == 1e-300).sum())
        assert np.array_equal(r["idx"][:k], np.flatnonzero(w.hk == 1e-300))
    assert_same(r, tree)
    assert_same(result(w), tree)
    if n < 50000:
        assert_oracle(w, r)


@pytest.mark.parametrize("distance", [2.0, 10.0, 70.0])
@pytest.mark.parametrize("case", ["one term", "two terms"])
def test_large_exponents(distance, case):
    """2 / gamma = 10^6: every left-hand side lies between 1 and 1.05, from
    components that differ from 1 by less than 10^-6."""
    n, e = 5000, 1e6
    w = dataclasses.replace(line(n, steps=3), neighbor_distance=distance, alpha=0.0, beta=2.0 / e, gamma=2.0 / e)
    lhs = 1.0 + np.random.default_rng(8).permutation(np.linspace(1e-3, 0.05, n))
    if case == "one term":
        w.H, w.c = np.array([[0.2, 0.0], [0.1, 0.0], [-0.2, 0.0]]), np.inf
        w.hk = 0.2 / np.exp(np.log(lhs) / e)
    else:
        w.H = np.array([[0.2, 0.0], [0.1, 0.0], [-0.2, 0.2]])
        w.hk = 0.2 / np.exp(np.log(lhs / 2.0) / e)
    r, tree = spec_and_tree(w)
    assert r["flips"] == n
    assert_same(r, tree)
    assert_oracle(w, r)
