"""Speculative batches by tiles (up to 2^20 magnets, 17 to 64 neighbours):
flips, spins and fields bit for bit those of the one-at-a-time relax on the max
tree, at the sizes and parameters where they can go wrong."""
import dataclasses

import numpy as np
import pytest

from paper_2002_11401_amd import asi
from paper_2002_11401_amd import workloads as W
from test_relax_lds import LDS_MAX_N, assert_oracle, assert_same, result
from test_relax_lds import line as narrow_line

pytestmark = pytest.mark.gpu
SMALL_TILES_MAX_N, MANY_MAX_N = 1 << 19, 1 << 20
TREE = dict(spec_min=10**12)  # no speculation: the max tree where keys are not in LDS


def line(n, distance=10.0, **kw):
    return dataclasses.replace(narrow_line(n, **kw), neighbor_distance=distance)


def spec_and_tree(w, **kw):
    """Batches from the first flippable magnet on (never fewer than two), and
    the max tree alone (one wavefront less keeps small instances off LDS keys)."""
    tree = TREE if w.n > LDS_MAX_N else dict(relax_waves=1)
    return result(w, tuning=dict(spec_min=1), **kw), result(w, tuning=tree, **kw)


# part of a tile, a tile and one more, the rows once and once more, the largest
# size of small tiles and the next, the largest size and the first beyond it
@pytest.mark.parametrize("n", [21, 64, 65, 8191, LDS_MAX_N + 1, 65536, 65537,
                               SMALL_TILES_MAX_N, SMALL_TILES_MAX_N + 1, MANY_MAX_N, MANY_MAX_N + 1])
def test_sizes(n):
    w = line(n, steps=3 if n > 100000 else 10)
    r, tree = spec_and_tree(w)
    assert r["flips"] > 0
    if n > 4096:
        assert_same(r, tree)
    if n < 50000:
        assert_oracle(w, r)


@pytest.mark.parametrize("mode", ["carry", "dirty", "full"])
@pytest.mark.parametrize("case", ["row16", "row18", "kagome3", "row32", "row34", "row64", "row66", "hot"])
def test_same_as_other_paths(case, mode):
    """Neighbours at the edges of the degrees taken and of half a wavefront."""
    if case.startswith("row"):
        w = line(40000, int(case[3:]) / 2.0, steps=8)
    else:
        H = W.rotating(12, 0.08, 40)
        w = W.family_instance("kagome", 38000, 3.0, 9, H,
                              0.01 if case == "hot" else 0.0, 9)
    r, tree = spec_and_tree(w, field_mode=mode)
    assert r["flips"] > 100
    assert_same(r, tree)


# no disorder: whole sublattices tie at every flip; ties between tiles; extreme
# exponents; large keys; no hard-axis term; h_k tiny
@pytest.mark.parametrize("case", ["ties", "few ties", "exponents", "strong", "parallel", "tiny"])
def test_key_ranges(case):
    H = W.linear_ramp(5, 0.27, -0.27, 33.0)
    w = W.family_instance("square", 2 * 140 * 141, 2.0, 3, H)
    assert w.n > LDS_MAX_N
    if case == "ties":
        w.hk = np.full(w.n, 0.2)
    elif case == "few ties":
        w.hk[: w.n // 2] = w.hk[w.n // 2 : 2 * (w.n // 2)]
    elif case == "exponents":
        w = dataclasses.replace(w, beta=0.3, gamma=9.5)
    elif case == "strong":
        w.H = w.H * 400.0
    elif case == "parallel":
        w = dataclasses.replace(w, **asi.PARALLEL_CRITERION)
    else:
        w = dataclasses.replace(w, hk=w.hk * 1e-30, H=w.H * 1e-30, alpha=w.alpha * 1e-30)
    r, tree = spec_and_tree(w)
    assert r["flips"] > 0
    assert_same(r, tree)


def test_flip_limit_leaves_no_trace():
    """A run with exactly enough flips, one that ends at the limit, and the
    same handle again."""
    w = line(LDS_MAX_N + 300, steps=6)
    plain = result(w)
    most = int(np.bincount(plain["step"]).max())
    sim = asi.Sim.from_workload(w, max_flips_per_step=most)  # exactly enough
    assert sim.run() == plain["flips"] and sim.flip_log()["hash"] == plain["hash"]
    sim.close()
    sim = asi.Sim.from_workload(w, max_flips_per_step=most - 1)
    for _ in range(2):
        with pytest.raises(asi.AsiError) as e:
            sim.run()
        assert e.value.status == asi.ASI_ELOOP
        k = sim.flip_log()["idx"]
        assert np.array_equal(k, plain["idx"][: len(k)]) and len(k) >= most - 1
        sim.set_state(w.spin0, -1)
    sim.close()


def test_batch_of_every_path():
    """Instances of every path in one batch, each mode."""
    wide = line(LDS_MAX_N + 5, 65.0, steps=5)
    ws = [line(50, steps=5), wide, line(LDS_MAX_N + 70, steps=5), line(LDS_MAX_N + 9, 2.0, steps=5),
          line(5000, steps=5)]
    plain = [result(w) for w in ws]
    for mode in ("lockstep", "graph", "fused"):
        sims = [asi.Sim.from_workload(w) for w in ws]
        flips = asi.batch_run(sims, mode)
        for s, f, p in zip(sims, flips, plain):
            assert f == p["flips"] and s.flip_log()["hash"] == p["hash"]
            assert np.array_equal(s.state()[0], p["s"])
            s.close()


@pytest.mark.parametrize("ties", [False, True])
def test_paused_mid_step(ties):
    """Server bursts of a fraction of a step: the relax is interrupted within
    steps and taken up again; with every key tied, on the exact path too."""
    ws = [line(LDS_MAX_N + 77, seed=s, steps=4) for s in (1, 2)]
    for w in ws:
        w.H[:] = np.linspace(0.05, -0.3, 4)[:, None] * w.H[0] / np.abs(w.H[0]).max()
        if ties:
            w.hk[:] = 0.2
    plain = [result(w) for w in ws]
    assert max(np.bincount(p["step"]).max() for p in plain) > 3000
    srv = asi.Server(hbm_budget_bytes=4 << 30, max_slots=4)
    ids = [srv.submit(w) for w in ws]
    for _ in range(20000):
        if not srv.step(budget_ms=0.3):
            break
    for i, p in zip(ids, plain):
        res = srv.take(i)
        assert (res["flips"], res["hash"]) == (p["flips"], p["hash"])
        assert np.array_equal(res["spins"], p["s"])
    srv.close()


@pytest.mark.parametrize("n", [4096, 4097])
def test_default_threshold(n):
    """On both sides of the size up to which the default threshold stays with
    one flip at a time."""
    w = line(n)
    assert_same(result(w), result(w, tuning=dict(spec_min=1)))
