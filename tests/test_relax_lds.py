"""Relax with every key in LDS (one flip at a time): flips, spins and fields
against the oracle, and bit for bit against the paths that hold their keys in
memory, at the sizes and parameters where it can go wrong."""
import dataclasses

import numpy as np
import pytest

from oracle import native as N
from paper_2002_11401_amd import asi
from paper_2002_11401_amd import workloads as W

pytestmark = pytest.mark.gpu
LDS_MAX_N = 36864


def result(w, tuning=None, **kw):
    sim = asi.Sim.from_workload(w, **kw)
    if tuning:
        t = sim.tuning()
        sim.set_tuning(tuning.get("relax_waves", t["relax_waves"]), t["l1_shift"],
                       tuning.get("spec_min", t["spec_min"]))
    flips = sim.run()
    log, (s, hp, hq, _) = sim.flip_log(), sim.state()
    sim.close()
    return dict(flips=flips, step=log["step"], idx=log["idx"], hash=log["hash"], s=s, hp=hp, hq=hq)


def assert_same(a, b):
    for k in a:
        assert np.array_equal(a[k], b[k]), k


def assert_oracle(w, r):
    o = N.Oracle.from_workload(w)
    o.set_spins(w.spin0)
    e = o.run(w.H)
    assert r["flips"] == e["n_flips"] > 0
    assert np.array_equal(r["idx"], e["idx"]) and np.array_equal(r["step"], e["step"])
    assert np.array_equal(r["s"], o.spins())


def line(n, seed=5, steps=12):
    xy, theta = W.ising(n, 1)
    H = W.linear_ramp(steps, 0.3, -0.3, 20.0)
    return W.Workload("line", xy, theta, W.polarised_spins(theta, H[0]),
                      W.disorder_hk(n, 0.2, 0.05, seed), H, alpha=0.01, neighbor_distance=2.0,
                      b=1.0, c=1.0, beta=3.0, gamma=3.0)


# one magnet, a partial tile, a whole wavefront, the step of the tile size at
# 1024 threads (4096, 32768), the largest size and the first beyond it
@pytest.mark.parametrize("n", [1, 3, 64, 4095, 4097, 32769, LDS_MAX_N, LDS_MAX_N + 1])
def test_sizes_match_the_oracle(n):
    w = line(n)
    assert_oracle(w, result(w))


@pytest.mark.parametrize("mode", ["carry", "dirty", "full"])
@pytest.mark.parametrize("case", ["d1", "d10", "wide", "hot"])
def test_same_as_keys_in_memory(case, mode):
    """Against the speculative relax, or (degree above 128) the max tree,
    which one wavefront holds for more than 4096 magnets."""
    fam, side, d, phys = {"d1": ("square", 40, 1.0, {}), "d10": ("pinwheel", 48, 10.0, {}),
                          "wide": ("square", 47, 19.0, {}), "hot": ("kagome", 40, 3.0, {})}[case]
    H = W.rotating(20, 0.08, 20) if fam == "kagome" else W.linear_ramp(20, 0.25, -0.25, 33.0)
    w = W.family_instance(fam, 2 * side * side, d, 9, H, 0.05 if case == "hot" else 0.0, 9)
    other = dict(spec_min=1) if d <= 3.0 else dict(relax_waves=1)
    assert d <= 3.0 or w.n > 4096
    r = result(w, field_mode=mode)
    assert r["flips"] > 0
    assert_same(r, result(w, tuning=other, field_mode=mode))


# no disorder: whole sublattices tie at every flip; exponents outside the
# approximation's range; keys past its range; no hard-axis term; h_k tiny
@pytest.mark.parametrize("case", ["ties", "exponents", "strong", "parallel", "tiny"])
def test_key_ranges(case):
    H = W.linear_ramp(8, 0.3, -0.3, 33.0)
    w = W.family_instance("square", 2 * 20 * 21, 1.0, 3, H)
    if case == "ties":
        w.hk = np.full(w.n, 0.2)
    elif case == "exponents":
        w = dataclasses.replace(w, beta=0.3, gamma=9.5)
    elif case == "strong":
        w.H = w.H * 400.0
    elif case == "parallel":
        w = dataclasses.replace(w, **asi.PARALLEL_CRITERION)
    else:
        w = dataclasses.replace(w, hk=w.hk * 1e-30, H=w.H * 1e-30, alpha=w.alpha * 1e-30)
    r = result(w)
    assert r["flips"] > 0
    assert_same(r, result(w, tuning=dict(spec_min=1)))
    if case != "ties":  # the oracle's sums round differently: equal keys there are not equal here
        assert_oracle(w, r)


def test_fields_after_a_run_and_the_flip_limit():
    w = W.family_instance("pinwheel", 2 * 20 * 21, 3.0, 4, W.linear_ramp(10, 0.1, -0.1, 30.0))
    sim = asi.Sim.from_workload(w, field_mode="full")
    sim.run()
    s, hp, hq, t = sim.state()
    o = N.Oracle.from_workload(w)
    o.set_spins(s)
    ep, eq, scale = o.fields(w.H[t], t)
    assert np.all(np.abs(hp - ep) <= 1e-12 * scale) and np.all(np.abs(hq - eq) <= 1e-12 * scale)
    sim.close()
    sim = asi.Sim.from_workload(w, max_flips_per_step=5)
    with pytest.raises(asi.AsiError) as e:
        sim.run()
    assert e.value.status == asi.ASI_ELOOP
    sim.close()


def test_batch_of_both_groups():
    """Instances on both sides of the size limit in one batch, each mode."""
    ws = [line(n, seed=n % 7, steps=6) for n in (50, LDS_MAX_N + 5, 5000, LDS_MAX_N)]
    plain = [result(w) for w in ws]
    for mode in ("lockstep", "graph", "fused"):
        sims = [asi.Sim.from_workload(w) for w in ws]
        flips = asi.batch_run(sims, mode)
        for s, f, p in zip(sims, flips, plain):
            assert f == p["flips"] and s.flip_log()["hash"] == p["hash"]
            assert np.array_equal(s.state()[0], p["s"])
            s.close()
