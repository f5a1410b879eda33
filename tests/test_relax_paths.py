"""Which relax runs and how it is launched; and every path, whole and paused
within steps, against one that shares none of its code: the max tree, which is
on its own where one wavefront holds too few magnets' keys in LDS (more than
3,840) or the exponents lie outside the codes' range, and the oracle."""
import dataclasses
from time import perf_counter

import numpy as np
import pytest

from paper_2002_11401_amd import asi
from paper_2002_11401_amd import workloads as W
from test_relax_lds import LDS_MAX_N, assert_oracle, assert_same, line, result

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["lockstep", "graph", "fused"])
def test_batch_of_both_kinds_costs_no_more_than_its_parts(mode):
    """Steps without flips, launches and waits alone: instances with keys in
    LDS and others in one batch, against the two batches one after the other."""
    H = np.zeros((300, 2))
    ws = [line(LDS_MAX_N + 900)] + [line(500, seed=k) for k in range(8)]
    for w in ws:
        w.H = H
    sims = [asi.Sim.from_workload(w) for w in ws]

    def best(part):
        times = []
        for _ in range(5):
            for s in part:
                s.set_state(np.ones(s.n, np.int8), -1)
            t0 = perf_counter()
            asi.batch_run(part, mode)
            times.append(perf_counter() - t0)
        return min(times)

    both, parts = best(sims), best(sims[:1]) + best(sims[1:])
    for s in sims:
        s.close()
    assert both <= parts, (both, parts)


@pytest.mark.parametrize("n,never", [(4096, True), (4097, False)])
def test_threshold_in_force(n, never):
    """The handle reports the threshold that its steps are held to, and takes
    every value literally, the usual default of 32 as well."""
    w = dataclasses.replace(line(n), neighbor_distance=10.0)
    sim = asi.Sim.from_workload(w)
    t = sim.tuning()
    assert t["spec_min"] == (2**63 - 1 if never else 32)
    sim.set_tuning(t["relax_waves"], t["l1_shift"], 32)
    assert sim.tuning()["spec_min"] == 32
    sim.close()
    assert_same(result(w), result(w, tuning=dict(spec_min=32)))


def test_shapes_are_not_carried_over_to_another_path(tmp_path, monkeypatch):
    """10,000 and 16,000 magnets are of one size class, but 4 wavefronts hold
    only the former's keys in LDS; the file keeps an entry for each."""
    monkeypatch.setenv("ASI_TUNE_CACHE", str(tmp_path / "shapes.txt"))
    sims = [asi.Sim.from_workload(dataclasses.replace(line(n, steps=4), neighbor_distance=70.0))
            for n in (10000, 16000, 15000)]
    first, other, same = [s.tune(sample_steps=2) for s in sims]
    assert first["trials"] > 0 and other["trials"] > 0
    assert same["trials"] == 0 and same["relax_waves"] == first["relax_waves"]
    words = (tmp_path / "shapes.txt").read_text().split()
    assert len(words) == 16 and words[0] != words[8] and words[1:4] == words[9:12]
    for s in sims:
        s.close()


TREE = dict(relax_waves=1)
NO_CODES = dict(beta=0.3, gamma=9.5)  # exponents outside the range of the codes


@pytest.mark.parametrize("mode", ["carry", "dirty", "full"])
@pytest.mark.parametrize("case", ["d1", "d1 ties", "d3", "d3 ties", "hot", "wide ties"])
def test_same_as_the_tree(case, mode):
    """The default, batches whenever they can start, and one flip at a time
    with keys in LDS alone."""
    fam, n, d = {"d1": ("square", 4400, 1.0), "d3": ("square", 4400, 3.0), "hot": ("kagome", 4400, 3.0),
                 "wide": ("pinwheel", 4400, 8.0)}[case.split()[0]]
    H = W.rotating(16, 0.08, 16) if fam == "kagome" else W.linear_ramp(16, 0.25, -0.25, 33.0)
    w = W.family_instance(fam, n, d, 9, H, 0.05 if case == "hot" else 0.0, 9)
    assert 3840 < w.n <= LDS_MAX_N
    if "ties" in case:
        w.hk = np.full(w.n, 0.2 if fam == "square" else 0.17)
    tree = result(w, tuning=TREE, field_mode=mode)
    assert tree["flips"] > 1000
    for tuning in (None, dict(spec_min=1), dict(spec_min=2**62)):
        assert_same(result(w, tuning=tuning, field_mode=mode), tree)


# flat root (up to 32,768 magnets) and two levels, 16 wavefronts and one, rows of
# one slot a thread and of several
@pytest.mark.parametrize("n,distance", [(4500, 70.0), (32768, 70.0), (32769, 70.0), (2600, 530.0), (4500, 10.0)])
def test_tree_against_the_oracle(n, distance):
    w = dataclasses.replace(line(n, steps=8), neighbor_distance=distance, **NO_CODES)
    never = dict(spec_min=2**62)
    r = result(w, tuning=never)
    assert_oracle(w, r)
    assert_same(r, result(w, tuning=dict(TREE, **never)))


def paused(ws, budget_ms=0.3):
    """The jobs served in bursts far shorter than a step, against plain runs."""
    plain = [result(w) for w in ws]
    srv = asi.Server(hbm_budget_bytes=8 << 30, max_slots=len(ws))
    ids = [srv.submit(w) for w in ws]
    for _ in range(20000):
        if not srv.step(budget_ms=budget_ms):
            break
    for i, p in zip(ids, plain):
        res = srv.take(i)
        assert (res["flips"], res["hash"]) == (p["flips"], p["hash"])
        assert np.array_equal(res["spins"], p["s"])
    pauses = srv.stats()["pauses"]
    srv.close()
    return pauses


def path(name, seed=1):
    """A few steps, most of the flips in one of them."""
    n, distance, kw = {"lds": (20000, 70.0, {}), "lds4": (4000, 70.0, {}), "many lds": (30000, 10.0, {}),
                       "tree": (12000, 70.0, NO_CODES), "window": (LDS_MAX_N + 77, 2.0, {}),
                       "many": (LDS_MAX_N + 77, 10.0, {})}[name.replace(" ties", "")]
    w = dataclasses.replace(line(n, seed=seed, steps=4), neighbor_distance=distance, **kw)
    w.H[:] = np.linspace(0.05, -0.3, 4)[:, None] * w.H[0] / np.abs(w.H[0]).max()
    if "ties" in name:
        w.hk = np.full(n, 0.2)
    return w


@pytest.mark.parametrize("name", ["lds", "lds ties", "lds4", "lds4 ties", "many lds", "many lds ties", "tree",
                                  "tree ties", "window", "window ties", "many", "many ties"])
def test_paused_within_steps(name):
    w = path(name)
    flips = result(w)
    assert np.bincount(flips["step"]).max() > 2000
    assert paused([w]) > 3


def test_paused_on_every_path_at_once():
    assert paused([path(p, seed=k) for k, p in enumerate(("lds", "tree", "window", "many", "many lds", "lds4"))]) > 20


@pytest.mark.parametrize("mode", ["lockstep", "graph", "fused"])
def test_batch_on_every_path(mode):
    """In the launch that holds every path, the max tree with rows of more
    slots than threads too; and a batch of the tree's instances and the
    window's alone."""
    wide = dataclasses.replace(line(2600, steps=4), neighbor_distance=530.0, **NO_CODES)
    ws = [path("lds"), path("tree"), wide, path("window"), path("many"), path("many lds"), path("lds4 ties")]
    for part in (ws, ws[1:4]):
        sims = [asi.Sim.from_workload(w) for w in part]
        flips = asi.batch_run(sims, mode)
        for w, s, f in zip(part, sims, flips):
            plain, (spins, hp, hq, _) = result(w), s.state()
            assert f == plain["flips"] > 0 and s.flip_log()["hash"] == plain["hash"]
            for a, b in ((spins, plain["s"]), (hp, plain["hp"]), (hq, plain["hq"])):
                assert np.array_equal(a, b)
            s.close()
