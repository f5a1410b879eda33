"""Which relax runs, and how it is launched."""
import dataclasses
from time import perf_counter

import numpy as np
import pytest

from paper_2002_11401_amd import asi
from test_relax_lds import LDS_MAX_N, assert_same, line, result

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
