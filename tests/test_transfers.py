"""Results on their way to the caller through pinned buffers: sizes at which a
transfer is cut into pieces, single outputs, several threads at a time."""
import ctypes as C
import threading

import numpy as np
import pytest

from oracle import native as N
from paper_2002_11401_amd import asi
from paper_2002_11401_amd import workloads as W

pytestmark = pytest.mark.gpu
PIECE = 1 << 20  # bytes


def line(n):
    xy, theta = W.ising(n, 1)
    H = W.linear_ramp(3, 0.3, -0.3, 20.0)
    return W.Workload("line", xy, theta, W.polarised_spins(theta, H[0]),
                      W.disorder_hk(n, 0.2, 0.05, n), H, alpha=0.01, neighbor_distance=1.0,
                      b=1.0, c=1.0, beta=3.0, gamma=3.0)


def only(sim, par):
    out = np.full(sim.n, np.nan)
    p = out.ctypes.data_as(C.POINTER(C.c_double))
    lib = asi.library()
    none = C.POINTER(C.c_double)()
    assert lib.asi_get_state(sim.handle, None, p if par else none, none if par else p, None) == 0
    return out


# a component is 8 bytes a magnet, the field 16: one piece, just below and at
# two, three with a remainder, the most pieces and more bytes than those
@pytest.mark.parametrize("n", [1, 7, PIECE // 8 - 1, PIECE // 8, 3 * PIECE // 16 + 5, PIECE, PIECE + 333])
def test_state_and_logs(n):
    w = line(n)
    sim = asi.Sim.from_workload(w, field_mode="full", flip_log_capacity=n)
    flips = sim.run()
    s, hp, hq, t = sim.state()
    assert np.array_equal(only(sim, True), hp) and np.array_equal(only(sim, False), hq)
    o = N.Oracle.from_workload(w)
    o.set_spins(s)
    ep, eq, scale = o.fields(w.H[t], t)
    assert np.all(np.abs(hp - ep) <= 1e-12 * scale) and np.all(np.abs(hq - eq) <= 1e-12 * scale)
    log = sim.flip_log()
    flipped = np.bincount(log["idx"], minlength=n)
    assert len(log["idx"]) == flips > 0 and np.array_equal(flipped % 2 == 1, s != w.spin0)
    first = np.full(n, np.iinfo(np.int64).max)
    np.minimum.at(first, log["idx"], np.arange(flips))
    order = sim.switching_order()
    assert np.array_equal(order[flipped > 0], first[flipped > 0])
    spins = np.where(np.arange(n) % 3 == 0, -1, 1).astype(np.int8)
    sim.set_state(spins, -1)
    assert np.array_equal(sim.state()[0], spins)
    bad = spins.copy()
    bad[-1] = 0
    with pytest.raises(asi.AsiError) as e:
        sim.set_state(bad, -1)
    assert e.value.status == asi.ASI_EINVAL and np.array_equal(sim.state()[0], spins)
    sim.close()


def test_threads():
    """Handles of several threads read at the same time, some closed meanwhile."""
    want, got, bad = {}, {}, []
    sizes = (300, 70001, 140003, 200000)
    for n in sizes:
        sim = asi.Sim.from_workload(line(n))
        sim.run()
        want[n] = sim.state()
        sim.close()

    def work(n):
        try:
            for _ in range(3):
                sim = asi.Sim.from_workload(line(n))
                sim.run()
                for _ in range(4):
                    got[n] = sim.state()
                    assert all(np.array_equal(a, b) for a, b in zip(got[n], want[n]))
                sim.close()
        except BaseException as e:  # reported by the test's own thread
            bad.append((n, repr(e)))

    ts = [threading.Thread(target=work, args=(n,)) for n in sizes]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad and set(got) == set(sizes)
