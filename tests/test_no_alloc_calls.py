"""asi_switching_rho_noalloc makes none of HIP's allocating and freeing calls,
counted by a library that stands between libasi.so and the HIP runtime."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

COUNTER = """
#include <stddef.h>
void* real[4];
long calls[4];
int hipMalloc(void** p, size_t n) { ++calls[0]; return ((int (*)(void**, size_t))real[0])(p, n); }
int hipFree(void* p) { ++calls[1]; return ((int (*)(void*))real[1])(p); }
int hipHostMalloc(void** p, size_t n, unsigned f) {
  ++calls[2];
  return ((int (*)(void**, size_t, unsigned))real[2])(p, n, f);
}
int hipHostFree(void* p) { ++calls[3]; return ((int (*)(void*))real[3])(p); }
"""

CHILD = """
import ctypes as C, sys
import torch
torch.zeros(1, device="cuda")
counter = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
hip = C.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))
real, calls = (C.c_void_p * 4).in_dll(counter, "real"), (C.c_long * 4).in_dll(counter, "calls")
for k, name in enumerate(("hipMalloc", "hipFree", "hipHostMalloc", "hipHostFree")):
    real[k] = C.cast(getattr(hip, name), C.c_void_p).value
from paper_2002_11401_amd import asi
sys.path.insert(0, "tests")
from test_relax_lds import line
# 70,000 magnets: the buffers that creation leaves behind, if any, are larger
# than the few bytes read here
a, b = (asi.Sim.from_workload(line(70000, seed=s), device="hip") for s in (1, 2))
before = list(calls)
asi.switching_rho_noalloc(a, b)
assert list(calls) == before, (before, list(calls))
a.run()
b.run()
before = list(calls)
assert before[0] > 0  # the counter is in the way
rho = asi.switching_rho_noalloc(a, b)
assert list(calls) == before, (before, list(calls))
assert asi.switching_rho(a, b) == rho and list(calls) != before
print("counted", before, list(calls))
"""


def test_no_allocating_call(tmp_path):
    src, lib = tmp_path / "counter.c", tmp_path / "libcounter.so"
    src.write_text(COUNTER)
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-O1", str(src), "-o", str(lib)])
    r = subprocess.run([sys.executable, "-u", "-c", CHILD, str(lib)], cwd=ROOT, capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0 and "counted" in r.stdout, r.stdout + r.stderr
