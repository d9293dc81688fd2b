"""Results come back where the system pins no host memory: a child process whose
hipHostMalloc (a stand-in loaded ahead of the library) always refuses reads the
same positions, features, velocities, error state, counters and flags."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2003_01061_amd import binding
from paper_2003_01061_amd import workload as wk

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STAND_IN = """#include <stddef.h>
int calls;
int hipHostMalloc(void **p, size_t n, unsigned flags) { ++calls; return 2; /* hipErrorOutOfMemory */ }
"""
CHILD = """
import ctypes, sys
stand_in = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import numpy as np
sys.path.insert(0, sys.argv[2] + "/tests")
import test_gpu_no_pinned as t
out = t.results(int(sys.argv[4]))
assert ctypes.c_int.in_dll(stand_in, "calls").value > 0, "the stand-in was not called"
np.savez(sys.argv[3], **out)
"""


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(gpu):
    return gpu


def results(dim):
    wl = wk.scaled_hole_2d(60_011, seed=81, res=128) if dim == 2 else wk.scaled_ball_3d(3001, seed=81, res=24)
    g = binding.SphMesh(wl)
    g.step(3)
    x, f = g.positions(with_feature=True)
    e, c = g.error(), g.counters()
    spec = binding.JobSpec(wl)
    b = binding.SphBatch(dim, binding.SPH_FP64, max_particles=spec.n, max_cells=spec.cells(), max_jobs=2)
    j = b.add(spec)
    b.step(3)
    live, conv, steps = b.status()
    so, si, _ = g.neighbors()
    return dict(x=x, f=f, v=g.velocities(), e=np.array([e["e_sys"], e["phase"], e["converged"], e["step"]]),
                c=np.array([c["steps"], c["escaped"], c["interactions"], c["interactions_last"]]),
                bx=b.positions(j), live=live, conv=conv, steps=steps, so=so, si=si)


@pytest.mark.parametrize("dim", [2, 3])
def test_results_come_back_without_pinned_memory(dim, tmp_path):
    src, so, out = tmp_path / "stand_in.c", tmp_path / "stand_in.so", tmp_path / "out.npz"
    src.write_text(STAND_IN)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    res = subprocess.run([sys.executable, "-c", CHILD, str(so), ROOT, str(out), str(dim)], capture_output=True,
                         text=True, timeout=100)
    assert res.returncode == 0, res.stderr[-2000:]
    want, got = results(dim), np.load(out)
    assert set(got.files) == set(want)
    for k, v in want.items():
        assert np.array_equal(got[k], v), k
