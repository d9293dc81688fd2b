"""The scan tile where kernels read it: 2D jobs from 175,000 particles on without
Verlet lists, and their list builds from 200,000 on.  Every tile gives the same
bits in every precision, and the lists' pair count is the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2003_01061_amd import binding
from paper_2003_01061_amd import workload as wk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(gpu):
    return gpu


@pytest.fixture(scope="module")
def job():
    cache = {}

    def get(n):
        if n not in cache:
            wl = wk.scaled_hole_2d(n, seed=64, res=256)
            ref = oracle.RefJob(wl, openmp=True)
            ref.step(1)
            cache[n] = wl, ref.counters()["interactions_last"]
        return cache[n]
    return get


@pytest.mark.parametrize("precision", [binding.SPH_FP64, binding.SPH_FP32_MIXED, binding.SPH_FP32_COMPENSATED])
@pytest.mark.parametrize("n,skin", [(175_000, 0.0), (200_003, 0.0), (200_000, 0.5), (250_001, 0.8)])
def test_tiles_give_the_same_bits(job, n, skin, precision):
    wl, pairs = job(n)
    runs = []
    for tile in (2, 4, 8):
        g = binding.SphMesh(wl, precision=precision, use_graph=1, scan_tile=tile, verlet_skin=skin)
        g.step(1)
        assert g.counters()["interactions_last"] == pairs, tile
        g.step(12)
        runs.append((g.positions(), g.velocities(), g.counters()))
    for x, v, c in runs[1:]:
        assert np.array_equal(x, runs[0][0]) and np.array_equal(v, runs[0][1]) and c == runs[0][2]
