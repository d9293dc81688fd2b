"""The 2D sweeps on both sides of the line between several lanes per particle and
one, and past the 262,144 particles that one-lane blocks run at once, against
the oracle in every precision, with and without Verlet lists; and a batch of
jobs on both sides against each job alone, bit for bit.

Bars: interaction counts equal.  FP64: a and a^p, sums of at most a few hundred
terms that cancel, to 1e-12 of their value or of 1e-3 of the largest, positions
to 1e-12; the FP32 modes hold positions to 1e-5."""
import numpy as np
import pytest

import oracle
from paper_2003_01061_amd import binding
from paper_2003_01061_amd import workload as wk

pytestmark = pytest.mark.gpu

LINE = 175_000
_cache = {}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(gpu):
    return gpu


def _reference(n):
    if n not in _cache:
        wl = wk.scaled_hole_2d(n, seed=95, res=256)
        ref = oracle.RefJob(wl, openmp=True)
        ref.step(1)
        first = (ref.counters()["interactions_last"], ref.field(oracle.F_AP), ref.field(oracle.F_A))
        ref.step(2)
        _cache[n] = wl, first, ref.state()[0]
    return _cache[n]


@pytest.mark.parametrize("precision", [binding.SPH_FP64, binding.SPH_FP32_MIXED, binding.SPH_FP32_COMPENSATED])
@pytest.mark.parametrize("skin", [0.0, 0.5])
@pytest.mark.parametrize("n", [LINE - 1, LINE, LINE + 1, 262_147])
def test_both_sides_of_the_line_follow_the_oracle(n, skin, precision):
    wl, (pairs, ap, a), x = _reference(n)
    gpu = binding.SphMesh(wl, precision=precision, debug_fields=1, verlet_skin=skin)
    gpu.step(1)
    assert gpu.counters()["interactions_last"] == pairs
    if precision == binding.SPH_FP64:
        for g, r in ((gpu.field(binding.FIELD_AP), ap), (gpu.field(binding.FIELD_A), a)):
            assert np.all(np.abs(g - r) <= 1e-12 * np.maximum(np.abs(r), 1e-3 * np.abs(r).max()))
    gpu.step(2)
    assert np.abs(gpu.positions() - x).max() <= (1e-12 if precision == binding.SPH_FP64 else 1e-5)


@pytest.mark.parametrize("precision", [binding.SPH_FP64, binding.SPH_FP32_MIXED])
def test_jobs_of_both_sides_share_a_batch(precision):
    wls = [wk.scaled_hole_2d(n, seed=n, res=256) for n in (2003, LINE, LINE - 1, 67, LINE + 60_001)]
    specs = [binding.JobSpec(w) for w in wls]
    b = binding.SphBatch(2, precision, max_particles=sum(s.n for s in specs),
                         max_cells=sum(s.cells() for s in specs), max_jobs=len(specs))
    ids = [b.add(s) for s in specs]
    b.step(6)
    for w, j in zip(wls, ids):
        g = binding.SphMesh(w, precision=precision, use_graph=1)
        g.step(6)
        assert np.array_equal(g.positions(), b.positions(j)) and g.counters() == b.counters(j), w.n
