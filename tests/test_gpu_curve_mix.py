"""A 3D job with imported curves, whose patches take the pair-normal pass, shares
a batch with plain 3D jobs on both sides of the neighbour kernel's size line:
every job runs the kernels it runs alone and gets the same bits, with the curve
job resident and after it has left."""
import numpy as np
import pytest

from paper_2003_01061_amd import binding
from paper_2003_01061_amd import workload as wk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(gpu):
    return gpu


@pytest.mark.parametrize("precision", [binding.SPH_FP64, binding.SPH_FP32_MIXED, binding.SPH_FP32_COMPENSATED])
def test_jobs_beside_a_job_with_curves_keep_their_bits(precision):
    wls = [wk.level_cube_sharp(), wk.scaled_ball_3d(9001, seed=71, res=48),
           wk.scaled_ball_3d(200_009, seed=72, res=48), wk.level_torus(n_total=5000, res=48),
           wk.paper_sphere01(n_total=3000, res=32)]
    specs = [binding.JobSpec(w) for w in wls]
    b = binding.SphBatch(3, precision, max_particles=sum(s.n for s in specs),
                         max_cells=sum(s.cells() for s in specs), max_jobs=len(specs), max_neighbors=512)
    ids = [b.add(s) for s in specs]
    alone = [binding.SphMesh(w, precision=precision, use_graph=1, max_neighbors=512) for w in wls]
    b.step(6)
    for w, j, g in zip(wls, ids, alone):
        g.step(6)
        assert np.array_equal(b.positions(j), g.positions()), w.name
        assert b.counters(j) == g.counters(), w.name
    b.remove(ids[0])
    b.step(5)
    for w, j, g in list(zip(wls, ids, alone))[1:]:
        g.step(5)
        assert np.array_equal(b.positions(j), g.positions()), w.name
