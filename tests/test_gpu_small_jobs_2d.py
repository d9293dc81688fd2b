"""2D batches whose small jobs together fill the chip take one lane per particle
that adds as four do: every job gets the bits it gets alone, where four lanes
share a particle; with lists past the entries kept in LDS and past a block, with
curved boundaries, and as jobs leave and the batch falls below the line again.
And jobs of both sizes, in any order, in one batch."""
import numpy as np
import pytest

from paper_2003_01061_amd import binding
from paper_2003_01061_amd import workload as wk

pytestmark = pytest.mark.gpu

LINE = 175_000
PRECISIONS = [binding.SPH_FP64, binding.SPH_FP32_MIXED, binding.SPH_FP32_COMPENSATED]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(gpu):
    return gpu


def _run(wls, precision, cap=0, tile=0, removed=()):
    specs = [binding.JobSpec(w) for w in wls]
    b = binding.SphBatch(2, precision, max_particles=sum(s.n for s in specs),
                         max_cells=sum(s.cells() for s in specs), max_jobs=len(specs), max_neighbors=cap,
                         scan_tile=tile)
    ids = [b.add(s) for s in specs]
    alone = [binding.SphMesh(w, precision=precision, use_graph=1, max_neighbors=cap) for w in wls]
    gone = set()
    for leave in [()] + [(k,) for k in removed]:
        for k in leave:
            b.remove(ids[k])
            gone.add(k)
        b.step(6)
        for k, (w, j, g) in enumerate(zip(wls, ids, alone)):
            if k in gone:
                continue
            g.step(6)
            assert np.array_equal(g.positions(), b.positions(j)), (w.name, w.n, leave)
            assert g.counters() == b.counters(j), (w.name, w.n)


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("tile", [2, 4, 8])
def test_small_jobs_that_fill_the_chip(precision, tile):
    wls = [wk.scaled_hole_2d(n, seed=n, res=256) for n in (LINE - 1, 20_011, 67, 5003)]
    wls += [wk.zalesak_disc(n_total=2400), wk.level_peanut(n_total=1500, res=128), wk.square_lattice(n_side=32, seed=5)]
    assert sum(w.n for w in wls) >= LINE
    _run(wls, precision, tile=tile, removed=(1, 0))    # below the line without the largest


@pytest.mark.parametrize("precision", PRECISIONS)
def test_long_lists(precision):
    wls = [wk.scaled_hole_2d(n, seed=n, res=256, kernel_support=r, boundary_scale=2.0)
           for n, r in ((90_001, 5.0), (87_003, 3.0), (2003, 6.0))]
    _run(wls, precision, cap=256)


@pytest.mark.parametrize("precision", PRECISIONS)
def test_large_and_small_jobs_in_any_order(precision):
    sizes = (3001, LINE, 100_003, 2003, LINE + 5, 90_001, 300)
    wls = [wk.scaled_hole_2d(n, seed=n, res=256) for n in sizes]
    _run(wls, precision, removed=(2, 4))
