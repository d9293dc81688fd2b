"""Neighbour lists of particles that the caller has put far off the box along the
first axis, past 2^31 cells too: pairs there are on the lists of the cell scan
with several lanes per particle, bit-exact against the oracle's brute force."""
import numpy as np
import pytest

import oracle
from paper_2003_01061_amd import binding
from paper_2003_01061_amd import workload as wk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(gpu):
    return gpu


@pytest.mark.parametrize("far", [3.0, 1e6, 1e9, -1e9, 1e12, -1e12])
@pytest.mark.parametrize("dim", [2, 3])
def test_pairs_far_off_the_box_stay_on_the_lists(dim, far):
    wl = wk.square_lattice(n_side=24, seed=3) if dim == 2 else wk.scaled_ball_3d(5003, seed=3, res=24)
    if dim == 3:   # one h, as on the square
        wl.sizing = dict(kind=wk.H_CONST, h0=0.05, grad=0.0, dcap=np.inf, point=[0.0, 0.0, 0.0])
    rng = np.random.default_rng(5)
    vol = np.nonzero(wl.feature == 0)[0]
    moved = rng.choice(vol, 40, replace=False)
    x = wl.xyz.copy()
    x[moved, 0] += far
    # pairs of them closer than h
    x[moved[20:]] = x[moved[:20]]
    x[moved[20:], 1] += 0.4 * wl.sizing["h0"]
    ref = oracle.RefJob(wl, xyz=x)
    gpu = binding.SphMesh(wl)
    gpu.set_state(x, np.zeros_like(x))
    so, si, sr = gpu.neighbors()
    every = np.arange(wl.n)
    ro, ri, rr, _, _, _ = ref.sample(every, cap_per=400)
    assert np.all(np.diff(ro)[moved] >= 1)
    assert np.array_equal(so, ro) and np.array_equal(si, ri) and np.array_equal(sr, rr)
    # a step's lists, counted, with and without Verlet lists
    for skin in (0.0, 0.3):
        job = binding.SphMesh(wl, verlet_skin=skin)
        job.set_state(x, np.zeros_like(x))
        job.step(1)
        assert job.counters()["interactions_last"] == len(ri), skin
