"""The tuner and the scan tile (no GPU): the lines from which a kernel reads the
tile are the library's, and where none does its values are timed once, so that
noise between equal configurations decides nothing."""
import os
import re

import pytest

from paper_2003_01061_amd import autotune

HIP = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2003_01061_amd", "csrc",
                   "sph_mesh.hip")


class Spec:
    def __init__(self, n):
        self.n = n


def test_the_lines_are_the_librarys():
    src = open(HIP).read()
    assert int(re.search(r"constexpr int ONE_LANE = (\d+);", src).group(1)) == autotune.ONE_LANE
    assert int(re.search(r"constexpr int ONE_LANE_BUILD = (\d+);", src).group(1)) == autotune.ONE_LANE_BUILD


@pytest.mark.parametrize("dim,sizes,scan,lists", [
    (3, [2_000_000], False, False), (2, [174_999], False, False), (2, [175_000], True, False),
    (2, [100_000, 100_000], True, True), (2, [199_999], True, False), (2, [200_000], True, True),
    (2, [1000] * 8, False, False)])
def test_equal_configurations_are_timed_once(dim, sizes, scan, lists, monkeypatch):
    specs = [Spec(n) for n in sizes]
    assert autotune.tile_matters(specs, dim, 0.0) == scan
    assert autotune.tile_matters(specs, dim, 0.3) == lists
    calls = []

    def noisy(sp, d, precision, cf, tile, steps, warmup, max_neighbors, skin=0.0):
        calls.append((cf, tile, skin))
        return 1.0 + 0.2 * (len(calls) % 3)      # 20% "noise"
    monkeypatch.setattr(autotune, "_time_config", noisy)
    r = autotune.tune(specs, dim, 1)
    cfs, tiles, skins = autotune.CELL_FACTORS, autotune.SCAN_TILES, autotune.SKINS
    assert len(r.table) == (len(cfs) + len(skins)) * len(tiles)
    assert len(calls) == len(cfs) * (len(tiles) if scan else 1) + len(skins) * (len(tiles) if lists else 1)
    if not scan:
        for cf in cfs:
            assert len({t["ms_per_step"] for t in r.table if t["cell_factor"] == cf and t["verlet_skin"] == 0.0}) == 1
    if not scan and not lists:
        assert r.best["scan_tile"] == autotune.DEFAULT["scan_tile"]
