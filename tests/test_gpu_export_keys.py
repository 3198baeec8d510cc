"""Exported sort keys, below and above the size that goes through the pinned ring and over several of its chunks:
the tile-major index of each particle's cell, formed from the positions that were loaded."""
import numpy as np
import pytest

from paper_2501_07465_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,n,tile,count", [
    ("disk2d", [130, 71, 1], [16, 8, 1], 1), ("disk2d", [130, 71, 1], [16, 8, 1], 393_217),
    ("disk2d", [1000, 640, 1], [32, 16, 1], 2_200_003), ("sphere3d", [45, 50, 61], [4, 8, 4], 4_500_001)])
def test_keys_are_the_cells_in_tiles(name, n, tile, count):
    from paper_2501_07465_amd import pic
    print(f"case keys {name} n {n} tile {tile} count {count}", flush=True)
    w = W.small(name)
    d = w["dims"]
    w["n"], w["tile"], w["periodic"], w["source"], w["ion"] = n, tile, [True] * 3, {"kind": "none"}, "uniform"
    w["species"] = [W.free_electrons(1, 5.5, 300.0, reflect=False)]
    rng = np.random.default_rng(count)
    c = np.stack([rng.integers(0, n[a], count) if a < d else np.zeros(count, np.int64) for a in range(3)], axis=1)
    x = (c + np.where(np.arange(3) < d, rng.uniform(0.05, 0.95, (count, 3)), 0.0)) * np.array(w["dx"])
    zero = np.zeros((3, n[2], n[1], n[0]))
    sim = pic.Simulation(w, precision="fp32", states=[(x, np.zeros((count, 3)), None, 1e-3)], fields=(zero, zero), init_fields=False)
    nt = [-(-n[a] // tile[a]) for a in range(3)]
    t, r = c // tile, c % tile
    want = ((t[:, 2] * nt[1] + t[:, 1]) * nt[0] + t[:, 0]) * int(np.prod(tile)) + (r[:, 2] * tile[1] + r[:, 1]) * tile[0] + r[:, 0]
    assert np.array_equal(sim.keys(0), want)
