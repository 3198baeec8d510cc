"""Deposits across the seam of a periodic axis whose last particle tile is cut short (n not a multiple of the
tile): a field task reads and clears the current wherever the windows of an active tile reach it, also
from the other side of the seam.  All other tiles are empty, so that nothing else has the current read."""
import copy

import numpy as np
import pytest

from paper_2501_07465_amd import workloads as W

pytestmark = pytest.mark.gpu

ME, QE = 9.1093837015e-31, 1.602176634e-19

CASES = [("disk2d", [67, 72, 1], [8, 8, 1], 0), ("disk2d", [72, 67, 1], [8, 8, 1], 1),
         ("disk2d", [250, 40, 1], [8, 16, 1], 0), ("disk2d", [40, 1001, 1], [16, 16, 1], 1),
         ("sphere3d", [67, 16, 16], [8, 4, 4], 0), ("sphere3d", [16, 67, 16], [4, 8, 4], 1),
         ("sphere3d", [16, 16, 35], [4, 4, 8], 2), ("sphere3d", [40, 16, 131], [4, 4, 8], 2)]


@pytest.mark.parametrize("sign", [-1, 1])
@pytest.mark.parametrize("name,n,tile,axis", CASES)
def test_deposits_across_the_seam_of_a_cut_tile(oracle, name, n, tile, axis, sign):
    """Electrons leave the first tile downwards (0.9 cells in a sort period) or the cut last tile upwards (up
    to 4 cells, within the tile's nominal window), against the oracle before and after the next sort."""
    from paper_2501_07465_amd import pic
    print(f"case {name} n {n} tile {tile} axis {axis} sign {sign}", flush=True)
    w = W.small(name)
    d = w["dims"]
    w["n"], w["tile"], w["periodic"], w["source"] = list(n), list(tile), [True] * 3, {"kind": "none"}
    w["species"] = [dict(w["species"][0], kind="free", q=-QE, m=ME, region={"kind": "all"}, reflect=False)]
    w["ion"], w["sort_every"] = "local", 20
    rng = np.random.default_rng(5)
    k = 60
    x, v = np.zeros((k, 3)), np.zeros((k, 3))
    for a in range(d):
        x[:, a] = rng.uniform(2.0, 5.0, k)
    step = (0.045 if sign < 0 else 0.19) * rng.uniform(0.6, 1.0, k)
    x[:, axis] = rng.uniform(0.01, 0.6, k) if sign < 0 else n[axis] - rng.uniform(0.01, 0.6, k)
    v[:, axis] = sign * step * w["dx"][axis] / w["dt"]
    x *= np.array(w["dx"])
    ref = oracle.Sim(w)
    ref.add_species(w["species"][0], 1e-3, x, v, np.zeros((k, 3)))
    ref.set_ion_background(False)
    sim = pic.Simulation(copy.deepcopy(w), precision="fp64", states=ref.state(), fields=ref.fields(), graphs=False)
    for steps in (15, 20):
        sim.step(steps)
        ref.step(steps)
        assert sim.overflow() == 0
        for g, r in zip(sim.fields(), ref.fields()):
            scale = np.abs(r).max()
            err = np.abs(g - r).max() / scale
            print(f"  step {sim.steps_done}: scale {scale:.2e}, off by {err:.2e}", flush=True)
            assert scale > 0 and err <= 1e-11
