"""FP32 rounding that a run of many particles depends on: the gather holds the weighted sum of the field nodes to
the rounding of its own terms, and the current does not depend on how the library splits tiles into work
units.  (Where either changes at the rounding level, an electron at a reflecting surface may turn a step
earlier or later, and the runs part there by the kick of a whole step.)"""
import copy

import numpy as np
import pytest

from paper_2501_07465_amd import workloads as W

pytestmark = pytest.mark.gpu

ME, QE = 9.1093837015e-31, 1.602176634e-19


@pytest.mark.parametrize("name", ["slab1d", "disk2d", "sphere3d"])
def test_gather_beside_a_large_node(name):
    """E_y falls from about 2^30 to about 2^10 V/m within a cell, with an electron 2^-20 cells from the small end:
    the field there is the sum of two terms of about 2^10, each rounded once (the nodes' difference would be
    rounded to a multiple of 64).  Against FP64: the two products, their sum, the half kick's factor, its
    two uses and the two sums of the velocity are at most 8 roundings of 2^-24."""
    from paper_2501_07465_amd import pic
    w = W.small(name)
    d = w["dims"]
    print(f"case {name}", flush=True)
    sp = dict(w["species"][0], kind="free", q=-QE, m=ME, region={"kind": "all"}, reflect=False)
    w["species"], w["source"], w["periodic"] = [sp], {"kind": "none"}, [True, True, True]
    w["ion"] = "local"
    u = 1.0 - 2.0 ** -20
    i = 20
    dx = np.array(w["dx"])
    x = np.zeros((1, 3))
    for a, off in enumerate((i + u, 14.5, 18.0)[:d]):  # E_y: located at the nodes of x and z, half a cell up in y
        x[0, a] = off * dx[a]
    L = W.field_extent(w)
    e = np.zeros((3, L[2], L[1], L[0]))
    big, small = 2.0 ** 30 + 128.0, 1055.0  # FP32 numbers
    e[1, :, :, i], e[1, :, :, i + 1] = big, small
    sim = pic.Simulation(w, precision="fp32", states=[(x, np.zeros((1, 3)), np.zeros((1, 3)), 1e-6)],
                         fields=(e, np.zeros_like(e)), init_fields=False, graphs=False)
    xf = sim.particles(0)[0][0, 0] / dx[0] - i
    assert abs(xf - u) < 1e-12  # (the offset is an FP32 number)
    sim.step(1)
    v = sim.particles(0)[1][0, 1]
    want = -QE / ME * w["dt"] * (big * (1.0 - u) + small * u)
    print(f"  v {v:.9e} want {want:.9e} off by {abs(v / want - 1):.2e}", flush=True)
    assert abs(v / want - 1) <= 8 * 2.0 ** -24


@pytest.mark.parametrize("name,tile,ppc,block", [
    ("slab1d", None, 400, 256),
    ("disk2d", [16, 8, 1], 45, 256),
    ("disk2d", [32, 32, 1], 13, 512),
    ("sphere3d", [8, 8, 4], 21, 256),
    ("sphere3d", [4, 4, 4], 37, 128),
])
def test_chosen_units_give_the_bits_of_whole_tiles(name, tile, ppc, block):
    from paper_2501_07465_amd import pic
    w = W.small(name)
    w["tile"] = tile or w["tile"]
    for s in w["species"]:
        s["ppc"] = ppc
    print(f"case {name} tile {w['tile']} ppc {ppc}", flush=True)
    out = []
    for unit in (1 << 20, 0):
        sim = pic.Simulation(copy.deepcopy(w), precision="fp32", block=block, unit=unit, series_cap=64)
        sim.step(40)
        assert sim.overflow() == 0
        out.append([*sim.fields(), *(a for s in sim.species for a in sim.particles(s))])
    assert np.abs(out[0][0]).max() > 0
    for a, b in zip(*out):
        assert np.array_equal(a, b)
