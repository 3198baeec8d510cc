"""Work units whose size the library chooses (unit = 0): the unit lists of one round and of many rounds,
with fewer and with more active tiles than the device holds blocks, give the run that units of a stated
size give.  The current's sums do not depend on how a tile's particles are split but for the rounding of
the sums within a group of lanes, so the FP64 runs agree to the 1e-12 that the form is held to."""
import copy

import numpy as np
import pytest

from paper_2501_07465_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(w, block, unit, steps):
    from paper_2501_07465_amd import pic
    sim = pic.Simulation(copy.deepcopy(w), precision="fp64", block=block, unit=unit, series_cap=steps + 8)
    sim.step(steps)
    out = {"fields": np.stack(sim.fields()), "series": sim.current_series()}
    for s in sim.species:
        out[f"x{s}"], out[f"v{s}"], _ = sim.particles(s)
    out["overflow"] = sim.overflow()
    return out


@pytest.mark.parametrize("label,n,tile,block", [
    ("one round of tiles", [72, 68, 1], [16, 8, 1], 256),        # units below a tile's particles
    ("many rounds, few active", [1000, 72, 1], [2, 2, 1], 256),  # 18000 tiles
    ("more tiles than blocks", [72, 68, 1], [2, 2, 1], 512),     # about 350 active, 256 blocks of 512
])
def test_chosen_units_match_stated_units(label, n, tile, block):
    print(f"case {label}: n {n} tile {tile} block {block}", flush=True)
    w = W.small("disk2d")
    w["n"], w["tile"] = n, tile
    w["species"][0]["ppc"] = w["species"][1]["ppc"] = 40
    ref = _run(w, block, 64, 40)
    got = _run(w, block, 0, 40)
    assert got["overflow"] == 0
    for k in ref:
        if k == "overflow":
            continue
        scale = np.abs(ref[k]).max()
        err = np.abs(got[k] - ref[k]).max() / scale
        print(f"  {k}: {err:.2e}", flush=True)
        assert err <= 1e-12, k


@pytest.mark.parametrize("members,unit", [(9, 64), (5, 0), (3, 512)])
def test_runs_of_units_in_a_batch_match_runs_alone(members, unit):
    """A batch's blocks take runs of units (9 members in units of 64: several units a run, runs that end
    inside a tile and cross from member to member) from ranges equal in work (members of very different
    size): every member is bit for bit the run of its own."""
    from paper_2501_07465_amd import pic
    steps = 40
    ws = []
    for i in range(members):
        w = W.small("disk2d")
        w["n"], w["tile"] = [136, 72, 1], [32, 16, 1]
        w["species"][0]["ppc"] = w["species"][1]["ppc"] = (4, 30, 90)[i % 3]
        w["seed"] = 100 + i
        ws.append(w)

    def export(sim):
        out = list(sim.fields())
        for s in sim.species:
            out += list(sim.particles(s))
        return out + [sim.current_series()]

    kw = dict(precision="fp32", block=256, unit=unit, series_cap=steps + 8)
    alone = []
    for w in ws:
        sim = pic.Simulation(copy.deepcopy(w), **kw)
        sim.step(steps)
        alone.append(export(sim))
    batch = pic.Batch(members, 2, "fp32")
    sims = [pic.Simulation(copy.deepcopy(w), stream=batch.stream, **kw) for w in ws]
    for sim in sims:
        batch.add(sim)
    batch.step(steps)
    batch.stream.synchronize()
    for i, sim in enumerate(sims):
        print(f"member {i}", flush=True)
        for a, b in zip(alone[i], export(sim)):
            assert np.array_equal(a, b)
