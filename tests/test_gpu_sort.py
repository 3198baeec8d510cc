"""The cell sort at the edges of its launch rules: one to three passes of 6 to 10 bits, one block and many,
the histogram scanned by the scatter's blocks (up to 32 of them) or on its own, one and four keys a thread,
digit totals by atomics or by rows.  The particles leave in the order of a stable argsort of their cell
keys, bit for bit; velocities and fields are zero, so the step that follows the sort moves nothing."""
import numpy as np
import pytest

from paper_2501_07465_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,tile,count", [
    ([8, 8, 8], [4, 4, 4], 50_000),           # 9 bits: one pass
    ([16, 16, 16], [4, 4, 4], 1),             # 12 bits: two passes of 6
    ([16, 16, 16], [4, 4, 4], 1025),          # a second block of one key
    ([40, 36, 44], [8, 8, 4], 32 * 1024),     # 17 bits; 32 blocks
    ([40, 36, 44], [8, 8, 4], 32 * 1024 + 1),  # 33
    ([1000, 1000, 1], [16, 16, 1], 600_001),  # 20 bits: two passes of 10
    ([2048, 4096, 1], [32, 32, 1], 2_200_003),  # 23 bits: three passes of 8, four keys a thread
    ([2048, 4096, 1], [32, 32, 1], 4_300_001),  # digit totals by rows
])
def test_sort_is_stable(n, tile, count):
    from paper_2501_07465_amd import pic
    dims = 2 if n[2] == 1 else 3
    w = W.disk2d(n=64, radius=9.0, ppc_free=1, ppc_bound=1) if dims == 2 else W.sphere3d(n=64, steps=1)
    w["n"], w["tile"] = n, tile
    w["periodic"] = [1, 1, 1 if dims == 3 else 0]
    w.pop("source")
    w["species"] = [W.free_electrons(1, 5.5, 300.0, reflect=False)]
    w["sort_every"] = 1
    w["ion"] = "uniform"
    rng = np.random.default_rng(count)
    x = rng.random((count, 3)) * (np.array(n) * np.array(w["dx"]))
    x[:, dims:] = 0.0
    zero = np.zeros((3, n[2], n[1], n[0]))
    print(f"case sort n {n} tile {tile} count {count}", flush=True)
    sim = pic.Simulation(w, precision="fp32", states=[(x, np.zeros((count, 3)), None, 1.0)], fields=(zero, zero), graphs=False)
    x0, _, _ = sim.particles(0)
    k0 = sim.keys(0)
    order = np.argsort(k0, kind="stable")
    sim.step(1)
    x1, _, _ = sim.particles(0)
    # (the positions alone: a particle whose FP32 offset rounds to a whole cell is in the next one after the step)
    assert np.array_equal(x1, x0[order])


@pytest.mark.parametrize("slots", [1, 3])
def test_batch_sorts_match_runs_alone(slots):
    """The shared sorts of a batch: members of one to three radix passes, one and two moving species, unit
    lists of one round and of many, joining one after the other, are bit for bit the runs alone."""
    from paper_2501_07465_amd import pic

    def disk(n, tile, two=False):
        w = W.small("disk2d")
        w["n"], w["tile"] = n + [1], tile + [1]
        for sp in w["species"]:
            sp["region"]["center"] = [n[0] / 2.0, n[1] / 2.0, 0.0]
            sp["ppc"] = 30
        if two:
            w["species"].append(dict(w["species"][0]))
        return w

    ws = [disk([64, 60], [16, 8]),            # 12 bits
          disk([72, 68], [16, 8], two=True),
          disk([1300, 1100], [4, 4])]         # 21 bits: three passes; 89375 tiles
    batch = pic.Batch(slots, 2, "fp32")
    sims = []
    for w in ws:
        if len(batch) == slots:
            batch.remove(batch.members[0])
        sims.append(pic.Simulation(w, precision="fp32", graphs=False, stream=batch.stream))
        batch.add(sims[-1])
        batch.step(40)
    for i, (w, sim) in enumerate(zip(ws, sims)):
        print(f"case shared sorts, slots {slots}, member {i}", flush=True)
        alone = pic.Simulation(w, precision="fp32", graphs=False)
        alone.step(sim.steps_done)
        assert all(np.array_equal(a, b) for a, b in zip(sim.fields(), alone.fields()))
        for k in sim.species:
            assert all(np.array_equal(a, b) for a, b in zip(sim.particles(k), alone.particles(k)))
