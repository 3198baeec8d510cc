"""The cell sort where its launches change form: two keys a thread, the histogram's columns scanned in sixteens
up to 512 blocks and in fours for up to 2048, and the same in the launches that the members of a batch share,
beside members of other forms.  The particles leave in the order of a stable argsort of their cell keys, bit
for bit."""
import numpy as np
import pytest

from paper_2501_07465_amd import workloads as W

pytestmark = pytest.mark.gpu


def _cloud(n, tile, count, seed):
    """A workload of one free species, and `count` particles at random places of its grid."""
    dims = 2 if n[2] == 1 else 3
    w = W.disk2d(n=64, radius=9.0, ppc_free=1, ppc_bound=1) if dims == 2 else W.sphere3d(n=64, steps=1)
    w["n"], w["tile"] = n, tile
    w["periodic"] = [1, 1, 1 if dims == 3 else 0]
    w.pop("source")
    w["species"] = [W.free_electrons(1, 5.5, 300.0, reflect=False)]
    w["sort_every"], w["ion"], w["steps"] = 1, "uniform", 16
    x = np.random.default_rng(seed).random((count, 3)) * (np.array(n) * np.array(w["dx"]))
    x[:, dims:] = 0.0
    return w, [(x, np.zeros((count, 3)), None, 1.0)]


def _zero(n):
    return (np.zeros((3, n[2], n[1], n[0])),) * 2


@pytest.mark.parametrize("n,tile,count", [
    ([512, 512, 1], [16, 16, 1], 1_100_003),   # 18 bits, digits of 9: two keys a thread
    ([512, 512, 1], [16, 16, 1], 2_200_003),
    ([2048, 4096, 1], [32, 32, 1], 1_500_001),  # digits of 8, too few keys for four a thread
    ([1000, 1000, 1], [16, 16, 1], 512 * 1024),      # 512 blocks: columns in sixteens
    ([1000, 1000, 1], [16, 16, 1], 512 * 1024 + 1),  # 513: in fours
    ([64, 64, 64], [8, 8, 4], 8_388_607),      # 2048 blocks
])
def test_sort_is_stable(n, tile, count):
    """(velocities and fields are zero, so the step that follows the sort moves nothing)"""
    from paper_2501_07465_amd import pic
    print(f"case sort n {n} tile {tile} count {count}", flush=True)
    w, states = _cloud(n, tile, count, count)
    sim = pic.Simulation(w, precision="fp32", states=states, fields=_zero(n), graphs=False)
    x0 = sim.particles(0)[0]
    order = np.argsort(sim.keys(0), kind="stable")
    sim.step(1)
    assert np.array_equal(sim.particles(0)[0], x0[order])


def test_shared_sorts_of_members_of_other_forms():
    """Members of 1, 33, 513 and 1025 blocks join one after the other (each asks for another form of the shared
    scans), with keys of 12, 18, 20 and 23 bits.  Particles of next to no charge fly at up to 0.9 cells a step, so
    that every step scrambles the keys and keeps the velocities, by which their order is seen."""
    from paper_2501_07465_amd import pic
    shapes = [([64, 60, 1], [16, 8, 1], 1000), ([512, 512, 1], [16, 16, 1], 32 * 1024 + 1),
              ([1000, 1000, 1], [32, 32, 1], 512 * 1024 + 1), ([2048, 4096, 1], [32, 32, 1], 4 * 1024 * 1024 + 1)]
    batch = pic.Batch(4, 2, "fp32")
    sims = []
    for i, (n, tile, count) in enumerate(shapes):
        print(f"case shared sorts: {i + 1} members, the last of {count}", flush=True)
        w, [(x, v, _, _)] = _cloud(n, tile, count, 90 + i)
        v = (np.random.default_rng(i).random((count, 3)) * 2.0 - 1.0) * 0.9 * np.array(w["dx"]) / w["dt"]
        v[:, 2] = 0.0
        sims.append(pic.Simulation(w, precision="fp32", states=[(x, v, None, 1e-30)], fields=_zero(n), graphs=False, stream=batch.stream))
        batch.add(sims[-1])
        batch.step(1)
        for _ in range(2):
            before = [(sim.particles(0)[1], sim.keys(0)) for sim in sims]
            batch.step(1)
            for sim, (v0, k0) in zip(sims, before):
                assert count < 2000 or (np.diff(k0) < 0).any()  # not in order before the sort
                assert np.array_equal(sim.particles(0)[1], v0[np.argsort(k0, kind="stable")])
                assert sim.overflow() == 0
