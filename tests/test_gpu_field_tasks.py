"""The field kernel's task shapes: row groups of the 2D sweep (1 to 6 rows), plane chunks of the 3D march (chosen by rounds of wavefronts, so from 1 to
10 planes over these grids, with a short last chunk or none), and the masks of particle-tile columns found
at the sort, on tiles of 2 to 16 cells and on open and periodic axes.  FP64 runs from the oracle's state
stay within the 1e-12 that the form is held to."""
import numpy as np
import pytest

from paper_2501_07465_amd import workloads as W

pytestmark = pytest.mark.gpu


def _sphere(n, tile, periodic):
    w = W.small("sphere3d")
    w["n"], w["tile"], w["periodic"] = list(n), list(tile), list(periodic)
    c = [x / 2.0 for x in n]
    r = min(n) / 2.0 - 4.5
    for sp in w["species"]:
        sp["region"] = {"kind": "ball", "center": c, "radius": r}
        sp["ppc"] = 2
    w["source"]["index"] = [n[0] // 2, n[1] // 2, n[2] - 3]
    return w


@pytest.mark.parametrize("n,tile,periodic", [
    ([17, 15, 13], [4, 4, 4], [0, 0, 0]),    # chunks of one plane
    ([70, 21, 131], [4, 8, 4], [0, 1, 0]),   # two strips, periodic rows
    ([61, 16, 101], [2, 4, 4], [1, 0, 1]),   # one whole strip, periodic planes, one bit for all columns
    ([130, 90, 64], [4, 4, 8], [0, 0, 1]),   # chunks of 5 planes (8832 tasks of one), the last of 4
    ([130, 90, 40], [4, 4, 4], [1, 0, 0]),   # chunks of 3, the last of 1 and the face plane
])
def test_fp64_plane_chunks_match_oracle(oracle, n, tile, periodic):
    from paper_2501_07465_amd import pic
    print(f"case plane chunks: n {n} tile {tile} periodic {periodic}", flush=True)
    w = _sphere(n, tile, periodic)
    ref = oracle.build_workload(w)
    sim = pic.Simulation(w, precision="fp64", states=ref.state(), fields=ref.fields(), graphs=False)
    ref.step(3)
    sim.step(3)
    (eg, bg), (er, br) = sim.fields(), ref.fields()
    ee = np.abs(eg - er).max() / np.abs(er).max()
    eb = np.abs(bg - br).max() / max(np.abs(br).max(), np.abs(er).max() / 3e8)
    print(f"  E {ee:.2e} B {eb:.2e}", flush=True)
    assert ee < 1e-12 and eb < 1e-12


@pytest.mark.parametrize("n,tile,periodic,slots", [
    ([72, 67], [16, 8], [0, 0], 32),      # 1 row a task, 2 in the batch (the last task one)
    ([72, 67], [16, 8], [1, 1], 64),      # 1 and 3
    ([1220, 201], [16, 16], [0, 1], 24),  # 2 (the last task one) and 4
    ([1831, 250], [32, 8], [1, 0], 2),    # 3 and 6, the last task with the face row
    ([3000, 298], [16, 16], [0, 0], 32),  # 5 and 6
])
def test_fp64_row_groups_of_a_batch_match_alone(n, tile, periodic, slots):
    """A member of a batch of many slots takes taller tasks than a simulation on its own, whose runs on the
    small grid the other tests hold to the oracle: the fields are the same bit for bit, also after the
    member has left and steps on its own again."""
    from paper_2501_07465_amd import pic
    print(f"case row groups: n {n} tile {tile} periodic {periodic} slots {slots}", flush=True)
    w = W.small("disk2d")
    w["n"], w["tile"], w["periodic"] = n + [1], tile + [1], periodic + [0]
    for sp in w["species"]:
        sp["region"]["center"] = [n[0] / 2.0, n[1] / 2.0, 0.0]
    batch = pic.Batch(slots, 2, "fp64")
    member = pic.Simulation(w, precision="fp64", graphs=False, stream=batch.stream)
    alone = pic.Simulation(w, precision="fp64", graphs=False)
    batch.add(member)
    batch.step(20)
    alone.step(20)
    assert all(np.array_equal(a, b) for a, b in zip(member.fields(), alone.fields()))
    batch.step(20)
    batch.remove(member)
    member.step(20)
    alone.step(40)
    assert all(np.array_equal(a, b) for a, b in zip(member.fields(), alone.fields()))
