"""A deposit that overflows spoils its own nodes and no others in the FP64 form: a particle whose velocity along
an invariant axis has grown to where charge times velocity is no number, among ordinary ones in the cells
around it."""
import numpy as np
import pytest

from paper_2501_07465_amd import workloads as W

pytestmark = pytest.mark.gpu

ME, QE = 9.1093837015e-31, 1.602176634e-19


@pytest.mark.parametrize("name,comp", [("slab1d", 1), ("slab1d", 2), ("disk2d", 2)])
def test_overflowing_deposit_stays_at_its_nodes(name, comp):
    from paper_2501_07465_amd import pic
    print(f"case {name} comp {comp}", flush=True)
    w = W.small(name)
    d = w["dims"]
    w["periodic"], w["source"], w["ion"] = [True] * 3, {"kind": "none"}, "local"
    w["species"] = [dict(w["species"][0], kind="free", q=-QE, m=ME, region={"kind": "all"}, reflect=False)]
    k, at = 40, 20
    x, v = np.zeros((k, 3)), np.zeros((k, 3))
    for a in range(d):
        x[:, a] = 18.5
    x[:, 0] = 18.5 + np.arange(k) % 8  # 5 in each of the cells 18 .. 25
    v[:, comp] = 1e5
    bad = np.flatnonzero(np.floor(x[:, 0]) == at)[0]
    v[bad, comp] = 1.0e308
    x *= np.array(w["dx"])
    sim = pic.Simulation(w, precision="fp64", states=[(x, v, np.zeros((k, 3)), 1e20)], graphs=False)
    sim.step(1)
    e = sim.fields()[0][comp].reshape(-1, w["n"][0])
    col = np.isfinite(e).all(axis=0)
    print("  columns not finite", np.flatnonzero(~col).tolist(), flush=True)
    assert np.flatnonzero(~col).tolist() == [at, at + 1]
    assert np.all(e[:, [18, 19, 22, 23, 24, 25]].any(axis=0))  # the others' deposits are there
