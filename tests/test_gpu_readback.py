"""Exports below and above the size that goes through the pinned ring, on chunk boundaries and past them,
from one thread and from several at once: the exported state is the state that was loaded (positions to the
rounding of their cell and offset, the rest exactly), and the fields are those that were loaded."""
import threading

import numpy as np
import pytest

from paper_2501_07465_amd import workloads as W

pytestmark = pytest.mark.gpu


def _sim(n, count, precision, seed):
    from paper_2501_07465_amd import pic
    w = W.small("disk2d")
    w["n"], w["periodic"] = [n, n + 3, 1], [1, 1, 1]
    w["source"] = {"kind": "none"}
    for sp in w["species"]:
        sp["region"], sp["reflect"] = {"kind": "all"}, False
    x, v = W.random_particles(w, count, seed)
    v = v.astype(np.float32).astype(np.float64)
    xi = (1e-11 * np.random.default_rng(seed).normal(size=(count, 3))).astype(np.float32).astype(np.float64)
    states = [(x, v, np.zeros_like(x), 1.0), (x[::-1].copy(), v[::-1].copy(), xi, 1.0)]
    rng = np.random.default_rng(seed + 1)
    f = rng.normal(size=(2, 3, 1, n + 3, n)).astype(np.float32).astype(np.float64)
    sim = pic.Simulation(w, precision=precision, states=states, fields=f, graphs=False)
    return w, sim, states, f


def _check(w, sim, states, f, precision):
    e, b = sim.fields()
    assert np.array_equal(e, f[0]) and np.array_equal(b, f[1])
    tol = 1e-6 if precision == "fp32" else 1e-12  # cells: an offset in [0, 1) in the run's reals
    for sid, (x, v, xi, _) in enumerate(states):
        xg, vg, xig = sim.particles(sid)
        assert np.abs(xg - x).max() <= tol * w["dx"][0]
        assert np.array_equal(vg, v)
        assert np.array_equal(xig, xi)
    k = sim.keys(0)
    assert k.shape == (len(states[0][0]),) and k.min() >= 0


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,count", [(33, 1), (60, 4999), (430, 262144), (801, 700001)])
def test_export_is_what_was_loaded(n, count, precision):
    print(f"case export n {n} count {count} {precision}", flush=True)
    w, sim, states, f = _sim(n, count, precision, 7)
    _check(w, sim, states, f, precision)


def test_exports_of_several_threads():
    print("case exports from four threads", flush=True)
    sims = [_sim(431, 100003, "fp32", 20 + k) for k in range(4)]
    bad = []

    def work(k):
        try:
            for _ in range(3):
                _check(*sims[k], "fp32")
        except BaseException as exc:  # noqa: BLE001
            bad.append((k, exc))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
