"""The work a user has this library do: runs of the particle-in-cell step through ``pic.Simulation`` and
``pic.Batch``, each pass a stretch of a run up to its next read-back.

A pass advances the simulation by ``steps`` steps (sort, particle and field kernels) and reads back what
the serving path and the studies read: the current series and the energies, and (but for the batch, whose
members leave with these numbers alone) a snapshot of the fields as the library exports it, E and then B
in one array.  FP32 runs keep their read-back in single precision, FP64 runs in double.

A case is a dict of plain values:

* ``kind``: ``slab`` (1D periodic plasma slab), ``relax`` (3D periodic cube of bulk electrons), ``disk``
  (2D metal disk in a pulse), ``request`` (a request of the serving stream, by its number), ``sheet`` (2D
  Dirac sheet on a bound substrate), ``sphere`` (3D nanosphere), ``batch`` (several requests at once);
* the sizes of that kind, ``precision``, ``steps``, and ``option`` (a feature of the run);
* ``tile``, ``block``, ``unit``: 0 for what the library does by default, or the launch shape that a user
  has tuned for the workload.

``exact`` is the same run in 64 bits by plain torch operations: its own loader, gather, pushers, deposit
and field update, written from the method and the workload's description.
"""
import math

import numpy as np
import torch

from paper_2501_07465_amd import pic, workloads as W

QE, ME, CL, EPS0 = 1.602176634e-19, 9.1093837015e-31, 299792458.0, 8.8541878128e-12
HBAR, KB = 1.054571817e-34, 1.380649e-23
TENSOR = [[3.7, 0.37, 0.185], [0.37, 3.33, 0.185], [0.185, 0.185, 4.07]]


def _case(name, kind, steps, precision="fp32", option="none", tile="0", block=0, unit=0, **sizes):
    return {"name": name, "kind": kind, "steps": steps, "precision": precision, "option": option,
            "tile": tile, "block": block, "unit": unit, **sizes}


def listed():
    return [
        # the plasma slab of the paper's validation runs, as shipped: the smallest run, all latency
        _case("slab_fp64", "slab", 100, "fp64", n=256, ppc=64),
        # the relaxation study's cube in its tuned launch shape: few cells, many particles a cell
        _case("relax_tuned", "relax", 200, tile="4x4x4", block=256, unit=1024, n=16, ppc=128),
        # a ragged metal disk as a user types it in, no tuning: an ordinary small 2D run
        _case("disk_ragged", "disk", 200, n=333, radius=55.5, ppc=12),
        # the 2D benchmark disk with the library's defaults
        _case("disk_default", "disk", 200, n=1024, radius=100.0, ppc=16),
        # the same in its tuned launch shape: the benchmark's second workload
        _case("disk_tuned", "disk", 300, tile="32x32", block=512, unit=2048, n=1024, radius=100.0, ppc=16),
        # the same in the reference precision
        _case("disk_fp64", "disk", 100, "fp64", n=1024, radius=100.0, ppc=16),
        # the disk filled with an anisotropic dielectric (a full permittivity tensor)
        _case("disk_tensor", "disk", 200, option="tensor", n=1024, radius=100.0, ppc=16),
        # the graphene sheet on its substrate in its tuned launch shape: mostly bound particles
        _case("sheet_tuned", "sheet", 400, tile="32x16", block=512, unit=8192, n=2048, ny=512, ppc=64),
        # a 64^3 nanosphere with the library's defaults: a small 3D run
        _case("sphere64_default", "sphere", 200, n=64, radius=25.0, ppc=8),
        # a 3D run in the reference precision (the tile is the one its LDS windows allow)
        _case("sphere_fp64", "sphere", 60, "fp64", tile="4x8x4", n=96, radius=37.0, ppc=8),
        # the headline workload: 256^3 cells, 65.5 million particles
        _case("sphere256_tuned", "sphere", 200, tile="8x8x4", block=256, n=256, radius=100.0, ppc=8),
        # sixteen requests of the serving stream in one batch, in the server's tuned launch shape
        _case("batch16", "batch", 60, tile="32x32", block=512, unit=2048, first=0, members=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["slab", "relax", "disk", "disk", "request", "sheet", "sphere", "sphere", "batch"])
    fp64 = rng.random() < 0.3
    p = "fp64" if fp64 else "fp32"
    tuned = rng.random() < 0.4
    c = {"kind": kind, "steps": rng.choice([60, 100, 140, 200]), "precision": p, "option": "none", "tile": "0", "block": 0, "unit": 0}
    if kind == "slab":
        c.update(n=_log(rng, 200, 60000), ppc=rng.randint(16, 100))
    elif kind == "relax":
        c.update(precision="fp32", n=rng.randint(10, 40), ppc=_log(rng, 16, 256))
        if tuned:
            c.update(tile="4x4x4", block=256, unit=1024)
    elif kind == "disk":
        n = _log(rng, 150, 1400)
        c.update(n=n, radius=round(n * rng.uniform(0.08, 0.28), 1), ppc=rng.randint(6, 32),
                 option=rng.choice(["none", "none", "diagonal", "tensor", "diffuse", "barrier"]))
        if tuned and not fp64:
            c.update(tile="32x32", block=512, unit=2048)
    elif kind == "request":
        c.update(j=rng.randrange(512))
    elif kind == "sheet":
        c.update(n=_log(rng, 300, 3000), ny=rng.choice([256, 400, 512, 601]), ppc=rng.randint(16, 80),
                 option=rng.choice(["none", "mass"]))
        if tuned and not fp64:
            c.update(tile="32x16", block=512, unit=8192)
    elif kind == "sphere":
        n = _log(rng, 40, 150 if not fp64 else 100)
        c.update(n=n, radius=round(n * rng.uniform(0.2, 0.4), 1), ppc=rng.randint(3, 10))
        if fp64:
            c.update(tile="4x8x4")
        elif tuned:
            c.update(tile="8x8x4", block=256)
    else:
        c.update(precision="fp32", steps=rng.choice([20, 40, 60]), first=rng.randrange(480), members=rng.randint(3, 16),
                 tile="32x32", block=512, unit=2048)
    return c


# ---- the runs --------------------------------------------------------------------------------------
def _shape(c, w):
    """The case's launch shape: the workload with its tile and unit."""
    if c["tile"] != "0":
        t = [int(x) for x in c["tile"].split("x")]
        w["tile"] = t + [1] * (3 - len(t))
    if c["unit"]:
        w["unit"] = c["unit"]
    w["steps"] = 4096
    return w


def _workload(c, seed):
    k, n = c["kind"], c.get("n")
    if k == "slab":
        w = W.slab1d(n=n, ppc=c["ppc"])
    elif k == "relax":
        w = W.relax3d(density=6e28, ppc=c["ppc"], n=n, box_nm=0.125 * n)
    elif k == "disk":
        w = W.disk2d(n=n, radius=c["radius"], ppc_free=c["ppc"], ppc_bound=c["ppc"])
    elif k == "request":
        w = W.stream_request(c["j"])
    elif k == "sheet":
        w = W.sheet2d(nx=n, ny=c["ny"], sheet_y=c["ny"] * 300 // 512, ppc_sheet=c["ppc"], src_y=c["ny"] - 12)
    else:
        w = W.sphere3d(n=n, radius=c["radius"], ppc_free=c["ppc"], ppc_bound=c["ppc"],
                       src_gap=max(2, min(14, int(n / 2 - c["radius"]) - 4)))
    if c["option"] == "diagonal":
        w = W.with_dielectric(w, [3.7, 3.7, 3.7])
    elif c["option"] == "tensor":
        w = W.with_dielectric(w, TENSOR)
    elif c["option"] == "diffuse":
        w = W.with_diffuse_walls(w)
    elif c["option"] == "barrier":
        w = W.with_potential_wall(w, 9.8, 8.0)
    elif c["option"] == "mass":
        w["species"][0]["mass_per_particle"] = True
    w["seed"] = 1 + seed % (1 << 31)
    return _shape(c, w)


def _requests(c, seed):
    return [dict(_shape(c, W.stream_request(c["first"] + m)), seed=1 + (seed * 64 + m) % (1 << 31)) for m in range(c["members"])]


def prepare(case, seed):
    """The loaded simulation (or the batch with its members joined) that a program is about to step."""
    block = case["block"] or 256
    if case["kind"] == "batch":
        b = pic.Batch(case["members"], 2, case["precision"])
        sims = [pic.Simulation(w, precision=case["precision"], graphs=False, stream=b.stream, block=block)
                for w in _requests(case, seed)]
        for s in sims:
            b.add(s)
        return {"case": case, "batch": b, "sims": sims}
    return {"case": case, "sims": [pic.Simulation(_workload(case, seed), precision=case["precision"], block=block)]}


def run(state):
    """Advance by the case's steps and read the run back."""
    c = state["case"]
    kept = np.float32 if c["precision"] == "fp32" else np.float64
    if c["kind"] == "batch":
        state["batch"].step(c["steps"])
    else:
        state["sims"][0].step(c["steps"])
    out = []
    for s in state["sims"]:
        r = {}
        if c["kind"] != "batch":
            r["fields"] = pic.pic_diag(s.h, pic.DIAG_EXPORT_FIELDS).astype(kept, copy=False)
        r["series"] = s.current_series().astype(kept, copy=False)
        r["energies"] = np.array([s.field_energy()] + [s.kinetic_energy(i) for i in s.species], dtype=kept)
        out.append(r)
    return out


def _cells(w, sp):
    """Region cells of a species, counted by the region's volume."""
    r, dims = sp["region"], w["dims"]
    if r["kind"] == "ball":
        x = max(1.0, r["radius"] - 0.75)
        return math.pi * x * x if dims == 2 else 4.0 / 3.0 * math.pi * x ** 3
    if r["kind"] == "box":
        return math.prod(max(1.0, r["hi"][a] - r["lo"][a]) for a in range(dims))
    return math.prod(w["n"][:dims])


def work(case):
    """One pass: per step every particle's state read and written once (a bound particle's anchor only
    read), E and B read and written once; the read-back written once."""
    ws = _requests(case, 0) if case["kind"] == "batch" else [_workload(case, 0)]
    es = 8 if case["precision"] == "fp64" else 4
    b = f = 0.0
    for w in ws:
        d, nodes = w["dims"], math.prod(W.field_extent(w))
        per, fl = 2 * 6 * es * nodes, 40.0 * nodes
        for sp in w["species"]:
            n = _cells(w, sp) * sp["ppc"]
            moved = 2 * (4 + (d + 3) * es) if sp["kind"] != "bound" else 4 + d * es + 2 * 6 * es
            per += n * moved
            fl += n * {1: 90, 2: 180, 3: 300}[d]
        b += per * case["steps"] + (0 if case["kind"] == "batch" else 6 * es * nodes)
        f += fl * case["steps"]
    return {"bytes": b, "flops": f}


# ---- the same run in 64 bits ------------------------------------------------------------------------
def _philox(x, k0, k1):
    m0, m1, mask = np.uint64(0xD2511F53), np.uint64(0xCD9E8D57), np.uint64(0xFFFFFFFF)
    s32 = np.uint64(32)
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
        p0, p1 = m0 * x[0], m1 * x[2]
        x = [(p1 >> s32) ^ x[1] ^ np.uint64(k0), p1 & mask, (p0 >> s32) ^ x[3] ^ np.uint64(k1), p0 & mask]
    return x


def _uniforms(n, sid, seed):
    """Six uniforms a particle: three calls of Philox4x32-10 with counter (index, 0, species, call)."""
    out = []
    for call in range(3):
        z = np.zeros(n, np.uint64)
        x = _philox([np.arange(n, dtype=np.uint64), z, z + np.uint64(sid), z + np.uint64(call)], seed & 0xFFFFFFFF, seed >> 32)
        for a, b in ((x[0], x[1]), (x[2], x[3])):
            out.append((((a >> np.uint64(5)) << np.uint64(26) | (b >> np.uint64(6))).astype(np.float64) + 0.5) / 9007199254740992.0)
    return out


def _fd_energy(u, mu, kT):
    """Fermi-Dirac energies by the inverse CDF tabulated on x = sqrt(e / e_max)."""
    tab = 65536
    x = np.arange(tab + 1) / tab
    e_max = mu + 40.0 * kT
    p = x * x / (1.0 + np.exp((e_max * x * x - mu) / kT))
    cdf = np.concatenate([[0.0], np.cumsum(0.5 * (p[1:] + p[:-1]) / tab)])
    cdf /= cdf[-1]
    lo = np.clip(np.searchsorted(cdf, u, side="right") - 1, 0, tab - 1)
    span = cdf[lo + 1] - cdf[lo]
    frac = np.where(span > 0, (u - cdf[lo]) / np.where(span > 0, span, 1.0), 0.0)
    return e_max * ((lo + frac) / tab) ** 2


def _region_cells(w, reg):
    n, dims = w["n"], w["dims"]
    g = np.meshgrid(np.arange(n[2]), np.arange(n[1]), np.arange(n[0]), indexing="ij")[::-1]
    keep = np.ones(g[0].shape, bool)
    if reg["kind"] == "box":
        for a in range(dims):
            keep &= (g[a] >= reg["lo"][a]) & (g[a] + 1 <= reg["hi"][a])
    elif reg["kind"] == "ball":
        far = sum(np.maximum((g[a] - reg["center"][a]) ** 2, (g[a] + 1 - reg["center"][a]) ** 2) for a in range(dims))
        keep &= far <= reg["radius"] ** 2
    return [x[keep] for x in g]


class _Run:
    """A run in 64 bits: positions as a cell and an offset in it, fields as [3][z][y][x]."""

    def __init__(self, w):
        self.w, self.dims, self.n = w, w["dims"], w["n"]
        self.dev = torch.device("cuda")
        self.dx, self.dt = w["dx"], w["dt"]
        self.per = [bool(w["periodic"][a]) or a >= self.dims for a in range(3)]
        self.L = [self.n[a] + (0 if self.per[a] else 1) for a in range(3)]
        f = lambda k: torch.zeros([k] + self.L[::-1], dtype=torch.float64, device=self.dev)  # noqa: E731
        self.E, self.B, self.step = f(3), f(3), 0
        self.einv = self.off = None
        if w.get("dielectric"):
            self._dielectric(w["dielectric"])
        self.sp = [self._load(i, s) for i, s in enumerate(w["species"])]
        if w.get("gauss_init"):
            s, n = self.sp[0], self.n[0]
            rho = torch.zeros(n, dtype=torch.float64, device=self.dev)
            for d, wt in ((0, 1.0 - s["o"][0]), (1, s["o"][0])):
                rho.index_add_(0, (s["c"][0] + d) % n, s["qw"] / self.dx[0] * wt)
            run = torch.cumsum(self.dx[0] * (rho - rho.mean()) / EPS0, 0)
            self.E[0, 0, 0] = run - run.mean()

    def t(self, x):
        return torch.as_tensor(x, device=self.dev)

    def _dielectric(self, d):
        eps = np.asarray(d["eps"], float)
        inv = np.diag(1.0 / eps) if eps.ndim == 1 else np.linalg.inv(eps)
        g = np.meshgrid(*[np.arange(self.L[a], dtype=float) for a in (2, 1, 0)], indexing="ij")[::-1]
        keep = np.ones(g[0].shape, bool)
        for a in range(self.dims):
            if not self.per[a]:
                keep &= (g[a] >= 2) & (g[a] <= self.n[a] - 2)
        ins = []
        for c in range(3):
            pos = [g[a] + (0.5 if a == c and c < self.dims else 0.0) for a in range(3)]
            ins.append(sum((pos[a] - d["region"]["center"][a]) ** 2 for a in range(self.dims)) <= d["region"]["radius"] ** 2)
        self.einv = self.t(np.stack([np.where(ins[c], inv[c, c], 1.0) for c in range(3)]))
        if eps.ndim == 2:
            self.off = {(a, b): self.t(np.where(ins[a] & keep, inv[a, b], 0.0)) for a in range(3) for b in range(3) if a != b}

    def _load(self, sid, sp):
        w, dims = self.w, self.dims
        cells = _region_cells(w, sp["region"])
        ppc, nc = sp["ppc"], len(cells[0])
        n = nc * ppc
        u = _uniforms(n, sid, w["seed"])
        c = [np.repeat(x, ppc) for x in cells]
        o = [u[a] if a < dims else np.zeros(n) for a in range(3)]
        m, v, xi = sp.get("m", 0.0), np.zeros((3, n)), np.zeros((3, n))
        dens = sp.get("density", 0.0)
        if sp.get("loading") == "quiet":
            x0 = c[0] + (np.arange(n) % ppc + 0.5) / ppc
            kw = 2.0 * math.pi * sp["pert_mode"] / self.n[0]
            X = x0 + sp["pert_amp"] / kw * np.sin(kw * x0)
            c[0], o[0] = np.floor(X).astype(np.int64) % self.n[0], X - np.floor(X)
        if sp["kind"] == "dirac":
            vf, nrm = sp["v_f"], sp["sheet_normal"]
            m = sp["e_fermi"] / vf / (2.0 * vf)
            dens = (sp["e_fermi"] / (HBAR * vf)) ** 2 / math.pi / self.dx[nrm]
            e1, e2 = [a for a in range(3) if a != nrm]
            v[e1], v[e2] = vf * np.cos(2 * math.pi * u[3]), vf * np.sin(2 * math.pi * u[3])
        else:
            if not dens:
                dens = (2.0 * m * sp["e_fermi"] / HBAR ** 2) ** 1.5 / (3.0 * math.pi ** 2)
            ct, ph = 2.0 * u[4] - 1.0, 2.0 * math.pi * u[5]
            way = np.stack([np.sqrt(1.0 - ct * ct) * np.cos(ph), np.sqrt(1.0 - ct * ct) * np.sin(ph), ct])
            if sp["kind"] == "free":
                v = np.sqrt(2.0 * _fd_energy(u[3], sp["e_fermi"], KB * sp["temperature"]) / m) * way
            else:
                xi = sp["xi_radius"] * np.cbrt(u[3]) * way
        wt = dens * math.prod(self.dx[:dims]) / ppc
        return {"sp": sp, "m": m, "q": sp["q"], "qw": sp["q"] * wt, "mw": m * wt, "c": [self.t(x) for x in c],
                "o": [self.t(x) for x in o], "v": list(self.t(v)), "xi": list(self.t(xi))}

    # nodes: flat index and whether they are on the grid
    def _node(self, g):
        ok, flat = None, 0
        for a in (2, 1, 0):
            x = g[a]
            if self.per[a]:
                x = x % self.n[a]
            else:
                inside = (x >= 0) & (x < self.L[a])
                ok, x = inside if ok is None else ok & inside, x.clamp(0, self.L[a] - 1)
            flat = flat * self.L[a] + x
        return flat, ok

    def _gather(self, F, half, c, o):
        base, up = [], []
        for a in range(3):
            if a >= self.dims:
                base.append(c[a])
                up.append(None)
            elif half[a]:
                s = (o[a] < 0.5).to(torch.int64)
                base.append(c[a] - s)
                up.append(o[a] - 0.5 + s)
            else:
                base.append(c[a])
                up.append(o[a])
        F, out = F.reshape(-1), 0.0
        for k in range(1 << self.dims):
            bit = [(k >> a) & 1 for a in range(3)]
            flat, ok = self._node([base[a] + bit[a] for a in range(3)])
            wt = 1.0
            for a in range(self.dims):
                wt = wt * (up[a] if bit[a] else 1.0 - up[a])
            x = wt * F[flat]
            out = out + (x if ok is None else torch.where(ok, x, 0.0))
        return out

    def _push(self, s, c, o):
        d, sp, dt = self.dims, s["sp"], self.dt
        E = [self._gather(self.E[k], [a == k for a in range(3)], c, o) for k in range(3)]
        v, qm = s["v"], s["q"] / s["m"]
        if sp["kind"] == "bound":
            acc = [qm * E[a] - sp["omega0"][a] ** 2 * s["xi"][a] for a in range(3)]
            g = [0.5 * sp["gamma"][a] * dt for a in range(3)]
            return [(1 - g[a]) / (1 + g[a]) * (v[a] + 0.5 * dt * acc[a]) + 0.5 * dt * acc[a] for a in range(3)]
        B = [self._gather(self.B[k], [a != k and a < d for a in range(3)], c, o) for k in range(3)]
        h = 0.5 * qm * dt
        vm, b = [v[a] + h * E[a] for a in range(3)], [h * B[a] for a in range(3)]
        bb = sum(x * x for x in b)
        bv = sum(x * y for x, y in zip(b, vm))
        cr = [vm[(a + 1) % 3] * b[(a + 2) % 3] - vm[(a + 2) % 3] * b[(a + 1) % 3] for a in range(3)]
        out = [((1 - bb) * vm[a] + 2 * bv * b[a] + 2 * cr[a]) / (1 + bb) + h * E[a] for a in range(3)]
        if sp["kind"] == "dirac":
            out[sp["sheet_normal"]] = torch.zeros_like(out[0])
            k = sp["v_f"] / torch.sqrt(sum(x * x for x in out))
            out = [x * k for x in out]
        return out

    def _mirror(self, sp, c, x1, v):
        reg, d = sp["region"], self.dims
        X = [c[a] + x1[a] for a in range(d)]
        if reg["kind"] == "ball":
            rel = [X[a] - reg["center"][a] for a in range(d)]
            r = torch.sqrt(sum(x * x for x in rel))
            out = r * r > reg["radius"] ** 2
            rh = [x / r for x in rel]
            vn = sum(v[a] * rh[a] for a in range(d))
            for a in range(d):
                x1[a] = torch.where(out, reg["center"][a] + (2 * reg["radius"] - r) * rh[a] - c[a], x1[a])
                v[a] = torch.where(out, v[a] - 2 * vn * rh[a], v[a])
        elif reg["kind"] == "box":
            for a in range(d):
                for out, at in ((X[a] > reg["hi"][a], reg["hi"][a]), (X[a] < reg["lo"][a], reg["lo"][a])):
                    x1[a] = torch.where(out, 2 * at - X[a] - c[a], x1[a])
                    v[a] = torch.where(out, -v[a], v[a])

    def _deposit(self, J, s, c, x0, x1, v):
        """Charge-conserving deposit on the nodes c - 1 .. c + 2 of each axis."""
        d, dx, dt, qw = self.dims, self.dx, self.dt, s["qw"]
        shape = lambda x, m: (1.0 - (x - (m - 1)).abs()).clamp(min=0.0)  # noqa: E731
        S = [[shape(x0[a], m) for m in range(4)] for a in range(d)]
        D = [[shape(x1[a], m) - S[a][m] for m in range(4)] for a in range(d)]
        area = math.prod(dx[:d])

        def mean(a, b, i, j):
            return S[a][i] * S[b][j] + 0.5 * (D[a][i] * S[b][j] + S[a][i] * D[b][j]) + D[a][i] * D[b][j] / 3.0

        run = [None] * d  # minus the running sum of the change along each axis
        for a in range(d):
            acc, run[a] = 0.0, []
            for m in range(4):
                acc = acc - D[a][m]
                run[a].append(acc)
        for k in range(4 ** d):
            m = [(k >> (2 * a)) & 3 for a in range(d)]
            flat, ok = self._node([c[a] + (m[a] - 1 if a < d else 0) for a in range(3)])
            for comp in range(3):
                if comp >= d:
                    wt = S[0][m[0]] + 0.5 * D[0][m[0]] if d == 1 else mean(0, 1, m[0], m[1])
                    x = qw / area * v[comp] * wt
                elif m[comp] == 3:
                    continue
                else:
                    oth = [a for a in range(d) if a != comp]
                    wt = 1.0 if d == 1 else (S[oth[0]][m[oth[0]]] + 0.5 * D[oth[0]][m[oth[0]]] if d == 2
                                             else mean(oth[0], oth[1], m[oth[0]], m[oth[1]]))
                    x = qw * dx[comp] / (dt * area) * run[comp][m[comp]] * wt
                J[comp].reshape(-1).index_add_(0, flat, x if ok is None else torch.where(ok, x, 0.0))

    def _particles(self, J):
        d, cur = self.dims, [0.0, 0.0, 0.0]
        for s in self.sp:
            n = s["v"][0].numel()
            for at in range(0, n, 1 << 20):
                k = slice(at, min(n, at + (1 << 20)))
                p = dict(s, c=[x[k] for x in s["c"]], o=[x[k] for x in s["o"]], v=[x[k] for x in s["v"]], xi=[x[k] for x in s["xi"]])
                c, x0 = list(p["c"]), list(p["o"])
                if s["sp"]["kind"] == "bound":
                    for a in range(d):
                        x = x0[a] + p["xi"][a] / self.dx[a]
                        c[a], x0[a] = c[a] + torch.floor(x).to(torch.int64), x - torch.floor(x)
                v = self._push(p, c, x0)
                x1 = [x0[a] + v[a] * (self.dt / self.dx[a]) for a in range(d)]
                if s["sp"].get("reflect"):
                    self._mirror(s["sp"], c, x1, v)
                self._deposit(J, s, c, x0, x1, v)
                for a in range(3):
                    s["v"][a][k] = v[a]
                    cur[a] += s["qw"] * v[a].sum()
                    if s["sp"]["kind"] == "bound":
                        s["xi"][a][k] += self.dt * v[a]
                    elif a < d:
                        f = torch.floor(x1[a])
                        c1 = c[a] + f.to(torch.int64)
                        s["c"][a][k] = c1 % self.n[a] if self.per[a] else c1
                        s["o"][a][k] = x1[a] - f
        return torch.stack([torch.as_tensor(x, dtype=torch.float64, device=self.dev) for x in cur])

    def _curl(self, F, way):
        """Curl by forward (+1) or backward (-1) differences; entries past an open face are not used."""
        out = torch.zeros_like(F)
        for c in range(3):
            for a, b, sg in (((c + 1) % 3, (c + 2) % 3, 1.0), ((c + 2) % 3, (c + 1) % 3, -1.0)):
                if a < self.dims:
                    out[c] += sg * way * (torch.roll(F[b], -way, 2 - a) - F[b]) / self.dx[a]
        return out

    def _pad(self, F, half):
        for c in range(3):
            for a in range(self.dims):
                if not self.per[a] and half(c, a):
                    F[c].narrow(2 - a, self.n[a], 1).zero_()

    def advance(self):
        J = torch.zeros_like(self.E)
        cur = self._particles(J)
        src = self.w.get("source", {"kind": "none"})
        t = (self.step + 0.5) * self.dt
        if src["kind"] != "none" and t <= src["tau"]:
            at = [slice(None)] * 3
            for a in range(self.dims):
                if src["kind"] == "point" or a == src["axis"]:
                    at[2 - a] = src["index"][a]
            J[src["comp"]][tuple(at)] += src["j0"] * math.sin(math.pi * t / src["tau"]) ** 2 * math.sin(src["omega"] * t)
        on_b = lambda c, a: a != c and a < self.dims  # noqa: E731
        self.B -= 0.5 * self.dt * self._curl(self.E, 1)
        self._pad(self.B, on_b)
        U = CL * CL * self._curl(self.B, -1) - J / EPS0
        E1 = self.E + self.dt * (U if self.einv is None else self.einv * U)
        if self.off is not None:
            for (a, b), e in self.off.items():
                ns, nt = 1 + (a < self.dims), 1 + (b < self.dims)
                acc = 0.0
                for i in range(ns):
                    for j in range(nt):
                        x = torch.roll(U[b], -i, 2 - a) if i else U[b]
                        acc = acc + (torch.roll(x, j, 2 - b) if j else x)
                E1[a] += self.dt * e * acc / (ns * nt)
        # first-order Mur on open faces, from the inward node along the lowest open axis; an inward
        # node that lies on a face itself counts with its old value
        faces = [(a, i, 1 if i == 0 else self.n[a] - 1) for a in range(self.dims) if not self.per[a] for i in (0, self.n[a])]
        for c in range(3):
            mine = [f for f in faces if f[0] != c]
            for a, i, _ in mine:
                E1[c].select(2 - a, i).copy_(self.E[c].select(2 - a, i))
            new = E1[c].clone()
            for a, i, inward in reversed(mine):
                k = (CL * self.dt - self.dx[a]) / (CL * self.dt + self.dx[a])
                old = self.E[c].select(2 - a, inward)
                new.select(2 - a, i).copy_(old + k * (E1[c].select(2 - a, inward) - self.E[c].select(2 - a, i)))
            E1[c] = new
        self._pad(E1, lambda c, a: a == c)
        self.E = E1
        self.B -= 0.5 * self.dt * self._curl(self.E, 1)
        self._pad(self.B, on_b)
        self.step += 1
        return cur

    def energies(self):
        dv = math.prod(self.dx[:self.dims])
        e = self.E ** 2 if self.einv is None else self.E ** 2 / self.einv
        out = [(0.5 * EPS0 * e.sum() + 0.5 * EPS0 * CL * CL * (self.B ** 2).sum()) * dv]
        out += [0.5 * s["mw"] * sum((x * x).sum() for x in s["v"]) for s in self.sp]
        return torch.stack(out)


def exact(case, seed):
    """None for the runs whose draws at the walls, barrier field or carrier masses are not restated
    here, and for those that would take too long."""
    if case["option"] in ("diffuse", "barrier", "mass"):
        return None
    ws = _requests(case, seed) if case["kind"] == "batch" else [_workload(case, seed)]
    moves = case["steps"] * sum(_cells(w, sp) * sp["ppc"] for w in ws for sp in w["species"] if w["dims"] < 3) + \
        4 * case["steps"] * sum(_cells(w, sp) * sp["ppc"] for w in ws for sp in w["species"] if w["dims"] == 3)
    if moves > 1.5e9:
        return None
    out = []
    for w in ws:
        r = _Run(w)
        series = torch.stack([r.advance() for _ in range(case["steps"])])
        one = {"series": series, "energies": r.energies()}
        if case["kind"] != "batch":
            one["fields"] = torch.cat([r.E.reshape(-1), r.B.reshape(-1)])
        out.append(one)
    return out
