"""Workloads whose speed is measured, the way programs of this package run
them: the statistical runs of the paper's Sec. 3 (many steps of a small box,
then its series), the large boxes of the benchmark, the mixed ensemble, the
diagnostics (structure factor, velocity PDFs), state saved and resumed, and a
program that reads the fields after every step.

``listed`` gives the fixed cases, ``draw`` more of the same ranges,
``prepare`` what such a program holds, ``run`` one pass, ``work`` what a pass
cannot do without and ``exact`` the FP64 values of its outputs, computed here
in plain torch from the method's definitions.
"""
import math

import numpy as np
import torch

from paper_2602_16486_amd import Ensemble, Lattice, external_bytes, rate_vector
from paper_2602_16486_amd import workloads as W

STORAGE_BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
STORAGE_TORCH = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16,
                 "bf16": torch.bfloat16}
# arithmetic operations a site needs per step (moments, normals, collision,
# back transformation)
SITE_OPS = {9: 340, 19: 670, 27: 900}
CS2 = 1.0 / 3.0


def _case(kind, q, shape, storage="f32", steps=1, **kw):
    nx, ny, nz = W.shape3(shape)
    c = {"kind": kind, "q": q, "nx": nx, "ny": ny, "nz": nz, "storage": storage, "steps": steps,
         "tau": 0.8, "kT": 1e-4, "rho0": 1.0, "rates": "paper", "in_place": False, "tuned": False}
    c.update(kw)
    return c


def listed():
    return [
        # a program that uses the fields after every step: the smallest call
        dict(_case("couple", 9, (96, 61), steps=1, kT=1 / 3000), name="couple_d2q9_96x61"),
        # Test 2: Taylor-Green decay in FP64, no noise, no series
        dict(_case("decay", 9, (64, 64), "f64", steps=512, tau=0.692, kT=0.0), name="decay_d2q9_64_f64"),
        # Tests 3-6: 200 x 200, hundreds of thousands of steps in chunks
        dict(_case("run", 9, (200, 200), steps=512, kT=1 / 3000), name="run_d2q9_200"),
        # the kT x tau sweep in FP64
        dict(_case("run", 9, (1024, 1024), "f64", steps=64, tau=0.6, kT=1e-5), name="run_d2q9_1024_f64"),
        # Test 7, box C1 (rows that are no whole cache lines)
        dict(_case("run", 27, (50, 50, 50), steps=128, kT=1 / 3000), name="run_d3q27_50"),
        # the benchmark's box, tuned as the benchmark tunes it
        dict(_case("run", 27, (256, 256, 256), steps=20, tuned=True), name="run_d3q27_256"),
        # the 16-bit storage run of the same box
        dict(_case("run", 27, (256, 256, 256), "f16", steps=20, tau=0.51), name="run_d3q27_256_f16"),
        # the reduced lattice in half the memory, one viscosity for all
        # second-order modes (general rates), ragged rows
        dict(_case("run", 19, (150, 144, 160), steps=24, rates="isotropic", in_place=True),
             name="run_d3q19_aa_isotropic"),
        # 256 D2Q9 and 64 D3Q27 replicas in one launch per step
        dict(_case("ensemble", 0, (1, 1), steps=40, n2d=256, n3d=64, manifest=2026, tuned=True),
             name="ensemble_320"),
        # structure factor sampled along a run
        dict(_case("spectrum", 27, (128, 128, 128), steps=10, samples=6, nbins=48, tau=0.55),
             name="spectrum_d3q27_128"),
        # velocity PDFs of a final state (Fig. 8)
        dict(_case("pdf", 27, (128, 128, 128), nbins=40, kT=1 / 3000), name="pdf_d3q27_128"),
        # a run resumed from saved populations and saved again
        dict(_case("checkpoint", 27, (64, 64, 64)), name="checkpoint_d3q27_64"),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _box(rng, dims, lo, hi):
    """Edges around a log-uniform side in [lo, hi], some of them multiples of
    32, most odd or ragged."""
    side = _log_uniform(rng, lo, hi)
    edges = [max(8, min(int(hi), round(side * math.exp(rng.uniform(-0.4, 0.4))))) for _ in range(dims)]
    if rng.random() < 0.4:
        edges[0] = max(32, edges[0] // 32 * 32)
    return tuple(edges)


def draw(rng):
    kind = rng.choice(["run"] * 5 + ["couple", "decay", "ensemble", "spectrum", "pdf", "checkpoint"])
    if kind == "ensemble":
        return _case("ensemble", 0, (1, 1), rng.choice(["f32", "f32", "f16", "f64"]),
                     steps=rng.randrange(8, 41), n2d=rng.randrange(4, 97), n3d=rng.randrange(0, 25),
                     manifest=rng.randrange(1, 1 << 20))
    if kind == "decay":
        n = round(_log_uniform(rng, 16, 256))
        return _case("decay", 9, (n, n), rng.choice(["f64", "f32"]), steps=rng.randrange(64, 513),
                     tau=rng.uniform(0.55, 1.0), kT=0.0)
    q = rng.choice([9, 9, 27, 27, 19])
    small = kind in ("couple", "checkpoint")
    shape = _box(rng, 2, 24, 512 if small else 1024) if q == 9 else _box(rng, 3, 12, 72 if small else 192)
    kw = {"tau": rng.uniform(0.6, 2.0), "kT": _log_uniform(rng, 1e-6, 1e-3),
          "rho0": rng.choice([0.5, 1.0, 1.0, 2.0])}
    storage = rng.choice(["f32", "f32", "f32", "f64", "f16", "bf16"])
    if kind == "run":
        sites = W.n_sites(shape)
        kw["steps"] = rng.randrange(*((100, 513) if sites < 60_000 else (16, 97) if sites < 1_500_000 else (8, 21)))
        kw["rates"] = rng.choice(["paper", "paper", "paper", "isotropic", "single"])
        kw["in_place"] = rng.random() < 0.2
        kw["tuned"] = rng.random() < 0.2
    elif kind == "couple":
        kw["steps"] = rng.choice([1, 1, 2, 5])
    elif kind == "spectrum":
        kw.update(steps=rng.randrange(4, 21), samples=rng.randrange(3, 9), nbins=rng.choice([32, 48, 64]))
    elif kind == "pdf":
        kw["nbins"] = rng.choice([40, 64, 200])
    return _case(kind, q, shape, storage, **kw)


def _shape(case):
    return (case["nx"], case["ny"], case["nz"])


def _manifest(case, seed):
    reps = W.ensemble_manifest(seed=case["manifest"], n2d=case["n2d"], n3d=case["n3d"])
    for r, rep in enumerate(reps):
        rep["seed"] = 1000 * (seed + 1) + r
    return reps


def _lattice(case, seed, **kw):
    lam = None if case["rates"] == "paper" else rate_vector(case["q"], case["tau"], case["rates"])
    return Lattice(case["q"], _shape(case), storage=case["storage"], rho0=case["rho0"], tau=case["tau"],
                   kT=case["kT"], lam=lam, seed=seed, in_place=case["in_place"], **kw)


def _thermal_fields(case, seed):
    """Density and velocity of a thermal state (N), (3, N), host FP64."""
    rng = np.random.default_rng(seed)
    n = W.n_sites(_shape(case))
    rho = case["rho0"] + math.sqrt(case["rho0"] * case["kT"] / CS2) * rng.standard_normal(n)
    u = math.sqrt(case["kT"] / case["rho0"]) * rng.standard_normal((3, n))
    if case["q"] == 9:
        u[2] = 0.0
    return rho, u


def _vortex(case, seed):
    """The Test 2 vortex, its phase from the seed."""
    rng = np.random.default_rng(seed)
    nx, ny, _ = _shape(case)
    k, px, py = 2 * math.pi / ny, *rng.uniform(0, 2 * math.pi, 2)
    x, y = np.arange(nx)[None, :] * k + px, np.arange(ny)[:, None] * k + py
    u = np.zeros((3, nx * ny))
    u[0] = (-1e-3 * np.cos(x) * np.sin(y)).ravel()
    u[1] = (1e-3 * np.sin(x) * np.cos(y)).ravel()
    return u


def _populations(case, seed):
    """Equilibrium populations (q, N), host FP64: w rho0 and their spread."""
    rng = np.random.default_rng(seed)
    w = np.array(weights(case["q"]))[:, None]
    z = rng.standard_normal((case["q"], W.n_sites(_shape(case))))
    return w * case["rho0"] + np.sqrt(case["rho0"] * case["kT"] * w / CS2) * z


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "steps": case["steps"]}
    if kind == "ensemble":
        s["ens"] = Ensemble(_manifest(case, seed), storage=case["storage"], series_capacity=case["steps"])
        if case["tuned"]:
            s["ens"].autotune(steps_per_trial=4)
        return s
    if kind == "run":
        n = external_bytes(case["q"], _shape(case), case["storage"], case["in_place"])
        s["buf"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        s["lat"] = _lattice(case, seed, external=(s["buf"].data_ptr(), n))
        values = s["buf"].view(STORAGE_TORCH[case["storage"]])
        count = case["q"] * W.n_sites(_shape(case))
        half = 0 if case["in_place"] else values.numel() // 2
        s["halves"], s["parity"] = [values[:count], values[half:half + count]], 0
        if case["tuned"]:
            s["lat"].autotune(steps_per_trial=10)
    elif kind == "couple":
        n = W.n_sites(_shape(case))
        s["lat"] = _lattice(case, seed)
        s["rho"] = torch.empty(n, dtype=torch.float32, device="cuda")
        s["u"] = torch.empty((3, n), dtype=torch.float32, device="cuda")
    elif kind == "decay":
        s["lat"] = _lattice(case, seed, flags=2)  # no series, as in Test 2
        s["lat"].init_equilibrium(u=_vortex(case, seed))
    elif kind == "spectrum":
        s["lat"] = _lattice(case, seed)
        s["lat"].sk_reset(case["nbins"])
    elif kind == "pdf":
        s["lat"] = _lattice(case, seed)
        s["lat"].init_equilibrium(*_thermal_fields(case, seed))
    elif kind == "checkpoint":
        s["lat"] = _lattice(case, seed)
        s["f"] = _populations(case, seed)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "ensemble":
        ens = s["ens"]
        ens.step(s["steps"])
        series = np.stack([ens.stats(k) for k in range(ens.n)])
        return {"series": series, "first": ens.get_populations(0), "last": ens.get_populations(ens.n - 1)}
    lat = s["lat"]
    if kind == "run":
        lat.step(s["steps"])
        s["parity"] ^= s["steps"] & 1
        return {"series": lat.stats(), "state": s["halves"][s["parity"]]}
    if kind == "couple":
        lat.step(s["steps"])
        lat.sample_macro(s["rho"].data_ptr(), s["u"].data_ptr())
        return {"rho": s["rho"], "u": s["u"]}
    if kind == "decay":
        lat.step(s["steps"])
        return dict(zip(("rho", "u"), lat.macroscopic()))
    if kind == "spectrum":
        for _ in range(case["samples"]):
            lat.step(s["steps"])
            lat.sk_accumulate()
        return {"shells": lat.sk_shells()[0], "series": lat.stats()}
    if kind == "pdf":
        return dict(zip(("moments", "counts"), lat.velocity_pdf(case["nbins"], 5.0)))
    lat.set_populations(s["f"])
    return {"f": lat.get_populations()}


def work(case):
    """Bytes and operations of one pass: a step reads and writes every stored
    population once (a lattice larger than the chip's memories cannot keep
    them between steps); a diagnostic reads the state once and writes its
    result; the canonical populations are FP64."""
    kind = case["kind"]
    if kind == "ensemble":
        site_q = [(W.n_sites(r["shape"]), r["q"]) for r in _manifest(case, 0)]
    else:
        site_q = [(W.n_sites(_shape(case)), case["q"])]
    b = STORAGE_BYTES[case["storage"]]
    state = sum(n * q * b for n, q in site_q)
    n = sum(n for n, _ in site_q)
    ops = sum(n * SITE_OPS[q] for n, q in site_q)
    macro = sum(n * 2 * q for n, q in site_q)
    steps = case["steps"]
    if kind in ("run", "ensemble"):
        return {"bytes": 2 * state * steps, "flops": ops * steps}
    if kind == "couple":
        return {"bytes": 2 * state * steps + state + 16 * n, "flops": ops * steps + macro}
    if kind == "decay":
        return {"bytes": 2 * state * steps + state + 32 * n, "flops": ops * steps + macro}
    if kind == "spectrum":
        # per sample: the state, and the four fields' |F|^2 into FP64 sums
        # (half spectrum, read and written)
        k = case["samples"]
        return {"bytes": k * (2 * state * steps + state + 32 * n) + 16 * n,
                "flops": k * (ops * steps + macro + 10 * n * math.log2(max(2, n)))}
    if kind == "pdf":
        return {"bytes": state, "flops": macro + 40 * n}
    return {"bytes": 2 * (state + 8 * site_q[0][0] * case["q"]), "flops": 4 * site_q[0][0] * case["q"]}


# ---------------------------------------------------------------------------
# the method in FP64, from its definitions (Sec. 2.2-2.4), for `exact`
# ---------------------------------------------------------------------------
VEL = {
    9: ([0, 1, 0, -1, 0, 1, -1, -1, 1], [0, 0, 1, 0, -1, 1, 1, -1, -1], [0] * 9),
    27: ([0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1],
         [0, 0, 0, 1, -1, 0, 0, 1, 1, -1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, 1, -1, -1, 1, 1, -1, -1],
         [0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, 1, -1, -1, 1, 1, -1, -1, 1, 1, 1, 1, -1, -1, -1, -1]),
}
VEL[19] = tuple(c[:19] for c in VEL[27])
# powers (p_x, p_y, p_z) of the one-axis polynomials 1, c, c^2 - c_s^2 of the
# tensor modes; D2Q9 modes 3 and 4 are the sum and difference of (2, 0) and (0, 2)
MODES = {
    9: [(0, 0, 0), (1, 0, 0), (0, 1, 0), None, None, (1, 1, 0), (2, 1, 0), (1, 2, 0), (2, 2, 0)],
    27: [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (2, 0, 0), (0, 2, 0), (0, 0, 2), (1, 1, 0),
         (1, 0, 1), (0, 1, 1), (2, 1, 0), (2, 0, 1), (1, 2, 0), (1, 0, 2), (0, 1, 2), (0, 2, 1),
         (1, 1, 1), (2, 2, 0), (2, 0, 2), (0, 2, 2), (1, 1, 2), (1, 2, 1), (2, 1, 1), (2, 1, 2),
         (2, 2, 1), (1, 2, 2), (2, 2, 2)],
}
AXIS_NORM = (1.0, 1 / 3, 2 / 9)


def weights(q):
    cx, cy, cz = VEL[q]
    if q == 19:
        return [1 / 3 if i == 0 else 1 / 18 if i <= 6 else 1 / 36 for i in range(19)]
    w1 = {0: 2 / 3, 1: 1 / 6, -1: 1 / 6}
    return [w1[cx[i]] * w1[cy[i]] * (w1[cz[i]] if q == 27 else 1.0) for i in range(q)]


def _basis19(x, y, z):
    c2 = x * x + y * y + z * z
    return [x * 0 + 1, x, y, z, c2 - 1, 3 * x * x - c2, y * y - z * z, x * y, y * z, x * z,
            x * (3 * c2 - 5), y * (3 * c2 - 5), z * (3 * c2 - 5), x * (y * y - z * z),
            y * (z * z - x * x), z * (x * x - y * y), 3 * c2 * c2 - 6 * c2 + 1,
            (2 * c2 - 3) * (3 * x * x - c2), (2 * c2 - 3) * (y * y - z * z)]


def _basis19_at_velocities():
    cx, cy, cz = VEL[19]
    return np.array([_basis19(float(cx[i]), float(cy[i]), float(cz[i])) for i in range(19)]).T


def _norms(q):
    if q == 19:
        return list((_basis19_at_velocities() ** 2) @ np.array(weights(19)))
    return [4 / 9 if m is None else AXIS_NORM[m[0]] * AXIS_NORM[m[1]] * AXIS_NORM[m[2]] for m in MODES[q]]


class _Exact:
    """A flat list of boxes of one lattice (one lattice, or the replicas of
    an ensemble) stepped in FP64 torch from rest; per-box parameters as
    per-site tensors, or numbers for a single box."""

    def __init__(self, q, boxes, rates="paper"):
        self.q, self.dev = q, "cuda" if torch.cuda.is_available() else "cpu"
        self.first = 3 if q == 9 else 4
        cx, cy, cz = VEL[q]
        self.sizes = [W.n_sites(b["shape"]) for b in boxes]
        starts = np.concatenate([[0], np.cumsum(self.sizes)])
        self.n = int(starts[-1])
        dev = self.dev

        def per_site(key, dtype=torch.float64):
            v = [b[key] for b in boxes]
            if len(v) == 1:
                return torch.tensor(v, dtype=dtype, device=dev)
            return torch.repeat_interleave(torch.tensor(v, dtype=dtype, device=dev),
                                           torch.tensor(self.sizes, device=dev))

        self.rho0, self.kT = per_site("rho0"), per_site("kT")
        omega = 1.0 / per_site("tau")
        self.replica, seeds = per_site("replica", torch.int64), per_site("seed", torch.int64)
        self.key = [seeds & 0xFFFFFFFF, seeds >> 32]
        one = torch.ones(1, dtype=torch.float64, device=dev)
        at_omega = (range(q) if rates == "single" else (4, 5) if q == 9 else
                    range(4, 10) if rates == "isotropic" else (7, 8, 9))
        self.lam = [omega if v in at_omega else one for v in range(q)]
        b = _norms(q)
        self.amp = [(self.lam[v] * (2 - self.lam[v]) * b[v] / CS2 * self.kT).clamp(min=0).sqrt() for v in range(q)]
        self.site = torch.cat([torch.arange(n, device=dev) for n in self.sizes])
        self.segment = None if len(boxes) == 1 else torch.repeat_interleave(
            torch.arange(len(boxes), device=dev), torch.tensor(self.sizes, device=dev))
        # flat index of x - c_i for every population
        self.source = []
        coords = []
        for s0, box in zip(starts, boxes):
            nx, ny, nz = W.shape3(box["shape"])
            s = torch.arange(nx * ny * nz, device=dev)
            coords.append((int(s0), nx, ny, nz, s % nx, s // nx % ny, s // (nx * ny)))
        for i in range(q):
            self.source.append(torch.cat([
                s0 + (x - cx[i]) % nx + nx * ((y - cy[i]) % ny + ny * ((z - cz[i]) % nz))
                for s0, nx, ny, nz, x, y, z in coords]))
        del coords
        self.d = [torch.zeros(self.n, dtype=torch.float64, device=dev) for _ in range(q)]
        self.post = self.d
        self.step_index = 0
        if q == 19:
            self.minv = np.linalg.inv(_basis19_at_velocities())

    def macro(self):
        drho = sum(self.d)
        rho = self.rho0 + drho
        j = [sum(c[i] * self.d[i] for i in range(self.q) if c[i]) + torch.zeros_like(drho) for c in VEL[self.q]]
        return drho, rho, j, [x / rho for x in j]

    def normals(self):
        """Philox4x32-10 and Box-Muller, one normal per noisy mode."""
        def mul(a, m):
            t = a * (m & 0xFFFF)
            return ((a * (m >> 16) + (t >> 16)) >> 16), (a * m) & 0xFFFFFFFF
        count, out = self.q - self.first, []
        for blk in range((count + 3) // 4):
            c = [self.site, torch.full_like(self.site, self.step_index & 0xFFFFFFFF),
                 self.replica.expand_as(self.site), torch.full_like(self.site, blk + ((self.step_index >> 32) << 8))]
            k0, k1 = self.key
            for _ in range(10):
                (h0, l0), (h1, l1) = mul(c[0], 0xD2511F53), mul(c[2], 0xCD9E8D57)
                c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
                k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
            for a, b in ((c[0], c[1]), (c[2], c[3])):
                r = (-2 * torch.log(((a >> 8) + 1).double() * 2.0 ** -24)).sqrt()
                t = 2 * math.pi * ((b >> 8).double() * 2.0 ** -24)
                out += [r * t.cos(), r * t.sin()]
        return out[:count]

    # moments of g about u in the lattice's basis and back
    def forward(self, g, u):
        if self.q == 19:
            k = [0.0] * 19
            for i in range(19):
                p = _basis19(*[VEL[19][a][i] - u[a] for a in range(3)])
                k = [k[v] + p[v] * g[i] for v in range(19)]
            return k
        t = {(VEL[self.q][0][i], VEL[self.q][1][i], VEL[self.q][2][i]): g[i] for i in range(self.q)}
        dims = 2 if self.q == 9 else 3
        for a in range(dims):
            new = {}
            for key in {k[:a] + (0,) + k[a + 1:] for k in t}:
                gm, g0, gp = (t[key[:a] + (c,) + key[a + 1:]] for c in (-1, 0, 1))
                m0, m1, m2 = gm + g0 + gp, gp - gm, gp + gm
                val = (m0, m1 - u[a] * m0, m2 - 2 * u[a] * m1 + (u[a] * u[a] - CS2) * m0)
                for p in range(3):
                    new[key[:a] + (p,) + key[a + 1:]] = val[p]
            t = new
        if self.q == 9:
            return [t[2, 0, 0] + t[0, 2, 0] if v == 3 else t[2, 0, 0] - t[0, 2, 0] if v == 4 else t[MODES[9][v]]
                    for v in range(9)]
        return [t[m] for m in MODES[27]]

    def backward(self, k, u):
        if self.q == 19:
            def pops(x):
                return [sum(float(self.minv[i, v]) * x[v] for v in range(19)) for i in range(19)]
            x = list(k)  # T(u) M^-1 = 1 + (nilpotent by degree): x = k - (T M^-1 - 1) x
            for _ in range(5):
                y = self.forward(pops(x), u)
                x = [k[v] - (y[v] - x[v]) for v in range(19)]
            return pops(x)
        if self.q == 9:
            t = {m: k[v] for v, m in enumerate(MODES[9]) if m}
            t[2, 0, 0], t[0, 2, 0] = (k[3] + k[4]) / 2, (k[3] - k[4]) / 2
        else:
            t = dict(zip(MODES[27], k))
        dims = 2 if self.q == 9 else 3
        for a in range(dims):
            new = {}
            for key in {x[:a] + (0,) + x[a + 1:] for x in t}:
                m0, m1, m2 = (t[key[:a] + (p,) + key[a + 1:]] for p in range(3))
                r1 = m1 + u[a] * m0
                r2 = m2 + (u[a] * u[a] + CS2) * m0 + 2 * u[a] * m1
                for c, val in ((-1, (r2 - r1) / 2), (0, m0 - r2), (1, (r2 + r1) / 2)):
                    new[key[:a] + (c,) + key[a + 1:]] = val
            t = new
        return [t[c] for c in zip(*VEL[self.q])]

    def row(self, drho, rho, j, u):
        cols = [rho] + j + u + [x * x for x in u]
        if self.segment is None:
            return torch.stack([self.row0()] + [c.sum() for c in cols] + [torch.zeros((), device=self.dev)])[None]
        m = len(self.sizes)
        sums = [torch.zeros(m, dtype=torch.float64, device=self.dev).index_add_(0, self.segment, c) for c in cols]
        return torch.stack([self.row0().expand(m)] + sums + [torch.zeros(m, device=self.dev)], dim=1)

    def row0(self):
        return torch.tensor(float(self.step_index), dtype=torch.float64, device=self.dev)

    def step(self):
        q, w = self.q, weights(self.q)
        drho, rho, j, u = self.macro()
        row = self.row(drho, rho, j, u)
        k = self.forward([self.d[i] + w[i] * self.rho0 for i in range(q)], u)
        noisy = bool((self.kT > 0).any())
        eta = self.normals() if noisy else None
        ks = [k[v] * (1 - self.lam[v]) + (rho * self.lam[0] if v == 0 else 0.0)
              + (self.amp[v] * rho.sqrt() * eta[v - self.first] if noisy and v >= self.first else 0.0)
              for v in range(q)]
        del k, eta
        f = self.backward(ks, u)
        del ks
        self.post = [f[i] - w[i] * self.rho0 for i in range(q)]
        del f
        self.d = [self.post[i][self.source[i]] for i in range(q)]
        self.step_index += 1
        return row

    def set_equilibrium(self, u):
        """rho = rho0 and velocity u: f = T(u)^-1 (rho, 0, ...)."""
        u = [torch.as_tensor(x, device=self.dev) for x in u]
        zero = torch.zeros(self.n, dtype=torch.float64, device=self.dev)
        f = self.backward([zero + self.rho0] + [zero] * (self.q - 1), u)
        self.d = [f[i] - w * self.rho0 for i, w in enumerate(weights(self.q))]


def _stored(sim, case, steps):
    """The population buffer in its documented order after `steps` steps."""
    q, (nx, ny, nz) = case["q"], _shape(case)
    vel = list(zip(*VEL[q]))
    order = list(range(9)) if q == 9 else sorted(range(q), key=lambda i: vel[i][::-1])
    if not case["in_place"]:
        rows = [sim.post[i] for i in order]
    elif steps % 2 == 0:
        rows = [sim.d[i] for i in order]
    else:
        rows = [sim.post[vel.index(tuple(-c for c in vel[i]))] for i in order]
    if case["storage"] in ("f16", "bf16"):
        scale = [2.0 ** math.ceil(math.log2(math.sqrt(case["rho0"] * case["kT"] * w / CS2))) for w in weights(q)]
        rows = [r / scale[i] for r, i in zip(rows, order)]
    return torch.stack([r.view(ny * nz, nx) for r in rows], dim=1).reshape(-1)


def _shells(case, samples):
    """Shell averages of the sampled (drho, u) fields."""
    nx, ny, nz = _shape(case)
    n, nbins, dev = nx * ny * nz, case["nbins"], samples[0][0].device
    acc = 0
    for fields in samples:
        acc = acc + torch.stack([torch.fft.rfftn(f.view(nz, ny, nx)).abs() ** 2 / n for f in fields])

    def wave(m, edge):
        return 2 * math.pi * torch.where(m <= edge // 2, m, m - edge).double() / edge
    kx = 2 * math.pi * torch.arange(nx // 2 + 1, device=dev).double() / nx
    ky, kz = (wave(torch.arange(e, device=dev), e) for e in (ny, nz))
    k = (kx[None, None] ** 2 + ky[None, :, None] ** 2 + kz[:, None, None] ** 2).sqrt().reshape(-1)
    ix = torch.arange(nx // 2 + 1, device=dev)
    w = torch.where((ix == 0) | ((nx % 2 == 0) & (ix == nx // 2)), 1.0, 2.0).double()
    w = w.expand(nz, ny, nx // 2 + 1).reshape(-1).clone()
    w[0] = 0.0
    kmax = math.pi * math.sqrt(sum(e > 1 for e in (nx, ny, nz))) * (1 + 1e-12)
    b = (k / kmax * nbins).long().clamp(max=nbins - 1)

    def binned(v):
        return torch.zeros(nbins, dtype=torch.float64, device=dev).index_add_(0, b, v)
    modes = binned(w)
    div = modes.clamp(min=1)
    cols = [binned(w * k) / div, modes] + [binned(w * a.reshape(-1)) / div / len(samples) for a in acc]
    return torch.stack(cols, dim=1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "checkpoint":
        return {"f": _populations(case, seed)}
    if kind == "pdf":
        _, u = _thermal_fields(case, seed)
        c = u - u.mean(axis=1, keepdims=True)
        var = (c ** 2).mean(axis=1)
        safe = np.where(var > 0, var, 1.0)
        mom = [u.mean(axis=1), var, (c ** 3).mean(axis=1) / safe ** 1.5, (c ** 4).mean(axis=1) / safe ** 2]
        return {"moments": np.stack(mom, axis=1), "counts": None}
    if kind == "ensemble":
        reps = _manifest(case, seed)
        rows = []
        for q in (9, 27):
            part = [r for r in reps if r["q"] == q]
            if not part:
                continue
            sim = _Exact(q, part)
            rows.append(torch.stack([sim.step() for _ in range(case["steps"])], dim=1))
            w = torch.tensor(weights(q), dtype=torch.float64, device=sim.dev)[:, None]
            d = torch.stack([x[:sim.sizes[0]] for x in sim.d]) if q == 9 else None
            if q == 9:
                first = w * part[0]["rho0"] + d
            last = w * part[-1]["rho0"] + torch.stack([x[sim.n - sim.sizes[-1]:] for x in sim.d])
            del sim, d
        return {"series": torch.cat(rows), "first": first, "last": last}
    box = dict(case, shape=_shape(case), seed=seed, replica=0)
    sim = _Exact(case["q"], [box], case["rates"])
    if kind == "decay":
        sim.set_equilibrium(_vortex(case, seed))
        for _ in range(case["steps"]):
            sim.step()
        _, rho, _, u = sim.macro()
        return {"rho": rho, "u": torch.stack(u)}
    if kind == "spectrum":
        rows, samples = [], []
        for _ in range(case["samples"]):
            rows += [sim.step() for _ in range(case["steps"])]
            drho, _, _, u = sim.macro()
            samples.append([drho] + u)
        return {"shells": _shells(case, samples), "series": torch.cat(rows)}
    rows = [sim.step() for _ in range(case["steps"])]
    if kind == "couple":
        _, rho, _, u = sim.macro()
        return {"rho": rho, "u": torch.stack(u)}
    return {"series": torch.cat(rows), "state": _stored(sim, case, case["steps"])}
