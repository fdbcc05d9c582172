"""Speed cases of the dose engine: the calls a planning or research program makes, from a two-thousand-history probe to a
256-beamlet plan, each through the public binding (``paper_1101_1245_amd.gpumcd``).

A case is a dict of plain values; ``prepare`` makes what a program holds before the call (context, tables, phantom, beams),
``run`` is one call, ``work`` the bytes and operations the call cannot do without.  Histories draw from counter-based
streams and deposits are integer sums, so a case's outputs are the same bits on every run: doses, uncertainties, and the
counts of events, steps and secondaries.
"""
import math

import numpy as np
import torch

from paper_1101_1245_amd import gpumcd as G
from paper_1101_1245_amd import inputs as I

LSB = 1.0 / 134217728.0          # MeV per energy unit of the integer tallies
J_PER_MEV = 1.602176634e-13
COUNTS = ("n_photon_events", "n_photon_interactions", "n_e_steps", "n_hard", "n_secondaries", "s_rel")

# One context and one server serve a whole program, as its handle does.
_held = {}


def _context():
    if "ctx" not in _held:
        _held["ctx"] = G.Context(0)
    return _held["ctx"]


def _server():
    if "srv" not in _held:
        c = G.Context(0)
        c.server_start(max_slots=4)
        _held["srv"] = c
    return _held["srv"]


class _Loaded:
    """Tables and phantom ids on a context, released with the state that holds them."""

    def __init__(self, ctx, materials, physics, phantoms):
        self.ctx = ctx
        self.tid = ctx.load_tables(materials, physics)
        self.pids = [ctx.load_phantom(p) for p in phantoms]
        self.pid = self.pids[0]

    def __del__(self):
        try:
            for h in self.pids + [self.tid]:
                self.ctx.release(h)
        except Exception:
            pass


# ------------------------------------------------------------------ cases
def listed():
    return [
        # a first look at a beam on a small ragged grid: launches and host round trips, hardly any transport
        {"name": "probe_electron_2e3", "kind": "plain", "phantom": "ellipsoids", "nx": 33, "ny": 29, "nz": 17, "voxel": 0.5,
         "particle": 1, "spectrum": "mono", "e": 12.0, "field": 3.0, "n": 2000, "ecut": 0.7, "out": "numpy"},
        # the smallest set-up of the tests: a 1 MeV pencil of photons in water, low cutoffs, results on the host
        {"name": "photon_1MeV_water32_1e5", "kind": "plain", "phantom": "water", "nx": 32, "ny": 32, "nz": 32, "voxel": 0.5,
         "particle": 0, "spectrum": "mono", "e": 1.0, "field": 0.5, "n": 100_000, "ecut": 0.2, "out": "numpy"},
        # Table IV of the paper: 1e6 electrons of 15 MeV on 64^3 water
        {"name": "electron_15MeV_water64_1e6", "kind": "plain", "phantom": "water", "nx": 64, "ny": 64, "nz": 64,
         "voxel": 0.5, "particle": 1, "spectrum": "mono", "e": 15.0, "field": 10.0, "n": 1_000_000, "ecut": 0.7,
         "out": "torch"},
        # the second geometry of the paper: 4e6 photons on water with a lung box (two materials)
        {"name": "photon_15MeV_lungbox64_4e6", "kind": "plain", "phantom": "lungbox", "nx": 64, "ny": 64, "nz": 64,
         "voxel": 0.5, "particle": 0, "spectrum": "mono", "e": 15.0, "field": 10.0, "n": 4_000_000, "ecut": 0.7,
         "out": "torch"},
        # one shard of a run split over GPUs: raw integer batch tallies of a history range, three materials
        {"name": "electron_slabs64_shard_1e6", "kind": "shard", "phantom": "tissue_lung_bone", "nx": 64, "ny": 64, "nz": 64,
         "voxel": 0.5, "particle": 1, "spectrum": "mono", "e": 15.0, "field": 10.0, "n": 1_000_000, "ecut": 0.7,
         "first": 3_000_001},
        # the benchmark's workload: the electron and the photon beam, each at 1% uncertainty, in one batched job
        {"name": "water64_both_beams_1pct", "kind": "pair", "phantom": "water", "nx": 64, "ny": 64, "nz": 64, "voxel": 0.5,
         "e": 15.0, "field": 10.0, "n_e": 5_250_000, "n_g": 65_000_000, "ecut": 0.7},
        # a linac spectrum on the largest grid of the request stream: clearing and finalizing 4.3 GB of tallies counts
        {"name": "photon_tri_256cube_1e6", "kind": "plain", "phantom": "ellipsoids", "nx": 256, "ny": 256, "nz": 256,
         "voxel": 0.3, "particle": 0, "spectrum": "triangular", "e": 10.0, "field": 7.0, "n": 1_000_000, "ecut": 0.7,
         "out": "torch"},
        # the heterogeneous slab phantom: 4e7 photons of 6 MeV on 128^3, three materials
        {"name": "photon_6MeV_slabs128_4e7", "kind": "plain", "phantom": "slabs", "nx": 128, "ny": 128, "nz": 128,
         "voxel": 0.25, "particle": 0, "spectrum": "mono", "e": 6.0, "field": 10.0, "n": 40_000_000, "ecut": 0.7,
         "out": "torch"},
        # a treatment plan: 256 pencil beamlets with the dose of each, four materials
        {"name": "beamlets_256_per_beam", "kind": "beamlets", "nx": 200, "ny": 200, "nz": 160, "voxel": 0.25, "beams": 256,
         "lo": 4.0, "hi": 6.0, "ecut": 0.7, "sigma_per_beam": False},
        # a small plan on a ragged grid, with the uncertainty of each beam too (a batched tally per beam)
        {"name": "beamlets_16_sigma_ragged", "kind": "beamlets", "nx": 101, "ny": 96, "nz": 83, "voxel": 0.3, "beams": 16,
         "lo": 4.0, "hi": 5.0, "ecut": 0.7, "sigma_per_beam": True},
        # dose requests submitted together to the server: mixed grids, spectra, fields and history counts
        {"name": "served_24_requests", "kind": "served", "requests": 24, "pool": 4, "g_lo": 32, "g_hi": 160, "lo": 4.0,
         "hi": 6.7},
        # the shards of a run added up: batch tallies already on the GPU to dose, sigma and s
        {"name": "finalize_128cube_32_batches", "kind": "finalize", "nx": 128, "ny": 128, "nz": 128, "voxel": 0.25,
         "batches": 32, "n": 40_000_000, "first": 1_000_003},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _grid(rng, lo, hi):
    n = _log(rng, lo, hi)
    return {k: max(lo, min(hi, int(round(n * rng.uniform(0.8, 1.25))))) for k in ("nx", "ny", "nz")}


def draw(rng):
    kind = rng.choice(["plain"] * 8 + ["shard", "pair", "pair", "beamlets", "beamlets", "served", "finalize", "finalize"])
    if kind == "finalize":
        c = {"kind": kind, **_grid(rng, 17, 128), "batches": rng.choice([1, 4, 10, 16, 32, 32, 32, 40])}
        return {**c, "voxel": rng.uniform(0.2, 0.5), "n": int(_log(rng, 1e4, 1e8)), "first": rng.choice([0, rng.randrange(1 << 20)])}
    if kind == "served":
        return {"kind": kind, "requests": rng.randint(2, 24), "pool": rng.randint(1, 4), "g_lo": 32,
                "g_hi": int(_log(rng, 40, 160)), "lo": 4.0, "hi": rng.uniform(5.0, 6.7)}
    if kind == "beamlets":
        return {"kind": kind, **_grid(rng, 40, 128), "voxel": rng.uniform(0.25, 0.4), "beams": int(_log(rng, 4, 65)), "lo": 4.0,
                "hi": rng.uniform(4.5, 5.7), "ecut": 0.7, "sigma_per_beam": rng.random() < 0.5}
    c = {"kind": kind, "phantom": rng.choice(["water", "ellipsoids", "ellipsoids", "slabs"]), **_grid(rng, 17, 200),
         "voxel": rng.uniform(0.25, 0.5), "e": rng.uniform(1.0, 20.0), "field": rng.uniform(0.5, 10.0),
         "ecut": rng.choice([0.7, 0.7, 0.7, 0.2, 0.189])}
    if kind == "pair":
        n = _log(rng, 2e4, 2e7)
        return {**c, "n_e": int(n * rng.uniform(0.05, 0.3)), "n_g": int(n)}
    c["particle"] = 1 if rng.random() < 0.4 else 0
    c["n"] = int(_log(rng, 2e3, 1.5e7 if c["particle"] == 0 else 4e6))
    c["spectrum"] = rng.choice(["mono", "mono", "triangular", "tabulated"])
    if kind == "shard":
        return {**c, "first": rng.randrange(1 << 24)}
    return {**c, "out": rng.choice(["numpy", "torch"])}


# ------------------------------------------------------------------ inputs
def _phantom(c, seed):
    """(materials, phantom) of a case."""
    n, h = (c["nx"], c["ny"], c["nz"]), c["voxel"]
    kind = c["phantom"]
    if kind == "water":
        return (I.WATER,), I.homogeneous(n, h, 0)
    if kind == "lungbox":
        w = I.lung_box(c["particle"])
        return w.materials, w.phantom
    if kind == "tissue_lung_bone":
        w = I.tissue_lung_bone(c["particle"])
        return w.materials, w.phantom
    if kind == "slabs":
        z = n[2] * h   # the slab phantom's proportions: 3, 2 and 7 of 32 cm, then water
        return (I.WATER, I.BONE, I.LUNG), I.z_slabs(n, h, [(z * 3 / 32, 0, 1.0), (z * 5 / 32, 1, 1.85),
                                                           (z * 12 / 32, 2, 0.26), (z, 0, 1.0)])
    return I.DEFAULT_MATERIALS, I.ellipsoids(n, h, seed=seed)


def _source(c, particle, seed, beam_id=0):
    s = I.Source(particle, I.MONO, c["e"], wx=c["field"], wy=c["field"], beam_id=beam_id,
                 first_history=c.get("first", 0))
    if c.get("spectrum") == "triangular":
        s.spectrum, s.e_lo, s.e_mode, s.e_hi = I.TRIANGULAR, 0.2 * c["e"], c["e"], min(1.8 * c["e"], 30.0)
    elif c.get("spectrum") == "tabulated":
        edges = np.linspace(0.05 * c["e"], 1.2 * c["e"], 25)
        mid = 0.5 * (edges[1:] + edges[:-1])
        s.spectrum, s.tab_e = I.TABULATED, edges
        s.tab_w = (1.0 - np.exp(-4.0 * mid / c["e"])) * np.exp(-2.0 * mid / c["e"]) \
            * np.random.default_rng(seed).uniform(0.9, 1.1, mid.size)
    return s


def _tally(c, seed):
    """Integer batch tallies [K, nz, ny, nx] as a broad beam leaves them: a lit column with statistical spread over
    the batches, scatter around it, most voxels outside untouched."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    K, nz, ny, nx = c["batches"], c["nz"], c["ny"], c["nx"]
    ax = lambda n: (torch.arange(n, device="cuda", dtype=torch.float32) + 0.5) / n - 0.5   # noqa: E731
    lit = torch.exp(-40.0 * (ax(ny)[:, None] ** 2 + ax(nx)[None, :] ** 2))[None] \
        * torch.exp(-1.5 * (ax(nz) + 0.5))[:, None, None]
    mean = lit * (float(c["n"]) / K * 2.0 ** 20)
    t = torch.empty((K, nz, ny, nx), dtype=torch.int64, device="cuda")
    for k in range(K):
        t[k] = (mean * (1.0 + 0.1 * torch.randn((nz, ny, nx), generator=g, device="cuda")).clamp_(min=0.0)).to(torch.int64)
    t[:, lit < 1e-4] = 0
    return t


def _finalize_phantom(c, seed):
    return I.ellipsoids((c["nx"], c["ny"], c["nz"]), c["voxel"], seed=seed)


def prepare(case, seed):
    c = case
    if c["kind"] == "finalize":
        ld = _Loaded(_context(), I.DEFAULT_MATERIALS, I.Physics(ecut=0.7, n_batches=c["batches"]), [_finalize_phantom(c, seed)])
        t = _tally(c, seed)
        d = torch.empty(t.shape[1:], dtype=torch.float64, device="cuda")
        return {"c": c, "ld": ld, "tally": t, "dose": d, "sigma": torch.empty_like(d)}
    if c["kind"] == "served":
        # the request stream's beams on a pool of cubic grids from g_lo to g_hi, counts spread evenly over the decades
        rng, nr, npool = np.random.default_rng(seed), c["requests"], c["pool"]
        grids = [int(round(g)) for g in np.linspace(c["g_lo"], c["g_hi"], npool)]
        pool = [I.ellipsoids(g, 0.25 + 0.25 * (i + 1) / (npool + 1), seed=seed + i) for i, g in enumerate(grids)]
        counts = rng.permutation(np.round(10.0 ** np.linspace(c["lo"], c["hi"], nr)).astype(np.int64))
        reqs = []
        for j in range(nr):
            side = float(rng.uniform(1.0, 10.0))
            src = I.Source(I.ELECTRON if j % 4 == 3 else I.PHOTON, I.MONO, float(rng.uniform(1.0, 20.0)), wx=side, wy=side,
                           beam_id=j)
            if j % 2:
                src.spectrum, src.e, src.e_lo, src.e_mode, src.e_hi = I.TRIANGULAR, 10.0, 2.0, 10.0, 18.0
            reqs.append(I.DoseRequest((7 * j) % npool, I.centred(pool[(7 * j) % npool], src), int(counts[j]), seed + j))
        return {"c": c, "ld": _Loaded(_server(), I.DEFAULT_MATERIALS, I.serving_physics(), pool), "reqs": reqs}
    if c["kind"] == "beamlets":
        ph = I.ellipsoids((c["nx"], c["ny"], c["nz"]), c["voxel"], seed=seed)
        # the plan's beamlets: a square grid of pencils over the middle of the entry face, counts spread evenly over the decades
        rng, nb = np.random.default_rng(seed), c["beams"]
        side = int(math.ceil(math.sqrt(nb)))
        ex, ey, _z = ph.extent
        pitch = min(1.0, 0.9 * min(ex, ey) / side)
        kinds = rng.permutation([I.PHOTON] * (nb - nb // 4) + [I.ELECTRON] * (nb // 4))
        counts = rng.permutation(np.round(10.0 ** np.linspace(c["lo"], c["hi"], nb)).astype(np.int64))
        energy = rng.permutation(np.linspace(1.0, 20.0, nb))
        srcs = [I.Source(int(kinds[i]), I.MONO, float(energy[i]), cx=ex / 2 + (i % side - (side - 1) / 2) * pitch,
                         cy=ey / 2 + (i // side - (side - 1) / 2) * pitch, wx=0.5, wy=0.5, beam_id=i) for i in range(nb)]
        ld = _Loaded(_context(), I.DEFAULT_MATERIALS, I.Physics(ecut=c["ecut"], pcut=0.01), [ph])
        return {"c": c, "ld": ld, "srcs": srcs, "counts": [int(n) for n in counts], "seed": seed}
    mats, ph = _phantom(c, seed)
    ld = _Loaded(_context(), mats, I.Physics(ecut=c["ecut"], pcut=0.01), [ph])
    if c["kind"] == "pair":
        srcs = [I.centred(ph, _source(c, I.ELECTRON, seed, 0)), I.centred(ph, _source(c, I.PHOTON, seed, 1))]
        return {"c": c, "ld": ld, "srcs": srcs, "counts": [c["n_e"], c["n_g"]], "seed": seed}
    return {"c": c, "ld": ld, "src": I.centred(ph, _source(c, c["particle"], seed)), "seed": seed}


def run(state):
    c, ld = state["c"], state["ld"]
    ctx = ld.ctx
    if c["kind"] == "finalize":
        s = ctx.finalize_tally_noalloc(ld.pid, ld.tid, state["tally"], c["first"], c["first"] + c["n"], state["dose"],
                                       state["sigma"])
        return {"dose": state["dose"], "sigma": state["sigma"], "s": s}
    if c["kind"] == "served":
        tickets = [ctx.submit(ld.pids[r.phantom], ld.tid, r.source, r.n_hist, r.seed) for r in state["reqs"]]
        done = [ctx.poll(t, wait=True, out="torch") for t in tickets]
        return [{"dose": d, "sigma": s} for _, d, s, _ in done]
    if c["kind"] == "shard":
        t, st = ctx.run_beam_tally(ld.pid, ld.tid, state["src"], c["n"], state["seed"], out="torch")
        return {"tally": t, **{k: st[k] for k in COUNTS if k != "s_rel"}}
    if c["kind"] in ("pair", "beamlets"):
        # the default settings ({}): a null tuning would run the search first
        pb, ps, d, s, st = ctx.run_beams(ld.pid, ld.tid, state["srcs"], state["counts"], state["seed"], tuning={},
                                         per_beam=c["kind"] == "beamlets", per_beam_sigma=c.get("sigma_per_beam", False),
                                         out="torch")
        out = {"dose": d, "sigma": s, **{k: st[k] for k in COUNTS}}
        if pb is not None:
            out["per_beam"] = pb
        if ps is not None:
            out["per_beam_sigma"] = ps
        return out
    d, s, st = ctx.run_beam(ld.pid, ld.tid, state["src"], c["n"], state["seed"], out=c["out"])
    return {"dose": d, "sigma": s, **{k: st[k] for k in COUNTS}}


# ------------------------------------------------------------------ work and reference
def _flops(particle, e, n, voxel, depth, ecut):
    """Operations of n histories: about 400 for one condensed step, 1.7 steps per voxel of an electron's path (2 MeV lost
    per cm) and a few hard events; about 175 for a photon's flight and 500 for an interaction, the attenuation being
    0.02 to 0.07 per cm, and half of the energy of an interaction given to electrons."""
    steps = lambda t: 400.0 * (1.7 * max(t - ecut, 0.0) / 2.0 / voxel + 2.0)   # noqa: E731
    if particle == I.ELECTRON:
        return n * (steps(e) + 0.5 * 175.0)
    hits = depth * max(0.02, 0.07 / math.sqrt(e))
    hits = (1.0 - math.exp(-hits)) * 2.0
    return n * ((hits + 1.0) * 175.0 + hits * (500.0 + steps(0.5 * e)))


def work(case):
    c = case
    if c["kind"] == "finalize":
        nv = c["nx"] * c["ny"] * c["nz"]
        return {"bytes": nv * (8.0 * c["batches"] + 8.0 + 16.0), "flops": nv * (5.0 * c["batches"] + 10.0)}
    if c["kind"] == "served":
        n = c["requests"] * (10.0 ** c["hi"] - 10.0 ** c["lo"]) / math.log(10.0) / (c["hi"] - c["lo"])
        g, e, voxel = 0.5 * (c["g_lo"] + c["g_hi"]), 10.0, 0.375
        fl = sum(w * _flops(p, e, n, voxel, g * voxel, 0.7) for p, w in ((I.PHOTON, 0.75), (I.ELECTRON, 0.25)))
        return {"bytes": (c["requests"] * 16.0 + c["pool"] * 8.0) * g ** 3, "flops": fl}
    nv = c["nx"] * c["ny"] * c["nz"]
    depth = c["nz"] * c["voxel"]
    if c["kind"] == "beamlets":
        n = c["beams"] * (10.0 ** c["hi"] - 10.0 ** c["lo"]) / math.log(10.0) / (c["hi"] - c["lo"])
        fl = sum(w * _flops(p, 10.5, n, c["voxel"], depth, c["ecut"]) for p, w in ((I.PHOTON, 0.75), (I.ELECTRON, 0.25)))
        per = 8.0 * c["beams"] * (2.0 if c["sigma_per_beam"] else 1.0)
        return {"bytes": nv * (8.0 + 16.0 + per), "flops": fl}
    if c["kind"] == "pair":
        fl = _flops(I.ELECTRON, c["e"], c["n_e"], c["voxel"], depth, c["ecut"]) \
            + _flops(I.PHOTON, c["e"], c["n_g"], c["voxel"], depth, c["ecut"])
        return {"bytes": nv * 24.0, "flops": fl}
    fl = _flops(c["particle"], c["e"], c["n"], c["voxel"], depth, c["ecut"])
    out = 32 * 8.0 if c["kind"] == "shard" else 16.0
    return {"bytes": nv * (8.0 + out), "flops": fl}


def exact(case, seed):
    """The finalize in double precision: D = sum_k T_k / N, sigma^2 = sum_k (T_k - n_k D)^2 / (N^2 (K - 1) / K), in Gy per
    history, and s, the mean of sigma / D over the voxels above a fifth of the largest dose.  Transport itself has no
    closed form: its outputs are fixed by the streams."""
    c = case
    if c["kind"] != "finalize":
        return None
    K, n, h0 = c["batches"], c["n"], c["first"]
    t = _tally(c, seed).double()
    rho = torch.from_numpy(_finalize_phantom(c, seed).rho).cuda().double()
    conv = LSB * J_PER_MEV / (c["voxel"] ** 3 * 1e-3) / rho
    m = t.sum(0) / n
    acc = torch.zeros_like(m)
    for k in range(K):
        nk = (h0 + n + K - 1 - k) // K - (h0 + K - 1 - k) // K
        acc += (t[k] - nk * m) ** 2
    dose = m * conv
    sigma = torch.sqrt(acc / (float(n) ** 2 * (K - 1) / K)) * conv if K > 1 else torch.zeros_like(m)
    hot = dose > 0.2 * dose.max()
    s = float((sigma[hot] / dose[hot]).mean()) if bool(hot.any()) else float("nan")
    return {"dose": dose, "sigma": sigma, "s": s}
