"""The work a program has this library do, as cases that can be timed and compared.

Each case is a dict of plain values; its "kind" says which calls a pass makes:

  step      one emission step (gather, push, trials, photon append, recoil, move) and its
            epilogue (ledger row and photon spectrum), with a re-sort every few steps where
            the case asks for one, as a simulation in a prescribed field runs it
  noalloc   one emission step through the entry point that allocates nothing (a serving loop)
  steps     many steps of a uniform field in one launch (the paper's single-particle figures)
  pic       one step of the closed PIC loop: emission, current, field solve, photon advance
  charge    the tile sort of an ensemble and the charge density of the sorted one
  diag      what is looked at between steps: angular map, spectrum, validity flags
  train     one Adam step of the learned sampler on a fresh batch
  forward   the learned sampler's network on a long list of samples

Fields of the prescribed cases are a standing wave and the same wave half a period later,
used in turn, so that the electrons stay as energetic and as spread out as they were
however often a pass is repeated.  `exact` is the same physics in plain torch, in 64 bits.
"""
import functools
import math

import numpy as np
import torch

from paper_1409_5574_amd import _lib as L
from paper_1409_5574_amd import api

TWO_PI = 2.0 * math.pi
ALPHA = 7.2973525643e-3
HBAR_LASER = 3.0327e-6     # hbar omega / mc^2 of a 0.8 um laser
HBAR_B = 2.2656e-5         # hbar omega / mc^2 with omega = eB/m at 1e5 T
SEED = 0x5EED
YEE = ((0.5, 0.0, 0.0), (0.0, 0.5, 0.0), (0.0, 0.0, 0.5),
       (0.0, 0.5, 0.5), (0.5, 0.0, 0.5), (0.5, 0.5, 0.0))
SAMPLERS = {"S": L.SR_SAMPLER_S, "table": L.SR_SAMPLER_TABLE, "learned": L.SR_SAMPLER_MLP,
            "quantum": L.SR_SAMPLER_QUANTUM}
RECOILS = {"none": L.SR_RECOIL_NONE, "photon": L.SR_RECOIL_PHOTON, "ll": L.SR_RECOIL_LL}
BINS, EPS_LO, EPS_HI = 64, 1e-8, 1e5
N_THETA, N_PHI = 32, 64
CHI_LO, CHI_HI = -4.0, 2.0
LOG2X_FLOOR = -16.609640
DEV = "cuda"


def _step(name, dim, n, nx, ny, nz, a0, K, **more):
    c = {"name": name, "kind": "step", "dim": dim, "n": n, "nx": nx, "ny": ny, "nz": nz, "a0": a0,
         "K": K, "pp": K, "sampler": "S", "kin_cut": dim == 3, "recoil": "photon", "f64": False,
         "floor": False, "ragged": False, "cells_per_lambda": 64, "slab": 1.0, "g_lo": 10.0,
         "g_hi": 500.0, "spread": 0.3, "sort_every": 0}
    c.update(more)
    return c


def listed():
    return [
        # a few hundred test electrons in a constant field, one call a step: latency counts
        {"name": "uniform_noalloc_1000", "kind": "noalloc", "dim": 0, "n": 1000, "K": 1, "pp": 1,
         "sampler": "S", "kin_cut": False, "recoil": "photon", "g_lo": 10.0, "g_hi": 1e4},
        # the same field, all thousand steps of a run in one launch
        {"name": "uniform_steps_16k", "kind": "steps", "dim": 0, "n": 16384, "steps": 1000, "K": 1,
         "pp": 4, "sampler": "S", "kin_cut": False, "recoil": "photon", "g_lo": 10.0, "g_hi": 1e4},
        # the 2D3V workload: 2048^2 cells, a million electrons
        _step("step_2d_2048_1M", 2, 1 << 20, 2048, 2048, 1, 300.0, 1, pp=4, sort_every=10),
        # the 3D workload of the headline benchmark: 512^3 cells, 16M electrons in two
        # wavelengths of eight, eight trials, the kinematic cut
        _step("step_3d_512_16M_K8", 3, 1 << 24, 512, 512, 512, 500.0, 8, slab=0.25, sort_every=4),
        # strong fields: quantum-corrected kernel, grid-frequency floor, ragged explicit chunks
        _step("step_3d_quantum_ragged", 3, 300007, 128, 96, 81, 500.0, 4, sampler="quantum",
              floor=True, ragged=True, sort_every=10),
        # the FP64 path, the reference a precision study runs beside the FP32 one
        _step("step_3d_f64_1M", 3, 1 << 20, 192, 192, 96, 800.0, 1, f64=True, g_lo=1.0, g_hi=3e4,
              spread=0.0),
        # the learned sampler with half of its chi bins on the table
        _step("step_3d_learned_1M_K8", 3, 1 << 20, 256, 128, 128, 500.0, 8, sampler="learned",
              slab=0.5, sort_every=4),
        # the closed PIC loop on the wakefield-shaped workload
        {"name": "pic_3d_512x128x64_8M", "kind": "pic", "dim": 3, "n": 1 << 23, "nx": 512, "ny": 128,
         "nz": 64, "K": 1, "pp": 1, "sampler": "S", "kin_cut": True, "recoil": "photon",
         "cells_per_lambda": 32, "a0": 50.0, "sort_every": 10, "box": True},
        # start of a run, or a repartition: sort an ensemble and take its charge
        {"name": "charge_sorted_256_4M", "kind": "charge", "dim": 3, "n": 4000037, "nx": 256,
         "ny": 256, "nz": 256, "cells_per_lambda": 32, "drift": 1.0},
        # diagnostics of one output time
        {"name": "diagnostics_1M", "kind": "diag", "dim": 3, "n": 1 << 20, "nx": 128, "ny": 128,
         "nz": 128, "pp": 8, "mean_photons": 24.0, "a0": 500.0, "cells_per_lambda": 64,
         "g_lo": 10.0, "g_hi": 3e3},
        # one training step of the learned sampler, and its network on a list of samples
        {"name": "train_step_65536", "kind": "train", "batch": 65536},
        {"name": "forward_3M", "kind": "forward", "M": 3145801},
    ]


def draw(rng):
    def loguni(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def dims(dim, lo, hi):
        return [loguni(lo, hi) for _ in range(dim)] + [1] * (3 - dim)

    kind = rng.choice(["step"] * 5 + ["noalloc", "steps", "pic", "charge", "diag", "train", "forward"])
    if kind == "step":
        dim = rng.choice([2, 3, 3])
        nx, ny, nz = dims(dim, 64, 2048) if dim == 2 else dims(dim, 32, 256)
        K = rng.choice([1, 1, 2, 4, 8, 8, 16])
        f64 = rng.random() < 0.15
        sampler = rng.choice(["S", "S", "S", "table", "quantum"] + ([] if f64 else ["learned"]))
        ragged = rng.random() < 0.15
        c = _step("", dim, loguni(3000, 1 << 22), nx, ny, nz, rng.choice([50.0, 300.0, 500.0, 800.0]), K,
                  sampler=sampler, f64=f64, ragged=ragged,
                  kin_cut=sampler in ("learned", "quantum") or rng.random() < 0.6,
                  recoil=rng.choice(["photon", "photon", "photon", "ll", "none"]),
                  floor=sampler != "learned" and rng.random() < 0.2,
                  slab=rng.choice([1.0, 0.5, 0.25]),
                  g_hi=rng.choice([500.0, 3e3, 3e4]), spread=rng.choice([0.0, 0.3]),
                  sort_every=0 if f64 else rng.choice([4, 10]))
    elif kind in ("noalloc", "steps"):
        n = loguni(100, 65536)
        c = {"kind": kind, "dim": 0, "n": n, "K": rng.choice([1, 1, 2, 4]), "pp": 4,
             "sampler": rng.choice(["S", "S", "table", "quantum"]), "kin_cut": rng.random() < 0.3,
             "recoil": rng.choice(["photon", "ll"]), "g_lo": 10.0, "g_hi": 1e4}
        if kind == "steps":
            c["steps"] = loguni(20, 1000)
            c["kin_cut"] = c["kin_cut"] or c["sampler"] == "quantum"
    elif kind == "pic":
        dim = rng.choice([2, 3, 3])
        nx, ny, nz = dims(dim, 64, 1024) if dim == 2 else dims(dim, 32, 160)
        ppc = rng.uniform(0.5, 4.0)
        c = {"kind": kind, "dim": dim, "n": max(1000, min(1 << 23, int(ppc * nx * ny * nz))), "nx": nx,
             "ny": ny, "nz": nz, "K": 1, "pp": 1, "sampler": "S", "kin_cut": True, "recoil": "photon",
             "cells_per_lambda": 32, "a0": rng.choice([5.0, 50.0]), "sort_every": 10,
             "box": rng.random() < 0.5}
    elif kind == "charge":
        dim = rng.choice([2, 3])
        nx, ny, nz = dims(dim, 64, 2048) if dim == 2 else dims(dim, 32, 256)
        c = {"kind": kind, "dim": dim, "n": loguni(5000, 1 << 22), "nx": nx, "ny": ny, "nz": nz,
             "cells_per_lambda": 32, "drift": rng.choice([1.0, 3.0, 1e4])}
    elif kind == "diag":
        nx, ny, nz = dims(3, 32, 192)
        c = {"kind": kind, "dim": 3, "n": loguni(5000, 1 << 21), "nx": nx, "ny": ny, "nz": nz,
             "pp": rng.choice([1, 4, 8]), "mean_photons": rng.uniform(0.5, 40.0), "a0": 500.0,
             "cells_per_lambda": 64, "g_lo": 10.0, "g_hi": 3e3}
    elif kind == "train":
        c = {"kind": kind, "batch": loguni(1000, 131072)}
    else:
        c = {"kind": kind, "M": loguni(1000, 1 << 22)}
    c.pop("name", None)
    return c


# ------------------------------------------------------------------ inputs
def _dx(c):
    return TWO_PI / c["cells_per_lambda"]


def _dt(c):
    return 0.01 * TWO_PI if c["dim"] == 0 else 0.5 * _dx(c)


def _hbar(c):
    return HBAR_B if c["dim"] == 0 else HBAR_LASER


def _grid_n(c):
    return (c["nx"], c["ny"], c["nz"])


def _floor(c):
    return 64.0 * c["cells_per_lambda"] if c.get("floor") else 0.0


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _momenta(c, n, g, phase=None):
    """log10 gamma uniform on [g_lo, g_hi]; isotropic, or, where the case names a spread,
    that far off the direction of the wave's fields, which the electrons follow."""
    u = torch.rand(3, n, generator=g, device=DEV, dtype=torch.float64)
    lo, hi = math.log10(c["g_lo"]), math.log10(c["g_hi"])
    gam = 10.0 ** (lo + (hi - lo) * u[0])
    pm = (gam * gam - 1.0).clamp_min(0.0).sqrt()
    if c.get("spread"):
        d = c["spread"] * torch.randn(3, n, generator=g, device=DEV, dtype=torch.float64)
        d[1] += math.cos(phase)
        d[2] -= math.sin(phase)
        return list(pm / (d * d).sum(0).sqrt() * d)
    ct, phi = 2.0 * u[1] - 1.0, TWO_PI * u[2]
    st = (1.0 - ct * ct).clamp_min(0.0).sqrt()
    return [pm * st * phi.cos(), pm * st * phi.sin(), pm * ct]


TILE = {"step2": (64, 4, 1), "step3": (16, 4, 4), "pic2": (8, 8, 1), "pic3": (4, 4, 4)}


def _tile(c):
    return TILE[("pic" if c["kind"] == "pic" else "step") + str(c["dim"])]


def _tile_keys(c, x):
    key, mul = torch.zeros(x[0].numel(), device=DEV, dtype=torch.int64), 1
    for a in range(c["dim"]):
        n, t = _grid_n(c)[a], _tile(c)[a]
        cell = (x[a].double() / _dx(c)).floor().long().clamp(0, n - 1)
        key += cell // t * mul
        mul *= (n + t - 1) // t
    return key


def _positions(c, g, drift, slab=1.0):
    """Uniform over the box (or the middle `slab` of it along x), in tile order, and then
    moved by about `drift` cells: the particles of a run some steps after its last sort."""
    n, dim, dx = c["n"], c["dim"], _dx(c)
    box = [v * dx for v in _grid_n(c)]
    x = [torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * box[a] for a in range(dim)]
    x[0] = x[0] * slab + 0.5 * (1.0 - slab) * box[0]
    if drift < 100.0:
        order = torch.argsort(_tile_keys(c, x), stable=True)
        x = [v[order] for v in x]
        for a in range(dim):
            x[a] += drift * dx * torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    out = []
    for a in range(dim):
        v = torch.remainder(x[a], box[a]).float()
        v[v >= np.float32(box[a])] = 0.0
        out.append(v)
    return out


def _wave(c, t):
    """The standing wave at time t on the Yee points: six arrays, x fastest."""
    nx, ny, nz = _grid_n(c)
    out = []
    for q in range(6):
        x = (torch.arange(nx, device=DEV, dtype=torch.float64) + YEE[q][0]) * _dx(c)
        amp = 2.0 * c["a0"] * (torch.cos(x) if q < 3 else torch.sin(x))
        prof = amp * (0.0, math.cos(t), -math.sin(t), 0.0, -math.cos(t), math.sin(t))[q]
        out.append(prof.float().view(1, 1, nx).expand(nz, ny, nx).contiguous().view(-1))
    return out


def _pulse(c, phase):
    """A laser pulse launched along x into the plasma (E along y), six Yee arrays."""
    nx, ny, nz = _grid_n(c)
    dx, out = _dx(c), []
    box = [v * dx for v in _grid_n(c)]
    for q in range(6):
        if q not in (1, 5):
            out.append(torch.zeros(nx * ny * nz, device=DEV))
            continue
        ax = [(torch.arange(m, device=DEV, dtype=torch.float64) + o) * dx
              for m, o in zip((nx, ny, nz), YEE[q])]
        f = c["a0"] * torch.cos(ax[0] - phase) * torch.exp(-0.5 * ((ax[0] - 0.25 * box[0]) / (0.1 * box[0])) ** 2)
        fy = torch.exp(-0.5 * ((ax[1] - 0.5 * box[1]) / (0.25 * box[1])) ** 2)
        fz = torch.exp(-0.5 * ((ax[2] - 0.5 * box[2]) / (0.5 * box[2])) ** 2)
        out.append((fz.view(-1, 1, 1) * fy.view(1, -1, 1) * f.view(1, 1, -1)).float().reshape(-1))
    return out


def _network(seed):
    """FP32 parameters of a network that follows log2 x of the photon spectrum roughly:
    3 log2 u below the median, nearly flat above it, and small random weights elsewhere."""
    r = np.random.RandomState(int(seed) % (1 << 31))
    h = 64
    W1, W2, W3 = 0.3 * r.randn(h, 2), 0.02 * r.randn(h, h), 0.02 * r.randn(h, h)
    b1, b2, b3 = 0.1 * r.randn(h), 0.02 * r.randn(h), 0.02 * r.randn(h)
    W4 = 0.02 * r.randn(h)
    for W in (W2, W3):
        W[:3] = 0.0
        W[0, 0], W[0, 1], W[1, 0], W[1, 1] = 1.0, -1.0, -1.0, 1.0
    W1[0], W1[1], b1[:2], b2[:2], b3[:3] = (0.0, 16.0), (0.0, -16.0), 0.0, 0.0, 0.0
    W2[2, 0], W2[2, 1], b2[2] = 1.0, -1.0, -1.0
    W3[2, 2] = 1.0
    W4[:3] = (4.33, -4.33, -4.2)
    return np.concatenate([np.asarray(v).reshape(-1) for v in (W1, b1, W2, b2, W3, b3, W4, [-3.7])]).astype(np.float32)


FALLBACK = [0 if 7 <= b < 19 else 1 for b in range(24)]     # log10 chi in [-2.25, 0.75) on the network


def _starts(c, g):
    """Explicit chunks of uneven length (sixty particles on average, empty ones among them)."""
    cuts = torch.randint(0, c["n"] + 1, (c["n"] // 60,), generator=g, device=DEV).sort().values
    return torch.cat([cuts.new_zeros(1), cuts, cuts.new_full((1,), c["n"])])


def _inputs(c, seed):
    """Every input of a case, from the seed alone."""
    g, kind, s = _gen(seed), c["kind"], {}
    if kind in ("train", "forward"):
        if kind == "train":
            r = np.random.RandomState(int(seed) % (1 << 31))
            h = 64
            w = [r.randn(h * 2), np.zeros(h), r.randn(h * h) * (2 / h) ** 0.5, np.zeros(h),
                 r.randn(h * h) * (2 / h) ** 0.5, np.zeros(h), r.randn(h) * (1 / h) ** 0.5, np.zeros(1)]
            s["master"] = np.concatenate(w).astype(np.float32)
        else:
            s["master"] = _network(seed)
            u = torch.rand(c["M"], generator=g, device=DEV, dtype=torch.float64).clamp(1e-7, 1 - 1e-7)
            f0 = 2.0 * torch.rand(c["M"], generator=g, device=DEV, dtype=torch.float64) - 1.0
            s["feats"] = torch.stack([f0, (u / (1 - u)).log() / 16.0], 1).float().contiguous()
        return s
    n = c["n"]
    s["id"] = torch.randperm(n, generator=g, device=DEV).to(torch.int32)
    if kind in ("noalloc", "steps"):
        s["x"] = [torch.zeros(n, device=DEV) for _ in range(3)]
        s["p"] = [v.float() for v in _momenta(c, n, g)]
        s["w"] = torch.ones(n, device=DEV)
        return s
    if kind == "charge":
        s["x"] = _positions(c, g, c["drift"])
        s["p"] = [torch.randn(n, generator=g, device=DEV) * 0.05 for _ in range(3)]
        s["w"] = 0.5 + torch.rand(n, generator=g, device=DEV)
        return s
    phase = float(torch.rand(1, generator=g, device=DEV, dtype=torch.float64)) * TWO_PI
    if kind == "pic":
        s["x"] = _positions(c, g, 0.3)
        s["p"] = [torch.randn(n, generator=g, device=DEV) * 0.05 for _ in range(3)]
        vol = math.prod(v * _dx(c) for v in _grid_n(c)[:c["dim"]])
        s["w"] = torch.full((n,), 0.01 * vol / n, device=DEV)
        s["fields"] = [_pulse(c, phase)]
        return s
    # (the library sorts no FP64 set, so that one is in no order)
    s["x"] = _positions(c, g, 1e4 if c.get("f64") else 0.6, c.get("slab", 1.0))
    s["p"] = _momenta(c, n, g, phase)
    if c.get("f64"):
        s["x"] = [v.double() for v in s["x"]]
    else:
        s["p"] = [v.float() for v in s["p"]]
    s["w"] = torch.ones(n, device=DEV, dtype=torch.float64 if c.get("f64") else torch.float32)
    s["fields"] = [_wave(c, phase), _wave(c, phase + math.pi)]
    if kind == "diag":
        s["fields"] = s["fields"][:1]
        s["photons"] = _photon_inputs(c, g)
        return s
    if c["ragged"]:
        s["start"] = _starts(c, g)
    if c["sampler"] == "learned":
        s["master"] = _network(17)
    return s


def _photon_inputs(c, g):
    """A photon buffer as a step leaves it: per chunk a Poisson number of photons, energies
    log-uniform, directions around the forward axis."""
    n, pp = c["n"], c["pp"]
    nc, cap = (n + 63) // 64, n * pp
    lam = torch.full((nc,), c["mean_photons"], device=DEV)
    count = torch.poisson(lam, generator=g).to(torch.int32)
    u = torch.rand(4, cap, generator=g, device=DEV)
    ct = 1.0 - 2.0 * u[0] ** 3
    st, phi = (1.0 - ct * ct).clamp_min(0.0).sqrt(), TWO_PI * u[1]
    return {"count": count, "eps": 10.0 ** (-7.0 + 10.0 * u[2]), "w": 0.1 + u[3],
            "dir": [ct, st * phi.cos(), st * phi.sin()]}


# ------------------------------------------------------------------ a program's state
@functools.lru_cache(maxsize=None)
def _table():
    return api.Table()


def _blank(photons):
    """Unused slots hold zeros, so that a buffer can be compared whole."""
    for t in [photons.eps, photons.w, photons.parent, photons.k, photons.step] + photons.dir + photons.pos:
        if t is not None:
            t.zero_()
    return photons


def _particles(c, s):
    x = s["x"] + [None] * (3 - len(s["x"]))
    return api.Particles(x, s["p"], s["w"], s["id"])


def _fields(arrays):
    f = api.Fields(ncells=1)
    f.e, f.b = arrays[:3], arrays[3:]
    return f


def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    st = {"case": c, "i": 0, "seed": SEED + int(seed)}
    kind = c["kind"]
    if kind == "train":
        st["mlp"], st["table"] = api.Mlp(s["master"]), _table()
        return st
    if kind == "forward":
        st["mlp"], st["feats"] = api.Mlp(s["master"]), s["feats"]
        return st
    n, dim = c["n"], c["dim"]
    st["parts"] = _particles(c, s)
    if dim == 0:
        st["grid"] = api.grid_struct(0, b0=(0.0, 0.0, 1.0))
    else:
        st["grid"] = api.grid_struct(dim, n=_grid_n(c), dx=(_dx(c),) * 3)
    if kind == "charge":
        st["alt"] = st["parts"].empty_like()
        st["sort_work"] = api.sort_work(st["grid"], _tile(c), n)
        st["rho"] = torch.zeros(math.prod(_grid_n(c)), device=DEV)
        return st
    st["hist"], st["hist_work"] = torch.zeros(2 * BINS, device=DEV, dtype=torch.float64), api.hist_work(BINS)
    if kind == "diag":
        st["fields"] = _fields(s["fields"][0])
        ph = _blank(api.PhotonBuffer(n, c["pp"], dim=3))
        ph.seg_count.copy_(s["photons"]["count"])
        ph.eps.copy_(s["photons"]["eps"])
        ph.w.copy_(s["photons"]["w"])
        for a in range(3):
            ph.dir[a].copy_(s["photons"]["dir"][a])
        st["photons"] = ph
        st["angular"] = torch.zeros(N_THETA * N_PHI + 1, device=DEV, dtype=torch.float64)
        st["angular_work"] = api.angular_work(N_THETA, N_PHI)
        return st
    st["table"] = _table()
    start = s.get("start")
    st["start"] = start
    n_chunks = api.n_chunks_uniform(n) if start is None else start.numel() - 1
    st["n_chunks"] = n_chunks
    steps = c.get("steps", 1)
    st["photons"] = _blank(api.PhotonBuffer(n, c["pp"], n_chunks=n_chunks, dim=3 if dim == 0 else dim,
                                            with_step=kind == "steps"))
    mlp = None
    if c["sampler"] == "learned":
        mlp = api.Mlp(s["master"])
        mlp.kin_cut = c["kin_cut"]
        mlp.set_fallback(FALLBACK)
        st["mlp"] = mlp
    st["prm"] = api.params_struct(_hbar(c), ALPHA, c["K"], SAMPLERS[c["sampler"]], RECOILS[c["recoil"]],
                                  kin_cut=c["kin_cut"], mlp=mlp, omega_grid=_floor(c),
                                  gather=L.SR_GATHER_BOX if c.get("box") else L.SR_GATHER_DIRECT)
    if kind == "noalloc":
        st["row"] = torch.zeros(L.SR_LEDGER_COLS, device=DEV, dtype=torch.float64)
        st["status"] = torch.zeros(1, device=DEV, dtype=torch.int32)
        return st
    st["ledger"] = api.LedgerBuf(steps, n_chunks, steps_per_call=steps)
    if kind == "steps":
        return st
    st["fields"] = [_fields(f) for f in s["fields"]]
    st["alt"] = st["parts"].empty_like()
    if c["sort_every"]:
        st["sort_work"] = api.sort_work(st["grid"], _tile(c), n)
    if kind == "pic":
        cells = math.prod(_grid_n(c))
        st["x_old"] = [None if t is None else torch.empty_like(t) for t in st["parts"].x]
        st["J"] = [torch.zeros(cells, device=DEV) for _ in range(3)]
        st["status"] = torch.zeros(1, device=DEV, dtype=torch.int32)
        return st
    # the C structs of a step, built once for each of the two particle sets and fields
    st["structs"] = {(id(p), j): api.make_structs(p, f, st["photons"], st["ledger"], start)
                     for p in (st["parts"], st["alt"]) for j, f in enumerate(st["fields"])}
    return st


# ------------------------------------------------------------------ one pass
def _particle_out(parts, dim):
    return {"x": parts.x[:3 if dim != 2 else 2], "p": parts.p}


def _photon_out(ph):
    out = {"count": ph.seg_count, "eps": ph.eps, "w": ph.w, "dir": ph.dir,
           "pos": [t for t in ph.pos if t is not None], "parent": ph.parent, "k": ph.k}
    if ph.step is not None:
        out["step"] = ph.step
    return out


def _resort(st):
    c = st["case"]
    if c["sort_every"] and st["i"] % c["sort_every"] == 0:
        api.sort_particles(st["parts"], st["alt"], st["grid"], _tile(c), st["sort_work"])
        st["parts"], st["alt"] = st["alt"], st["parts"]


def _run_step(st):
    c, i, j = st["case"], st["i"], st["i"] & 1
    parts, photons, ledger = st["parts"], st["photons"], st["ledger"]
    structs = st["structs"][(id(parts), j)]
    api.gather_push_emit(parts, st["fields"][j], st["grid"], _dt(c), st["seed"], i, st["prm"], st["table"],
                         photons, ledger, None, structs=structs)
    api.step_epilogue(ledger, st["n_chunks"], 0, photons, c["n"], EPS_LO, EPS_HI, BINS, st["hist"],
                      st["hist_work"], start=st["start"], ls=structs[4])
    st["i"] = i + 1
    out = {"particles": _particle_out(parts, c["dim"]), "photons": _photon_out(photons),
           "ledger": ledger.rows, "hist": st["hist"]}
    _resort(st)     # the order inside a tile is open, so what is returned is the set before it
    return out


def _run_noalloc(st):
    c = st["case"]
    api.gather_push_emit_noalloc(st["parts"], None, st["grid"], _dt(c), st["seed"], st["i"], st["prm"],
                                 st["table"], st["photons"], st["row"], st["status"])
    st["i"] += 1
    return {"particles": _particle_out(st["parts"], 0), "photons": _photon_out(st["photons"]),
            "ledger": st["row"], "status": st["status"]}


def _run_steps(st):
    c = st["case"]
    api.gather_push_emit_steps(st["parts"], st["grid"], _dt(c), st["seed"], st["i"], c["steps"], st["prm"],
                               st["table"], st["photons"], st["ledger"])
    st["i"] += c["steps"]
    return {"particles": _particle_out(st["parts"], 0), "photons": _photon_out(st["photons"]),
            "ledger": st["ledger"].rows}


def _run_pic(st):
    c, parts, photons, ledger = st["case"], st["parts"], st["photons"], st["ledger"]
    fields, grid, dt = st["fields"][0], st["grid"], _dt(c)
    for d, s in zip(st["x_old"], parts.x):
        if d is not None:
            d.copy_(s)
    api.gather_push_emit(parts, fields, grid, dt, st["seed"], st["i"], st["prm"], st["table"], photons,
                         ledger, 0)
    for t in st["J"]:
        t.zero_()
    api.deposit_current(parts, st["x_old"], grid, dt, -1.0, st["J"], st["status"])
    api.field_step(fields, grid, dt, st["J"])
    api.photon_advance(photons, c["n"], grid, dt)
    st["i"] += 1
    out = {"particles": _particle_out(parts, c["dim"]), "photons": _photon_out(photons),
           "ledger": ledger.rows, "E": fields.e, "B": fields.b, "J": st["J"], "status": st["status"]}
    _resort(st)     # the order inside a tile is open, so what is returned is the set before it
    return out


def _run_charge(st):
    c = st["case"]
    api.sort_particles(st["parts"], st["alt"], st["grid"], _tile(c), st["sort_work"])
    st["rho"].zero_()
    api.deposit_rho(st["alt"], st["grid"], -1.0, st["rho"])
    return {"rho": st["rho"]}     # the sorted order inside a tile is open: the charge is not


def _run_diag(st):
    c, ph = st["case"], st["photons"]
    api.angular_histogram(ph, c["n"], (1.0, 0.0, 0.0), (0.0, 1.0, 0.0), N_THETA, N_PHI, st["angular"],
                          st["angular_work"])
    api.spectrum_histogram(ph, c["n"], EPS_LO, EPS_HI, BINS, st["hist"], st["hist_work"])
    flags, sums = api.validity(st["parts"], st["fields"], st["grid"], _dt(c), HBAR_LASER, ALPHA, 1.0)
    return {"angular": st["angular"], "hist": st["hist"], "flags": flags, "sums": sums}


def _run_train(st):
    mlp = st["mlp"]
    feats, target = mlp.make_batch(st["table"], st["seed"], st["i"], st["case"]["batch"])
    grads = mlp.mse_grad(feats, target)
    mlp.adam(1e-3)
    st["i"] += 1
    return {"feats": feats, "target": target, "grads": grads, "master": mlp.master, "m": mlp.m,
            "v": mlp.v, "params": mlp.params}


def _run_forward(st):
    return {"y": st["mlp"].forward(st["feats"])}


_RUN = {"step": _run_step, "noalloc": _run_noalloc, "steps": _run_steps, "pic": _run_pic,
        "charge": _run_charge, "diag": _run_diag, "train": _run_train, "forward": _run_forward}


def run(state):
    return _RUN[state["case"]["kind"]](state)


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    c, kind = case, case["kind"]
    if kind == "forward":
        return {"bytes": 12.0 * c["M"] + 17154, "flops": 2.0 * c["M"] * (2 * 64 + 2 * 4096 + 64)}
    if kind == "train":
        # features and targets written and read once, weights and moments read and written
        return {"bytes": 24.0 * c["batch"] + 36.0 * 8577, "flops": 6.0 * c["batch"] * (2 * 64 + 2 * 4096 + 64)}
    n, dim = c["n"], c["dim"]
    cells = math.prod(_grid_n(c)) if dim else 0
    real = 8.0 if c.get("f64") else 4.0
    if kind == "charge":
        return {"bytes": n * (4.0 * (dim + 5)) * 2 + n * 4.0 * (dim + 1) + 4.0 * cells, "flops": 30.0 * n}
    ppc = n / (cells * c.get("slab", 1.0)) if cells else 0.0
    grid_bytes = 24.0 * cells * c.get("slab", 1.0) * (1.0 - math.exp(-ppc * 2 ** dim)) if cells else 0.0
    if kind == "diag":
        photons = c["mean_photons"] * n / 64
        return {"bytes": 28.0 * photons + n * (28.0 + 1.0) + grid_bytes, "flops": 300.0 * n + 60.0 * photons}
    nd = 3 if dim != 2 else 2
    steps = c.get("steps", 1)
    # about one trial in twenty emits in the grid cases, one in four thousand in the uniform ones
    photons = n * c["K"] * steps * (0.05 if dim else 2.5e-4)
    b = n * (real * (2 * nd + 6 + 1) + 4.0) + grid_bytes + photons * (4.0 * (6 + nd) + 1) + 64.0 * steps
    flops = n * steps * (200.0 + 60.0 * c["K"])
    if kind == "pic":
        # positions kept (read by the current beside the new ones), J written and read, the
        # field solve's E and B read and written once, stored photons moved
        b += n * (8.0 * nd + 4.0) + cells * (24.0 + 48.0) + photons * 4.0 * 3 * nd
        flops += 400.0 * n + 60.0 * cells
    return {"bytes": b, "flops": flops}


# ------------------------------------------------------------------ the same in 64 bits
M32 = 0xFFFFFFFF


def _philox(ctr, seed):
    """Philox4x32-10 of four int64 tensors holding 32-bit words."""
    k0, k1 = seed & M32, (seed >> 32) & M32
    x, y, z, w = ctr
    for r in range(10):
        m0, m1 = x * 0xD2511F53, z * 0xCD9E8D57
        x, y, z, w = ((m1 >> 32) & M32) ^ y ^ k0, m1 & M32, ((m0 >> 32) & M32) ^ w ^ k1, m0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return x, y, z, w


def _branch():
    a = 0.69
    for _ in range(60):
        f = a ** (4 / 3) + 7 / 9 * math.exp(-a) - 1
        a -= f / (4 / 3 * a ** (1 / 3) - 7 / 9 * math.exp(-a))
    return float(np.float32(a ** (4 / 3)))


def _laplace(x, weight, h=0.2):
    """int_0^inf exp(-x cosh s) weight(s) ds by the trapezoid rule (the integrand is
    analytic in a strip, so a step of 1/5 reaches 64-bit rounding)."""
    out = torch.zeros_like(x)
    if not x.numel():
        return out
    xmin = max(float(x.min()), 1e-30)
    top = math.acosh(max(800.0 / xmin, 2.0))
    for o, v in zip(out.split(1 << 21), x.split(1 << 21)):
        s = 0.0
        while s <= top:
            o.add_(torch.mul(v, -math.cosh(s)).exp_(), alpha=weight(s) * h * (0.5 if s == 0 else 1.0))
            s += h
    return out


def _f_over_x(x):
    return _laplace(x, lambda s: math.cosh(5 * s / 3) / math.cosh(s))


N_INF = 5 * math.pi / 3


def _number_tail(x):
    return _laplace(x, lambda s: math.cosh(5 * s / 3) / math.cosh(s) ** 2)


def _cut_tail(chi):
    """1 - r(chi): the share of the photon-number spectrum above x = 2/(3 chi)."""
    xc = (2.0 / (3.0 * chi.clamp_min(1e-30))).clamp_max(1e6)
    low = xc < 700.0
    out = torch.zeros_like(chi)
    out[low] = _number_tail(xc[low]) / N_INF
    return out


def _log2_x(one_minus_U):
    """log2 of the x above which lies the share one_minus_U of the photons."""
    lo, hi = torch.full_like(one_minus_U, -80.0), torch.full_like(one_minus_U, 5.5)
    for _ in range(52):
        mid = 0.5 * (lo + hi)
        above = _number_tail(torch.exp2(mid)) > one_minus_U * N_INF
        lo, hi = torch.where(above, mid, lo), torch.where(above, hi, mid)
    return 0.5 * (lo + hi)


def _split_params(master):
    p = torch.as_tensor(master).to(DEV).to(torch.bfloat16).double()
    W1, b1, W2, b2, W3, b3, W4, b4 = p.split([128, 64, 4096, 64, 4096, 64, 64, 1])
    return [W1.view(64, 2), b1, W2.view(64, 64), b2, W3.view(64, 64), b3, W4, b4]


def _net(q, f):
    silu = torch.nn.functional.silu
    h = silu(f @ q[0].t() + q[1])
    h = silu(h @ q[2].t() + q[3])
    h = silu(h @ q[4].t() + q[5])
    return h @ q[6] + q[7]


def _gather(f, off, x, c):
    """Cloud-in-cell value of a component at the particles."""
    dim, n = c["dim"], _grid_n(c)
    idx, fr = [], []
    for a in range(dim):
        u = x[a] / _dx(c) - off[a]
        i = u.floor()
        idx.append(torch.remainder(i.long(), n[a]))
        fr.append(u - i)
    out = torch.zeros_like(x[0])
    for corner in range(1 << dim):
        w, flat, mul = 1.0, 0, 1
        for a in range(dim):
            up = (corner >> a) & 1
            w = w * (fr[a] if up else 1.0 - fr[a])
            flat = flat + torch.remainder(idx[a] + up, n[a]) * mul
            mul *= n[a]
        out += w * f[flat].double()
    return out


def _cross(a, b):
    return [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]]


def _dot(a, b):
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]


def _push(c, s, fields):
    """Boris push, H_eff and chi of every particle."""
    dt = _dt(c)
    if c["dim"] == 0:
        z = torch.zeros_like(s["p"][0])
        E, B = [z, z, z], [z, z, z + 1.0]
    else:
        f = [_gather(fields[q], YEE[q], s["x"], c) for q in range(6)]
        E, B = f[:3], f[3:]
    h, p0 = -0.5 * dt, s["p"]
    um = [p0[a] + h * E[a] for a in range(3)]
    gm = (1.0 + _dot(um, um)).sqrt()
    t = [h * B[a] / gm for a in range(3)]
    sv = [2.0 * v / (1.0 + _dot(t, t)) for v in t]
    up = [u + v for u, v in zip(um, _cross(um, t))]
    d = [v + 2.0 * h * E[a] for a, v in enumerate(_cross(up, sv))]
    pn = [p0[a] + d[a] for a in range(3)]
    pb = [p0[a] + 0.5 * d[a] for a in range(3)]
    p2 = _dot(pb, pb)
    cr = _cross(pb, d)
    g_new = (1.0 + _dot(pn, pn)).sqrt()
    gb = 0.5 * ((1.0 + _dot(p0, p0)).sqrt() + g_new)
    H = torch.where(p2 > 0, gb / dt * (_dot(cr, cr).sqrt() / p2).clamp_max(1.0), 0.0)
    return {"pn": pn, "pb": pb, "p2": p2, "gb": gb, "g_new": g_new, "H": H, "chi": _hbar(c) * H * gb}


def _trials(c, s, q, step, seed):
    """(decision, share of the weight, x) of each trial: three lists over k."""
    n, K, dt, chi = c["n"], c["K"], _dt(c), q["chi"]
    ids, zero, pa = s["id"].long() & M32, torch.zeros(n, device=DEV, dtype=torch.int64), _branch()
    eps_unit = 1.5 * chi * q["gb"]
    tail = None
    if c["sampler"] in ("table", "learned"):
        tail = _cut_tail(chi) if c["kin_cut"] else torch.zeros_like(chi)
        rate = dt * 5.0 / (2.0 * math.sqrt(3.0)) * ALPHA * q["H"] * (1.0 - tail)
        net = torch.zeros(n, device=DEV, dtype=torch.bool)
        lchi = chi.clamp_min(1e-30).log10()
        if c["sampler"] == "learned":
            b = (lchi - CHI_LO) * (24 / (CHI_HI - CHI_LO))
            fb = torch.tensor(FALLBACK, device=DEV)
            net = (b >= 0) & (b < 24) & (fb[b.clamp(0, 23).long()] == 0)
    else:
        rate = dt * math.sqrt(3.0) / TWO_PI * ALPHA * q["H"]
    emits, fracs, xs, words = [], [], [], None
    for k in range(K):
        if k % 2 == 0:
            words = _philox((ids, zero + (step & M32), zero + k // 2, zero), seed)
        wa, wb = words[2 * (k & 1)], words[2 * (k & 1) + 1]
        rp = ((wa >> 9) * 2 + 1).double() * 2.0 ** -24
        if tail is None:
            low = rp <= pa
            x = torch.where(low, rp ** 0.75, -(9.0 / 7.0 * (1.0 - rp)).log())
            S = torch.where(low, 4.0 / 3.0 * rp ** 0.25, 1.0 - rp)
            if c["sampler"] == "S":
                dn = rate * _f_over_x(x) / S
                if c["kin_cut"]:
                    dn = torch.where(1.5 * chi * x > 1.0, 0.0, dn)
            else:
                om = 1.0 - 1.5 * chi * x
                ok = om > 0.0
                xi = torch.where(ok, x / om.clamp_min(1e-300), 1e9)
                live = xi < 128.0
                Q = torch.zeros_like(x)
                z, o = xi[live], om[live]
                Q[live] = (o + 1.0 / o) * _laplace(z, lambda t: math.cosh(2 * t / 3)) - \
                    _laplace(z, lambda t: math.cosh(t / 3) / math.cosh(t))
                dn = rate * Q / S
            if _floor(c) > 0.0:
                dn = torch.where(eps_unit * x < _hbar(c) * _floor(c), 0.0, dn)
        else:
            x, dn = torch.zeros_like(rp), rate
        emit = (dn >= 1.0) | (wb.double() < (dn * 4294967296.0).floor())
        if tail is not None:
            one_minus_U = (1.0 - rp) + rp * tail
            tab = emit & ~net
            x[tab] = torch.exp2(_log2_x(one_minus_U[tab]))
            on = emit & net
            if bool(on.any()):
                f = torch.stack([(lchi[on] + 1.0) / 3.0, (rp[on] / (1.0 - rp[on])).log() / 16.0], 1)
                x[on] = torch.exp2(_net(_split_params(s["master"]), f))
            if _floor(c) > 0.0:
                emit = emit & (eps_unit * x >= _hbar(c) * _floor(c))
        emits.append(emit)
        fracs.append(torch.where(dn >= 1.0, dn, 1.0) / K)
        xs.append(x)
    return emits, fracs, xs


def _new_photons(c, n_chunks, with_step):
    cap, f = c["n"] * c["pp"], dict(device=DEV, dtype=torch.float64)
    nd = 3 if c["dim"] != 2 else 2
    ph = {"count": torch.zeros(n_chunks, device=DEV, dtype=torch.int64), "eps": torch.zeros(cap, **f),
          "w": torch.zeros(cap, **f), "dir": [torch.zeros(cap, **f) for _ in range(3)],
          "pos": [torch.zeros(cap, **f) for _ in range(nd)],
          "parent": None, "k": None}
    if with_step:
        ph["step"] = None
    return ph


def _exact_step(c, s, fields, step, seed, start, ph):
    """One emission step in place on s; photons into ph; returns the ledger row."""
    n, K, w, dt = c["n"], c["K"], s["w"], _dt(c)
    q = _push(c, s, fields)
    emits, fracs, xs = _trials(c, s, q, step, seed)
    eps_unit = 1.5 * q["chi"] * q["gb"]
    # the slots: in a chunk its rounds of 64 particles, in a round its trials, then the lanes
    i = torch.arange(n, device=DEV)
    chunk = i // 64 if start is None else torch.searchsorted(start, i, right=True) - 1
    first = chunk * 64 if start is None else start[chunk]
    begin = (i - first) % 64 == 0
    group = begin.long().cumsum(0)
    who, trial = [], []
    delta = torch.zeros_like(w)
    for k in range(K):
        at = emits[k].nonzero().squeeze(1)
        who.append(at)
        trial.append(torch.full_like(at, k))
        delta += torch.where(emits[k], fracs[k] * eps_unit * xs[k], 0.0)
    who, trial = torch.cat(who), torch.cat(trial)
    order = torch.argsort(group[who], stable=True)
    who, trial = who[order], trial[order]
    mine = chunk[who]
    count = torch.bincount(mine, minlength=ph["count"].numel())
    slot = torch.arange(who.numel(), device=DEV) - (count.cumsum(0) - count)[mine] + ph["count"][mine]
    room = torch.diff(start) * c["pp"] if start is not None else \
        (torch.arange(count.numel(), device=DEV) * 64).neg().add(n).clamp_max(64) * c["pp"]
    ph["count"] += count
    frac, x = torch.stack(fracs)[trial, who], torch.stack(xs)[trial, who]
    eps, wph = eps_unit[who] * x, w[who] * frac
    keep = slot < room[mine]
    o = first[who][keep] * c["pp"] + slot[keep]
    pbm = q["p2"].sqrt()
    ph["eps"][o], ph["w"][o] = eps[keep], wph[keep]
    for a in range(3):
        ph["dir"][a][o] = (q["pb"][a] / pbm)[who][keep]
    for a in range(len(ph["pos"])):
        ph["pos"][a][o] = s["x"][a][who][keep]
    # recoil, ledger, move
    beta2 = q["p2"] / (q["gb"] * q["gb"])
    ll = 2.0 / 3.0 * ALPHA / _hbar(c) * dt * q["chi"] ** 2
    removed = {"none": torch.zeros_like(w), "photon": delta, "ll": ll * pbm / q["gb"]}[c["recoil"]]
    pm = _dot(q["pn"], q["pn"]).sqrt()
    took = torch.minimum(removed, pm)
    scale = torch.where(pm > 0, 1.0 - took / pm.clamp_min(1e-300), 0.0)
    pn = [v * torch.where(removed > 0, scale, 1.0) for v in q["pn"]]
    after = pm - took
    g_after = torch.where(removed > 0, (1.0 + after * after).sqrt(), q["g_new"])
    row = torch.stack([(w * delta).sum(), (w * ll * beta2).sum(),
                       (-w * took * (after + pm) / (g_after + q["g_new"])).sum(),
                       (w * (removed - took)).sum(), (wph * eps)[~keep].sum(), count.sum().double(), w.sum(),
                       q["chi"].max()])
    for a in range(len(s["x"])):
        s["x"][a] = s["x"][a] + dt / g_after * pn[a]
        if c["dim"]:
            s["x"][a] = torch.remainder(s["x"][a], _grid_n(c)[a] * _dx(c))
    s["p"] = pn
    return row


def _bin_photons(c, eps, w, hist):
    u = ((eps.log2() - math.log2(EPS_LO)) * (BINS / (math.log2(EPS_HI) - math.log2(EPS_LO))))
    ok = (u >= 0) & (u < BINS)
    b = u[ok].long()
    hist[:BINS].index_add_(0, b, (w * eps)[ok])
    hist[BINS:].index_add_(0, b, w[ok])


def _doubles(s):
    d = dict(s)
    d["x"], d["p"] = [v.double() for v in s["x"]], [v.double() for v in s["p"]]
    d["w"] = s["w"].double()
    return d


def _exact_emission(c, seed):
    s, steps = _doubles(_inputs(c, seed)), c.get("steps", 1)
    start = s.get("start")
    n_chunks = (c["n"] + 63) // 64 if start is None else start.numel() - 1
    ph = _new_photons(c, n_chunks, c["kind"] == "steps")
    fields = s["fields"][0] if "fields" in s else None
    rows = torch.stack([_exact_step(c, s, fields, i, SEED + int(seed), start, ph) for i in range(steps)])
    ph["count"] = None
    out = {"particles": {"x": s["x"], "p": s["p"]}, "photons": ph,
           "ledger": rows[0] if c["kind"] == "noalloc" else rows}
    if c["kind"] == "noalloc":
        out["status"] = None
    if c["kind"] == "step":
        out["hist"] = torch.zeros(2 * BINS, device=DEV, dtype=torch.float64)
        on = ph["eps"] > 0
        _bin_photons(c, ph["eps"][on], ph["w"][on], out["hist"])
    return out


def _shape(r, k):
    return (1.0 - (r - k).abs()).clamp_min(0.0)


def _exact_current(c, x0, s):
    """Esirkepov's current of the moves x0 -> s["x"], on the Yee points."""
    dim, n, dx, dt = c["dim"], _grid_n(c), _dx(c), _dt(c)
    S0, D, node = [], [], []
    for a in range(dim):
        L_a = n[a] * dx
        d = torch.remainder(s["x"][a] - x0[a] + 0.5 * L_a, L_a) - 0.5 * L_a
        u = x0[a] / dx
        i = u.floor()
        r0, r1 = u - i, u - i + d / dx
        S0.append([_shape(r0, k) for k in (-1, 0, 1, 2)])
        D.append([_shape(r1, k) - o for k, o in zip((-1, 0, 1, 2), S0[a])])
        node.append([torch.remainder(i.long() + k, n[a]) for k in (-1, 0, 1, 2)])
    q = -1.0 * s["w"] / dx ** dim
    J = [torch.zeros(math.prod(n), device=DEV, dtype=torch.float64) for _ in range(3)]

    def add(comp, at, v):
        flat, mul = 0, 1
        for a in range(dim):
            flat, mul = flat + node[a][at[a]] * mul, mul * n[a]
        J[comp].index_add_(0, flat, v)

    def cross2(a, j, b, k):
        return S0[a][j] * S0[b][k] + 0.5 * D[a][j] * S0[b][k] + 0.5 * S0[a][j] * D[b][k] + \
            D[a][j] * D[b][k] / 3.0

    for a in range(dim):
        others = [b for b in range(dim) if b != a]
        for j in range(4):
            for k in range(4) if dim == 3 else (0,):
                t = cross2(others[0], j, others[1], k) if dim == 3 else S0[others[0]][j] + 0.5 * D[others[0]][j]
                acc = torch.zeros_like(q)
                for i in range(3):
                    acc = acc - q * dx / dt * D[a][i] * t
                    at = [0, 0, 0]
                    at[a], at[others[0]] = i, j
                    if dim == 3:
                        at[others[1]] = k
                    add(a, at, acc)
    if dim == 2:
        vz = s["p"][2] / (1.0 + _dot(s["p"], s["p"])).sqrt()
        for i in range(4):
            for j in range(4):
                add(2, [i, j], q * vz * cross2(0, i, 1, j))
    return J


def _exact_fields(c, fields, J):
    nx, ny, nz = _grid_n(c)
    dt, dx = _dt(c), _dx(c)
    f = [v.double().view(nz, ny, nx) for v in fields]
    J = [v.view(nz, ny, nx) for v in J]
    E, B = f[:3], f[3:]

    def diff(v, axis, forward):
        if axis == 2 and c["dim"] == 2:
            return torch.zeros_like(v)
        o = torch.roll(v, -1 if forward else 1, dims=2 - axis)
        return (o - v if forward else v - o) / dx

    def curl(v, forward):
        return [diff(v[2], 1, forward) - diff(v[1], 2, forward),
                diff(v[0], 2, forward) - diff(v[2], 0, forward),
                diff(v[1], 0, forward) - diff(v[0], 1, forward)]

    B = [b - 0.5 * dt * k for b, k in zip(B, curl(E, True))]
    E = [e + dt * (k - j) for e, k, j in zip(E, curl(B, False), J)]
    B = [b - 0.5 * dt * k for b, k in zip(B, curl(E, True))]
    return [v.reshape(-1) for v in E], [v.reshape(-1) for v in B]


def _exact_pic(c, seed):
    s = _doubles(_inputs(c, seed))
    ph = _new_photons(c, (c["n"] + 63) // 64, False)
    x0 = list(s["x"])
    row = _exact_step(c, s, s["fields"][0], 0, SEED + int(seed), None, ph)
    J = _exact_current(c, x0, s)
    E, B = _exact_fields(c, s["fields"][0], J)
    on = ph["eps"] > 0
    for a in range(c["dim"]):
        ph["pos"][a][on] = torch.remainder(ph["pos"][a][on] + _dt(c) * ph["dir"][a][on], _grid_n(c)[a] * _dx(c))
    ph["count"] = None
    return {"particles": {"x": s["x"], "p": s["p"]}, "photons": ph, "ledger": row.view(1, -1), "E": E,
            "B": B, "J": J, "status": None}


def _exact_charge(c, seed):
    s = _doubles(_inputs(c, seed))
    dim, n, dx = c["dim"], _grid_n(c), _dx(c)
    rho = torch.zeros(math.prod(n), device=DEV, dtype=torch.float64)
    u = [v / dx for v in s["x"]]
    for corner in range(1 << dim):
        w, flat, mul = -s["w"] / dx ** dim, 0, 1
        for a in range(dim):
            i, up = u[a].floor(), (corner >> a) & 1
            w = w * (u[a] - i if up else 1.0 - (u[a] - i))
            flat, mul = flat + torch.remainder(i.long() + up, n[a]) * mul, mul * n[a]
        rho.index_add_(0, flat, w)
    return {"rho": rho}


def _exact_diag(c, seed):
    s = _doubles(_inputs(c, seed))
    ph, n, pp = s["photons"], c["n"], c["pp"]
    at = torch.arange(n * pp, device=DEV)
    chunk = at // (64 * pp)
    on = at - chunk * 64 * pp < ph["count"][chunk]
    eps, w, d = ph["eps"][on].double(), ph["w"][on].double(), [v[on].double() for v in ph["dir"]]
    hist = torch.zeros(2 * BINS, device=DEV, dtype=torch.float64)
    _bin_photons(c, eps, w, hist)
    theta, phi = d[0].clamp(-1, 1).acos(), torch.remainder(torch.atan2(d[2], d[1]), TWO_PI)
    b = (theta * (2 * N_THETA / math.pi)).long().clamp_max(N_THETA - 1) * N_PHI + \
        (phi * (N_PHI / TWO_PI)).long().clamp_max(N_PHI - 1)
    b = torch.where(d[0] > 0, b, N_THETA * N_PHI)
    angular = torch.zeros(N_THETA * N_PHI + 1, device=DEV, dtype=torch.float64).index_add_(0, b, eps * w)
    q = _push(c, s, s["fields"][0])
    quantum, wiggle = q["chi"] >= 1.0, (q["H"] > 0) & (q["H"] <= 1.0)
    ll = s["w"] * 2.0 / 3.0 * ALPHA / HBAR_LASER * _dt(c) * q["chi"] ** 2 * q["p2"] / q["gb"] ** 2
    sums = torch.stack([v.sum() for v in (s["w"], s["w"][quantum], s["w"][wiggle], ll, ll[quantum], ll[wiggle])])
    return {"angular": angular, "hist": hist, "flags": None, "sums": sums}


def _exact_train(c, seed):
    master = torch.from_numpy(_inputs(c, seed)["master"]).to(DEV).double()
    M = c["batch"]
    i = torch.arange(M, device=DEV)
    zero = torch.zeros_like(i)
    w = _philox((i, zero, zero, zero + 3), SEED + int(seed))
    lchi = CHI_LO + (CHI_HI - CHI_LO) * (w[0] >> 8).double() * 2.0 ** -24
    u = ((w[1] >> 9) * 2 + 1).double() * 2.0 ** -24
    target = _log2_x((1.0 - u) + u * _cut_tail(10.0 ** lchi)).clamp_min(LOG2X_FLOOR)
    feats = torch.stack([(lchi + 1.0) / 3.0, (u / (1.0 - u)).log() / 16.0], 1)
    params = [v.clone().requires_grad_(True) for v in _split_params(master.float())]
    weight = torch.exp2(target) * (15.0 * math.sqrt(3.0) / 8.0)
    loss = (weight * (_net(params, feats) - target) ** 2).mean()
    g = torch.cat([v.reshape(-1) for v in torch.autograd.grad(loss, params)])
    m, v = 0.1 * g, 0.001 * g * g
    master = master - 1e-3 * (m / 0.1) / ((v / 0.001).sqrt() + 1e-8)
    return {"feats": feats, "target": target, "grads": g, "master": master, "m": m, "v": v, "params": master}


def _exact_forward(c, seed):
    s = _inputs(c, seed)
    q = _split_params(s["master"])
    return {"y": torch.cat([_net(q, f.double()) for f in s["feats"].split(1 << 18)])}


def exact(case, seed):
    kind = case["kind"]
    f = {"step": _exact_emission, "noalloc": _exact_emission, "steps": _exact_emission, "pic": _exact_pic,
         "charge": _exact_charge, "diag": _exact_diag, "train": _exact_train, "forward": _exact_forward}
    return f[kind](case, seed)
