"""The work users have this package do, as cases that a timing program can run.

A case is a dict of plain values.  Kinds:

  step    new positions in, accelerations out: ShortRange.build + forward, the
          call of every time step (prefill of a plan and its evaluation)
  grad    the same, then ShortRange.adjoint: gradients with respect to
          positions and masses of sum_i w_i . a_i
  batch   several independent boxes in one plan: ShortRange.build_batch + forward
  mesh    the long-range mesh force of the split: Context.long_range
  sim     one kick-drift-kick step of Simulation (short range, mesh, kicks, drift)

Particles: ``n_side``^3 of them in a periodic box of side 100 with the force
split of the package's workloads (N_PM = n_side, r_s = 1.2 mesh cells, r_cut =
4.5 r_s), uniform or a Zel'dovich grid with a part of the particles in Plummer
halos (the recipe of ``inputs.py``, drawn on the GPU).  A program that chose
the float32 pair forms holds its particles in float32 and takes the
accelerations and gradients back in that type, as ShortRangeForce gives them;
the float64 forms take and give float64.
"""

from __future__ import annotations

import math
import random

import torch

from paper_2107_14008_amd import api
from paper_2107_14008_amd import binding as B

BOX = 100.0

# pair forms: name -> evaluation parameters (float32 r^2 table: the headline
# form of bench.py; the Taylor tables: the paper's; exact: the default)
FORMS = {
    "fp32_r2": dict(precision="fp32", trunc="r2", table_size=64, table_level=2),
    "fp32_table": dict(precision="fp32", trunc="table", table_size=512, table_level=2),
    "fp32_exact": dict(precision="fp32", trunc="exact"),
    "fp64_r2": dict(precision="fp64", trunc="r2", table_size=64, table_level=6),
    "fp64_table": dict(precision="fp64", trunc="table", table_size=2048, table_level=4),
    "fp64_exact": dict(precision="fp64", trunc="exact"),
}

# beyond this many particles the pair-by-pair reference takes too long
MOST_EXACT = 4_500_000


def _case(name, kind, n_side, form="", **kw):
    c = dict(kind=kind, n_side=n_side, form=form, clustered=True, halo_frac=0.2, max_leaf=64,
             order=-1, theta=0.0)
    if name:
        c["name"] = name
    c.update(kw)
    return c


FAR = dict(order=4, theta=0.25)


def listed():
    return [
        # the smallest box of a batch run on its own (4,096 particles, all of
        # it launches and round trips)
        _case("clustered16_fp32", "step", 16, "fp32_r2", **FAR),
        # a small uniform box in the default form, every pair summed
        _case("uniform32_fp64", "step", 32, "fp64_exact", clustered=False, max_leaf=32),
        # the workload of bench.py, in its headline form ...
        _case("clustered128_fp32", "step", 128, "fp32_r2", **FAR),
        # ... and in plain float64, the run that checks the float32 one
        _case("clustered128_fp64", "step", 128, "fp64_exact", **FAR),
        # an ordinary float64 production run; a size whose leaves are ragged
        _case("clustered100_fp64_r2", "step", 100, "fp64_r2", **FAR),
        # the paper's own single-precision form
        _case("clustered90_fp32_table", "step", 90, "fp32_table", **FAR),
        # the largest box of bench.py
        _case("clustered256_fp32", "step", 256, "fp32_r2", halo_frac=0.3, **FAR),
        # an ensemble of uneven boxes in one launch
        _case("batch24_fp32", "batch", 96, "fp32_r2", n_box=24, low_side=16, sides=7),
        # field-level inference: force and gradient per step, float32
        _case("grad64_fp32", "grad", 64, "fp32_r2"),
        # the gradient of the full expansion in float64 (checks, small fits)
        _case("grad40_fp64_far", "grad", 40, "fp64_exact", **FAR),
        # the other half of the split at the headline size
        _case("mesh128", "mesh", 128, n_pm=128),
        # a float64 time step of a whole simulation, ragged leaves
        _case("sim48_fp64", "sim", 48, "fp64_exact", n_pm=48, **FAR),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "grad", "batch", "mesh", "sim"])
    far = rng.choice([FAR, FAR, dict(order=-1, theta=0.0)])
    if kind == "step":
        form = rng.choice(sorted(FORMS) + ["fp32_r2", "fp32_r2"])
        hi = 200 if form == "fp32_r2" else 150 if form != "fp64_exact" else 128
        return _case("", kind, _log_int(rng, 12, hi), form, clustered=rng.random() < 0.8,
                     halo_frac=round(rng.uniform(0.1, 0.3), 3),
                     max_leaf=rng.choice([32, 48, 64, 64, 64]), **far)
    if kind == "grad":
        form = rng.choice(["fp32_r2", "fp32_r2", "fp32_exact", "fp64_exact"])
        return _case("", kind, _log_int(rng, 12, 96 if form == "fp32_r2" else 64), form, **far)
    if kind == "batch":
        return _case("", kind, _log_int(rng, 24, 96), rng.choice(["fp32_r2", "fp64_r2"]),
                     n_box=rng.randint(2, 32), low_side=rng.randint(12, 24),
                     sides=rng.randrange(1 << 16))
    n = _log_int(rng, 12, 160 if kind == "mesh" else 96)
    n_pm = max(8, 2 * int(round(n * rng.choice([0.25, 0.5, 0.5]))))
    if kind == "mesh":
        return _case("", kind, n, n_pm=n_pm, clustered=rng.random() < 0.8)
    return _case("", kind, n, rng.choice(["fp64_exact", "fp64_r2"]), n_pm=n_pm, **far)


# ------------------------------------------------------------------ inputs

def _split(n_side):
    r_s = 1.2 * BOX / n_side
    return r_s, 4.5 * r_s


def _wrap(x):
    x = torch.remainder(x, BOX)
    return torch.where(x >= BOX, torch.zeros_like(x), x)


def _positions(n_side, clustered, halo_frac, gen):
    dev, f64 = "cuda", torch.float64
    n = n_side ** 3
    if not clustered:
        return torch.rand((n, 3), generator=gen, device=dev, dtype=f64) * BOX
    # Zel'dovich grid, density contrast ~ k^-1, displacements of 0.5 spacings rms
    wk = torch.fft.rfftn(torch.randn((n_side,) * 3, generator=gen, device=dev, dtype=f64))
    f = torch.fft.fftfreq(n_side, 1.0 / n_side, device=dev, dtype=f64)
    fz = torch.fft.rfftfreq(n_side, 1.0 / n_side, device=dev, dtype=f64)
    k = (f[:, None, None], f[None, :, None], fz[None, None, :])
    k2 = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    zero = k2 == 0
    if n_side % 2 == 0:
        for a in k:
            zero = zero | (a.abs() == n_side // 2)
    amp = torch.where(zero, torch.zeros_like(k2), torch.where(zero, torch.ones_like(k2), k2) ** -1.5)
    disp = torch.stack([torch.fft.irfftn(1j * a * amp * wk, s=(n_side,) * 3) for a in k], -1)
    dg = BOX / n_side
    disp *= 0.5 * dg / disp.square().sum(-1).mean().sqrt()
    g = (torch.arange(n_side, device=dev, dtype=f64) + 0.5) * dg
    x = (torch.stack(torch.meshgrid(g, g, g, indexing="ij"), -1) + disp).reshape(-1, 3)
    # Plummer halos, scale 0.3 spacings, cut at ten scales
    move = int(round(halo_frac * n))
    if move:
        halos = max(4, round(halo_frac * n / 2100))
        pick = torch.randperm(n, generator=gen, device=dev)[:move]
        weight = 10.0 ** torch.rand(halos, generator=gen, device=dev, dtype=f64)
        cum = torch.cumsum(weight, 0) / weight.sum()
        of = torch.searchsorted(cum, torch.rand(move, generator=gen, device=dev, dtype=f64))
        centre = torch.rand((halos, 3), generator=gen, device=dev, dtype=f64) * BOX
        u = torch.rand(move, generator=gen, device=dev, dtype=f64) * (1000.0 / 101.0 ** 1.5)
        r = 0.3 * dg / (u.clamp_min(1e-12) ** (-2.0 / 3.0) - 1.0).sqrt()
        v = torch.randn((move, 3), generator=gen, device=dev, dtype=f64)
        x[pick] = centre[of.clamp_max(halos - 1)] + r[:, None] * v / v.norm(dim=1, keepdim=True)
    return x


def _sides(case):
    """The boxes of a batch: sides log-uniform in [low_side, n_side]."""
    if case["kind"] != "batch":
        return [case["n_side"]]
    rng = random.Random(case["sides"])
    return [_log_int(rng, case["low_side"], case["n_side"]) for _ in range(case["n_box"])]


def _inputs(case, seed):
    """Positions, masses (equal, 1 / n) and the gradient's or the motion's vectors."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dtype = torch.float32 if case["form"].startswith("fp32") else torch.float64
    pos, mass = [], []
    for n_side in _sides(case):
        x = _positions(n_side, case["clustered"], case["halo_frac"], gen)
        pos.append(_wrap(_wrap(x).to(dtype)))
        mass.append(torch.full((len(x),), 1.0 / len(x), device="cuda", dtype=dtype))
    pos, mass = torch.cat(pos), torch.cat(mass)
    vec = torch.randn(pos.shape, generator=gen, device="cuda", dtype=torch.float64).to(dtype)
    return pos, mass, vec


def _params(case):
    r_s, r_cut = _split(case["n_side"])
    return dict(box=BOX, r_s=r_s, r_cut=r_cut, max_leaf=case["max_leaf"], order=case["order"],
                theta=case["theta"])


def _motion(case, vec):
    """Velocities and the time step of a simulation: about 0.003 spacings a step."""
    dg = BOX / case["n_side"]
    return 5e-5 * dg * vec, 50.0


# ------------------------------------------------------------------ the cases

def prepare(case, seed):
    pos, mass, vec = _inputs(case, seed)
    s = dict(case=case, pos=pos, mass=mass)
    if case["kind"] == "mesh":
        r_s, r_cut = _split(case["n_side"])
        s["ctx"] = B.Context(box=BOX, r_s=r_s, r_cut=r_cut)
        s["out"] = torch.empty_like(pos)
    elif case["kind"] == "sim":
        vel, s["dt"] = _motion(case, vec)
        s["sim"] = api.Simulation(pos, vel.contiguous(), mass, n_pm=case["n_pm"], **_params(case),
                                  **FORMS[case["form"]])
    else:
        s["w"] = vec
        if case["kind"] == "batch":
            sides = _sides(case)
            s["boxes"] = [dict(box=BOX, r_s=_split(n)[0], r_cut=_split(n)[1],
                               max_leaf=case["max_leaf"], order=-1, theta=0.0) for n in sides]
            s["counts"] = [n ** 3 for n in sides]
            s["sr"] = api.ShortRange(**FORMS[case["form"]])
        else:
            s["sr"] = api.ShortRange(**_params(case), **FORMS[case["form"]])
    return s


def run(state):
    kind = state["case"]["kind"]
    pos, mass = state["pos"], state["mass"]
    if kind == "mesh":
        state["ctx"].long_range(state["case"]["n_pm"], pos, mass, state["out"],
                                torch.cuda.current_stream())
        return state["out"]
    if kind == "sim":
        sim = state["sim"]
        p, v = sim.step(state["dt"])
        return [p, v, sim.acc]
    sr = state["sr"]
    if kind == "batch":
        sr.build_batch(state["boxes"], state["counts"], pos, mass)
    else:
        sr.build(pos, mass)
    acc = sr.forward().to(pos.dtype)
    if kind != "grad":
        return acc
    gp, gm = sr.adjoint(state["w"])
    return [acc, gp.to(pos.dtype), gm.to(pos.dtype)]


def work(case):
    """Particles read and results written once; operations of the pairs inside
    the cutoff (all others can be known to be beyond it), each transcendental
    function counted as one."""
    sides = _sides(case)
    n = sum(s ** 3 for s in sides)
    size = 4 if case["form"].startswith("fp32") else 8
    words = {"step": 7, "batch": 7, "grad": 14, "mesh": 7, "sim": 22}[case["kind"]]
    flops = 0.0
    if case["kind"] != "mesh":
        per_pair = {"r2": 23, "table": 27, "exact": 27}[case["form"].split("_")[1]]
        if case["kind"] == "grad":
            per_pair += 59
        for s in sides:
            # mean-density neighbours inside r_cut = 5.4 spacings, and those
            # of a halo particle in its own halo
            pairs = 4.0 / 3.0 * math.pi * 5.4 ** 3
            if case["clustered"]:
                m = case["halo_frac"] * s ** 3
                pairs += case["halo_frac"] * m / max(4, round(m / 2100))
            flops += per_pair * pairs * s ** 3
    if "n_pm" in case:
        m = case["n_pm"] ** 3
        flops += 4 * 2.5 * m * math.log2(m) + 30 * m + 100 * n
    return {"bytes": float(words * size * n), "flops": float(flops)}


# ------------------------------------------------------------------ reference

def _direct(pos, mass, r_s, r_cut, w=None):
    """The truncated pair sum (G = 1) of one box over a grid of cells of side
    >= r_cut, pair by pair in float64; with w also the gradient."""
    n, dev = len(pos), pos.device
    nc = max(1, int(BOX / r_cut))
    nc = nc if nc >= 3 else 1
    cell = (pos * (nc / BOX)).long().clamp_(0, nc - 1)
    cid = (cell[:, 0] * nc + cell[:, 1]) * nc + cell[:, 2]
    order = torch.argsort(cid)
    start = torch.zeros(nc ** 3 + 1, dtype=torch.long, device=dev)
    start[1:] = torch.cumsum(torch.bincount(cid, minlength=nc ** 3), 0)
    p, m, c = pos[order], mass[order], cell[order]
    wv = None if w is None else w[order]
    acc = torch.zeros((n, 3), dtype=torch.float64, device=dev)
    gp, gm = torch.zeros_like(acc), torch.zeros(n, dtype=torch.float64, device=dev)
    steps = [(x, y, z) for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1)] if nc > 1 \
        else [(0, 0, 0)]
    for off in steps:
        nb = (c + torch.tensor(off, device=dev)) % nc
        nb = (nb[:, 0] * nc + nb[:, 1]) * nc + nb[:, 2]
        first, count = start[nb], start[nb + 1] - start[nb]
        cum = torch.cumsum(count, 0)
        lo = 0
        while lo < n:
            base = int(cum[lo - 1]) if lo else 0
            hi = max(lo + 1, int(torch.searchsorted(cum, base + (1 << 25), right=True)))
            i = torch.repeat_interleave(torch.arange(lo, hi, device=dev), count[lo:hi])
            j = torch.arange(len(i), device=dev) + (first - (cum - count))[i] + base
            d = p[j] - p[i]
            d -= BOX * torch.round(d / BOX)
            r2 = d.square().sum(1)
            ok = torch.nonzero((r2 > 0) & (r2 < r_cut * r_cut))[:, 0]
            i, j, d, r2 = i[ok], j[ok], d[ok], r2[ok]
            r = r2.sqrt()
            x = r / (2.0 * r_s)
            ex = torch.exp(-x * x)
            t = torch.special.erfc(x) + (2.0 / math.sqrt(math.pi)) * x * ex
            g = t / (r2 * r)
            acc.index_add_(0, i, (m[j] * g)[:, None] * d)
            if wv is not None:
                h = -(3.0 * t + (4.0 / math.sqrt(math.pi)) * x ** 3 * ex) / (r2 * r2 * r)
                dl, dk = (d * wv[j]).sum(1), (d * wv[i]).sum(1)
                gp.index_add_(0, i, m[i][:, None] * (g[:, None] * wv[j] + (h * dl)[:, None] * d)
                              - m[j][:, None] * (g[:, None] * wv[i] + (h * dk)[:, None] * d))
                gm.index_add_(0, i, -g * dl)
            lo = hi
    back = torch.empty_like(order)
    back[order] = torch.arange(n, device=dev)
    return acc[back], gp[back], gm[back]


def _mesh(pos, mass, r_s, n):
    """The long-range mesh force: CIC in, filtered Green's function, CIC out."""
    u = pos * (n / BOX)
    g = torch.floor(u)
    f = u - g
    g = g.long()
    corners = []
    for s in range(8):
        b = (s & 1, s >> 1 & 1, s >> 2)
        node, wt = torch.zeros(len(pos), dtype=torch.long, device=pos.device), 1.0
        for a in range(3):
            node = node * n + (g[:, a] + b[a]) % n
            wt = wt * (f[:, a] if b[a] else 1.0 - f[:, a])
        corners.append((node, wt))
    rho = torch.zeros(n ** 3, dtype=torch.float64, device=pos.device)
    for node, wt in corners:
        rho.index_add_(0, node, mass * wt)
    rk = torch.fft.fftn((rho * (n / BOX) ** 3).reshape(n, n, n))
    k1 = 2.0 * math.pi / BOX * torch.fft.fftfreq(n, 1.0 / n, device=pos.device, dtype=torch.float64)
    k = (k1[:, None, None], k1[None, :, None], k1[None, None, :])
    k2 = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    window = torch.ones_like(k2)
    for a in k:
        window = window * torch.sinc(a * (0.5 * BOX / n / math.pi)) ** 2
    green = -4.0 * math.pi * torch.exp(-k2 * r_s * r_s) / torch.where(k2 > 0, k2, 1.0) / window ** 2
    phi = rk * torch.where(k2 > 0, green, 0.0)
    acc = torch.zeros_like(pos)
    for a in range(3):
        ka = k[a].clone()
        ka.reshape(-1)[n // 2] = 0.0
        field = torch.fft.ifftn(-1j * ka * phi).real.reshape(-1)
        for node, wt in corners:
            acc[:, a] += wt * field[node]
    return acc


def exact(case, seed):
    pos, mass, vec = _inputs(case, seed)
    if len(pos) > MOST_EXACT and case["kind"] != "mesh":
        return None
    pos, mass, vec = pos.double(), mass.double(), vec.double()
    r_s, r_cut = _split(case["n_side"])
    if case["kind"] == "mesh":
        return _mesh(pos, mass, r_s, case["n_pm"])
    if case["kind"] == "sim":
        vel, dt = _motion(case, vec)

        def force(p):
            return _direct(p, mass, r_s, r_cut)[0] + _mesh(p, mass, r_s, case["n_pm"])
        vel = vel + 0.5 * dt * force(pos)
        pos = _wrap(pos + dt * vel)
        acc = force(pos)
        return [pos, vel + 0.5 * dt * acc, acc]
    if case["kind"] == "batch":
        out, at = [], 0
        for n_side in _sides(case):
            k = slice(at, at + n_side ** 3)
            out.append(_direct(pos[k], mass[k], *_split(n_side))[0])
            at += n_side ** 3
        return torch.cat(out)
    acc, gp, gm = _direct(pos, mass, r_s, r_cut, vec if case["kind"] == "grad" else None)
    return [acc, gp, gm] if case["kind"] == "grad" else acc
