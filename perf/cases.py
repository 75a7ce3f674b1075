"""Performance cases of the halo finder.

Each case is work that a program has this library do: whole passes of the hot
path, and its stages through their own entry points.  Sizes run from a halo
of a few thousand particles to the 256^3 box of the benchmark.

  listed()        the standing cases, by name
  draw(rng)       one more case of the same ranges
  prepare(c, s)   device inputs of case c from seed s, with the context,
                  weights and tables that a program keeps
  run(state)      one pass through the public entry points; its outputs
  work(c)         bytes and flops a pass cannot do without
  exact(c, s)     outputs that a formula gives, in 64 bits, in plain torch

Boxes are drawn on the GPU with the distributions of synth.cosmo_box and
synth.two_species: 45% of the particles in NFW halos of sizes
dN/dlnN ~ N^-0.9, a tenth of each in Plummer subhalos, the rest uniform.
"""
import functools
import math
import os

import numpy as np
import torch

from paper_1902_01010_amd import pipeline, surrogate, synth, vr

DEV = "cuda"
BITS = synth.GRID_BITS
SPACING = 100.0 / 256.0                 # Mpc/h between particles of the 256^3 box
ELLX = 0.2 * SPACING
M_P = synth.OMEGA_M * synth.RHO_CRIT * SPACING ** 3
HOST_MIN, N_MIN = 256, 20
TUNE = os.path.join(os.path.dirname(os.path.abspath(vr.__file__)), "data", "autotune_gfx950.json")


def listed():
    return [
        # the smallest whole pass: one resolved halo, as in a zoom run's early outputs
        dict(name="halo_12k", kind="halo", n_host=12000, n_sub=3, levels=1),
        # the isolated halo of 100k particles and its five subhalos, searched two levels deep
        dict(name="halo_100k", kind="halo", n_host=100000, n_sub=5, levels=2),
        # the benchmark's snapshot
        dict(name="box_256", kind="box", n=256 ** 3),
        # field halos by adaptive 6D FOF (the paper's default field search), a ragged snapshot
        dict(name="field_6d", kind="field", n=3000017),
        # cells and R at the paper's own neighbour counts
        dict(name="background_256_32", kind="background", n=1000003, n_se=256, n_v=32, masses=False),
        # cells and R at the default counts over hosts of unequal particle masses
        dict(name="background_masses", kind="background", n=4000037, n_se=32, n_v=8, masses=True),
        # R alone for given moments, more neighbours than the default
        dict(name="ratio_48_16", kind="ratio", n=500009, n_se=48, n_v=16, masses=True),
        # learned R of a snapshot's host members: features and network
        dict(name="surrogate_2m", kind="surrogate", n=2097152),
        # one optimiser step of the network at its training batch
        dict(name="train_8192", kind="train", batch=8192),
        # normalised ratio, the paper's substructure linker with growth, cleaning
        dict(name="sub_paper", kind="sub", n=2000003),
        # dark matter and stars: seeded FOF and baryons to substructure
        dict(name="species", kind="species", n=1000003),
        # unbinding of a heavy-tailed group set: the largest split over the chip, hundreds of small ones
        dict(name="unbind_heavy", kind="unbind", n_groups=600, largest=100000, masses=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["halo", "box", "field", "background", "background", "ratio", "surrogate", "train", "sub",
                       "species", "unbind", "unbind"])
    if kind == "halo":
        return dict(kind=kind, n_host=_log(rng, 4000, 300000), n_sub=rng.randint(1, 6), levels=rng.randint(1, 2))
    if kind == "box":
        return dict(kind=kind, n=_log(rng, 200000, 256 ** 3 - 1))
    if kind == "field":
        return dict(kind=kind, n=_log(rng, 100000, 3000000))
    if kind == "background":
        n_se, n_v = rng.choice([(32, 8), (32, 8), (48, 16), (64, 16), (256, 32)])
        return dict(kind=kind, n=_log(rng, 100000, 1000000 if n_se > 64 else 4000000), n_se=n_se, n_v=n_v,
                    masses=rng.random() < 0.5)
    if kind == "ratio":
        n_se, n_v = rng.choice([(32, 8), (48, 16), (100, 20)])
        return dict(kind=kind, n=_log(rng, 50000, 500000), n_se=n_se, n_v=n_v, masses=rng.random() < 0.5)
    if kind == "surrogate":
        return dict(kind=kind, n=_log(rng, 100000, 2097152))
    if kind == "train":
        return dict(kind=kind, batch=_log(rng, 256, 65536))
    if kind == "sub":
        return dict(kind=kind, n=_log(rng, 100000, 2000000))
    if kind == "species":
        return dict(kind=kind, n=_log(rng, 100000, 1000000))
    largest = _log(rng, 300, 100000)
    return dict(kind=kind, n_groups=_log(rng, 1, max(2, min(20000, 3000000 // int(math.sqrt(20 * largest))))),
                largest=largest, masses=rng.random() < 0.5)


@functools.lru_cache(maxsize=None)
def _context():
    """The one context a program keeps, with the launch knobs shipped for this GPU."""
    ctx = vr.Context(0)
    ctx.autotune(TUNE)
    return ctx


# ---------------------------------------------------------------------------
# inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _unit(g, n):
    u = torch.randn((3, n), device=DEV, generator=g, dtype=torch.float64)
    return u / u.norm(dim=0, keepdim=True)


def _rand(g, *shape):
    return torch.rand(shape, device=DEV, generator=g, dtype=torch.float64)


def _nfw_radii(g, r200, c):
    """Radii of NFW profiles truncated at r200: the enclosed mass inverted by a table."""
    x = torch.cat([torch.zeros(1, device=DEV, dtype=torch.float64),
                   torch.logspace(-5, math.log10(16.0), 8191, device=DEV, dtype=torch.float64)])
    mu = torch.log1p(x) - x / (1 + x)
    t = _rand(g, len(c)) * (torch.log1p(c) - c / (1 + c))
    k = torch.searchsorted(mu, t).clamp_(1, len(x) - 1)
    f = ((t - mu[k - 1]) / (mu[k] - mu[k - 1])).clamp_(0, 1)
    return (x[k - 1] + f * (x[k] - x[k - 1])) * (r200 / c)


def _sizes(rng, lo, hi, total):
    """Sizes of dN/dlnN ~ N^-0.9 on [lo, hi] that sum to `total`."""
    a, b = lo ** -0.9, hi ** -0.9
    out, acc = [], 0
    while acc < total:
        s = np.floor((a - rng.random(max(16, min(65536, int(total - acc) // 100))) * (a - b)) ** (-1 / 0.9))
        out.append(np.clip(s, lo, hi).astype(np.int64))
        acc += int(out[-1].sum())
    s = np.concatenate(out)
    c = np.cumsum(s)
    k = int(np.searchsorted(c, total))
    s = s[:k + 1].copy()
    s[-1] -= c[k] - total
    return s[s > 0]


def _t(a, dtype=None):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV, dtype)


class _Box:
    """Particles of a synthetic box, their halo and subhalo, and the halo table."""


def _box(seed, n, masses=False, stars=False, n_max=None):
    rng = np.random.default_rng(seed)
    g = _gen(seed)
    b = _Box()
    b.box = box = SPACING * n ** (1.0 / 3.0)
    if n_max is None:
        n_max = int(min(2_000_000, max(1000, 2_000_000 * n / 256 ** 3)))
    size = _sizes(rng, 20, n_max, int(round(0.45 * n)))
    nh = len(size)
    r200 = (3 * size * M_P / (800 * np.pi * synth.RHO_CRIT)) ** (1 / 3)
    sig = 300.0 * (size / 1e5) ** (1 / 3)
    conc = rng.uniform(5.0, 15.0, nh)
    centre, bulk = rng.random((3, nh)) * box, rng.normal(0.0, 400.0, (3, nh))
    sh, ss = [], []
    for h in np.nonzero(size >= 200)[0]:
        s = _sizes(rng, 20, max(20, size[h] // 10), size[h] // 10)
        sh.append(np.full(len(s), h))
        ss.append(s)
    sh = np.concatenate(sh) if sh else np.zeros(0, np.int64)
    ss = np.concatenate(ss) if ss else np.zeros(0, np.int64)
    nfw = size - np.bincount(sh, weights=ss, minlength=nh).astype(np.int64)
    R, S, C, X, V = _t(r200), _t(sig), _t(conc), _t(centre), _t(bulk)
    ids = torch.arange(nh, device=DEV)
    h0 = torch.repeat_interleave(ids, _t(nfw))
    r = _nfw_radii(g, R[h0], C[h0])
    pos = [X[:, h0] + _unit(g, len(h0)) * r]
    vel = [V[:, h0] + torch.randn((3, len(h0)), device=DEV, generator=g, dtype=torch.float64) * S[h0]]
    ns = len(ss)
    SH = _t(sh)
    s1 = torch.repeat_interleave(torch.arange(ns, device=DEV), _t(ss))
    a = (0.005 + 0.01 * _rand(g, ns)) * R[SH] / 0.3
    sc = X[:, SH] + _unit(g, ns) * (0.1 + 0.73 * _rand(g, ns)) * R[SH]
    sv = (10 + 20 * _rand(g, ns)) * S[SH] / 200.0
    sb = V[:, SH] + torch.randn((3, ns), device=DEV, generator=g, dtype=torch.float64) * S[SH]
    rr = a[s1] / torch.sqrt((_rand(g, len(s1)) * 0.985).clamp_min(1e-12) ** (-2.0 / 3.0) - 1)
    pos.append(sc[:, s1] + _unit(g, len(s1)) * rr)
    vel.append(sb[:, s1] + torch.randn((3, len(s1)), device=DEV, generator=g, dtype=torch.float64) * sv[s1])
    nb = n - len(h0) - len(s1)
    pos.append(_rand(g, 3, nb) * box)
    vel.append(300.0 * torch.randn((3, nb), device=DEV, generator=g, dtype=torch.float64))
    neg = torch.full((max(nb, len(h0)),), -1, device=DEV, dtype=torch.int64)
    halo, sub = [h0, SH[s1], neg[:nb]], [neg[:len(h0)], s1, neg[:nb]]
    star = [torch.zeros(n, device=DEV, dtype=torch.uint8)]
    if stars:
        # 0.662 stars per halo particle: 70% in exponential discs, the rest on the halo's profile
        k = np.rint(0.662 * size).astype(np.int64)
        kd = np.rint(0.7 * k).astype(np.int64)
        hd, hs = (torch.repeat_interleave(ids, _t(v)) for v in (kd, k - kd))
        scale = 0.03 * R[hd]
        rad = -torch.log((_rand(g, len(hd)) * _rand(g, len(hd))).clamp_min(1e-300)) * scale
        z = -0.1 * scale * torch.log(_rand(g, len(hd)).clamp_min(1e-300)) * torch.sign(_rand(g, len(hd)) - 0.5)
        ph = 2 * math.pi * _rand(g, len(hd))
        nrm = _unit(g, nh)
        e1 = torch.linalg.cross(nrm, _unit(g, nh), dim=0)
        e1 = e1 / e1.norm(dim=0, keepdim=True)
        e2 = torch.linalg.cross(nrm, e1, dim=0)
        e1, e2, nrm = e1[:, hd], e2[:, hd], nrm[:, hd]
        pos.append(X[:, hd] + rad * (e1 * torch.cos(ph) + e2 * torch.sin(ph)) + nrm * z)
        vel.append(V[:, hd] + 150.0 * (e2 * torch.cos(ph) - e1 * torch.sin(ph))
                   + 20.0 * torch.randn((3, len(hd)), device=DEV, generator=g, dtype=torch.float64))
        pos.append(X[:, hs] + _unit(g, len(hs)) * _nfw_radii(g, R[hs], C[hs]))
        vel.append(V[:, hs] + 0.8 * S[hs] * torch.randn((3, len(hs)), device=DEV, generator=g, dtype=torch.float64))
        kn = len(hd) + len(hs)
        halo += [hd, hs]
        sub.append(torch.full((kn,), -1, device=DEV, dtype=torch.int64))
        star.append(torch.ones(kn, device=DEV, dtype=torch.uint8))
    pos, vel, halo, sub, star = (torch.cat(v, dim=-1) for v in (pos, vel, halo, sub, star))
    # the stars are cut to a count that the particle number alone sets
    p = torch.randperm(n + int(0.295 * n) if stars else n, device=DEV, generator=g)
    x = torch.remainder(pos[:, p], box).float()
    b.x = torch.where(x >= box * (1 - 1e-7), torch.zeros_like(x), x).contiguous()
    b.v = vel[:, p].float().contiguous()
    b.halo, b.sub, b.star = halo[p], sub[p], star[p].contiguous()
    b.n = b.x.shape[1]
    b.mass = None
    if masses:
        b.mass = (M_P * (0.5 + _rand(g, b.n))).float()
    elif stars:
        b.mass = torch.where(b.star > 0, 0.1 * M_P, M_P).float()
    b.bulk, b.sig, b.r200, b.centre, b.gen = V, S, R, X, g
    return b


def _hosts(b):
    """Halos of >= HOST_MIN members as a group table: larger first, then by
    smallest member; members ascending.  Also each particle's host or -1."""
    nh = b.bulk.shape[1]
    ok = b.halo >= 0
    h = b.halo.clamp_min(0)
    cnt = torch.bincount(h[ok], minlength=nh)
    idx = torch.arange(b.n, device=DEV)
    first = torch.full((nh,), b.n, device=DEV, dtype=torch.int64).scatter_reduce_(0, h[ok], idx[ok], "amin")
    order = torch.argsort(first, stable=True)
    order = order[torch.argsort(cnt[order], descending=True, stable=True)]
    k = int((cnt >= HOST_MIN).sum())
    rank = torch.full((nh,), -1, device=DEV, dtype=torch.int64)
    rank[order[:k]] = torch.arange(k, device=DEV)
    host_of = torch.where(ok, rank[h], torch.full_like(h, -1))
    sel = torch.nonzero(host_of >= 0)[:, 0]
    members = sel[torch.argsort(host_of[sel], stable=True)].to(torch.int32)
    off = torch.zeros(k + 1, device=DEV, dtype=torch.int32)
    off[1:] = torch.cumsum(cnt[order[:k]], 0).to(torch.int32)
    return off, members, host_of.to(torch.int32), k


def _moments(b):
    """Per-particle local mean velocity [n][3] and dispersion [n][6]: the
    halo's bulk and dispersion, varying over the halo and its particles."""
    h = b.halo.clamp_min(0)
    d = b.x.double() - b.centre[:, h]
    d = d - b.box * torch.round(d / b.box)
    u = d / b.r200[h].clamp_min(1e-9)
    s2 = b.sig[h] ** 2
    vbar = (b.bulk[:, h] + 0.1 * b.sig[h] * torch.sin(2 * u)).t().float().contiguous()
    w = torch.cos(u)
    sigma = torch.stack([s2 * (1 + 0.2 * w[0]), s2 * (1 + 0.2 * w[1]), s2 * (1 + 0.2 * w[2]), 0.10 * s2 * w[2],
                         0.10 * s2 * w[1], 0.10 * s2 * w[0]], 1).float().contiguous()
    return vbar, sigma


def _particles(ctx, b):
    return vr.Particles(ctx.quantize(b.x, b.box, BITS), b.v, b.mass, M_P, b.box, BITS)


def _group_sizes(c):
    """Sizes N_k ~ k^-1.1 from `largest` down to 20 members, n_groups of them."""
    k = np.arange(1, c["n_groups"] + 1, dtype=np.float64)
    return np.maximum(20, (c["largest"] * k ** -1.1)).astype(np.int64)


def _unbind_inputs(c, seed):
    w = synth.unbind_groups(seed=seed, sizes=_group_sizes(c))
    off, mem = w.groups
    mass = None
    if c["masses"]:
        mass = (w.mass_value * (0.5 + np.random.default_rng(seed + 1).random(w.n))).astype(np.float32)
    return w, off, mem, mass


def _train_inputs(c, seed):
    g = _gen(seed)
    n = 4 * c["batch"]
    f = torch.randn((n, 12), device=DEV, generator=g)
    feat = f.to(torch.bfloat16)
    target = (0.3 + f[:, 1] ** 2 - 0.4 * f[:, 0] + 0.5 * f[:, 4] * f[:, 8]
              + torch.randn(n, device=DEV, generator=g)).clamp(*surrogate.TARGET_CLIP)
    rows = torch.randperm(n, device=DEV, generator=g)[:c["batch"]].to(torch.int32)
    weights = _t(synth.mlp_init(seed))
    state = torch.cat([1e-2 * torch.randn(vr.MLP_PARAMS, device=DEV, generator=g),
                       1e-3 * (0.5 + torch.rand(vr.MLP_PARAMS, device=DEV, generator=g))])
    return feat, target, rows, weights, state


TRAIN_STEP, TRAIN_LR = 1000, 1e-3


def prepare(case, seed):
    c, kind = case, case["kind"]
    ctx = _context()
    if kind == "halo":
        k = max(20, c["n_host"] // 18)
        w = synth.isolated_halo(seed=seed, n_host=c["n_host"], n_sub=c["n_sub"], sub_range=(k, k))
        x, v, m = pipeline.device_inputs(w)
        prm = pipeline.Params.from_workload(w)
        prm.levels = c["levels"]
        return dict(c=c, ctx=ctx, x=x, v=v, mass=m, mass_value=w.mass_value, box=w.box, prm=prm)
    if kind in ("box", "field"):
        b = _box(seed, c["n"])
        prm = pipeline.Params(ellx=ELLX, eps=0.02 * SPACING, field_6d=kind == "field")
        return dict(c=c, ctx=ctx, x=b.x, v=b.v, mass=None, mass_value=M_P, box=b.box, prm=prm)
    if kind == "train":
        feat, target, rows, weights, state = _train_inputs(c, seed)
        return dict(c=c, ctx=ctx, feat=feat.view(torch.int16), target=target, rows=rows, weights=weights, adam=state,
                    loss=torch.zeros(1, device=DEV))
    if kind == "unbind":
        w, off, mem, mass = _unbind_inputs(c, seed)
        P = vr.Particles(ctx.quantize(_t(w.x), w.box, w.grid_bits), _t(w.v), None if mass is None else _t(mass),
                         w.mass_value, w.box, w.grid_bits)
        return dict(c=c, ctx=ctx, P=P, off=_t(off), mem=_t(mem), G=w.params["G"], eps=w.params["eps"])
    n_max = 20000 if kind == "ratio" else None
    b = _box(seed, c["n"], masses=c.get("masses", False), stars=kind == "species", n_max=n_max)
    off, mem, host_of, nh = _hosts(b)
    s = dict(c=c, ctx=ctx, P=_particles(ctx, b), off=off, mem=mem, host_of=host_of, nh=nh)
    if kind in ("ratio", "surrogate", "sub"):
        s["vbar"], s["sigma"] = (t.t() for t in _moments(b))
    if kind == "surrogate":
        prm = pipeline.Params(ellx=ELLX)
        s["model"] = surrogate.SurrogateModel.load(device=DEV).bind(prm, b.box, BITS)
        h = b.halo.clamp_min(0)
        s["rho"] = (M_P * 10.0 ** (2.5 + 2.5 * _rand(b.gen, b.n)) / b.r200[h] ** 3).float()
        s["feat"] = torch.zeros((b.n, 12), dtype=torch.int16, device=DEV)
        s["rhat"] = torch.zeros(b.n, device=DEV)
    if kind == "sub":
        # R of a smooth background (mean 0.27, longer lower tail), higher in subhalos
        z = torch.randn(b.n, device=DEV, generator=b.gen)
        R = 0.27 + torch.where(z < 0, 0.9 * z, 0.8 * z)
        s["R"] = torch.where(b.sub >= 0, 2.0 + 1.5 * z.abs(), R).where(b.halo >= 0, torch.full_like(z, float("nan")))
    if kind == "species":
        # the subhalo of each dark-matter particle, named by its smallest one
        ok = b.sub >= 0
        idx = torch.arange(b.n, device=DEV)
        first = torch.full((int(b.sub.max()) + 2,), b.n, device=DEV, dtype=torch.int64)
        first.scatter_reduce_(0, b.sub.clamp_min(0)[ok], idx[ok], "amin")
        s["sub"] = torch.where(ok, first[b.sub.clamp_min(0)], torch.full_like(idx, -1)).to(torch.int32)
        s["star"] = b.star
    return s


# ---------------------------------------------------------------------------
# passes

def _table(t, n):
    """A table of the groups found, in the capacity that n particles need."""
    return torch.nn.functional.pad(t, (0, 0) * (t.dim() - 1) + (0, n // N_MIN + 2 - t.shape[0]))


def _pass(s):
    out, _ = pipeline.run(s["ctx"], s["x"], s["v"], s["mass"], s["mass_value"], s["box"], BITS, s["prm"])
    n = s["x"].shape[1]
    res = dict(label=out["label"], R=out["R"])
    levels = [out] + out.get("levels", [])
    for k in range(s["prm"].levels):
        lev = levels[k] if k < len(levels) else {}
        ub = lev.get("unbind") or dict(bound=torch.zeros(n, dtype=torch.uint8, device=DEV),
                                       phi=torch.zeros(n, dtype=torch.float64, device=DEV),
                                       iters=torch.zeros(0, dtype=torch.int32, device=DEV))
        res[f"label6_{k}"] = lev["label6"] if lev else torch.zeros(n, dtype=torch.int32, device=DEV)
        res[f"ellv_{k}"] = _table(lev["ellv"] if lev else torch.zeros(0, dtype=torch.float64, device=DEV), n)
        res.update({f"bound_{k}": ub["bound"], f"phi_{k}": ub["phi"], f"iters_{k}": _table(ub["iters"], n)})
    return res


def run(state):
    s, c, ctx = state, state["c"], state["ctx"]
    kind = c["kind"]
    if kind in ("halo", "box"):
        return _pass(s)
    if kind == "field":
        prm = s["prm"]
        ctx.new_snapshot()
        P = vr.Particles(ctx.quantize(s["x"], s["box"], BITS), s["v"], None, M_P, s["box"], BITS)
        label3d = ctx.fof3d(P, prm.ellx)
        ng, group_of, off, mem = ctx.groups(label3d, prm.n_min)
        ellv = ctx.host_ellv(P, off, mem, prm.alpha_v)
        label = ctx.fof6d(P, group_of, ellv, prm.ellx, None)
        ng, group_of, off, mem = ctx.groups(label, prm.n_min)
        mem[int(off[-1]):] = -1
        return dict(label3d=label3d, ellv=_table(ellv, P.n), label=label, group_of=group_of, offsets=_table(off, P.n),
                    members=mem)
    if kind == "background":
        ctx.new_snapshot()
        cm = ctx.cell_moments(s["P"], s["off"], s["mem"], want_table=False, want_cell_of=False)
        R = ctx.local_vdensity(s["P"], s["off"], s["mem"], cm["vbar"], cm["sigma"], c["n_se"], c["n_v"])
        return dict(vbar=cm["vbar"], sigma=cm["sigma"], rho=cm["rho_cell"], R=R)
    if kind == "ratio":
        ctx.new_snapshot()
        return dict(R=ctx.local_vdensity(s["P"], s["off"], s["mem"], s["vbar"], s["sigma"], c["n_se"], c["n_v"]))
    if kind == "surrogate":
        m = s["model"]
        ctx.new_snapshot()
        feat = ctx.rs_features(s["P"], s["off"], s["mem"], s["vbar"], s["sigma"], s["rho"], 32, m.cell_bits, m.shift,
                               m.scale, feat=s["feat"])
        ctx.mlp_forward(m.weights, feat, out=s["rhat"])
        return dict(feat=s["feat"], rhat=s["rhat"])
    if kind == "train":
        ctx.mlp_train_step(s["weights"], s["adam"], s["feat"], s["target"], TRAIN_STEP, rows=s["rows"], lr=TRAIN_LR,
                           loss=s["loss"])
        return dict(weights=s["weights"], adam=s["adam"], loss=s["loss"])
    if kind == "sub":
        ef = ctx.ell_fit(s["R"], s["off"], s["mem"])
        label = ctx.fof_sub(s["P"], s["host_of"], s["nh"], s["vbar"], 0.5 * ELLX, ef["ell"])
        label, rounds = ctx.sub_grow(s["P"], s["host_of"], s["nh"], s["vbar"], ef["ell"], label, 0.5 * ELLX)
        grown = label.clone()
        nc, _, off, mem = ctx.groups(label, N_MIN)
        removed = None
        if nc > 0:
            label, removed = ctx.ell_clean(ef["ell"], off, mem, label)
        n = s["P"].n
        removed = torch.zeros(0, dtype=torch.int32, device=DEV) if removed is None else removed
        return dict(fit=_table(ef["fit"], n), status=_table(ef["status"], n), merge=_table(ef["merge"], n),
                    ell=ef["ell"], grown=grown, rounds=rounds, label=label, removed=_table(removed, n))
    if kind == "species":
        ctx.new_snapshot()
        label = ctx.fof3d_dm(s["P"], ELLX, s["star"])
        off, mem = ctx.select_members(s["P"].n, s["off"], s["mem"], s["star"])
        ellv = ctx.host_ellv(s["P"], off, mem)
        lab, used = ctx.assign_baryons(s["P"], s["off"], s["mem"], s["star"], s["sub"], ELLX, 0.0, ellv_host=ellv)
        return dict(label=label, ellv=_table(ellv, s["P"].n), assigned=lab, sigma_v=used, final=ctx.relabel_min(lab, 1))
    ub = ctx.unbind(s["P"], s["off"], s["mem"], s["G"], s["eps"])
    return dict(bound=ub["bound"], phi=ub["phi"], iters=ub["iters"])


# ---------------------------------------------------------------------------
# floors

def work(case):
    c, kind = case, case["kind"]
    n = c.get("n", 0)
    hosted = 0.4 * n                    # members of halos of >= HOST_MIN particles
    if kind == "halo":
        n = 1.25 * c["n_host"]
        # x, v in; label, R, 6D label, bound, phi out; n_se neighbours' kernel sums, pair terms of the subhalos
        return dict(bytes=n * (24 + 4 + 4 + 4 + 1 + 8), flops=n * 32 * 20.0)
    if kind == "box":
        return dict(bytes=n * (24 + 4 + 4 + 4 + 1 + 8), flops=hosted * 32 * 20.0)
    if kind == "field":
        return dict(bytes=n * (24 + 4 + 4 + 4) + 4 * 0.45 * n, flops=0.45 * n * 20.0)
    if kind == "background":
        m = 4 if c["masses"] else 0
        return dict(bytes=hosted * (24 + m + 4) + hosted * (12 + 24 + 4 + 4), flops=hosted * c["n_se"] * 20.0)
    if kind == "ratio":
        m = 4 if c["masses"] else 0
        return dict(bytes=hosted * (24 + m + 4 + 36) + hosted * 4, flops=hosted * c["n_se"] * 20.0)
    if kind == "surrogate":
        return dict(bytes=hosted * (24 + 36 + 4 + 4) + hosted * 28, flops=hosted * 18048.0)
    if kind == "train":
        return dict(bytes=c["batch"] * 32 + 4.0 * 6 * vr.MLP_PARAMS, flops=c["batch"] * 18048.0 * 3)
    if kind == "sub":
        # R, member, ell; positions, u of the outliers; labels before and after cleaning
        return dict(bytes=hosted * 12 + n * 8 + 0.06 * n * 28, flops=hosted * 10.0)
    if kind == "species":
        n = 1.3 * n
        return dict(bytes=n * (12 + 1 + 4) + 0.6 * n * (28 + 4) + 4 * n, flops=0.23 * n * 20.0)
    sizes = 1.2 * _group_sizes(c)
    return dict(bytes=float(sizes.sum()) * (28 + 1 + 8), flops=6.0 * float((sizes ** 2).sum()))


# ---------------------------------------------------------------------------
# 64-bit values

def _grid(x, box):
    return torch.floor(x.double() * (2.0 ** BITS / box)).to(torch.int64) % (1 << BITS)


def _rel(q, first):
    """Grid offsets from `first` in the periodic box."""
    half, full = 1 << (BITS - 1), 1 << BITS
    return ((q - first + half) % full) - half


def _exact_ratio(c, seed):
    b = _box(seed, c["n"], masses=c["masses"], n_max=20000)
    off, mem, _, nh = _hosts(b)
    vbar, sigma = (t.double() for t in _moments(b))
    off, q = off.tolist(), _grid(b.x, b.box)
    v = b.v.double()
    mass = torch.full((b.n,), M_P, device=DEV, dtype=torch.float64) if b.mass is None else b.mass.double()
    R = torch.full((b.n,), float("nan"), device=DEV, dtype=torch.float64)
    n_se, n_v = c["n_se"], c["n_v"]
    for h in range(nh):
        i = mem[off[h]:off[h + 1]].long()
        N = len(i)
        p = _rel(q[:, i], q[:, i[:1]])
        rows = max(1, 60_000_000 // N)
        rank = torch.arange(N, device=DEV)
        for r in range(0, N, rows):
            k = rank[r:r + rows]
            d = sum((p[a][k][:, None] - p[a][None, :]) ** 2 for a in range(3))
            s = torch.topk(d * N + rank, n_se, dim=1, largest=False).values % N
            dv = ((v[:, i[s]] - v[:, i[k]][:, :, None]) ** 2).sum(0)
            w, pick = torch.topk(dv, n_v, dim=1, largest=False, sorted=True)
            ms = mass[i[s]]
            h2 = w[:, -1]
            fl = (ms.gather(1, pick) * 15 / (8 * math.pi) * (1 - w / h2[:, None])).sum(1)
            R[i[k]] = torch.log(fl) - 1.5 * torch.log(h2) - torch.log(ms.sum(1))
    i = mem.long()
    e = sigma[i]
    S = torch.stack([e[:, [0, 3, 4]], e[:, [3, 1, 5]], e[:, [4, 5, 2]]], 1)
    L = torch.linalg.cholesky(S)
    y = torch.linalg.solve_triangular(L, (v[:, i].t() - vbar[i])[:, :, None], upper=False)[:, :, 0]
    R[i] -= (-0.5 * (y ** 2).sum(1) - 1.5 * math.log(2 * math.pi)
             - torch.log(torch.diagonal(L, dim1=1, dim2=2)).sum(1))
    return dict(R=R)


def _exact_train(c, seed):
    feat, target, rows, weights, state = _train_inputs(c, seed)
    W = weights.double().requires_grad_(True)
    x, y = feat[rows.long()].double(), target[rows.long()].double()
    at, a = 0, x
    for k, (i, o) in enumerate(((12, 64), (64, 64), (64, 64), (64, 1))):
        a = a @ W[at:at + i * o].view(i, o) + W[at + i * o:at + i * o + o]
        at += i * o + o
        if k < 3:
            a = torch.relu(a)
    loss = ((a[:, 0] - y) ** 2).mean()
    loss.backward()
    g, m, v = W.grad, state[:vr.MLP_PARAMS].double(), state[vr.MLP_PARAMS:].double()
    m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
    new = W.detach() - TRAIN_LR * (m / (1 - 0.9 ** TRAIN_STEP)) / (torch.sqrt(v / (1 - 0.999 ** TRAIN_STEP)) + 1e-8)
    return dict(weights=new, adam=torch.cat([m, v]), loss=loss.detach().view(1))


def _pair_sums(xi, xj, mj, eps2):
    """sum_j m_j / sqrt(r_ij^2 + eps^2), pairs at zero distance with eps = 0 left out."""
    out = torch.zeros(xi.shape[1], device=DEV, dtype=torch.float64)
    rows = max(1, 40_000_000 // max(1, xj.shape[1]))
    for r in range(0, xi.shape[1], rows):
        r2 = sum((xi[d, r:r + rows, None] - xj[d][None, :]) ** 2 for d in range(3)) + eps2
        out[r:r + rows] = (mj * torch.rsqrt(r2)).sum(1)
    return out


def _exact_unbind(c, seed):
    sizes = 1.2 * _group_sizes(c)
    if float((sizes ** 2).sum()) > 6e10 or len(sizes) > 1500:
        return None
    w, off, mem, mass = _unbind_inputs(c, seed)
    q, v = _grid(_t(w.x), w.box), _t(w.v).double()
    m = torch.full((w.n,), w.mass_value, device=DEV, dtype=torch.float64) if mass is None else _t(mass).double()
    phi = torch.full((w.n,), float("nan"), device=DEV, dtype=torch.float64)
    G, eps2, unit = w.params["G"], w.params["eps"] ** 2, w.box / 2.0 ** BITS
    for g in range(len(off) - 1):
        S = _t(mem[off[g]:off[g + 1]]).long()
        if len(S) < N_MIN:
            continue
        p = _rel(q[:, S], q[:, S[:1]])
        x = p.double() * unit
        sums = _pair_sums(x, x, m[S], eps2) - m[S] / math.sqrt(eps2)
        while True:
            f = -G * sums
            phi[S] = f
            k = int(torch.argmin(f))
            n = len(S)
            ref = min(n, max(10, math.ceil(0.1 * n)))
            d = ((p - p[:, k:k + 1]) ** 2).sum(0)
            near = torch.topk(d * n + torch.arange(n, device=DEV), ref, largest=False).values % n
            mr = m[S[near]]
            u = (mr * v[:, S[near]]).sum(1, keepdim=True) / mr.sum()
            keep = ~(0.95 * 0.5 * ((v[:, S] - u) ** 2).sum(0) + f >= 0)
            left = int(keep.sum())
            if left == n or left < N_MIN:
                break
            sums = (sums - _pair_sums(x, x[:, ~keep], m[S[~keep]], eps2))[keep]
            S, p, x = S[keep], p[:, keep], x[:, keep]
    return dict(bound=None, phi=phi, iters=None)


def exact(case, seed):
    """R for given moments, the optimiser step and the potentials; the other
    stages' numbers follow from trees and groups, not from a formula."""
    kind = case["kind"]
    if kind == "ratio":
        return _exact_ratio(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "unbind":
        return _exact_unbind(case, seed)
    return None
