"""Performance cases of the meshless hydro library: whole calls through its public
entry points, over the particle sets, sizes, schemes and directions that programs
use it for.

A case names a particle set (``set``, ``side``), the call a program makes on it
(``call``) and the options of the context.  The sets are those of
``paper_1712_01294_amd.workloads`` drawn on the GPU:

* ``lattice``     jittered side^3 lattice with a sine density (periodic)
* ``tube``        the planar shock tube, side x side lattice cross-section
* ``turbulence``  jittered side^3 lattice with a Mach-2 k^-4 velocity field
* ``clustered``   side^3 particles drawn from a log-normal density field
* ``open``        side^3 uniform random particles in an open 1 x 1/2 x 1 box
"""
from __future__ import annotations

import math

import torch

from paper_1712_01294_amd import mfm
from paper_1712_01294_amd.autodiff import Evolution, MFMSteps
from paper_1712_01294_amd.workloads import Workload

F64 = torch.float64
N_NGB = 32.0
MAX_BIN = 3            # hierarchical steps: T = 8 smallest steps
HIER_CFL = 0.05        # their Courant factor: the clustered set is far from equilibrium at its start
EXACT_MAX_N = 3_000_000


def _case(name, set_, side, call, **kw):
    c = {"name": name, "set": set_, "side": side, "call": call, "scheme": "mfm", "precision": "fp64", "limiter": 0,
         "max_ngb": 256, "steps": 0}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a whole pass queued without a context or any allocation (serving loops, graph capture)
        _case("noalloc_4k", "lattice", 16, "noalloc"),
        # a small pass and its reverse: gradients of one force evaluation inside a fitting loop
        _case("pass_adjoint_8k", "lattice", 20, "pass_adjoint"),
        # a small open, ragged set in the finite-volume form, results handed back in the caller's order
        _case("open_mfv_10k", "open", 21, "pass_unpermute", scheme="mfv"),
        # small adaptive set: kernel lengths over a factor of fifty, long lists
        _case("clustered_32k", "clustered", 32, "pass", max_ngb=1024),
        # forward and backward of a ten-step differentiable evolution
        _case("adjoint_262k", "lattice", 64, "evolve", steps=10),
        # production loop: one kick-drift-kick step at the Courant step, kernel lengths warm
        _case("tube_step_295k", "tube", 32, "step", steps=1),
        # the mixed form on a start from a snapshot (cold kernel lengths)
        _case("tube_mixed_295k", "tube", 32, "pass", precision="mixed"),
        # fixed steps of the finite-volume form on a flow
        _case("turbulence_mfv_912k", "turbulence", 97, "step", scheme="mfv", steps=2),
        # ordinary large set, cold start
        _case("turbulence_2M", "turbulence", 128, "pass"),
        # the optional limiters on a strongly clustered set
        _case("clustered_limited_2M", "clustered", 128, "pass", limiter=1),
        # hierarchical time steps with active subsets, from a snapshot: pass, bins, system step
        _case("hier_2M", "clustered", 128, "hier"),
        # the largest: a clustered medium, cold start
        _case("clustered_16M", "clustered", 256, "pass"),
    ]


def draw(rng):
    def side(lo, hi):   # sizes spread over the logarithm of the range
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("noalloc", "pass_adjoint", "open", "clustered", "evolve", "tube", "mixed", "turbulence", "hier"))
    scheme = rng.choice(("mfm", "mfv"))
    lim = rng.choice((0, 0, 1))
    if kind == "noalloc":
        c = _case("", "lattice", side(8, 20), "noalloc", scheme=scheme, limiter=lim)
    elif kind == "pass_adjoint":
        c = _case("", "lattice", side(10, 80), "pass_adjoint")
    elif kind == "open":
        c = _case("", "open", side(12, 60), "pass_unpermute", scheme=scheme, limiter=lim)
    elif kind == "clustered":
        c = _case("", "clustered", side(24, 200), "pass", scheme=scheme, limiter=lim, max_ngb=rng.choice((384, 512)))
    elif kind == "evolve":
        c = _case("", "lattice", side(12, 64), "evolve", steps=rng.randint(1, 10))
    elif kind == "tube":
        c = _case("", "tube", 2 * side(6, 24), "step", scheme=scheme, limiter=lim, steps=rng.randint(1, 3))
    elif kind == "mixed":
        c = _case("", rng.choice(("tube", "turbulence")), 2 * side(8, 18), "pass", precision="mixed", scheme="mfm")
    elif kind == "turbulence":
        c = _case("", "turbulence", side(24, 160), rng.choice(("pass", "step")), scheme=scheme, limiter=lim,
                  steps=rng.randint(1, 3))
    else:
        c = _case("", "clustered", side(32, 128), "hier")
    del c["name"]
    return c


# ------------------------------------------------------------------ particle sets
def _lattice(nx, ny, nz, sp, gen, jitter=0.2, origin=0.0):
    i = [torch.arange(k, device="cuda", dtype=F64) for k in (nx, ny, nz)]
    X = torch.stack([g.reshape(-1) for g in torch.meshgrid(*i, indexing="ij")])
    X = (X + 0.5) * sp
    X[0] += origin
    return X + jitter * sp * (2.0 * torch.rand(X.shape, generator=gen, device="cuda", dtype=F64) - 1.0)


def _wrap(X, box):
    b = torch.tensor(box, device="cuda", dtype=F64)[:, None]
    X = torch.remainder(X, b)
    return torch.where(X >= b, torch.zeros_like(X), X)


def _field(n, power, kmin, kmax, gen):
    k1 = torch.fft.fftfreq(n, d=1.0 / n, device="cuda", dtype=F64)
    k3 = torch.fft.rfftfreq(n, d=1.0 / n, device="cuda", dtype=F64)
    kk = torch.sqrt(k1[:, None, None] ** 2 + k1[None, :, None] ** 2 + k3[None, None, :] ** 2)
    filt = torch.where((kk >= kmin) & (kk <= kmax), kk.clamp(min=0.5) ** (0.5 * power), torch.zeros_like(kk))
    white = torch.randn(n, n, n, generator=gen, device="cuda", dtype=F64)
    return torch.fft.irfftn(torch.fft.rfftn(white) * filt, s=(n, n, n))


def particles(case, seed):
    """x (3, n), m, v (3, n), u, gamma, box, periodic of a case, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    s, gamma, box, per = case["side"], 5.0 / 3.0, (1.0, 1.0, 1.0), (1, 1, 1)
    if case["set"] == "lattice":
        x = _wrap(_lattice(s, s, s, 1.0 / s, gen), box)
        rho = 1.0 + 0.1 * torch.sin(2.0 * math.pi * x[0])
        m = rho / s ** 3
        v = 0.1 * torch.randn(x.shape, generator=gen, device="cuda", dtype=F64)
        u = 1.0 / ((gamma - 1.0) * rho)
    elif case["set"] == "tube":
        l_yz = s / 256.0
        box, dl = (2.0, l_yz, l_yz), 1.0 / 256.0
        x = torch.cat([_lattice(256, s, s, dl, gen), _lattice(128, s // 2, s // 2, 2 * dl, gen, origin=1.0)], 1)
        left = torch.arange(x.shape[1], device="cuda") < 256 * s * s
        perm = torch.randperm(x.shape[1], generator=gen, device="cuda")
        x, left = _wrap(x, box)[:, perm].contiguous(), left[perm]
        m = torch.full((x.shape[1],), dl ** 3, device="cuda", dtype=F64)
        rho = torch.where(left, 1.0, 0.125).to(F64)
        u = torch.where(left, 1.0, 0.1).to(F64) / ((gamma - 1.0) * rho)
        v = torch.zeros_like(x)
    elif case["set"] == "turbulence":
        gamma = 1.001
        x = _wrap(_lattice(s, s, s, 1.0 / s, gen), box)
        v = torch.stack([_field(s, -4.0, 1.0, 8.0, gen).reshape(-1) for _ in range(3)])
        v *= 2.0 / torch.sqrt((v * v).sum(0).mean())
        m = torch.full((s ** 3,), 1.0 / s ** 3, device="cuda", dtype=F64)
        u = torch.full((s ** 3,), 1.0 / (gamma * (gamma - 1.0)), device="cuda", dtype=F64)
    elif case["set"] == "clustered":
        n = s ** 3
        delta = _field(s, -3.0, 1.0, s / 2.0, gen).reshape(-1)
        rho = torch.exp(delta * (2.0 / delta.std()))
        rho /= rho.mean()
        cdf = torch.cumsum(rho, 0)
        cell = torch.searchsorted(cdf, torch.rand(n, generator=gen, device="cuda", dtype=F64) * cdf[-1])
        cell.clamp_(max=n - 1)
        c = torch.stack([cell // (s * s), (cell // s) % s, cell % s]).to(F64)
        x = _wrap((c + torch.rand(3, n, generator=gen, device="cuda", dtype=F64)) / s, box)
        v = 0.3 * torch.randn(3, n, generator=gen, device="cuda", dtype=F64)
        u = rho[cell] ** (2.0 / 3.0) / (gamma - 1.0)
        m = torch.full((n,), 1.0 / n, device="cuda", dtype=F64)
    else:
        gamma, box, per, n = 1.4, (1.0, 0.5, 1.0), (0, 0, 0), s ** 3
        x = torch.rand(3, n, generator=gen, device="cuda", dtype=F64)
        x[1] *= 0.5
        m = (0.5 + torch.rand(n, generator=gen, device="cuda", dtype=F64)) / n
        v = 0.2 * torch.randn(3, n, generator=gen, device="cuda", dtype=F64)
        u = 1.0 + torch.rand(n, generator=gen, device="cuda", dtype=F64)
    return {"x": x, "m": m, "v": v, "u": u, "gamma": gamma, "box": box, "periodic": per}


def _config(case, p):
    lim = dict(limiter=1, beta=2.0, beta_min=1.0, cond_lo=10.0, cond_hi=1000.0) if case["limiter"] else {}
    return mfm.Config(gamma=p["gamma"], box=p["box"], periodic=p["periodic"], n_ngb=N_NGB, u_floor=1e-10,
                      cfl=HIER_CFL if case["call"] == "hier" else 0.25,
                      precision=mfm.MIXED if case["precision"] == "mixed" else mfm.FP64, max_ngb=case["max_ngb"],
                      scheme=mfm.SCHEME_MFV if case["scheme"] == "mfv" else mfm.SCHEME_MFM, **lim)


def _arrays(p):
    return {"x": p["x"][0].contiguous(), "y": p["x"][1].contiguous(), "z": p["x"][2].contiguous(), "m": p["m"],
            "vx": p["v"][0].contiguous(), "vy": p["v"][1].contiguous(), "vz": p["v"][2].contiguous(), "u": p["u"]}


def _fixed_dt(case):
    # steps of the turbulent set are fixed (a fifth of a spacing at Mach 2); the tube takes the Courant step
    return 0.1 / case["side"] * 0.1 if case["set"] == "turbulence" else 0.0


# ------------------------------------------------------------------ the measured calls
STATE = ("x", "y", "z", "m", "vx", "vy", "vz", "u", "H", "dp", "dE", "vsig", "dm")


def prepare(case, seed):
    p = particles(case, seed)
    n = p["x"].shape[1]
    cfg = _config(case, p)
    if case["call"] == "evolve":
        w = Workload(name="evolve", gamma=p["gamma"], box=p["box"], periodic=p["periodic"], **_arrays(p))
        evo = Evolution(w, case["steps"], 1.0e-3, cfg)
        return {"case": case, "evo": evo, "v0": p["v"].contiguous(), "u0": p["u"], "m": p["m"]}
    st = mfm.State.from_arrays(_arrays(p), dm=case["scheme"] == "mfv")
    s = {"case": case, "st": st, "cfg": cfg}
    if case["call"] == "noalloc":
        return s
    s["ctx"] = ctx = mfm.Context(cfg, n)
    if case["call"] == "pass_adjoint":
        gen = torch.Generator(device="cuda")
        gen.manual_seed(int(seed) + 1)
        s["adj_dp"] = torch.randn(3, n, generator=gen, device="cuda", dtype=F64)
        s["adj_dE"] = torch.randn(n, generator=gen, device="cuda", dtype=F64)
    elif case["call"] == "step":
        ctx.build_neighbours(st)
        ctx.hydro_pass(st)
    if case["call"] in ("step", "hier"):
        keys = [k for k in STATE if getattr(st, k) is not None] + ["id"]
        s["live"] = [getattr(st, k) for k in keys]
        s["start"] = [t.clone() for t in s["live"]]
    if case["call"] == "hier":
        s["bins"] = torch.zeros(n, dtype=torch.int64, device="cuda")
    return s


def _outputs(st):
    keys = ("id", "x", "y", "z", "m", "vx", "vy", "vz", "u", "H", "nk", "V", "B", "rho", "P", "grad", "dp", "dE",
            "vsig") + (("dm",) if st.dm is not None else ())
    return {k: getattr(st, k) for k in keys}


def _time_bins(s):
    """Each particle's bin from the smaller of its Courant step and the step in which its acceleration moves it
    by cfl H, then the neighbour limiter; the system step is 2^MAX_BIN of the smallest steps."""
    st, cfg = s["st"], s["cfg"]
    acc = torch.sqrt((st.dp * st.dp).sum(0)) / st.m
    dti = torch.minimum(cfg.cfl * st.H / st.vsig, torch.sqrt(2.0 * cfg.cfl * st.H / acc))
    dtmin = float(dti.min())
    s["bins"].copy_((MAX_BIN - torch.floor(torch.log2(dti / dtmin))).clamp(0, MAX_BIN))
    s["ctx"].limit_bins(st, s["bins"], MAX_BIN)
    return dtmin * (1 << MAX_BIN)


def run(s):
    case = s["case"]
    call = case["call"]
    if call == "evolve":
        v0 = s["v0"].clone().requires_grad_(True)
        u0 = s["u0"].clone().requires_grad_(True)
        vk, uk = MFMSteps.apply(v0, u0, s["evo"])
        (s["m"] * (vk * vk).sum(0)).sum().backward()
        return {"v": vk.detach(), "u": uk.detach(), "grad_v0": v0.grad, "grad_u0": u0.grad}
    st = s["st"]
    if call == "noalloc":
        st.H.zero_()
        mfm.hydro_pass_noalloc(s["cfg"], st, counters=False)
        return _outputs(st)
    ctx = s["ctx"]
    if call == "step":
        torch._foreach_copy_(s["live"][:-1], s["start"][:-1])
        s["live"][-1].copy_(s["start"][-1])
        dt = [ctx.step(st, _fixed_dt(case)) for _ in range(case["steps"])]
        return dict(_outputs(st), dt=dt)
    if call == "hier":
        torch._foreach_copy_(s["live"][:-1], s["start"][:-1])
        s["live"][-1].copy_(s["start"][-1])
    st.H.zero_()
    ctx.build_neighbours(st)
    ctx.hydro_pass(st)
    if call == "hier":
        T = _time_bins(s)
        ctx.step_hier(st, s["bins"], MAX_BIN, T, rebin=True, active=True)
        return dict(_outputs(st), bins=s["bins"], T=T)
    if call == "pass_adjoint":
        ax, av, au = ctx.pass_adjoint(st, s["adj_dp"], s["adj_dE"])
        return dict(_outputs(st), adj_x=ax, adj_v=av, adj_u=au)
    if call == "pass_unpermute":
        ctx.unpermute(st)
    return _outputs(st)


def _count(case):
    s = case["side"]
    return 256 * s * s + 128 * (s // 2) ** 2 if case["set"] == "tube" else s ** 3


def work(case):
    """Per particle: the state read once and the state and pass outputs written once (8-byte values), and the
    arithmetic of about 29 gather neighbours (five sums of 20 flops for the kernel length, 65 for the gradients)
    and 15.5 unordered pairs (400 flops, 475 in the finite-volume form)."""
    n = _count(case)
    mfv = case["scheme"] == "mfv"
    flops = 29 * (5 * 20 + 65) + 15.5 * (475 if mfv else 400)
    bytes_ = 8 * (10 + 41 + (2 if mfv else 0))
    if case["call"] == "step":
        bytes_, flops = case["steps"] * (bytes_ + 8 * 6), case["steps"] * flops
    elif case["call"] == "hier":   # the pass, the rebin's gradients and fluxes, the last boundary's pass
        bytes_, flops = 3 * bytes_, 3 * flops
    elif case["call"] == "pass_adjoint":
        bytes_, flops = bytes_ + 8 * 11, 4 * flops
    elif case["call"] == "evolve":
        k = case["steps"] + 1
        bytes_, flops = k * (bytes_ + 8 * 60), k * 4 * flops
    return {"bytes": float(bytes_ * n), "flops": float(flops * n)}


# ------------------------------------------------------------------ the same in 64 bits, in plain torch
def _w(q):
    t, h = (1.0 - q).clamp(min=0.0), (0.5 - q).clamp(min=0.0)
    return 2.0 * t ** 3 - 8.0 * h ** 3


def _qdw(q):
    t, h = (1.0 - q).clamp(min=0.0), (0.5 - q).clamp(min=0.0)
    return q * (24.0 * h * h - 6.0 * t * t)


C32 = 32.0 / 3.0


def _disp(x, i, j, p):
    d = x[:, j] - x[:, i]
    b = torch.tensor(p["box"], device="cuda", dtype=F64)[:, None]
    per = torch.tensor(p["periodic"], device="cuda", dtype=F64)[:, None]
    return d - per * b * torch.round(d.detach() / b)


def _roots(r):
    """Rows of radii (inf where there is none, self included) -> the H of each row, bracketed by (0, top]."""
    hi = torch.where(torch.isfinite(r), r, torch.zeros_like(r)).amax(1) * 1.0000001 + 1e-300
    lo = torch.zeros_like(hi)
    grow = C32 * _w(r / hi[:, None]).sum(1) < N_NGB
    while bool(grow.any()):
        hi = torch.where(grow, 1.5 * hi, hi)
        grow = C32 * _w(r / hi[:, None]).sum(1) < N_NGB
    for _ in range(40):
        mid = 0.5 * (lo + hi)
        up = C32 * _w(r / mid[:, None]).sum(1) >= N_NGB
        hi, lo = torch.where(up, mid, hi), torch.where(up, lo, mid)
    h = 0.5 * (lo + hi)
    for _ in range(4):
        q = r / h[:, None]
        q = torch.where(torch.isfinite(q), q, torch.full_like(q, 2.0))
        h = h + (C32 * _w(q).sum(1) - N_NGB) / (C32 * _qdw(q).sum(1) / h)
    return h


def _gather(x, p):
    """H and the directed gather pairs (i, j), r_ij < H_i, i != j: particles still unsolved look at the 27 cells
    around theirs on ever coarser grids, until the sphere of one cell side holds the root."""
    n = x.shape[1]
    box = torch.tensor(p["box"], device="cuda", dtype=F64)
    H = torch.zeros(n, device="cuda", dtype=F64)
    I, J = [], []
    left = torch.arange(n, device="cuda")
    side = 0.0 if n <= 8192 else 0.35 * float(box.prod() / n) ** (1.0 / 3.0)

    def settle(q, row, j, reach):
        """queries q with candidate entries (row into q, j); returns which are solved"""
        d = _disp(x, q[row], j, p)
        r = torch.sqrt((d * d).sum(0))
        keep = r < reach
        row, j, r = row[keep], j[keep], r[keep]
        cnt = torch.bincount(row, minlength=q.numel())
        start = torch.cumsum(cnt, 0) - cnt
        dense = torch.full((q.numel(), max(1, int(cnt.max()))), float("inf"), device="cuda", dtype=F64)
        dense[row, torch.arange(row.numel(), device="cuda") - start[row]] = r
        ok = C32 * _w(dense / reach).sum(1) >= N_NGB if math.isfinite(reach) else torch.ones_like(q, dtype=torch.bool)
        if bool(ok.any()):
            h = torch.zeros(q.numel(), device="cuda", dtype=F64)
            h[ok] = _roots(dense[ok])
            H[q[ok]] = h[ok]
            got = ok[row] & (r < h[row]) & (j != q[row])
            I.append(q[row[got]])
            J.append(j[got])
        return ok

    while left.numel():
        nc = [int(b / side) if side else 0 for b in p["box"]]
        if min(nc) < 3:   # few or large cells: every particle is a candidate
            step = max(1, 60_000_000 // n)
            for a in range(0, left.numel(), step):
                q = left[a:a + step]
                settle(q, torch.arange(q.numel(), device="cuda").repeat_interleave(n),
                       torch.arange(n, device="cuda").repeat(q.numel()), float("inf"))
            break
        nct = torch.tensor(nc, device="cuda")
        c = torch.minimum((x / box[:, None] * nct[:, None]).long(), nct[:, None] - 1)
        flat = (c[0] * nc[1] + c[1]) * nc[2] + c[2]
        order = torch.argsort(flat)
        cnt = torch.bincount(flat, minlength=nc[0] * nc[1] * nc[2])
        first = torch.cumsum(cnt, 0) - cnt
        offs = torch.stack(torch.meshgrid(*[torch.arange(-1, 2, device="cuda")] * 3, indexing="ij")).reshape(3, 27)
        cc = c[:, left][:, :, None] + offs[:, None, :]
        inside = torch.ones(cc.shape[1:], dtype=torch.bool, device="cuda")
        for d in range(3):
            if p["periodic"][d]:
                cc[d] %= nc[d]
            else:
                inside &= (cc[d] >= 0) & (cc[d] < nc[d])
                cc[d].clamp_(0, nc[d] - 1)
        cell = (cc[0] * nc[1] + cc[1]) * nc[2] + cc[2]
        num = cnt[cell] * inside
        tot = torch.cumsum(num.sum(1), 0)
        todo, a = [], 0
        while a < left.numel():
            base = int(tot[a - 1]) if a else 0
            b = max(a + 1, int(torch.searchsorted(tot, torch.tensor(base + 80_000_000, device="cuda"))))
            k = num[a:b].reshape(-1)
            rep = torch.arange(k.numel(), device="cuda").repeat_interleave(k)
            within = torch.arange(rep.numel(), device="cuda") - (torch.cumsum(k, 0) - k)[rep]
            j = order[first[cell[a:b].reshape(-1)][rep] + within]
            ok = settle(left[a:b], rep // 27, j, min(b_ / k_ for b_, k_ in zip(p["box"], nc)))
            todo.append(left[a:b][~ok])
            a = b
        left = torch.cat(todo)
        side *= 1.35
    return H, torch.cat(I), torch.cat(J)


def _sum(n, i, v):
    return torch.zeros((n,) + v.shape[1:], device="cuda", dtype=F64).index_add(0, i, v)


def _pair_bound(f, pk, po):
    """The pairwise bound of a face value: at most a quarter of the difference past the midpoint on the other
    side, at most half of it outside the centre range on its own, keeping the sign."""
    D, mid, below = (po - pk).abs(), 0.5 * (pk + po), pk < po
    v = torch.where(below, torch.minimum(f, mid + 0.25 * D), torch.maximum(f, mid - 0.25 * D))
    wide = torch.where(below, pk - 0.5 * D, pk + 0.5 * D)
    wide = torch.where(wide * pk > 0, wide, pk * pk.abs() / (pk.abs() + 0.5 * D).clamp(min=1e-300))
    return torch.where(pk == po, pk, torch.where(below, torch.maximum(v, wide), torch.minimum(v, wide)))


def _pass(case, p, x, v, u, m):
    n, gamma = x.shape[1], p["gamma"]
    with torch.no_grad():
        H0, i, j = _gather(x.detach(), p)
    d = _disp(x, i, j, p)
    r = torch.sqrt((d * d).sum(0))
    q0 = r / H0[i]
    # H by the implicit-function theorem (its value is the root's already)
    H = H0 - (C32 * (1.0 + _sum(n, i, _w(q0))) - N_NGB) / (-C32 * _sum(n, i, _qdw(q0)) / H0).detach()
    nrm = 8.0 / math.pi / H ** 3
    q = r / H[i]
    nk = nrm * (1.0 + _sum(n, i, _w(q)))
    V = 1.0 / nk
    rho = m * nk
    P = (gamma - 1.0) * rho * u
    phi = torch.stack([rho, v[0], v[1], v[2], P], 1)
    psi = nrm[i] * _w(q) * V[i]
    E = _sum(n, i, torch.stack([d[a] * d[b] * psi for a, b in ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))], 1))
    e = E.unbind(1)
    c = (e[3] * e[5] - e[4] * e[4], e[2] * e[4] - e[1] * e[5], e[1] * e[4] - e[2] * e[3],
         e[0] * e[5] - e[2] * e[2], e[1] * e[2] - e[0] * e[4], e[0] * e[3] - e[1] * e[1])
    B = torch.stack(c, 1) / (e[0] * c[0] + e[1] * c[1] + e[2] * c[2])[:, None]
    full = [0, 1, 2, 1, 3, 4, 2, 4, 5]
    Bf = B[:, full].reshape(n, 3, 3)
    df = (phi[j] - phi[i]) * psi[:, None]
    S = torch.stack([_sum(n, i, df * d[a][:, None]) for a in range(3)], 2)
    g = (Bf[:, None] * S[:, :, None, :]).sum(3)
    ii = i[:, None].expand(-1, 5)
    top = phi.scatter_reduce(0, ii, phi[j], "amax")
    low = phi.scatter_reduce(0, ii, phi[j], "amin")
    half = 0.5 * torch.zeros_like(H).scatter_reduce(0, i, r, "amax")
    beta = torch.ones_like(H)
    if case["limiter"]:
        cond = torch.sqrt((E[:, full] ** 2).sum(1)) * torch.sqrt((B[:, full] ** 2).sum(1))
        beta = 2.0 - ((torch.log10(cond) - 1.0) / 2.0).clamp(0.0, 1.0)
    gn = torch.sqrt((g * g).sum(2)).clamp(min=1e-300)
    al = beta[:, None] * torch.minimum(top - phi, phi - low) / (gn * half[:, None])
    g = al.clamp(max=1.0)[:, :, None] * g
    # every unordered pair of the flux set once
    keep = (i < j) | (r >= H[j])
    a, b, d, r = i[keep], j[keep], d[:, keep], r[keep]
    Wa, Wb = nrm[a] * _w(r / H[a]), nrm[b] * _w(r / H[b])
    A = ((V[a] ** 2 * Wa)[:, None, None] * Bf[a] + (V[b] ** 2 * Wb)[:, None, None] * Bf[b])
    A = (A * d.t()[:, None, :]).sum(2).t()
    Am = torch.sqrt((A * A).sum(0))
    nh = A / Am
    qL = phi[a] + 0.5 * (g[a] * d.t()[:, None, :]).sum(2)
    qR = phi[b] - 0.5 * (g[b] * d.t()[:, None, :]).sum(2)
    if case["limiter"]:
        qL, qR = _pair_bound(qL, phi[a], phi[b]), _pair_bound(qR, phi[b], phi[a])
    first = ((qL[:, 0] <= 0) | (qL[:, 4] <= 0) | (qR[:, 0] <= 0) | (qR[:, 4] <= 0))[:, None]
    qL, qR = torch.where(first, phi[a], qL).unbind(1), torch.where(first, phi[b], qR).unbind(1)
    w = 0.5 * (phi[a, 1:4] + phi[b, 1:4]).t()
    uL = sum((qL[1 + k] - w[k]) * nh[k] for k in range(3))
    uR = sum((qR[1 + k] - w[k]) * nh[k] for k in range(3))
    cL, cR = torch.sqrt(gamma * qL[4] / qL[0]), torch.sqrt(gamma * qR[4] / qR[0])
    SL, SR = torch.minimum(uL - cL, uR - cR), torch.maximum(uL + cL, uR + cR)
    mL, mR = qL[0] * (SL - uL), qR[0] * (SR - uR)
    Ss = (qR[4] - qL[4] + mL * uL - mR * uR) / (mL - mR)
    wn = (w * nh).sum(0)
    if case["scheme"] == "mfv":
        lft = (SL >= 0) | (Ss >= 0)
        star = torch.where(lft, SL < 0, SR >= 0)
        qk = [torch.where(lft, x_, y_) for x_, y_ in zip(qL, qR)]
        uk, Sk = torch.where(lft, uL, uR), torch.where(lft, SL, SR)
        vp = torch.stack(qk[1:4]) - w
        Ek = qk[4] / (gamma - 1.0) + 0.5 * qk[0] * (vp * vp).sum(0)
        Fm, Fp, FE = qk[0] * uk, qk[0] * vp * uk + qk[4] * nh, (Ek + qk[4]) * uk
        f, du = qk[0] * (Sk - uk) / (Sk - Ss), Ss - uk
        Fm = Fm + torch.where(star, Sk * (f - qk[0]), torch.zeros_like(Fm))
        Fp = Fp + torch.where(star, Sk * (f * (vp + du * nh) - qk[0] * vp), torch.zeros_like(Fp))
        Es = f * (Ek / qk[0] + du * (Ss + qk[4] / (qk[0] * (Sk - uk))))
        FE = FE + torch.where(star, Sk * (Es - Ek), torch.zeros_like(FE))
        FE = (FE + (w * Fp).sum(0) + 0.5 * (w * w).sum(0) * Fm) * Am
        Fp, Fm = (Fp + w * Fm) * Am, Fm * Am
    else:
        Ps = (0.5 * (qL[4] + qR[4] + mL * (Ss - uL) + mR * (Ss - uR))).clamp(min=0.0)
        Fm, Fp, FE = torch.zeros_like(Ps), Ps * A, Ps * (Ss + wn) * Am
    F = torch.stack([Fp[0], Fp[1], Fp[2], FE, Fm], 1)
    F = _sum(n, b, F) - _sum(n, a, F)
    cs = torch.sqrt(gamma * P / rho)
    sig = cs[a] + cs[b] + (((v[:, a] - v[:, b]) * d).sum(0) / r).clamp(min=0.0)
    vsig = torch.zeros_like(H).scatter_reduce(0, a, sig, "amax").scatter_reduce(0, b, sig, "amax")
    out = {"H": H, "nk": nk, "V": V, "B": B.t(), "rho": rho, "P": P, "grad": g.reshape(n, 15).t(),
           "dp": F[:, :3].t(), "dE": F[:, 3], "vsig": vsig}
    if case["scheme"] == "mfv":
        out["dm"] = F[:, 4]
    return out


def _step(case, p, s, o, dt):
    """One kick-drift-kick step of the state s = (x, v, u, m) with pass outputs o."""
    x, v, u, m = s
    h, dm = 0.5 * dt, o.get("dm", torch.zeros_like(m))
    Q, E = m * v, m * (u + 0.5 * (v * v).sum(0))
    Q1, E1, m1 = Q + h * o["dp"], E + h * o["dE"], m + h * dm
    x = _drift(x + dt * Q1 / m1, p)
    m2, v2 = m1 + h * dm, (Q1 + h * o["dp"]) / (m1 + h * dm)
    u2 = ((E1 + h * o["dE"]) / m2 - 0.5 * (v2 * v2).sum(0)).clamp(min=1e-10)
    o = _pass(case, p, x, v2, u2, m2)
    dm = o.get("dm", torch.zeros_like(m))
    m3, E3 = m1 + h * dm, E1 + h * o["dE"]
    v3 = (Q1 + h * o["dp"]) / m3
    return (x, v3, (E3 / m3 - 0.5 * (v3 * v3).sum(0)).clamp(min=1e-10), m3), o


def _drift(x, p):
    b = torch.tensor(p["box"], device="cuda", dtype=F64)[:, None]
    per = torch.tensor(p["periodic"], device="cuda", dtype=F64)[:, None]
    return x - per * b * torch.floor(x.detach() / b)


def _sorted(x, p, levels):
    """The library's particle order: per-axis Morton keys, axis by axis from the longest, stable."""
    top = max(p["box"])
    qb = [max(0, levels - round(math.log2(top / b))) for b in p["box"]]
    key = torch.zeros(x.shape[1], dtype=torch.int64, device="cuda")
    q = [torch.floor(x[d] * (2.0 ** qb[d] / p["box"][d])).long().clamp(0, 2 ** qb[d] - 1) for d in range(3)]
    for l in range(1, levels + 1):
        for d in range(3):
            if l > levels - qb[d]:
                key = (key << 1) | ((q[d] >> (levels - l)) & 1)
    return torch.sort(key, stable=True).indices


def exact(case, seed):
    n, call = _count(case), case["call"]
    if n > EXACT_MAX_N or call == "hier":
        return None
    p = particles(case, seed)
    x, v, u, m = p["x"], p["v"], p["u"], p["m"]
    if call == "evolve":
        v, u = v.clone().requires_grad_(True), u.clone().requires_grad_(True)
        s, o = (x, v, u, m), _pass(case, p, x, v, u, m)
        for _ in range(case["steps"]):
            s, o = _step(case, p, s, o, 1.0e-3)
        (m * (s[1] * s[1]).sum(0)).sum().backward()
        return {"v": s[1].detach(), "u": s[2].detach(), "grad_v0": v.grad, "grad_u0": u.grad}
    levels = 6 if call == "noalloc" else next(b for b in range(31) if 8 ** b >= n) + 2
    order = _sorted(x, p, levels)
    if call == "pass_unpermute":
        order = torch.arange(n, device="cuda")
    more = {}
    if call == "pass_adjoint":
        x, v, u = (t[..., order].clone().requires_grad_(True) for t in (x, v, u))
        m, ids, order = m[order], order, torch.arange(n, device="cuda")
        o = _pass(case, p, x, v, u, m)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(int(seed) + 1)
        adj_dp = torch.randn(3, n, generator=gen, device="cuda", dtype=F64)
        adj_dE = torch.randn(n, generator=gen, device="cuda", dtype=F64)
        ((o["dp"] * adj_dp).sum() + (o["dE"] * adj_dE).sum()).backward()
        more = {"adj_x": x.grad, "adj_v": v.grad, "adj_u": u.grad}
    else:
        o, ids = _pass(case, p, x, v, u, m), order
    if call == "step":
        dts = []
        for _ in range(case["steps"]):
            dt = _fixed_dt(case) or 0.25 * float((o["H"] / o["vsig"]).min())
            (x, v, u, m), o = _step(case, p, (x, v, u, m), o, dt)
            order = order[_sorted(x[:, order], p, levels)]
            dts.append(dt)
        more, ids = {"dt": dts}, order
    o = dict(o, x=x[0], y=x[1], z=x[2], vx=v[0], vy=v[1], vz=v[2], u=u, m=m)
    o = {k: t.detach()[..., order].contiguous() for k, t in o.items()}
    return dict(o, id=ids, **more)
