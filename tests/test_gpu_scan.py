"""The neighbour search of the kernel-length solve against brute force: every
flux list equals the set r < max(H_i, H_j) as integers, and every H solves
(32/3) sum_j w(r_ij / H) = n_ngb over all particles, on sets whose groups span
wide ranges of radii, distances and cell sizes."""
import numpy as np
import pytest

from paper_1712_01294_amd import workloads as W

pytestmark = pytest.mark.gpu

# a sum of at most a few hundred kernel weights <= 1, each rounded to 2^-53 of
# its value and the sum to n_ngb, relative to n_ngb: below 1e-13
TOL_COUNT = 1e-12


def _set(kind, n, seed):
    rng = np.random.default_rng(seed)
    box, per = (1.0, 1.0, 1.0), (1, 1, 1)
    if kind == "uniform":
        X = rng.uniform(0, 1, (3, n))
    elif kind == "slab":
        box = (4.0, 1.0, 0.25)
        X = rng.uniform(0, 1, (3, n)) * np.array(box)[:, None]
    else:
        # two tight clumps in a wide open box: finest cells hold thousands of
        # particles and lie far beyond the spheres of the clumps' members
        box, per = (1000.0, 1000.0, 1000.0), (0, 0, 0)
        X = rng.uniform(0, 1000, (3, n))
        k = min(n // 4, 1500)
        X[:, :k] = 300.0 + 0.5 * rng.normal(size=(3, k))
        X[:, k:2 * k] = 302.0 + 0.02 * rng.normal(size=(3, k))
    return W.Workload(name=kind, x=X[0].copy(), y=X[1].copy(), z=X[2].copy(), m=np.full(n, 1.0 / n),
                      vx=rng.normal(0, 0.1, n), vy=rng.normal(0, 0.1, n), vz=rng.normal(0, 0.1, n),
                      u=np.full(n, 1.5), gamma=5.0 / 3.0, box=box, periodic=per)


# n_ngb 55 and 100: about 64 and 120 radii a particle, up to and past what the root kernel keeps in registers
@pytest.mark.parametrize("kind,n,n_ngb", [("uniform", 300, 32.0), ("uniform", 70001, 32.0), ("slab", 66000, 32.0),
                                          ("clumps", 2500, 32.0), ("clumps", 70003, 32.0), ("slab", 40009, 55.0),
                                          ("uniform", 40009, 100.0),
                                          # the last size solved one wave a particle, the first of the group scan
                                          ("uniform", 49152, 32.0), ("uniform", 49153, 32.0), ("clumps", 49152, 32.0),
                                          ("clumps", 49153, 32.0), ("slab", 50001, 55.0), ("uniform", 50001, 100.0)])
def test_lists_and_kernel_lengths_equal_brute_force(kind, n, n_ngb):
    import dataclasses

    import torch

    from paper_1712_01294_amd import mfm
    w = dataclasses.replace(_set(kind, n, W.SEED_BASE + 700 + n), n_ngb=n_ngb)
    ctx = mfm.Context(mfm.config_of(w, max_ngb=4096), n)
    st = mfm.State.from_arrays(w.arrays())
    ctx.build_neighbours(st)
    ctx.hydro_pass(st)
    ctx.check(allow_illcond=True)
    counts, lst = ctx.flux_lists(n)
    X, H = torch.stack([st.x, st.y, st.z]), st.H
    box = torch.tensor(w.box, dtype=torch.float64, device="cuda")
    worst = 0.0
    step = max(1, 40_000_000 // n)
    for a in range(0, n, step):
        b = min(n, a + step)
        r2 = torch.zeros(b - a, n, dtype=torch.float64, device="cuda")
        for c in range(3):
            d = X[c][None, :] - X[c][a:b, None]
            if w.periodic[c]:
                d -= box[c] * torch.round(d / box[c])
            r2 += d * d
        r = torch.sqrt(r2)
        q = r / H[a:b, None]
        t, h = (1 - q).clamp(min=0), (0.5 - q).clamp(min=0)
        s = (32.0 / 3.0) * (2 * t ** 3 - 8 * h ** 3).sum(1)
        worst = max(worst, float((s / w.n_ngb - 1).abs().max()))
        want = r < torch.maximum(H[a:b, None], H[None, :])
        want[torch.arange(b - a, device="cuda"), torch.arange(a, b, device="cuda")] = False
        got = torch.zeros_like(want)
        k = torch.arange(lst.shape[0], device="cuda")[:, None]
        used = k < counts[a:b][None, :]
        got[torch.arange(b - a, device="cuda").expand_as(used)[used], lst[:, a:b][used].long()] = True
        assert torch.equal(counts[a:b].long(), want.sum(1)), (kind, a)
        assert torch.equal(got, want), (kind, a)
    print(f"{kind} {n}: residual of the neighbour-number equation {worst:.2e}", flush=True)
    assert worst <= TOL_COUNT


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("n", [63, 64, 65, 193])
def test_pass_at_the_edges_of_a_wave(n, precision):
    """Sets that end just before, at and after a wave of 64 particles, in an open
    box: every output against the oracle (the FP64 bar of the other pass tests,
    the mixed bar for the mixed fluxes)."""
    from oracle import oracle as O

    from .gpu_util import compare_pass, run_pass
    rng = np.random.default_rng(W.SEED_BASE + 760 + n)
    w = W.Workload(name="edge", x=rng.uniform(0, 1, n), y=rng.uniform(0, 1, n), z=rng.uniform(0, 1, n),
                   m=rng.uniform(0.5, 1.5, n) / n, vx=rng.normal(0, 0.2, n), vy=rng.normal(0, 0.2, n),
                   vz=rng.normal(0, 0.2, n), u=rng.uniform(1, 2, n), gamma=1.4, box=(1.0, 1.0, 1.0),
                   periodic=(0, 0, 0))
    ref = O.hydro_pass(O.Setup.of(w), w.arrays())
    ctx, st = run_pass(w, precision=precision)
    ctx.check()
    errs = compare_pass(st, ref)
    print(n, precision, " ".join(f"{k}={v:.1e}" for k, v in errs.items()), flush=True)
    for k, e in errs.items():
        if precision == 0 or k in ("H", "nk", "V", "rho", "P"):
            assert e <= 1e-12, (k, e)
        elif k in ("dp", "dE"):
            assert e <= 1e-5, (k, e)


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("n", [49152, 49153, 65536, 65537, 131072, 131073])
def test_pass_on_both_sides_of_the_lane_split(n, precision):
    """The sizes at which the number of lanes that share a particle's list
    changes in the gradients and the fluxes: the first, some middle and the last
    particles (the last, partly filled wave) of a random open set, against the
    oracle on the same sample (the bars of the full passes)."""
    from .gpu_util import in_input_order, nerr, oracle_sample, run_pass
    rng = np.random.default_rng(W.SEED_BASE + 780)
    w = W.Workload(name="split", x=rng.uniform(0, 1, n), y=rng.uniform(0, 1, n), z=rng.uniform(0, 1, n),
                   m=rng.uniform(0.5, 1.5, n) / n, vx=rng.normal(0, 0.2, n), vy=rng.normal(0, 0.2, n),
                   vz=rng.normal(0, 0.2, n), u=rng.uniform(1, 2, n), gamma=1.4, box=(1.0, 1.0, 1.0),
                   periodic=(1, 1, 1))
    ctx, st = run_pass(w, precision=precision)
    ctx.check(allow_illcond=True)
    ids = st.id.cpu().numpy()
    targets = np.concatenate([ids[:8], ids[n // 2:n // 2 + 8], ids[-16:]])
    ref = oracle_sample(w, targets)
    # E^-1 amplifies the rounding of the sums of E by cond(E)
    tol = max(1e-12, 32 * np.finfo(np.float64).eps * float(ref["cond"][targets].max()))
    for k in ("H", "nk", "rho", "P", "dp", "dE") + (() if precision else ("B", "grad", "vsig")):
        e = nerr(in_input_order(st, k)[..., targets], ref[k][..., targets])
        print(n, precision, k, f"{e:.1e}", flush=True)
        bar = 1e-12 if k not in ("B", "grad", "dp", "dE") else 1e-5 if precision else tol
        assert e <= bar, (k, e)
