"""The number of lanes that share a particle's list in the pass reverse changes
with the size of the set: a set at the last size of one form, alone and with a
second set far outside its reach (the other form), has the same adjoints."""
import numpy as np
import pytest

from paper_1712_01294_amd import workloads as W

pytestmark = pytest.mark.gpu

# sums of some hundred terms in another order, each rounded to 2^-53, amplified by
# cond(E) of a jittered lattice's faces and corners (below 1e2): below 1e-11
TOL = 1e-11


def _lattice(side, origin, rng):
    g = (np.arange(side) + 0.5) / side
    X = np.stack(np.meshgrid(g, g, g, indexing="ij")).reshape(3, -1)
    X = X + rng.uniform(-0.2, 0.2, X.shape) / side + np.array(origin)[:, None]
    n = X.shape[1]
    return X, rng.uniform(0.5, 1.5, n) / n, rng.normal(0, 0.2, (3, n)), rng.uniform(1, 2, n)


@pytest.mark.parametrize("side", [32, 12])
def test_pass_adjoint_of_two_sets_out_of_reach(side):
    import torch

    from paper_1712_01294_amd import mfm
    rng = np.random.default_rng(W.SEED_BASE + 795)
    A = _lattice(side, (0.5, 0.5, 0.5), rng)
    more = 32769 - side ** 3 if side < 32 else 125
    B = _lattice(int(np.ceil(more ** (1 / 3))), (6.0, 6.0, 6.0), rng)
    n = A[1].size
    out = []
    for sets in ((A,), (A, B)):
        X = np.concatenate([s[0] for s in sets], 1)
        m = np.concatenate([s[1] for s in sets])
        V = np.concatenate([s[2] for s in sets], 1)
        u = np.concatenate([s[3] for s in sets])
        w = W.Workload(name="two", x=X[0].copy(), y=X[1].copy(), z=X[2].copy(), m=m, vx=V[0].copy(), vy=V[1].copy(),
                       vz=V[2].copy(), u=u, gamma=1.4, box=(8.0, 8.0, 8.0), periodic=(0, 0, 0))
        ctx = mfm.Context(mfm.config_of(w, max_ngb=512), w.n)
        st = mfm.State.from_arrays(w.arrays())
        ctx.build_neighbours(st)
        ctx.hydro_pass(st)
        ctx.check(allow_illcond=True)
        ids = st.id
        g = torch.as_tensor(np.random.default_rng(7).normal(size=(4, n)), device="cuda")
        lam = torch.zeros(4, w.n, dtype=torch.float64, device="cuda")
        lam[:, :n] = g
        ax, av, au = ctx.pass_adjoint(st, lam[:3, ids].contiguous(), lam[3, ids].contiguous())
        got = []
        for t in (ax, av, au):
            full = torch.empty_like(t)
            full[..., ids] = t
            got.append(full[..., :n].cpu().numpy())
        out.append((w.n, got))
    assert out[0][0] <= 32768 < out[1][0]
    for k, a, b in zip(("x", "v", "u"), out[0][1], out[1][1]):
        e = np.abs(a - b).max() / np.abs(a).max()
        print(side, k, f"{e:.1e}", flush=True)
        assert e <= TOL, (k, e)
