"""The neighbour order against a stable sort of the Morton keys on the CPU, with
many particles to a cell, at the edges of the one-block sort's rounds and of its
range (16,384 particles; the tiled sort beyond)."""
import numpy as np
import pytest

from paper_1712_01294_amd import workloads as W

pytestmark = pytest.mark.gpu


def _keys(X, levels, box):
    q = [np.clip(np.floor(X[d] * ((1 << levels) / box)), 0, (1 << levels) - 1).astype(np.uint64) for d in range(3)]
    key = np.zeros(X.shape[1], np.uint64)
    for lev in range(levels - 1, -1, -1):
        for d in range(3):
            key = (key << np.uint64(1)) | ((q[d] >> np.uint64(lev)) & np.uint64(1))
    return key


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1025, 4095, 4096, 4097, 8192, 8193, 16383, 16384, 16385])
def test_order_is_the_stable_sort_of_the_keys(n):
    import torch

    from paper_1712_01294_amd import mfm
    rng = np.random.default_rng(W.SEED_BASE + 810 + n)
    X = rng.uniform(0, 1, (3, n))
    X[:, ::3] = np.round(X[:, ::3] * 4) / 4 * 0.999   # a third of them in 125 places
    levels = max(2, int(np.ceil(np.log2(np.cbrt(float(n))) - 1e-12)) + 2)
    w = W.Workload(name="sort", x=X[0].copy(), y=X[1].copy(), z=X[2].copy(), m=np.full(n, 1.0 / n),
                   vx=np.zeros(n), vy=np.zeros(n), vz=np.zeros(n), u=np.ones(n), gamma=1.4, box=(1.0, 1.0, 1.0),
                   periodic=(1, 1, 1))
    ctx = mfm.Context(mfm.config_of(w), n)
    st = mfm.State.from_arrays(w.arrays())
    for _ in range(2):   # a second build finds the particles sorted
        ctx.build_neighbours(st)
        torch.cuda.synchronize()
        want = np.argsort(_keys(X, levels, 1.0), kind="stable")
        assert np.array_equal(st.id.cpu().numpy(), want)
        for c, k in enumerate("xyz"):
            assert np.array_equal(getattr(st, k).cpu().numpy(), X[c][want])

