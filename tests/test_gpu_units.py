"""Passes in units far from one, against the oracle: masses and lengths scaled
by powers of two, so that squared distances leave the range of FP32 and density
times pressure that of the joint square roots and reciprocals of the flux
pairs, below and above."""
import dataclasses

import numpy as np
import pytest

from paper_1712_01294_amd import workloads as W

pytestmark = pytest.mark.gpu


# powers of two of the masses and of the lengths: rho P of about 2^-800, 2^720, 2^-540 and 2^-940
@pytest.mark.parametrize("scheme", ["mfm", "mfv"])
@pytest.mark.parametrize("mass,length", [(-400, 0), (0, -120), (0, 90), (-200, 90), (0, 0)])
def test_pass_in_far_units(mass, length, scheme):
    from oracle import oracle as O

    from paper_1712_01294_amd import mfm

    from .gpu_util import compare_pass, run_pass
    n = 300
    rng = np.random.default_rng(W.SEED_BASE + 790)
    s = 2.0 ** length
    X = rng.uniform(0, s, (3, n))
    w = W.Workload(name="units", x=X[0].copy(), y=X[1].copy(), z=X[2].copy(),
                   m=rng.uniform(0.5, 1.5, n) / n * 2.0 ** mass, vx=rng.normal(0, 0.2, n),
                   vy=rng.normal(0, 0.2, n), vz=rng.normal(0, 0.2, n), u=rng.uniform(1, 2, n), gamma=1.4,
                   box=(s, s, s), periodic=(0, 0, 0))
    kw = {} if scheme == "mfm" else {"scheme": mfm.SCHEME_MFV}
    ref = O.hydro_pass(dataclasses.replace(O.Setup.of(w), scheme=scheme), w.arrays())
    ctx, st = run_pass(w, **kw)
    ctx.check(allow_illcond=True)
    errs = compare_pass(st, ref)
    print(mass, length, scheme, " ".join(f"{k}={v:.1e}" for k, v in errs.items()), flush=True)
    for k, e in errs.items():
        assert e <= 1e-12, (k, e)   # the FP64 bar of the other pass tests
