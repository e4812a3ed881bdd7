"""The normal-equation solve at the sizes where its 16 x 16 blocking can go
wrong: one partial block, a whole number of blocks (the right-hand side then
has a block row of its own), one unknown into the next block, and both sides
of the limits at which more waves take over (48 and 112 unknowns), against the
oracle's fit of the same frames.  The stamp bar is the noisy-data bar of the
FP64 fit, scaled by the ratio of the Jacobi-scaled condition numbers to the
standard basis's where that is larger."""
import numpy as np
import pytest

import oracle
from paper_2207_14304_amd import argus
from test_gpu_stages import NOISY_STAMP_TOL, _fit, _jacobi_cond, _noisy_pair, _ospec, _spec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = argus.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("sigmas,degrees,D,Dbg,n", [
    ((1.5,), (0,), 0, 0, 2),
    ((1.5,), (4,), 0, 0, 16),
    ((0.8, 1.6), (4, 0), 0, 0, 17),
    ((1.5,), (4,), 1, 1, 48),
    ((0.8, 1.6), (4, 0), 1, 0, 49),
    ((0.8, 1.6, 2.6), (4, 1, 0), 1, 1, 60),
    ((0.8, 1.6), (4, 1), 2, 1, 111),
    ((0.8, 1.6), (4, 1), 2, 2, 114),
    ((0.7, 1.5, 3.0), (4, 3, 2), 2, 0, 187),
    ((0.7, 1.5, 3.0), (4, 3, 2), 2, 2, 192),
])
def test_solve_sizes(ctx, sigmas, degrees, D, Dbg, n):
    planes = _noisy_pair(300, 260, 91, n_stars=300)
    spec = argus.make_spec(sigmas=sigmas, degrees=degrees, half_width=7, spatial_degree=D,
                           bg_degree=Dbg, precision=argus.FP64)
    assert argus.kernel_dims(spec) == (n, 1)
    os_ = _ospec(spec)
    co, nf, st, stamps, _, _ = _fit(ctx, spec, planes)
    oco, ost, onf = oracle.fit_kernel(*planes, os_)
    assert st[0] == ost[0] == 0 and nf[0] == onf[0]
    assert co.shape == (1, n) and np.all(np.isfinite(co))
    o_stamps, _ = oracle.expand_kernel(oco, os_)
    err = np.abs(stamps - o_stamps).max() / np.abs(o_stamps).max()
    std = _ospec(_spec(half_width=7, spatial_degree=1, bg_degree=1))
    ratio = max(1.0, _jacobi_cond(planes, os_) / _jacobi_cond(planes, std))
    print(f"n {n}: stamp error {err:.3e}, condition ratio {ratio:.2f}")
    assert err <= NOISY_STAMP_TOL[argus.FP64] * ratio
