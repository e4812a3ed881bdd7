"""FP64 moments of degrees 0 and 1, each wave 16 pixels of a row and the powers
of y from running sums over the rows: strips of one column less, exactly and
one more than 64, odd and even row counts, several row chunks, and tiles of
their own solves, against the FP64 oracle.  Bars as for the other fits (FP64:
stamps 1e-5, chi^2 1e-8), scaled by the ratio of the normal matrix's condition
number to that of the frame the bars were set on: what is left is the FP32
rounding of the basis convolutions, which the system amplifies by it."""
import numpy as np
import pytest

import oracle
from paper_2207_14304_amd import argus
from test_gpu_stages import (NOISY_CHI2_TOL, NOISY_STAMP_TOL, _fit, _jacobi_cond, _noisy_pair, _ospec,
                             _spec)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = argus.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("D", [0, 1])
@pytest.mark.parametrize("W,H", [(77, 95), (78, 96), (79, 97), (143, 120), (333, 281)])
def test_strips_and_rows(ctx, D, W, H):
    planes = _noisy_pair(W, H, W + D, n_stars=max(60, W * H // 400))
    spec = _spec(half_width=7, spatial_degree=D, bg_degree=D, precision=argus.FP64)
    os_ = _ospec(spec)
    co, nf, st, stamps, bg, _ = _fit(ctx, spec, planes)
    oco, ost, onf = oracle.fit_kernel(*planes, os_)
    assert st[0] == ost[0] == 0 and nf[0] == onf[0]
    o_stamps, _ = oracle.expand_kernel(oco, os_)
    ref = _jacobi_cond(_noisy_pair(333, 280, 60 + D + 7, n_stars=250), os_)
    ratio = max(1.0, _jacobi_cond(planes, os_) / ref)
    assert np.abs(stamps - o_stamps).max() <= NOISY_STAMP_TOL[argus.FP64] * ratio * np.abs(o_stamps).max()
    assert abs(oracle.chi2(*planes, os_, co)[0] / oracle.chi2(*planes, os_, oco)[0] - 1) \
        <= NOISY_CHI2_TOL[argus.FP64] * ratio


def test_tiles_of_their_own(ctx):
    planes = _noisy_pair(290, 260, 77, n_stars=400)
    spec = _spec(half_width=7, tiles_x=2, tiles_y=2, mode=argus.FIT_PER_TILE, precision=argus.FP64)
    os_ = _ospec(spec)
    co, nf, st, stamps, bg, _ = _fit(ctx, spec, planes)
    oco, ost, onf = oracle.fit_kernel(*planes, os_)
    assert np.array_equal(st, ost) and np.array_equal(nf, onf)
    o_stamps, _ = oracle.expand_kernel(oco, os_)
    ref = _jacobi_cond(_noisy_pair(333, 280, 67, n_stars=250), _ospec(_spec(half_width=7)))
    from oracle import core
    A = np.asarray(core.normal_equations(*planes, os_)[0])
    cond = 0.0
    for a in A.reshape(-1, A.shape[-2], A.shape[-1]):
        d = np.sqrt(np.diag(a))
        ev = np.linalg.eigvalsh(a / np.outer(d, d))
        cond = max(cond, ev[-1] / ev[0])
    err = np.abs(stamps - o_stamps).max() / np.abs(o_stamps).max()
    assert err <= NOISY_STAMP_TOL[argus.FP64] * max(1.0, cond / ref)
