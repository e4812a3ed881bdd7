"""Solves that cover few columns of a wide frame (FP32, degree 2, 6144 columns):
one to seven 64-column strips as a tile of its own at the frame's centre, or as
the only unmasked columns of a GLOBAL fit.  In such a system every x-power about
the strip's centre is a diagonal of its own, so each has to be accurate in
itself.  Stamps and difference images against the FP64 oracle's solution.

Bars, as for the other wide fits: stamps 1e-4 times the ratio q of the
Jacobi-scaled condition numbers to the standard frame's where that is larger;
difference image RMS 1e-4 sigma times sqrt(q) (with r the moments' error, the
solution's is A^-1 r and the difference's square r' A^-1 r), maximum 1e-2 sigma."""
import numpy as np
import pytest

import oracle
from paper_2207_14304_amd import argus
from test_gpu_stages import (NOISY_STAMP_TOL, _fit, _jacobi_cond, _noisy_pair, _ospec,
                             _run_subtract, _spec)

pytestmark = pytest.mark.gpu

W, H, h = 6144, 140, 7


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = argus.Context(0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def planes():
    return _noisy_pair(W, H, 41, n_stars=2400)


@pytest.fixture(scope="module")
def std_cond():
    return _jacobi_cond(_noisy_pair(333, 280, 69, n_stars=250),
                        _ospec(_spec(half_width=7, spatial_degree=2, bg_degree=2)))


# (first column, columns): tiles of the frame cut into 96, 64, 48, 24 and 15
# columns of tiles, and masked GLOBAL fits in the middle of the frame and
# across a strip's edge
@pytest.mark.parametrize("mode,x0,cols", [
    (argus.FIT_PER_TILE, 3008, 64), (argus.FIT_PER_TILE, 3072, 96), (argus.FIT_PER_TILE, 2944, 128),
    (argus.FIT_PER_TILE, 3072, 256), (argus.FIT_PER_TILE, 2867, 409),
    (argus.FIT_GLOBAL, 3008, 128), (argus.FIT_GLOBAL, 3040, 90)])
def test_few_columns(ctx, planes, std_cond, mode, x0, cols):
    sel = list(planes)
    sel[5] = np.full_like(planes[5], oracle.BAD)        # science mask: only these columns fit
    sel[5][:, x0:x0 + cols] = planes[5][:, x0:x0 + cols]
    one = _spec(half_width=h, spatial_degree=2, bg_degree=2)
    os_ = _ospec(one)
    oco, ost, onf = oracle.fit_kernel(*sel, os_)
    o_stamps, o_bg = oracle.expand_kernel(oco, os_)
    assert ost[0] == 0
    if mode == argus.FIT_PER_TILE:
        tiles = W // cols
        t = -(-x0 * tiles // W)
        assert t * W // tiles == x0 and (t + 1) * W // tiles == x0 + cols
        spec = _spec(half_width=h, spatial_degree=2, bg_degree=2, tiles_x=tiles, tiles_y=1, mode=mode)
        co, nf, st, stamps, bg, _ = _fit(ctx, spec, planes)
    else:
        t = 0
        co, nf, st, stamps, bg, _ = _fit(ctx, one, sel)
    assert st[t] == 0 and nf[t] == onf[0]
    err = np.abs(stamps[t] - o_stamps[0]).max() / np.abs(o_stamps).max()
    ratio = max(1.0, _jacobi_cond(sel, os_) / std_cond)
    D, V, m, _, _ = _run_subtract(ctx, one, stamps[t:t + 1], bg[t:t + 1], sel)
    oD, _, _, _, _ = _run_subtract(ctx, one, o_stamps, o_bg, sel)
    ok = m == 0
    z = (D - oD)[ok] / np.sqrt(V[ok])
    rms, top = np.sqrt(np.mean(z.astype(np.float64) ** 2)), np.abs(z).max()
    print(f"{cols} columns at {x0}: stamp error {err:.2e} (condition ratio {ratio:.1f}), "
          f"difference RMS {rms:.2e} max {top:.2e} sigma")
    assert err <= NOISY_STAMP_TOL[argus.FP32] * ratio
    assert rms <= 1e-4 * np.sqrt(ratio) and top <= 1e-2
