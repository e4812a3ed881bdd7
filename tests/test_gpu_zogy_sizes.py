"""ZOGY at every tile side the transforms are built for (64..1024: each has its
own radix steps, thread groups and flag words), with flagged pixels at word
and tile edges, the smallest and the largest PSF half-width, an odd number of
tiles, and a tile partly off the frame, against the FP64 oracle (the bars of
the ZOGY parity test: masks bit-exact, D and SNR within 1e-6 of the image's
scale, sum P_D^2 within 1e-12)."""
import numpy as np
import pytest

from oracle import zogy
from paper_2207_14304_amd import argus
from gpu_util import dev, host, empty
from test_gpu_zogy import _psf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,r", [(64, 1), (64, 15), (128, 15), (256, 1), (512, 7), (1024, 15)])
def test_zogy_tile_sides(L, r):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = argus.Context(0)
    rng = np.random.default_rng(L + r)
    H, W = L + 40, L + 75
    N = (30.0 * rng.standard_normal((H, W))).astype(np.float32)
    R = (28.0 * rng.standard_normal((H, W))).astype(np.float32)
    N[L // 2, L // 3] += 5000.0
    mn, mr = (np.zeros((H, W), np.uint8) for _ in range(2))
    for y, x in ((0, 0), (L // 2 + 7, 63), (9, 64), (L + 10, L + 3)):
        mn[y, min(x, W - 1)] = 1
    mr[L // 4, L - 1] = 2
    org = np.array([[0, 0], [W - L, H - L], [-9, L // 2 + 5]], np.int32)
    Pn, Pr = _psf(r, 2.8).astype(np.float32), _psf(r, 2.0).astype(np.float32)
    Fn, Fr, sn, sr = 1.05, 1.0, 30.0, 28.0
    n = len(org)
    D, S, F = (empty((n, L, L), torch.float32) for _ in range(3))
    M, pd2 = empty((n, L, L), torch.uint8), empty(1, torch.float64)
    ctx.zogy(dev(N), dev(mn), dev(R), dev(mr), dev(org), L, dev(Pn), dev(Pr), r, Fn, Fr, sn, sr,
             D, S, F, M, pd2)
    gD, gS, gF, gM, gp = host(D), host(S), host(F), host(M), host(pd2)
    for t, (x0, y0) in enumerate(org):
        Nt, Rt, bad = np.zeros((L, L)), np.zeros((L, L)), np.ones((L, L), np.uint8)
        ys, xs = slice(max(y0, 0), min(y0 + L, H)), slice(max(x0, 0), min(x0 + L, W))
        sub = (slice(ys.start - y0, ys.stop - y0), slice(xs.start - x0, xs.stop - x0))
        Nt[sub], Rt[sub] = N[ys, xs], R[ys, xs]
        bad[sub] = (mn[ys, xs] != 0) | (mr[ys, xs] != 0)
        oD, oS, oF, FD, opd2, oM = zogy.zogy_tile(Nt, Rt, bad, np.zeros_like(bad),
                                                 Pn.astype(np.float64), Pr.astype(np.float64),
                                                 Fn, Fr, sn, sr)
        assert gp[0] == pytest.approx(opd2, rel=1e-12)
        assert np.array_equal(gM[t], oM), t
        assert np.abs(gD[t] - oD).max() <= 1e-6 * max(1.0, np.abs(oD).max())
        assert np.abs(gS[t] - oS).max() <= 1e-6 * max(1.0, np.abs(oS).max())
        assert np.abs(gF[t] - oF).max() * FD * np.sqrt(opd2) <= 1e-6 * max(1.0, np.abs(oS).max())
    ctx.close()
