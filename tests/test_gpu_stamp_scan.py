"""Stamp extraction by many workgroups per tile (the passes over the pixels in
their own kernels, scratch in X) against the one-workgroup form, which takes
over where X is not 4-byte aligned: bit-identical stamps, validity and overflow
for ragged tiles, tiles of a few pixels, masked tiles, odd and even numbers of
unmasked pixels, negative and constant skies, and more candidates than the
list holds."""
import numpy as np
import pytest

from paper_2207_14304_amd import argus
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


def _frame(W, H, seed, level, kind):
    rng = np.random.default_rng(seed)
    ref = np.full((H, W), level, np.float32)
    if kind != "flat":
        ref += (5.0 * rng.standard_normal((H, W))).astype(np.float32)
        for _ in range(max(3, W * H // 2000)):
            y, x = rng.integers(1, H - 1), rng.integers(1, W - 1)
            ref[y - 1:y + 2, x - 1:x + 2] += np.float32(rng.uniform(50, 4000)) * \
                np.array([[.3, .6, .3], [.6, 1, .6], [.3, .6, .3]], np.float32)
    sci = (ref * 1.03 + rng.standard_normal((H, W))).astype(np.float32)
    var = np.full((H, W), 25.0, np.float32)
    mask = (rng.random((H, W)) < 1e-3).astype(np.uint8)
    if kind == "masked":
        mask[: H // 2, : W // 2] = 1
    return ref, var, mask, sci


@pytest.mark.parametrize("W,H,TX,TY,snr,level,kind", [
    (333, 280, 3, 2, 10.0, 800.0, "stars"),
    (1001, 61, 4, 1, 10.0, -300.0, "stars"),
    (130, 127, 1, 1, 5.0, 0.0, "stars"),
    (256, 256, 2, 2, 10.0, 800.0, "masked"),
    (97, 80, 1, 1, 10.0, 800.0, "flat"),
    (70, 70, 35, 7, 10.0, 800.0, "stars"),
    (640, 640, 1, 1, 1e-6, 800.0, "stars"),     # more maxima than the list's 26 624
])
def test_scan_kernels_match_one_workgroup(W, H, TX, TY, snr, level, kind):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = argus.Context(0)
    ref, var, mask, sci = _frame(W, H, W + H, level, kind)
    planes = [dev(a) for a in (ref, var, mask, sci)]
    T, n = TX * TY, TX * TY * argus.CNN_STAMPS * argus.CNN_NPX * 2
    got = []
    for off in (0, 1):
        buf = torch.full((n + 2,), 7.0, dtype=torch.bfloat16, device="cuda")
        X = buf[off:off + n].view(T, argus.CNN_STAMPS, argus.CNN_NPX, 2)
        assert X.data_ptr() % 4 == 2 * off
        valid = torch.full((T, argus.CNN_STAMPS), 9, dtype=torch.uint8, device="cuda")
        ovf = torch.zeros(1, dtype=torch.int32, device="cuda")
        ctx.extract_stamps(planes[0], planes[1], planes[2], planes[3], planes[2], TX, TY, snr, X,
                           valid, ovf)
        got.append((host(X.contiguous().view(torch.int16)), host(valid), host(ovf)))
        assert float(buf[n + 1]) == 7.0
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    print(f"{W}x{H} {TX}x{TY}: {int(got[0][1].sum())} stamps, overflow {int(got[0][2][0])}")
    ctx.close()
