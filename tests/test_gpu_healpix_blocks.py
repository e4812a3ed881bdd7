"""Segment resampling where its 32 x 32 blocks and short series meet their
limits, against the oracle (the bars of the resampling parity test): segment
sides one under, at and over a block, each block size (segments as fine as the
frame, half as fine, coarser), blocks that the frame only touches,
tiles at a pole and wide-angle tiles (offsets beyond the series), the mixed
tiles on the polar cap's edge, a frame much finer than the segment (its box
does not fit) and frames one pixel wide or high."""
import numpy as np
import pytest

from oracle import healpix as hp
from paper_2207_14304_amd import argus
from gpu_util import dev, host, empty
from test_gpu_healpix import _near_boundary, _ulps, _wcs_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,ra0,dec0,rot,scale,nside,m", [
    (60, 50, 83.6, 22.0, 0.3, 1.38, 256, 31),
    (900, 700, 83.6, -40.2, 0.4, 1.38, 256, 301),
    (900, 700, 83.6, 70.0, 1.1, 1.38, 256, 601),
    (300, 260, 83.6, -22.0, 0.3, 30.0, 256, 32),
    (300, 260, 211.0, 41.8, 0.8, 25.0, 256, 33),
    (500, 400, 45.3, 89.93, 0.2, 5.0, 256, 160),
    (500, 400, 300.0, -89.99, 0.2, 5.0, 256, 160),
    (200, 180, 10.0, 60.0, 0.0, 900.0, 2, 70),
    (200, 180, 350.0, -5.0, 0.4, 900.0, 1, 90),
    (700, 640, 83.6, 35.0, 0.3, 0.25, 256, 300),
    (1, 300, 83.6, 22.0, 0.0, 4.0, 256, 200),
    (300, 1, 83.6, 22.0, 0.0, 4.0, 256, 200),
])
def test_blocks(W, H, ra0, dec0, rot, scale, nside, m):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = argus.Context(0)
    wo, wg = _wcs_pair(W, H, ra0, dec0, rot, scale)
    tiles = argus.healpix_tiles(wg, W, H, nside, 8)
    rng = np.random.default_rng(W + m)
    cal = rng.normal(100.0, 30.0, (H, W)).astype(np.float32)
    var = rng.uniform(10.0, 50.0, (H, W)).astype(np.float32)
    mask = (rng.random((H, W)) < 0.01).astype(np.uint8) * 4
    n = len(tiles)
    out, ov, om = (empty((n, m, m), torch.float32), empty((n, m, m), torch.float32),
                   empty((n, m, m), torch.uint8))
    ctx.resample_healpix(dev(cal), dev(var), dev(mask), wg, nside, m, dev(tiles.astype(np.int32)),
                         out, ov, om)
    ot = [tuple(t) for t in tiles.tolist()]
    val, vv, mm = hp.resample(cal, var, mask, wo, ot, nside, m)
    g, gv, gm = host(out), host(ov), host(om)
    near = _near_boundary(wo, ot, nside, m, W, H)
    ok = (mm == 0) & (gm == 0)
    print(f"{W}x{H} dec {dec0} nside {nside} m {m}: {n} tiles, {int(ok.sum())} pixels with data")
    assert near.sum() <= 4 or W == 1 or H == 1
    assert np.array_equal(gm[~near], mm[~near])
    if W > 1 and H > 1:
        assert ok.any()
    if ok.any():
        assert _ulps(g[ok], val[ok]).max() <= 2 and _ulps(gv[ok], vv[ok]).max() <= 2
    assert np.all(g[gm != 0] == 0) and np.all(gv[gm != 0] == 0)
    ctx.close()


@pytest.mark.parametrize("rot,m", [(0.785, 560), (0.1, 530), (0.785, 450), (0.3, 447)])
def test_larger_boxes(rot, m):
    """Segments a little coarser than the frame: boxes of 3000 and 4000 pixels,
    with the frame along the segment's diagonals (widest box) and across them."""
    test_blocks(700, 600, 83.6, 33.0, rot, 1.38, 256, m)
