"""Subtraction blocks of 64x16 pixels (four pixels a thread) and 128x16 (eight):
widths at and beside their edges, an odd pitch, the one and the other form of
the degree-0 kernel, tiles of their own solves, and the allocation-free entry,
against the FP64 oracle with the same stamps (the bars of the stage tests)."""
import numpy as np
import pytest

import oracle
from paper_2207_14304_amd import argus
from gpu_util import dev, empty, host
from test_gpu_stages import _check_subtract, _ospec, _run_subtract, _spec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = argus.Context(0)
    yield c
    c.close()


def _planes(W, H, seed):
    r = np.random.default_rng(seed)
    f = lambda a: a.astype(np.float32)
    img = lambda: f(200 + 15 * r.standard_normal((H, W)) + 3000 * (r.random((H, W)) < 0.01))
    var = lambda: f(200 + 20 * r.random((H, W)))
    flag = lambda p: np.where(r.random((H, W)) < p, oracle.BAD, 0).astype(np.uint8)
    return img(), var(), flag(1e-3), img(), var(), flag(2e-3)


def _stamps(spec, n_solves, seed):
    r = np.random.default_rng(seed)
    K = 2 * spec.half_width + 1
    n = (spec.spatial_degree + 1) * (spec.spatial_degree + 2) // 2
    u = np.arange(K) - spec.half_width
    g = np.exp(-(u[:, None] ** 2 + u[None] ** 2) / 8.0)
    g /= g.sum()
    st = g * (1 + 0.3 * r.standard_normal((n_solves, n, K, K)))
    st[:, 1:] *= 0.2
    nb = (spec.bg_degree + 1) * (spec.bg_degree + 2) // 2
    return st.astype(np.float32), (3 * r.standard_normal((n_solves, nb))).astype(np.float32)


@pytest.mark.parametrize("D,h,W,H,tiles", [
    (1, 7, 63, 40, 0), (1, 7, 64, 47, 0), (2, 7, 65, 49, 0), (2, 10, 127, 60, 0),
    (2, 4, 129, 33, 0), (1, 15, 191, 80, 0), (0, 7, 193, 64, 0), (0, 7, 66, 48, 0),
    (0, 5, 1037, 561, 0),            # 9 x 36 blocks of eight pixels
    (2, 3, 260, 150, 3), (0, 6, 333, 200, 4),
])
def test_block_edges(ctx, D, h, W, H, tiles):
    spec = _spec(half_width=h, spatial_degree=D, bg_degree=min(D, 1),
                 **(dict(tiles_x=tiles, tiles_y=2, mode=argus.FIT_PER_TILE) if tiles else {}))
    n = 2 * tiles if tiles else 1
    st, bg = _stamps(spec, n, W)
    planes = _planes(W, H, 7 * W + H)
    g = _run_subtract(ctx, spec, st, bg, planes)
    o = oracle.subtract(st, bg, *planes, _ospec(spec))
    _check_subtract(g, o)


@pytest.mark.parametrize("off", [0, 1, 3])
def test_unaligned_outputs_and_noalloc(ctx, off):
    """Outputs whose first pixel lies off a 16-byte boundary, and the
    allocation-free entry, give the bits of aligned outputs."""
    import torch
    W, H = 201, 57
    spec = _spec(half_width=6, spatial_degree=2, bg_degree=1)
    st, bg = _stamps(spec, 1, 3)
    d = [dev(p) for p in _planes(W, H, 11)]
    res = []
    for o, noalloc in ((0, False), (off, True)):
        fl = torch.zeros((2, W * H + 8), dtype=torch.float32, device="cuda")
        m = torch.zeros(W * H + 8, dtype=torch.uint8, device="cuda")
        D, V = (fl[i, o:o + W * H].view(H, W) for i in (0, 1))
        M = m[o:o + W * H].view(H, W)
        c2 = empty(1, torch.float64)
        ctx.subtract(spec, dev(st), dev(bg), *d, D, V, M, c2, noalloc=noalloc)
        torch.cuda.synchronize()
        res.append([host(x).copy() for x in (D, V, M, c2)])
    for a, b in zip(*res):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("D,h,W,H", [(0, 3, 1021, 256), (0, 4, 1024, 240), (2, 2, 1024, 512), (2, 2, 1024, 500),
                                     (1, 3, 2048, 1024), (2, 5, 2045, 1000)])
def test_narrow_kernels_turn_earlier(ctx, D, h, W, H):
    """On and one row of blocks under the block counts where narrow kernels go
    from four to eight pixels a thread."""
    spec = _spec(half_width=h, spatial_degree=D, bg_degree=min(D, 1))
    st, bg = _stamps(spec, 1, W)
    planes = _planes(W, H, W + H)
    g = _run_subtract(ctx, spec, st, bg, planes)
    _check_subtract(g, oracle.subtract(st, bg, *planes, _ospec(spec)))
