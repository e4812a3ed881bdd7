"""Background cells whose last column is 32 or 64 pixels wide but starts between
the 16-byte words of its row (boxes that are no multiple of 4), beside ones that
start on them: levels bit-exact against the oracle's medians."""
import numpy as np
import pytest

from oracle import background as bk
from paper_2207_14304_amd import argus
from gpu_util import dev, host, empty, padded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,box", [(82, 50), (65, 33), (95, 63), (150, 59), (84, 52), (128, 64)])
def test_last_cell_of_a_word_width(W, box):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = argus.Context(0)
    H = 70
    rng = np.random.default_rng(W)
    cal = rng.normal(800.0, 30.0, (H, W)).astype(np.float32)
    mask = (rng.random((H, W)) < 0.03).astype(np.uint8)
    pad = -W % 4 + 4                                   # a pitch of whole 16-byte words
    lev, grid = (empty((-(-H // box), -(-W // box)), torch.float32) for _ in range(2))
    ctx.background(padded(dev(cal), pad), padded(dev(mask), pad), box, grid, lev)
    o = bk.cell_levels(cal.astype(np.float64), mask, box).astype(np.float32)
    assert np.array_equal(host(lev), o)
    ctx.close()


# cells of at most a pixel a thread (256), one more, and 256 pixels in words
@pytest.mark.parametrize("W,H,box", [(61, 43, 4), (64, 48, 16), (68, 51, 17), (64, 40, 32)])
def test_small_cells(W, H, box):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = argus.Context(0)
    rng = np.random.default_rng(box)
    cal = rng.normal(800.0, 30.0, (H, W)).astype(np.float32)
    mask = (rng.random((H, W)) < 0.1).astype(np.uint8)
    lev, grid = (empty((-(-H // box), -(-W // box)), torch.float32) for _ in range(2))
    ctx.background(dev(cal), dev(mask), box, grid, lev)
    o = bk.cell_levels(cal.astype(np.float64), mask, box).astype(np.float32)
    assert np.array_equal(host(lev), o, equal_nan=True)
    ctx.close()
