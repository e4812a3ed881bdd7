"""Convolution workgroups stay on the chip and take several bands each once a
batch has more bands than resident workgroups (two per compute unit).  A batch
of 8 tiles with 384 valid stamps (768 bands) against its tiles run one by one:
the outputs are the same bits (a band's arithmetic does not depend on who
computes it), and the gradients are the mean of the tiles' gradients.  The loss
is a mean over tiles, so the batch's backward signal is each tile's divided by
8, exactly; what differs is the order of FP32 sums over at most 384 stamps and
961 pixels, rounding errors of about 6e-8 each that add like a random walk over
the 64 partial sums they pass through: 5e-7 of the gradient's norm, bar 1e-5."""
import numpy as np
import pytest

from paper_2207_14304_amd import argus, surrogate
from gpu_util import dev, host, empty

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [(64, 63, 1, 0, 64, 64, 64, 64), (1, 0, 0, 2, 0, 0, 0, 0)])
def test_bands_beyond_the_resident_workgroups(counts):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = argus.Context(0)
    T, S = len(counts), 64
    g = torch.Generator().manual_seed(3)
    X = torch.rand((T, S, 961, 2), generator=g).to(torch.bfloat16).cuda()
    valid = torch.zeros((T, S), dtype=torch.uint8)
    for t, c in enumerate(counts):
        valid[t, torch.randperm(S, generator=g)[:c]] = 1
    valid = valid.cuda()
    tgt = (0.1 * torch.randn((T, 31), generator=g)).cuda()
    flat = surrogate.init_weights(5).astype(np.float32)

    def run(sl):
        n = X[sl].shape[0]
        cnn = argus.CNN(ctx, n)
        cnn.set_weights(flat)
        out, loss = empty((n, 31), torch.float32), torch.zeros(1, dtype=torch.float64, device="cuda")
        x, v = X[sl].contiguous(), valid[sl].contiguous()
        cnn.forward(x, v, out)
        cnn.train_step(x, v, tgt[sl].contiguous(), 0.0, loss)
        r = host(out).copy(), cnn.get_grads().astype(np.float64), float(host(loss)[0])
        cnn.close()
        return r

    out, grad, loss = run(slice(0, T))
    parts = [run(slice(t, t + 1)) for t in range(T)]
    assert np.array_equal(out, np.concatenate([p[0] for p in parts]))
    assert abs(loss / np.mean([p[2] for p in parts]) - 1) <= 1e-6
    mean = np.mean([p[1] for p in parts], axis=0)
    assert np.isfinite(mean).all() and np.linalg.norm(mean) > 0
    assert np.linalg.norm(grad - mean) <= 1e-5 * np.linalg.norm(mean)
    ctx.close()
