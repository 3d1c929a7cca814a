"""The surrogate network at sizes where its tiles, its grid and its workspace change."""
import numpy as np
import pytest
import torch

import oracle.mlp as om
import paper_1702_05167_amd as pkg

pytestmark = pytest.mark.gpu


def test_forward_of_millions_of_samples(ctx):
    # more than 65,536 tiles of rows, of either height
    n, widths = 65536 * 64 + 7, (1, 1)
    net = pkg.MLP(ctx, widths)
    net.set_params(np.array([3.0, -1.0], np.float32))
    x = (torch.arange(n, device=ctx.torch_device) % 1021).to(torch.float32)[:, None]
    assert torch.equal(net.forward(x), 3.0 * x - 1.0)


# tiles of 32 rows below 1024 tiles of 64, of 64 rows from there on; whole numbers, exact in any order
@pytest.mark.parametrize("n,widths", [(1023 * 64, (3, 5)), (1024 * 64 - 63, (3, 5)), (1024 * 64 + 1, (9, 64)), (32769, (40, 65)),
                                      (16400, (7, 200)), (65, (8, 3)), (33, (33, 1))])
def test_forward_exact(ctx, n, widths):
    rng = np.random.default_rng(n)
    net = pkg.MLP(ctx, widths)
    p = rng.integers(-3, 4, net.get_params().numel()).astype(np.float32)
    net.set_params(p)
    x = rng.integers(-3, 4, (n, widths[0])).astype(np.float32)
    k, m = widths
    assert np.array_equal(net.forward(x).cpu().numpy(), x @ p[:k * m].reshape(m, k).T + p[k * m:])


def test_gradients_through_wide_tiles(ctx):
    # the gradient flowing back takes 64-row tiles as well
    n, widths = 66000, (4, 70, 3)
    rng = np.random.default_rng(2)
    net = pkg.MLP(ctx, widths)
    p = (0.3 * rng.standard_normal(net.get_params().numel())).astype(np.float32)
    net.set_params(p)
    x, t = rng.standard_normal((n, 4)).astype(np.float32), rng.standard_normal((n, 3)).astype(np.float32)
    g, _ = net.grads(x, t)
    ref = om.grads(p.astype(np.float64), widths, x.astype(np.float64), t.astype(np.float64))
    # FP32 sums of 66000 terms of one sign pattern at random: 2^-24 sqrt(66000) of the terms' rms, in practice less
    assert np.abs(g.cpu().numpy() - ref).max() <= 2e-5 * np.abs(ref).max()


def test_evaluation_allocates_no_gradients(ctx):
    dev = ctx.torch_device
    net = pkg.MLP(ctx, (1024, 1024))
    x = torch.zeros((2048, 1024), device=dev)
    y = torch.empty((2048, 1024), device=dev)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    y = net.forward(x)
    torch.cuda.synchronize()
    # the workspace of 2048 samples, 8 MiB a buffer, and the output; the gradients' chunks would be 63 MB more
    assert free - torch.cuda.mem_get_info()[0] <= 72 << 20
    g, _ = net.grads(x, torch.ones_like(y))
    assert float(g[-1]) == pytest.approx(-2.0 / 1024, rel=1e-5)
