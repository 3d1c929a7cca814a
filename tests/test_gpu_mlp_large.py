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
