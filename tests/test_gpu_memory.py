"""Solves where the workspace with kept residues does not fit the free memory: the same values from a plan without."""
import ctypes as C

import numpy as np
import pytest
import torch

import synth
import paper_1702_05167_amd as pkg
import paper_1702_05167_amd.hsc as H

pytestmark = pytest.mark.gpu


def _up(v, a):
    return -(-v // a) * a


def _kept_bytes(tree):
    """Residues that a plan keeps per energy: Psi, and Psi^T and A_ii^-1 of the separators"""
    t = tree.export()
    inner = set(t["parent"].tolist())
    total = 0
    for i, (p, n) in enumerate(zip(t["parent"].tolist(), t["size"].tolist())):
        f = int(t["front_ptr"][i + 1] - t["front_ptr"][i])
        if p < 0:
            continue
        if f >= 32:
            total += 64 * _up(n, 32) * _up(f, 64)
        if i in inner and n >= 32:
            total += 64 * (_up(f, 32) + _up(n, 32)) * _up(n, 64)
    return total


def test_batch_that_fits_without_kept_residues():
    dev = synth.config1_device(n_side=16)
    tree = pkg.Tree.from_device(dev, leaf_side=8)
    ne = 24
    E = torch.tensor(np.linspace(-4.0, 4.0, ne), device="cuda:0")
    kw = dict(eta=1e-8, kT=0.025, mu_L=0.1, mu_R=-0.1, want=H.HSC_DIAG_GR | H.HSC_DIAG_GL | H.HSC_TRANS, batch=ne)
    ctx = pkg.Context(0)
    ref = pkg.solve(ctx, tree, E, **kw)     # (torch's pool holds the outputs from here on)
    ctx.sync()
    ctx.close()
    del ctx
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx = pkg.Context(0)
    again = pkg.solve(ctx, tree, E, **kw)
    ctx.sync()
    used = free - torch.cuda.mem_get_info()[0]
    ctx.close()
    del ctx, again
    kept = ne * _kept_bytes(tree)
    assert 0 < kept < used
    torch.cuda.synchronize()
    room = used - kept // 2
    hip = C.CDLL("libamdhip64.so")
    hog = []
    ctx = pkg.Context(0)
    try:
        while torch.cuda.mem_get_info()[0] > room:   # (a large allocation may take less than was asked for)
            hog.append(C.c_void_p())
            assert hip.hipMalloc(C.byref(hog[-1]), C.c_size_t(max(torch.cuda.mem_get_info()[0] - room, 32 << 20))) == 0
        out = pkg.solve(ctx, tree, E, **kw)
        ctx.sync()
        for k in ("gr", "gl", "trans", "status"):
            assert torch.equal(out[k], ref[k]), k
    finally:
        ctx.close()
        for q in hog:
            hip.hipFree(q)
    assert torch.cuda.mem_get_info()[0] > free - (64 << 20)
