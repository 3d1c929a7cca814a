"""Kernels at the sizes where their splits change: edges of tiles, of panels and of chunks, remainders,
the smallest sizes.  References: exact rational arithmetic, NumPy in complex128, the float64 oracle."""
from fractions import Fraction as F

import numpy as np
import pytest
import torch

import oracle.mlp as om
import paper_1702_05167_amd as pkg
import paper_1702_05167_amd.hsc as H

pytestmark = pytest.mark.gpu


def _zdd(x):
    """(..., 4) double-double values of the complex128 array x"""
    out = np.zeros(x.shape + (4,))
    out[..., 0], out[..., 2] = x.real, x.imag
    return out


def _fr(v):
    return F(float(v[0])) + F(float(v[1])), F(float(v[2])) + F(float(v[3]))


def _dot(a, b):
    """exact sum of products of two vectors of double-double values"""
    re = im = F(0)
    for x, y in zip(a, b):
        xr, xi = _fr(x)
        yr, yi = _fr(y)
        re += xr * yr - xi * yi
        im += xr * yi + xi * yr
    return re, im


# Panels take 1, 2, 4 or 8 waves of one row a thread, then 2 rows, then panels of 4 columns with 4 rows (and of 2
# columns with 8); super-panels are 64 columns, their remainders up to 16 and 32 columns pack rows in the rank
# update; beyond 512 a third level of 256 columns.
@pytest.mark.parametrize("matrix_cores", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 63, 64, 65, 80, 81, 96, 97, 128, 129, 256, 257, 512, 513, 641, 1024, 1025, 2049])
def test_zinv_dd_sizes(ctx, n, matrix_cores):
    # a row permutation of 4 I + G, G with eigenvalues inside the unit circle: condition below 2, pivots off
    # the diagonal.  Each entry of A Y - I sums n products whose factors carry the errors of n elimination
    # steps at 2^-104 (or K 0.8 2^-104 of the residue products) with entries up to 5: 64 n 2^-104
    rng = np.random.default_rng(n)
    A = 4.0 * np.eye(n) + (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / np.sqrt(2.0 * n)
    A = _zdd(A[rng.permutation(n)])
    Y, st = H.kern_zinv_dd(ctx, torch.tensor(A, device=ctx.torch_device), matrix_cores=matrix_cores)
    Y = Y.cpu().numpy()
    assert int(st.cpu()[0]) == 0
    picks = {(i, j) for i in (0, n - 1) for j in (0, n - 1)}
    picks |= {(int(i), int(j)) for i, j in rng.integers(0, n, (12, 2))}
    picks |= {(i, i) for i in rng.integers(0, n, 6).tolist()}
    for i, j in sorted(picks):
        re, im = _dot(A[i], Y[:, j])
        err = max(abs(float(re - (1 if i == j else 0))), abs(float(im)))
        assert err <= 64 * n * 2.0 ** -104, (i, j, err)
    # and every entry in 64 bits: rounding of Y and of the product
    a, y = A[..., 0] + 1j * A[..., 2], Y[..., 0] + 1j * Y[..., 2]
    assert np.abs(a @ y - np.eye(n)).max() <= 64 * n * 2.0 ** -53


# residue products: 64 x 32 tiles, operands padded to 32 rows, k steps of 64 whose splits cover 512 or 1024 deep
# pieces, K rounded up to 64
@pytest.mark.parametrize("config", [3, 4])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (1, 33, 64), (32, 32, 65), (64, 32, 128), (65, 31, 63), (97, 1, 512), (16, 64, 513),
                                   (2, 3, 1024), (33, 2, 1087), (130, 66, 33)])
def test_residue_product_edges(ctx, M, N, K, config):
    rng = np.random.default_rng(M + 100 * N + K)
    a = _zdd(rng.standard_normal((M, K)) + 1j * rng.standard_normal((M, K)))
    b = _zdd(rng.standard_normal((K, N)) + 1j * rng.standard_normal((K, N)))
    a[..., 1], a[..., 3], b[..., 1], b[..., 3] = (0.4 * np.spacing(np.abs(v)) * s for v, s in
                                                  ((a[..., 0], 1), (a[..., 2], -1), (b[..., 0], -1), (b[..., 2], 1)))
    dev = ctx.torch_device
    D = H.kern_zgemm_dd(ctx, 0, 0, torch.tensor(a, device=dev), torch.tensor(b, device=dev), config=config).cpu().numpy()
    # operands rounded to S 7-bit digits below a power of two under twice the row's largest part: K products miss
    # 2 2^-7S of both largest each, real and imaginary sums of two; the result is rounded to double-double
    S = {3: 16, 4: 15}[config]
    part = lambda v: np.maximum(np.abs(v[..., 0]), np.abs(v[..., 2]))
    ra, cb = part(a).max(1), part(b).max(0)
    picks = {(i, j) for i in {0, M // 2, M - 1} for j in {0, N // 2, N - 1}} | {(int(i) % M, int(j) % N) for i, j in rng.integers(0, 4096, (6, 2))}
    for i, j in sorted(picks):
        re, im = _dot(a[i], b[:, j])
        got = _fr(D[i, j])
        bound = K * ra[i] * cb[j] * (16 * 2.0 ** (-7 * S) + 2.0 ** -104)
        assert max(abs(float(got[0] - re)), abs(float(got[1] - im))) <= bound, (i, j)


# complex128: blocks of 16 outputs that an edge tile leaves out, C read ahead of the product, every other edge
# tile with its waves in reverse order (N spans several tiles)
@pytest.mark.parametrize("tile", range(9))
@pytest.mark.parametrize("M", [1, 15, 16, 17, 48, 49, 64, 65, 81, 128])
def test_zgemm_edge_blocks(ctx, tile, M):
    dev = ctx.torch_device
    rng = np.random.default_rng(M + 1000 * tile)
    for N, K, opA in ((16, 5, 0), (97, 33, 1), (200, 1, 0), (130, 0, 0)):
        a = rng.standard_normal((M, K)) + 1j * rng.standard_normal((M, K))
        b = rng.standard_normal((K, N)) + 1j * rng.standard_normal((K, N))
        c = rng.standard_normal((M, N)) + 1j * rng.standard_normal((M, N))
        guard = torch.full((M + 2, N + 2), 7.0 - 3.0j, dtype=torch.complex128, device=dev)
        D = guard[1:M + 1, 1:N + 1]
        D.copy_(torch.tensor(c, device=dev))
        A = torch.tensor(a if opA == 0 else np.ascontiguousarray(a.T), device=dev)
        H.kern_zgemm(ctx, opA, 0, 1.0, A, torch.tensor(b, device=dev), beta=1, C_=D, D=D, tile=tile)
        # K products and K + 1 additions of complex values, three real products in tiles 4, 5 and 7: factor 6
        bound = 6 * (K + 2) * 2.0 ** -53 * (2 * (np.abs(a) @ np.abs(b)) + np.abs(c))
        assert (np.abs(D.cpu().numpy() - (a @ b + c)) <= bound).all(), (N, K)
        rim = guard.cpu().numpy()
        rim[1:-1, 1:-1] = 7.0 - 3.0j
        assert (rim == 7.0 - 3.0j).all()


# gradients summed over chunks of 64 samples or more, at most 64 of them and 15 for the widest layer (whose last
# is a short one): one linear layer with small whole numbers and a power of two of outputs, where every FP32
# operation is exact in any order, so the gradients are the oracle's bit for bit
@pytest.mark.parametrize("n,widths", [(1, (3, 1)), (64, (33, 1)), (64, (4, 2)), (128, (65, 4)), (1024, (31, 64)), (8192, (5, 2)),
                                      (2048, (1024, 1024))])
def test_mlp_gradient_chunks_exact(ctx, n, widths):
    rng = np.random.default_rng(n)
    net = pkg.MLP(ctx, widths)
    p = rng.integers(-1, 2, net.get_params().numel()).astype(np.float32)
    net.set_params(p)
    x = rng.integers(-1, 2, (n, widths[0])).astype(np.float32)
    t = rng.integers(-4, 5, (n, widths[1])).astype(np.float32)
    g, _ = net.grads(x, t)
    ref = om.grads(p.astype(np.float64), widths, x.astype(np.float64), t.astype(np.float64))
    assert np.array_equal(g.cpu().numpy().astype(np.float64), ref)
