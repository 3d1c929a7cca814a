"""Double-double pivot-block inverses where the choice of the pivot and the elimination's errors matter:
columns whose largest entries differ in the last bits, nearly singular blocks of several super-panels."""
from fractions import Fraction as F

import numpy as np
import pytest
import torch

import paper_1702_05167_amd.hsc as H

pytestmark = pytest.mark.gpu


# Rows in one thread, wave, workgroup pass and in different ones (two rows a thread from n = 513 on).
@pytest.mark.parametrize("gap", [2.0 ** -10, 2.0 ** -25, 2.0 ** -52, 0.0])
@pytest.mark.parametrize("n,r0,r1", [(2, 0, 1), (60, 3, 41), (130, 5, 127), (300, 0, 299), (600, 9, 521), (600, 9, 560), (1100, 20, 1090)])
def test_pivot_is_the_largest_entry(ctx, n, r0, r1, gap):
    # column 0 holds 1 (row r0) and 1 + gap (row r1); row r0 holds a value in column 1 that overflows when it is
    # multiplied by anything beyond 1: only the larger pivot leaves it alone
    A = np.zeros((n, n, 4))
    big = np.finfo(float).max * (1.0 - gap / 4)
    A[r0, 0, 0], A[r1, 0, 0], A[r0, 1, 0] = 1.0, 1.0 + gap, big
    if gap == 0.0:
        A[r1, 1, 0] = 1.0   # equal entries: the first row
    for j, r in zip(range(2, n), [r for r in range(n) if r not in (r0, r1)]):
        A[r, j, 0] = 1.0
    Y, st = H.kern_zinv_dd(ctx, torch.tensor(A, device=ctx.torch_device))
    Y = Y.cpu().numpy()
    assert np.isfinite(Y).all() and int(st.cpu()[0]) == 0
    if gap:
        # [[1, big], [1 + gap, 0]]^-1 = [[0, 1 / (1 + gap)], [1 / big, -1 / (big (1 + gap))]]
        assert abs(Y[0, r1, 0] * (1.0 + gap) - 1.0) <= 2.0 ** -52 and abs(Y[0, r0, 0]) <= 2.0 ** -100
        assert abs(Y[1, r0, 0] * big - 1.0) <= 1e-14   # (a subnormal number)


# One, two and several super-panels of 64 columns; beyond 512 the level of 256 columns, panels of 8 and 4 columns.
@pytest.mark.parametrize("matrix_cores", [0, 1])
@pytest.mark.parametrize("n", [40, 64, 65, 130, 257, 520, 700, 1030])
def test_nearly_singular_block(ctx, n, matrix_cores):
    # complex symmetric, one eigenvalue at 1e-9, the others of size 1 to 3.  Elimination with partial pivoting leaves
    # |A Y - I| at some n units of 2^-104 times |A| |Y| (growth of the entries by a few, residue products K 0.8 2^-104)
    rng = np.random.default_rng(n)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    lam = np.concatenate([[1e-9], rng.uniform(1.0, 3.0, n - 1) * rng.choice([-1.0, 1.0], n - 1)])
    a = (q * lam) @ q.T
    a = 0.5 * (a + a.T) + 1e-11j * np.eye(n)
    A = np.zeros((n, n, 4))
    A[..., 0], A[..., 2] = a.real, a.imag
    Y, st = H.kern_zinv_dd(ctx, torch.tensor(A, device=ctx.torch_device), matrix_cores=matrix_cores)
    Y = Y.cpu().numpy()
    assert int(st.cpu()[0]) == 0
    y64 = Y[..., 0] + 1j * Y[..., 2]
    assert np.abs(y64).max() > 1e9 / n
    bound = 64 * n * 2.0 ** -104 * 3.0 * np.linalg.norm(y64, 2)
    worst = 0.0
    for i, j in {(0, 0), (n - 1, 0), (0, n - 1), (n - 1, n - 1)} | {(int(i), int(j)) for i, j in rng.integers(0, n, (16, 2))}:
        re = im = F(0)
        for k in range(n):
            ar, ai = F(A[i, k, 0]), F(A[i, k, 2])
            yr, yi = F(Y[k, j, 0]) + F(Y[k, j, 1]), F(Y[k, j, 2]) + F(Y[k, j, 3])
            re += ar * yr - ai * yi
            im += ar * yi + ai * yr
        worst = max(worst, abs(float(re - (1 if i == j else 0))), abs(float(im)))
    print("n", n, "matrix cores", matrix_cores, "worst |A Y - I|", worst, "over its bound", worst / bound, flush=True)
    assert worst <= bound
