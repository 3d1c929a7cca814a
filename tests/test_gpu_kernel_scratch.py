"""The scratch that a context keeps for synchronous residue products: sizes in any order, several threads, given back."""
import threading

import pytest
import torch

import paper_1702_05167_amd as pkg
import paper_1702_05167_amd.hsc as H

pytestmark = pytest.mark.gpu


def _operands(M, N, K, seed):
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    make = lambda r, c: torch.randn((r, c, 4), dtype=torch.float64, device="cuda:0", generator=g) * \
        torch.tensor([1.0, 2.0 ** -55, 1.0, 2.0 ** -55], dtype=torch.float64, device="cuda:0")
    return make(M, K), make(K, N)


SIZES = [(40, 30, 64), (300, 200, 100), (16, 16, 32), (33, 2000, 500), (1100, 1100, 700), (5, 7, 1)]


def test_sizes_in_any_order_match_fresh_contexts(ctx):
    for s, (M, N, K) in enumerate(SIZES + SIZES[::-1]):
        A, B = _operands(M, N, K, s)
        D = H.kern_zgemm_dd(ctx, 0, 0, A, B, config=3)
        fresh = pkg.Context(0)
        assert torch.equal(D, H.kern_zgemm_dd(fresh, 0, 0, A, B, config=3)), (M, N, K)
        fresh.close()


def test_threads_on_one_context(ctx):
    work = [_operands(M, N, K, 50 + s) for s, (M, N, K) in enumerate(SIZES[:4])]
    ref = [H.kern_zgemm_dd(ctx, 0, 0, A, B, config=3) for A, B in work]
    torch.cuda.synchronize()
    bad = []

    def run(k):
        for _ in range(20):
            if not torch.equal(H.kern_zgemm_dd(ctx, 0, 0, *work[k], config=3), ref[k]):
                bad.append(k)

    threads = [threading.Thread(target=run, args=(k,)) for k in range(len(work))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


def test_scratch_is_bounded_and_given_back():
    own = pkg.Context(0)
    A, B = _operands(1400, 1400, 1000, 1)     # 180 MB of residues: not kept
    D = H.kern_zgemm_dd(own, 0, 0, A, B, config=3)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for M, N, K in SIZES:
        a, b = A[:M, :K].contiguous(), B[:K, :N].contiguous()
        H.kern_zgemm_dd(own, 0, 0, a, b, D=D[:M, :N], config=3)
    torch.cuda.synchronize()
    del a, b
    torch.cuda.empty_cache()
    assert free - torch.cuda.mem_get_info()[0] <= 98 << 20
    own.close()
    assert free - torch.cuda.mem_get_info()[0] <= 2 << 20
