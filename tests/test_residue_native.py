"""Tables of the residue products (csrc/residue.h, g++ on the CPU): the kernels' own steps -- chunks, residues,
products modulo each prime power, Chinese remainder sums -- replayed in exact integer arithmetic."""
import math
import os
import random
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SPLIT_BITS = 28


@pytest.fixture(scope="module")
def tab(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("residue") / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fconstexpr-ops-limit=1000000000", "-o", exe,
                    os.path.join(HERE, "native", "residue_driver.cpp")], check=True)
    lines = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.strip().split("\n")
    p = [int(v) for v in lines[0].split()]
    ns, nl, bits, hi, lo = lines[1].split()
    rows = [[int(v) for v in ln.split()] for ln in lines[2:]]
    split = [rows[32 * q:32 * (q + 1)] for q in range(4)]
    crt = [[rows[128 + (2 * part + g) * int(nl):128 + (2 * part + g + 1) * int(nl)] for g in range(2)]
           for part in range(2)]
    return dict(p=p, nsplit=int(ns), limbs=int(nl), bits=int(bits), hi=float.fromhex(hi), lo=float.fromhex(lo),
                split=split, crt=crt, bias=rows[-2], bias_off=rows[-1])


def _chunk_bytes(x):
    """Four chunks of 28 bits, rounded from the top, each as four signed bytes; the kernel's digits of x."""
    out = [0] * 16
    for b in range(3, -1, -1):
        w = 1 << (SPLIT_BITS * b)
        q = (2 * x + w) // (2 * w)
        x -= q * w
        assert abs(q) <= (1 << 27) + 1
        v = ((q + 0x00808080) ^ 0x00808080) & 0xffffffff
        for k in range(4):
            d = (v >> (8 * k)) & 0xff
            out[4 * b + k] = d - 256 if d > 127 else d
    assert x == 0
    return out


def _centred(c, p):
    r = c % p
    return r - p if 2 * r > p or (2 * r == p) else r


def _residues(tab, xr, xi):
    """[32][2] signed bytes: the two planes of every modulus."""
    dr, di = _chunk_bytes(xr), _chunk_bytes(xi)
    out = []
    for m, p in enumerate(tab["p"]):
        pl = []
        for h in range(2):
            s = sum(a * b for a, b in zip(dr, tab["split"][2 * h][m])) + \
                sum(a * b for a, b in zip(di, tab["split"][2 * h + 1][m]))
            assert abs(s) < 1 << 20
            r = _centred(s, p)
            assert -128 <= r <= 127
            pl.append(r)
        out.append(pl)
    return out


def test_moduli_cover_the_deepest_product(tab):
    p = tab["p"]
    assert len(p) == 32 and max(p) <= 256
    assert all(math.gcd(a, b) == 1 for i, a in enumerate(p) for b in p[:i])
    P = math.prod(p)
    assert P.bit_length() - 1 == tab["bits"]
    # operands |Re| + |Im| <= 2^111 + 1: 10880 terms of S = 16 (11648 of S = 15 are smaller) stay below P / 2
    assert 2 * 11648 * (2 ** 111 + 1) ** 2 < P
    assert abs(tab["lo"]) <= abs(tab["hi"]) * 2.0 ** -53
    from fractions import Fraction
    assert abs(Fraction(tab["hi"]) + Fraction(tab["lo"]) - Fraction(P, 2 ** tab["bits"])) < Fraction(2) ** -104


@pytest.mark.parametrize("depth", [1, 64, 10880])
def test_products_come_back_exactly(tab, depth):
    rng = random.Random(depth)
    p, ns = tab["p"], tab["nsplit"]
    P = math.prod(p)
    top = 2 ** 111
    cases = [((top, 0), (top, 0)), ((0, -top), (0, top)), ((top // 2, top // 2), (-(top // 2), top // 2)),
             ((0, 0), (top, 0)), ((1, -1), (-1, 1))]
    for _ in range(20):
        cases.append(tuple((rng.randrange(-top // 2, top // 2), rng.randrange(-top // 2, top // 2)) for _ in range(2)))
    for (ar, ai), (br, bi) in cases:
        # depth equal terms: the deepest sums of the kernel
        re, im = depth * (ar * br - ai * bi), depth * (ar * bi + ai * br)
        A, B = _residues(tab, ar, ai), _residues(tab, br, bi)
        parts = []
        for m, q in enumerate(p):
            (a0, a1), (b0, b1) = A[m], B[m]
            if m < ns:
                u, v = depth * a0 * b0, depth * a1 * b1
                x, y = u + v, u - v
            else:
                x, y = depth * (a0 * b0 - a1 * b1), depth * (a0 * b1 + a1 * b0)
            parts.append((_centred(x, q), _centred(y, q)))
        for part, want in ((0, re), (1, im)):
            limbs = [sum(tab["crt"][part][g][l][b] * parts[2 * b + g][part]
                         for g in range(2) for b in range(16)) for l in range(tab["limbs"])]
            assert max(abs(v) for v in limbs) <= 1 << 19
            bits = 8 * tab["limbs"]
            s = sum(v << (bits - 8 * (l + 1)) for l, v in enumerate(limbs)) % (1 << bits)
            if s >= 1 << (bits - 1):
                s -= 1 << bits
            # the weights are kept to 2^-160: s / 2^160 = X / P to 32 * 128 * 2^-160
            assert abs(s * P - (want << bits)) <= 4096 * P, (part, want)


def test_biased_sums_give_the_same_residues(tab):
    # sums of one element's digits (32 products of at most 128 x 121) and of products up to 128 deep
    top = 2 * 128 * 122 ** 2
    rng = np.random.default_rng(0)
    c = np.concatenate([np.arange(-3000, 3000), rng.integers(-top, top + 1, 20000), [-top, top]])
    for p, bias, off in zip(tab["p"], tab["bias"], tab["bias_off"]):
        bits = (bias + c).astype(np.int32)
        if p != 256:
            near = np.concatenate([k * p + np.arange(-2, 3) + p // 2 for k in rng.integers(-top // p + 2, top // p - 2, 400)])
            bits = np.concatenate([bits, (bias + near).astype(np.int32)])
        f = bits.view(np.float32)
        s = bits.astype(np.int64) - bias
        inv = np.float32(1.0) / np.float32(p)
        q = (f.astype(np.float64) * np.float64(inv) + off).astype(np.float32).view(np.int32).astype(np.int64)
        byte = (bits.astype(np.int64) - p * (q & 0xffffff)) & 0xff
        r = np.where(byte > 127, byte - 256, byte)
        assert ((r - s) % p == 0).all(), p
        if p != 256:
            assert (np.abs(f.astype(np.float64) - 2.0 ** 23 * 1.5) < 2 ** 22).all()
            assert np.abs(r).max() <= (p + 2) // 2
