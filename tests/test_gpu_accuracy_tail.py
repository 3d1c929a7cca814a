"""Out of the lead band, at the few energies where the elimination over a nested-dissection tree loses digits even in
double-double: products from residues lose no more of them than products on the vector units.  The reference is the
chain of slabs, whose elimination keeps them (chains along x and along z agree to 1e-20 at such energies)."""
import numpy as np
import pytest
import torch

import synth
import paper_1702_05167_amd as pkg
import paper_1702_05167_amd.hsc as H

pytestmark = pytest.mark.gpu

KW = dict(eta=1e-8, kT=0.025, mu_L=0.1, mu_R=-0.1)


def _errors(x, ref):
    x, ref = (v.reshape(len(v), -1) for v in (x, ref))
    return np.abs(x - ref).max(1) / np.abs(ref).max(1)


def test_residue_products_lose_no_more_than_the_vector_units():
    ctx = pkg.Context(0)   # (plans of chains are large: closed at the end)
    dims, ne = (29, 18, 37), 32
    err = {k: [] for k in ("vector units", "residues", "15 digits")}
    spectral = {k: [] for k in err}
    for seed in (14, 18, 24, 36):
        n = int(np.prod(dims))
        dev = synth.cuboid(*dims, onsite=np.random.default_rng((seed, 3)).uniform(-0.5, 0.5, n))
        rng = np.random.default_rng((seed, 77))
        E = rng.choice([-1, 1], ne) * rng.uniform(2.02, 5.8, ne)
        tree, chain = pkg.Tree.from_device(dev, leaf_side=8), pkg.Tree.slab_chain(dev)
        want = H.HSC_DIAG_GR | H.HSC_SPECTRAL_LR

        def run(t, e, want, **kw):
            out = pkg.solve(ctx, t, torch.tensor(e, device=ctx.torch_device), want=want, batch=8, **KW, **kw)
            return {k: v.cpu().numpy() for k, v in out.items() if k in ("gr", "spectral")}

        print("device", seed, flush=True)
        g = {"vector units": run(tree, E, want, precision=2), "residues": run(tree, E, want),
             "15 digits": run(tree, E, want, slices=15)}
        # energies whose digits are lost: the two paths differ by more than the outputs' own rounding
        lost = np.flatnonzero(_errors(g["residues"]["gr"], g["vector units"]["gr"]) > 1e-14)[:8]
        if not len(lost):
            continue
        ref = run(chain, E[lost], H.HSC_DIAG_GR, precision=2)["gr"]
        for k in err:
            err[k] += list(_errors(g[k]["gr"][lost], ref))
        # both contact spectral functions at the worst of them (on a chain every block reaches the contacts)
        worst = lost[np.argmax(_errors(g["residues"]["gr"][lost], g["vector units"]["gr"][lost]))][None]
        ref = run(chain, E[worst], want)["spectral"]
        for k in spectral:
            spectral[k] += list(_errors(g[k]["spectral"][worst], ref))
    ctx.close()
    for name, e in (("G^r", err), ("A_L, A_R", spectral)):
        base = np.log2(np.maximum(e["vector units"], 1e-16))
        mean = {k: float(np.mean(np.log2(np.maximum(e[k], 1e-16)) - base)) for k in e}
        print(name, len(base), "energies: errors over the vector units' 2^", mean, "largest", {k: max(e[k]) for k in e}, flush=True)
        assert len(base) >= 4
        # single energies scatter by some 2^1.5 either way: the mean of N by 2^(1.5 / sqrt N), twice that and 2^0.5 more
        assert mean["residues"] <= 0.5 + 3.0 / np.sqrt(len(base)), (name, mean)
