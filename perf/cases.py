"""The work that users of this solver have it do, as cases that can be timed and checked.

A case is a dict of plain values; `listed()` holds the fixed ones and `draw(rng)` makes more of the same ranges.
`prepare(case, seed)` builds what a program holds before the call (device Hamiltonian, cluster tree, context,
energies), `run(state)` is one pass through the public entry points, `work(case)` the bytes and operations that
the pass cannot do without, and `exact(case, seed)` the same outputs from plain torch / numpy in 64 bits.

Kinds of case
  solve   diag G^r, diag G^<, T (or the two spectral functions) of one cuboid over a list of energies
  wire    the same for a wire with several orbitals per site
  forest  several uneven small cuboids in one call, one common energy list
  scf     a few iterations of the self-consistent NEGF-Poisson loop
  grads   loss and gradients of the surrogate network (learned energy grid) on one batch of samples
"""
import math

import numpy as np
import torch

import paper_1702_05167_amd as hsc

ETA, KT, MU_L, MU_R = 1e-8, 0.025, 0.1, -0.1
E_RANGE = (-6.0, 6.0)   # the benchmark's energy range; the lead band is [-2, 2]
DENSE_SITES = 2600   # `exact` inverts the whole matrix up to this size (pivoted: accurate at every energy)


def listed():
    return [
        # one energy on the smallest device: the latency of a call (adaptive grids, root searches)
        dict(name="cube8_point", kind="solve", nx=8, ny=8, nz=8, leaf=4, ne=1, prec=3, dense=0, spectral=0,
             transverse=0),
        # the 8^3 device over its 16-point energy grid
        dict(name="cube8_grid", kind="solve", nx=8, ny=8, nz=8, leaf=4, ne=16, prec=3, dense=0, spectral=0,
             transverse=0),
        # a small device of odd sides, both contact spectral functions (learned-grid training data)
        dict(name="cuboid_spectral", kind="solve", nx=13, ny=11, nz=17, leaf=8, ne=8, prec=3, dense=0, spectral=1,
             transverse=0),
        # a medium cube over many energies, with the per-energy totals that a sweep reports
        dict(name="cube16_sweep", kind="solve", nx=16, ny=16, nz=16, leaf=8, ne=32, prec=3, dense=0, spectral=0,
             transverse=0),
        # whole-face leads: the dense self-energy blocks on an elongated device
        dict(name="faces16", kind="solve", nx=24, ny=16, nz=16, leaf=8, ne=8, prec=3, dense=1, spectral=0,
             transverse=0),
        # an uneven cuboid of the multi-device workload's size range (sides 16 to 48)
        dict(name="cuboid_uneven", kind="solve", nx=29, ny=18, nz=37, leaf=8, ne=4, prec=3, dense=0, spectral=0,
             transverse=0),
        # the benchmark cube, one batch of energies of its grid
        dict(name="cube32_batch", kind="solve", nx=32, ny=32, nz=32, leaf=8, ne=4, prec=3, dense=0, spectral=0,
             transverse=0),
        # complex128 on the FP64 matrix cores, transverse tree: the in-band production setting of that precision
        dict(name="cube24_c128", kind="solve", nx=24, ny=24, nz=24, leaf=4, ne=8, prec=0, dense=0, spectral=0,
             transverse=1),
        # uneven small cubes solved together as one forest
        dict(name="forest8", kind="forest", devices=8, lo=8, hi=16, ne=16, leaf=8),
        # a ten-orbital nanowire of 4 x 4 sites across
        dict(name="wire10", kind="wire", nx=32, ny=4, nz=4, orbitals=10, ne=8, leaf=8),
        # two iterations of the self-consistent loop on a small device
        dict(name="scf_small", kind="scf", nx=16, ny=9, nz=8, ne=16, leaf=8, iterations=2),
        # one gradient of the surrogate network on a training batch
        dict(name="mlp_grads", kind="grads", samples=2048, hidden=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "wire", "forest", "scf", "grads"])
    if kind == "solve":
        while True:
            nx, ny, nz = (_log_int(rng, 6, 32) for _ in range(3))
            ne = _log_int(rng, 1, 32)
            # below the largest listed case (cost ~ sites^2 per energy) and its memory
            if max(nx, ny, nz) <= 4 * min(nx, ny, nz) and (nx * ny * nz) ** 2 * ne <= 0.5 * 32768 ** 2 * 4 and \
                    nx * ny * nz <= 24000 and nx * ny * nz * ne <= 110000:
                break
        prec = rng.choice([3, 3, 3, 0])
        dense = int(prec == 3 and nx >= 4 and rng.random() < 0.25)
        return dict(kind="solve", nx=nx, ny=ny, nz=nz, leaf=4 if prec == 0 or nx * ny * nz < 900 else 8, ne=ne, prec=prec,
                    dense=dense, spectral=int(not dense and rng.random() < 0.25), transverse=int(prec == 0))
    if kind == "wire":
        return dict(kind="wire", nx=_log_int(rng, 8, 40), ny=rng.randint(3, 4), nz=rng.randint(3, 4),
                    orbitals=rng.randint(4, 10), ne=_log_int(rng, 2, 8), leaf=8)
    if kind == "forest":
        return dict(kind="forest", devices=rng.randint(3, 10), lo=8, hi=rng.randint(11, 16), ne=_log_int(rng, 4, 16),
                    leaf=8)
    if kind == "scf":
        return dict(kind="scf", nx=rng.randint(8, 16), ny=rng.randint(6, 10), nz=rng.randint(6, 10),
                    ne=_log_int(rng, 8, 24), leaf=8, iterations=rng.randint(1, 3))
    return dict(kind="grads", samples=_log_int(rng, 256, 8192), hidden=rng.choice([128, 256, 320]))


# ---- inputs ----------------------------------------------------------------------------------------

def _rng(case, seed, k=0):
    return np.random.default_rng((seed & 0x7FFFFFFF, k, 17))


def _csr(n, rows, cols, vals):
    rows, cols = np.concatenate(rows).astype(np.int64), np.concatenate(cols).astype(np.int64)
    vals = np.concatenate(vals).astype(np.complex128)
    order = np.lexsort((cols, rows))
    indptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int64)
    return indptr, cols[order].astype(np.int32), vals[order]


class _Device:
    """Cuboid of b orbitals per site (unknown o + b (x + nx (y + ny z))), nearest-neighbour coupling, leads on
    the x faces (one 1D lead per unknown, or a lead that continues the face lattice)."""

    def __init__(self, nx, ny, nz, rng, b=1, sigma=None):
        self.dims, self.b = (nx, ny, nz), b
        ns = nx * ny * nz
        self.n = n = ns * b
        site = np.arange(ns)
        xyz = np.stack([site % nx, (site // nx) % ny, site // (nx * ny)], 1)
        rows, cols, vals = [], [], []
        if b == 1:
            onsite = rng.uniform(-0.5, 0.5, ns) if sigma is None else rng.normal(0.0, sigma, ns)
            rows.append(site), cols.append(site), vals.append(onsite)
        else:
            m = np.triu(rng.normal(0.0, 0.3, (ns, b, b)), 1)
            blk = m + m.transpose(0, 2, 1) + np.diag(np.linspace(-3.0, 3.0, b))
            o, p = np.meshgrid(np.arange(b), np.arange(b), indexing="ij")
            rows.append((site[:, None, None] * b + o).ravel())
            cols.append((site[:, None, None] * b + p).ravel())
            vals.append(blk.ravel())
        for d, stride in enumerate((1, nx, nx * ny)):
            i = site[xyz[:, d] + 1 < self.dims[d]]
            if b == 1:
                rows += [i, i + stride]
                cols += [i + stride, i]
                vals += [np.full(len(i), -1.0)] * 2
            else:
                t = rng.normal(0.0, 1.0 / np.sqrt(b), (b, b))
                o, p = np.meshgrid(np.arange(b), np.arange(b), indexing="ij")
                a, c = (i[:, None, None] * b + o).ravel(), ((i + stride)[:, None, None] * b + p).ravel()
                v = np.broadcast_to(t, (len(i), b, b)).ravel()
                rows += [a, c]
                cols += [c, a]
                vals += [v, v]
        self.indptr, self.indices, self.values = _csr(n, rows, cols, vals)
        self.coords = np.repeat(xyz, b, axis=0).astype(np.int32)
        x = self.coords[:, 0]
        self.left, self.right = np.flatnonzero(x == 0), np.flatnonzero(x == nx - 1)

    def tree(self, leaf, dense=False, transverse=False):
        contacts = [(self.left, 0.0, -1.0, -1.0), (self.right, 0.0, -1.0, -1.0)]
        return hsc.Tree.build(self.n, self.indptr, self.indices, self.values, self.coords, contacts,
                              6 if transverse else 7, leaf, dense)

    def dense_h(self):
        h = np.zeros((self.n, self.n), np.complex128)
        h[np.repeat(np.arange(self.n), np.diff(self.indptr)), self.indices] = self.values
        return h


def _devices(case, seed):
    k = case["kind"]
    if k == "forest":
        out = []
        for d in range(case["devices"]):
            sides = np.random.default_rng((case["devices"], case["hi"], d)).integers(case["lo"], case["hi"] + 1, 3)
            out.append(_Device(*(int(s) for s in sides), _rng(case, seed, d + 1), sigma=0.3))
        return out
    return [_Device(case["nx"], case["ny"], case["nz"], _rng(case, seed, 1), case.get("orbitals", 1))]


def _energies(case, seed):
    ne = case["ne"]
    # complex128 is used inside the lead band; the loop's window ends above the chemical potentials
    lo, hi = (-1.9, 1.9) if case.get("prec") == 0 else (-4.5, 0.5) if case["kind"] == "scf" else E_RANGE
    # evenly spaced, each point moved inside its interval: sweeps and adaptive refinements alike
    return lo + (hi - lo) * (np.arange(ne) + _rng(case, seed).uniform(0.05, 0.95, ne)) / ne


def _network(case, seed):
    rng = _rng(case, seed, 5)
    widths = [4, case["hidden"], case["hidden"], 2]
    params = np.concatenate([np.concatenate([rng.normal(0.0, 1.0 / np.sqrt(a), a * b), np.zeros(b)])
                             for a, b in zip(widths[:-1], widths[1:])])
    x = rng.uniform(-1.0, 1.0, (case["samples"], 4))
    t = rng.normal(0.0, 1.0, (case["samples"], 2))
    return widths, params.astype(np.float32), x.astype(np.float32), t.astype(np.float32)


def prepare(case, seed):
    ctx = hsc.Context(0)
    state = dict(case=case, ctx=ctx)
    if case["kind"] == "grads":
        widths, params, x, t = _network(case, seed)
        state["net"] = hsc.MLP(ctx, widths)
        state["net"].set_params(params)
        state["x"] = torch.tensor(x, device=ctx.torch_device)
        state["t"] = torch.tensor(t, device=ctx.torch_device)
        return state
    state["trees"] = [d.tree(case["leaf"], bool(case.get("dense")), bool(case.get("transverse")))
                      for d in _devices(case, seed)]
    energies = _energies(case, seed)
    state["energies"] = torch.tensor(energies, dtype=torch.float64, device=ctx.torch_device)
    if case["kind"] == "scf":
        state["weights"] = torch.tensor(_weights(energies), dtype=torch.float64, device=ctx.torch_device)
    return state


def _weights(e):
    w = np.zeros(len(e))
    w[1:] += 0.5 * np.diff(e)
    w[:-1] += 0.5 * np.diff(e)
    return w


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "grads":
        g, loss = state["net"].grads(state["x"], state["t"])
        return {"grads": g, "loss": loss}
    if kind == "forest":
        return hsc.solve_batch(ctx, state["trees"], state["energies"], ETA, KT, MU_L, MU_R, batch=case["ne"])
    if kind == "scf":
        u, dens, res = hsc.scf(ctx, state["trees"][0], (case["nx"], case["ny"], case["nz"]), state["energies"],
                               state["weights"], u_left=0.05, u_right=-0.05, coupling=0.05, mixing=0.5,
                               max_iter=case["iterations"], batch=case["ne"])
        return {"u": u, "density": dens, "residuals": res}
    tree = state["trees"][0]
    if case.get("spectral"):
        out = hsc.solve(ctx, tree, state["energies"], ETA, KT, MU_L, MU_R,
                        want=hsc.HSC_DIAG_GR | hsc.HSC_DIAG_GL | hsc.HSC_SPECTRAL_LR | hsc.HSC_TRANS, batch=case["ne"],
                        precision=case["prec"])
    else:
        out = hsc.solve(ctx, tree, state["energies"], ETA, KT, MU_L, MU_R, batch=case["ne"],
                        precision=case.get("prec", 3))
    out["totals"] = hsc.totals(ctx, out, tree.n)
    return out


def work(case):
    """Operations: the multiply-adds of the block algorithms (8 real operations per complex one) that the case's
    cluster trees need; bytes: the Hamiltonian read once per call, each output written once."""
    if case["kind"] == "grads":
        h, s = case["hidden"], case["samples"]
        p = 4 * h + h + h * h + h + 2 * h + 2
        return {"bytes": 4.0 * (2 * p + 6 * s), "flops": 6.0 * s * (4 * h + h * h + 2 * h)}
    flops = by = 0.0
    calls = case.get("iterations", 1)
    for d in _devices(case, 0):
        t = d.tree(case["leaf"], bool(case.get("dense")), bool(case.get("transverse")))
        flops += calls * case["ne"] * t.stats()["flops_per_energy"]
        per = 16.0 if case["kind"] == "scf" else 48.0 if case.get("spectral") else 32.0
        by += calls * (20.0 * len(d.values) + case["ne"] * d.n * per)
        t.close()
    return {"bytes": by, "flops": flops}


# ---- 64-bit values without this repository's code ---------------------------------------------------

def _lead_g(z, eps):
    """Decaying root of g^2 - (z - eps) g + 1 = 0 (surface function of a chain with hopping -1)."""
    w = z - eps
    s = np.sqrt(w * w - 4.0 + 0j)
    a, b = 0.5 * (w + s), 0.5 * (w - s)
    return np.where(np.abs(a) < np.abs(b), a, b)


def _sigma(dev, z, dense):
    """Self-energy block of the sites of an x face (the same for both faces)."""
    m = len(dev.left)
    if not dense:
        return np.diag(np.full(m, complex(_lead_g(z, 0.0))))
    ny, nz = dev.dims[1:]
    modes = [np.sqrt(2.0 / (d + 1)) * np.sin(np.pi * np.outer(np.arange(1, d + 1), np.arange(1, d + 1)) / (d + 1))
             for d in (ny, nz)]
    eps = [-2.0 * np.cos(np.pi * np.arange(1, d + 1) / (d + 1)) for d in (ny, nz)]
    # face sites run y fastest, then z
    v = np.kron(modes[1], modes[0])
    return (v * _lead_g(z, (eps[1][:, None] + eps[0][None, :]).ravel())[None, :]) @ v.T


def _fermi(e, mu):
    x = (e - mu) / KT
    return math.exp(-x) / (1.0 + math.exp(-x)) if x > 0 else 1.0 / (1.0 + math.exp(x))


def _green(dev, e, dense, pot=None):
    """(diag G^r, A_L, A_R, T) at one energy, by block elimination over the x layers (dense inverse of the whole
    matrix when it is small)."""
    tdev = torch.device("cuda" if torch.cuda.is_available() else "cpu")

    def mat(a):
        return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.complex128, device=tdev)

    z = e + 1j * ETA
    s = _sigma(dev, z, dense)
    gam = mat(-2.0 * s.imag)
    if dev.n <= DENSE_SITES:
        a = -dev.dense_h()
        a[np.diag_indices(dev.n)] += z - (0.0 if pot is None else pot)
        a[np.ix_(dev.left, dev.left)] -= s
        a[np.ix_(dev.right, dev.right)] -= s
        g = torch.linalg.inv(mat(a))
        gl, gr = g[:, torch.as_tensor(dev.left, device=tdev)], g[:, torch.as_tensor(dev.right, device=tdev)]
        al, ar = ((gl @ gam) * gl.conj()).sum(1).real, ((gr @ gam) * gr.conj()).sum(1).real
        glr = gr[torch.as_tensor(dev.left, device=tdev)]
        t = ((gam @ glr @ gam) * glr.conj()).sum().real
        return [v.cpu().numpy() for v in (torch.diagonal(g), al, ar)] + [float(t)]
    x = dev.coords[:, 0]
    lay = [np.flatnonzero(x == k) for k in range(dev.dims[0])]
    loc = np.empty(dev.n, np.int64)
    for ix in lay:
        loc[ix] = np.arange(len(ix))
    rows = np.repeat(np.arange(dev.n), np.diff(dev.indptr))

    def block(a, b):
        m = np.zeros((len(lay[a]), len(lay[b])), np.complex128)
        sel = (x[rows] == a) & (x[dev.indices] == b)
        m[loc[rows[sel]], loc[dev.indices[sel]]] = -dev.values[sel]
        return m

    nl = len(lay)
    diag, up = [], []
    for k in range(nl):
        m = block(k, k)
        m[np.diag_indices(len(m))] += z - (0.0 if pot is None else pot[lay[k]])
        if k in (0, nl - 1):
            m -= s
        diag.append(mat(m))
        if k + 1 < nl:
            up.append(mat(block(k, k + 1)))
    inv = torch.linalg.inv
    fl, fr = [None] * nl, [None] * nl
    fl[0] = inv(diag[0])
    for k in range(1, nl):
        fl[k] = inv(diag[k] - up[k - 1].T @ fl[k - 1] @ up[k - 1])
    fr[-1] = inv(diag[-1])
    for k in range(nl - 2, -1, -1):
        fr[k] = inv(diag[k] - up[k] @ fr[k + 1] @ up[k].T)
    gd, cr, cl = [None] * nl, [None] * nl, [None] * nl
    gd[-1] = cr[-1] = fl[-1]
    for k in range(nl - 2, -1, -1):
        w = fl[k] @ up[k]
        gd[k] = fl[k] + w @ gd[k + 1] @ w.T
        cr[k] = -(w @ cr[k + 1])
    cl[0] = fr[0]
    for k in range(1, nl):
        cl[k] = -(fr[k] @ up[k - 1].T @ cl[k - 1])
    g, al, ar = np.zeros(dev.n, np.complex128), np.zeros(dev.n), np.zeros(dev.n)
    for k in range(nl):
        g[lay[k]] = torch.diagonal(gd[k]).cpu().numpy()
        al[lay[k]] = ((cl[k] @ gam) * cl[k].conj()).sum(1).real.cpu().numpy()
        ar[lay[k]] = ((cr[k] @ gam) * cr[k].conj()).sum(1).real.cpu().numpy()
    t = ((gam @ cr[0] @ gam) * cr[0].conj()).sum().real
    return g, al, ar, float(t)


def _solve_exact(dev, energies, dense=False, spectral=False, totals=True):
    gr, gl, tr, sp = [], [], [], []
    for e in energies:
        g, al, ar, t = _green(dev, float(e), dense)
        gr.append(g), tr.append(t), sp.append(np.stack([al, ar]))
        gl.append(1j * (_fermi(e, MU_L) * al + _fermi(e, MU_R) * ar))
    gr, gl, sp = np.stack(gr), np.stack(gl), np.stack(sp)
    out = {"gr": gr, "gl": gl, "trans": np.array(tr)}
    if spectral:
        out["spectral"] = sp
    out["status"] = None
    if totals:
        tot = np.zeros((len(gr), 3))
        tot[:, 0] = -gr.imag.sum(1) / np.pi
        tot[:, 1] = gl.imag.sum(1) / (2.0 * np.pi)
        if spectral:
            tot[:, 2] = sp.sum((1, 2)) / (2.0 * np.pi)
        out["totals"] = tot
    return out


def _poisson(dims, rho, ul, ur):
    ops = []
    for ax, d in enumerate(dims):
        m = 2.0 * np.eye(d) - np.eye(d, k=1) - np.eye(d, k=-1)
        if ax:
            m[0, 0] -= 1.0
            m[-1, -1] -= 1.0
        ops.append(m)
    i = [np.eye(d) for d in dims]
    op = np.kron(i[2], np.kron(i[1], ops[0])) + np.kron(i[2], np.kron(ops[1], i[0])) + np.kron(ops[2], np.kron(i[1], i[0]))
    b = rho.copy()
    x = np.arange(len(rho)) % dims[0]
    b[x == 0] += ul
    b[x == dims[0] - 1] += ur
    return np.linalg.solve(op, b)


def exact(case, seed):
    kind = case["kind"]
    if kind == "grads":
        widths, params, x, t = (v if isinstance(v, list) else v.astype(np.float64) for v in _network(case, seed))
        layers, o = [], 0
        for a, b in zip(widths[:-1], widths[1:]):
            layers.append((params[o:o + a * b].reshape(b, a), params[o + a * b:o + a * b + b]))
            o += a * b + b
        acts = [x]
        for k, (w, b) in enumerate(layers):
            y = acts[-1] @ w.T + b
            acts.append(np.tanh(y) if k + 1 < len(layers) else y)
        err = acts[-1] - t
        loss, d, grads = float((err ** 2).mean()), 2.0 * err / err.size, []
        for k in range(len(layers) - 1, -1, -1):
            grads.insert(0, np.concatenate([(d.T @ acts[k]).ravel(), d.sum(0)]))
            if k:
                d = (d @ layers[k][0]) * (1.0 - acts[k] ** 2)
        return {"grads": np.concatenate(grads), "loss": loss}
    devs, energies = _devices(case, seed), _energies(case, seed)
    cost = sum((d.dims[1] * d.dims[2] * d.b) ** 3 * d.dims[0] if d.n > DENSE_SITES else d.n ** 3 for d in devs)
    if cost * case["ne"] * case.get("iterations", 1) > 6e11:   # beyond some 20 seconds
        return None
    if kind == "forest":
        return [_solve_exact(d, energies, totals=False) for d in devs]
    if kind == "scf":
        dev, w = devs[0], _weights(energies)
        u, res = np.zeros(dev.n), []
        for _ in range(case["iterations"]):
            dens = np.zeros(dev.n)
            for e, we in zip(energies, w):
                _, al, ar, _ = _green(dev, float(e), False, u)
                dens += we * (_fermi(e, MU_L) * al + _fermi(e, MU_R) * ar) / (2.0 * np.pi)
            new = _poisson(dev.dims, 0.05 * dens, 0.05, -0.05)
            res.append(np.abs(new - u).max())
            u = u + 0.5 * (new - u)
        return {"u": u, "density": dens, "residuals": np.array(res)}
    return _solve_exact(devs[0], energies, bool(case.get("dense")), bool(case.get("spectral")))
