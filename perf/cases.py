"""Performance cases of the form-factor engine, through its Python entry points.

A case is a dict of plain values.  ``listed()`` gives the fixed ones, ``draw``
one more of the same ranges, ``prepare`` what a user's program holds before
the call (molecule, transition densities, context, output buffers), ``run``
one pass, ``work`` what the pass cannot do without and ``exact`` the same
outputs in FP64 from plain torch.

Kinds of case:

  grid    the whole step of the Cartesian method: molecule load, transitions
          from device memory, pair precompute, 1D tables and the q-grid, f and
          |f|^2 left in device memory
  serve   a burst of independent requests through the request server, results
          in host memory
  points  f at arbitrary q points of a loaded molecule (line cuts, shells)
  fft     the FFT method's step on a real-space box
  sph     the spherical method's step on radii and an angular grid
  lowq    transition dipoles, oscillator strengths and one separable integral
  fit     the angular-average fit of the low-momentum limit

Molecules are seeded synthetic ones (double-zeta-like Cartesian shells with
three primitives, exponents log-uniform in [0.1, 100]); transitions are
C_occ X C_vir^T with orthonormal C and ||X||_F = 1.
"""
from __future__ import annotations

import math
import random
from types import SimpleNamespace

import numpy as np
import torch

BOHR = 1.0 / 0.529177210903
CART = {0: [(0, 0, 0)], 1: [(1, 0, 0), (0, 1, 0), (0, 0, 1)],
        2: [(2, 0, 0), (1, 1, 0), (1, 0, 1), (0, 2, 0), (0, 1, 1), (0, 0, 2)]}
EPS = 1e-9   # screening threshold, as the benchmark sets it


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # the smallest call: a four-atom molecule, one transition, 32^3 (latency and launches)
        dict(name="grid_tiny_fp32", kind="grid", heavy=4, hyd=4, d=False, states=1, nx=32, ny=32, nz=32, qmax=5.0,
             precision="fp32", sym=False),
        # the ordinary step: ten heavy atoms, 12 transitions, 64^3
        dict(name="grid_mid_fp32", kind="grid", heavy=10, hyd=8, d=True, states=12, nx=64, ny=64, nz=64, qmax=6.0,
             precision="fp32", sym=False),
        # the same molecule class on an odd, ragged grid with the split-BF16 contraction
        dict(name="grid_ragged_bf16x3", kind="grid", heavy=10, hyd=8, d=True, states=9, nx=51, ny=47, nz=85, qmax=6.5,
             precision="bf16x3", sym=False),
        # the benchmark's size: 30 heavy atoms, 24 transitions, 96^3 (the largest)
        dict(name="grid_large_fp32", kind="grid", heavy=30, hyd=24, d=True, states=24, nx=96, ny=96, nz=96, qmax=8.0,
             precision="fp32", sym=False),
        # the same with the split-BF16 contraction
        dict(name="grid_large_bf16x3", kind="grid", heavy=30, hyd=24, d=True, states=24, nx=96, ny=96, nz=96, qmax=8.0,
             precision="bf16x3", sym=False),
        # a burst of mixed requests (2-30 heavy atoms, 1-24 transitions, 32^3-96^3) through the server
        dict(name="serve_burst_fp32", kind="serve", requests=6, mix=5, precision="fp32"),
        # a line cut or a set of detector momenta of a loaded molecule
        dict(name="points_1000", kind="points", heavy=10, hyd=8, d=True, states=12, points=1000, qmax=6.0),
        # the FFT method on the box of the ordinary molecule
        dict(name="fft_mid_fp32", kind="fft", heavy=10, hyd=8, d=True, states=12, nx=128, ny=128, nz=128,
             precision="fp32"),
        # the FFT method with split-BF16, a larger basis and few transitions on an uneven box
        dict(name="fft_uneven_bf16x3", kind="fft", heavy=20, hyd=16, d=True, states=5, nx=128, ny=64, nz=32,
             precision="bf16x3"),
        # the spherical method at the usual angular order
        dict(name="sph_mid", kind="sph", heavy=10, hyd=8, d=True, states=12, lmax=24, radii=24, n_theta=32, n_phi=64,
             qmax=6.0),
        # dipoles, oscillator strengths and one separable integral of the large molecule
        dict(name="lowq_large", kind="lowq", heavy=30, hyd=24, d=True, states=24, nx=96, ny=96, nz=96, qmax=8.0),
        # the paper's fit of the angular average for a small molecule
        dict(name="fit_small", kind="fit", heavy=4, hyd=4, d=True, states=3, qfit=0.1),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choices(["grid", "points", "fft", "sph", "lowq", "fit", "serve"], [10, 2, 3, 2, 1, 1, 1])[0]
    heavy = _logint(rng, 2, 30)
    c = dict(kind=kind, heavy=heavy, hyd=int(round(0.8 * heavy)), d=rng.random() < 0.8 or heavy > 6,
             states=_logint(rng, 1, 24))
    if kind == "grid":
        n = [_logint(rng, 16, 128) for _ in range(3)]
        # no more than the largest listed case: pairs kept x grid points
        while (heavy / 30.0) ** 1.2 * n[0] * n[1] * n[2] > 0.85 * 96 ** 3 * (1.0 if c["states"] > 16 else 1.5):
            n[n.index(max(n))] -= 7
        c.update(nx=n[0], ny=n[1], nz=n[2], qmax=round(rng.uniform(5.0, 8.0), 3),
                 precision=rng.choice(["fp32", "bf16x3"]), sym=rng.random() < 0.15)
    elif kind == "points":
        heavy = min(heavy, 10)
        c.update(heavy=heavy, hyd=int(round(0.8 * heavy)), points=_logint(rng, 32, 4096),
                 qmax=round(rng.uniform(3.0, 8.0), 3))
    elif kind == "fft":
        n = [2 ** rng.randint(4, 7) for _ in range(3)]
        if heavy > 16:
            n[0] = min(n[0], 64)
        c.update(nx=n[0], ny=n[1], nz=n[2], precision=rng.choice(["fp32", "bf16x3"]))
    elif kind == "sph":
        heavy = min(heavy, 10)
        lmax = rng.randint(4, 28)
        radii = _logint(rng, 2, 40)
        c.update(heavy=heavy, hyd=int(round(0.8 * heavy)), lmax=lmax, states=min(c["states"], 12), radii=radii,
                 n_theta=rng.randint(8, 48), n_phi=rng.randint(8, 96), qmax=round(rng.uniform(2.0, 6.0), 3))
    elif kind == "lowq":
        c.update(nx=rng.randint(16, 128), ny=rng.randint(16, 128), nz=rng.randint(16, 128),
                 qmax=round(rng.uniform(5.0, 8.0), 3))
    elif kind == "fit":
        heavy = min(heavy, 5)
        c.update(heavy=heavy, hyd=int(round(0.8 * heavy)), states=min(c["states"], 12),
                 qfit=round(rng.uniform(0.05, 0.2), 4))
    else:
        c = dict(kind="serve", requests=rng.randint(2, 6), mix=rng.randint(0, 1 << 20),
                 precision=rng.choice(["fp32", "bf16x3"]))
    return c


# ------------------------------------------------------------------ the inputs

def _molecule(case, rng):
    """Heavy atoms uniform in a box of constant density, H at 1.09 A from distinct heavy atoms."""
    nh, hyd, d = case["heavy"], min(case["hyd"], case["heavy"]), case["d"]
    edge = max(12.0 * (nh / 30.0) ** (1.0 / 3.0), 2.5) * BOHR
    pts = []
    while len(pts) < nh:
        p = (rng.random(3) - 0.5) * edge
        if all(np.linalg.norm(p - x) >= 1.2 * BOHR for x in pts):
            pts.append(p)
    hosts = rng.choice(nh, size=hyd, replace=False)
    for h in hosts:
        while True:
            v = rng.normal(size=3)
            p = pts[h] + 1.09 * BOHR * v / np.linalg.norm(v)
            if all(np.linalg.norm(p - x) >= 0.9 * BOHR for i, x in enumerate(pts) if i != h):
                pts.append(p)
                break
    Z = np.concatenate([rng.choice([6, 7, 8], size=nh), np.ones(hyd, dtype=np.int64)])
    atom, ls, ex, co = [], [], [], []
    for ia, z in enumerate(Z):
        for l in ([0, 0] + ([1] if d else []) if z == 1 else [0, 0, 0, 1, 1] + ([2] if d else [])):
            atom.append(ia)
            ls.append(l)
            ex.append(np.sort(np.exp(rng.uniform(np.log(0.1), np.log(100.0), size=3)))[::-1])
            co.append(rng.uniform(0.1, 1.0, size=3))
    return SimpleNamespace(Z=Z, xyz=np.array(pts), shell_atom=np.array(atom, np.int32), shell_l=np.array(ls, np.int32),
                           shell_nprim=np.full(len(ls), 3, np.int32), exps=np.concatenate(ex), coefs=np.concatenate(co))


def _transitions(mol, n_states, rng):
    nbf = sum((l + 1) * (l + 2) // 2 for l in mol.shell_l.tolist())
    C, R = np.linalg.qr(rng.normal(size=(nbf, nbf)))
    C = C * np.sign(np.diag(R))[None, :]
    no = min(int(mol.Z.sum()) // 2, nbf - 1)
    T = np.empty((n_states, nbf, nbf))
    for s in range(n_states):
        X = rng.normal(size=(no, nbf - no))
        T[s] = C[:, :no] @ (X / np.linalg.norm(X)) @ C[:, no:].T
    return T


def _requests(case):
    """The sizes of a burst: plain cases, from the case alone."""
    rng = random.Random(case["mix"])
    out = []
    for _ in range(case["requests"]):
        heavy, n = rng.randint(2, 30), rng.randint(32, 96)
        out.append(dict(kind="grid", heavy=heavy, hyd=int(round(0.8 * heavy)), d=True, states=rng.randint(1, 24), nx=n,
                        ny=n, nz=n, qmax=round(rng.uniform(5.0, 8.0), 3), precision=case["precision"], sym=False))
    return out


def _grid(case):
    return SimpleNamespace(n=(case["nx"], case["ny"], case["nz"]), qmin=(-case["qmax"],) * 3, qmax=(case["qmax"],) * 3)


def _box(mol, case):
    """Bounding box + 5 bohr, doubled about its centre."""
    lo, hi = mol.xyz.min(axis=0) - 5.0, mol.xyz.max(axis=0) + 5.0
    L = 2.0 * (hi - lo)
    xmin = 0.5 * (lo + hi) - 0.5 * L
    return (case["nx"], case["ny"], case["nz"]), tuple(map(float, xmin)), tuple(map(float, L))


def _inputs(case, seed):
    """Every host input of a case, from the seed alone."""
    rng = np.random.Generator(np.random.PCG64(seed))
    if case["kind"] == "serve":
        reqs = _requests(case)
        mols = [_molecule(r, rng) for r in reqs]
        return SimpleNamespace(reqs=reqs, mols=mols, Ts=[_transitions(m, r["states"], rng) for m, r in zip(mols, reqs)])
    mol = _molecule(case, rng)
    x = SimpleNamespace(mol=mol, T=_transitions(mol, case["states"], rng))
    if case["kind"] == "points":
        v = rng.normal(size=(case["points"], 3))
        x.q = v / np.linalg.norm(v, axis=1)[:, None] * case["qmax"] * rng.random((case["points"], 1)) ** (1.0 / 3.0)
    if case["kind"] == "sph":
        x.qs = case["qmax"] * (np.arange(case["radii"]) + 1.0) / case["radii"]
    if case["kind"] in ("lowq", "fit"):
        x.dE = rng.uniform(0.1, 0.4, size=case["states"])
    if case["kind"] == "lowq":
        # a Gaussian window times trapezoid weights on each axis, as a separable rate integral has
        x.w = []
        for n in (case["nx"], case["ny"], case["nz"]):
            q = np.linspace(-case["qmax"], case["qmax"], n)
            tr = np.full(n, q[1] - q[0])
            tr[0] *= 0.5
            tr[-1] *= 0.5
            x.w.append((np.exp(-0.5 * ((q - rng.uniform(-1, 1)) / rng.uniform(1.0, 3.0)) ** 2) * tr).astype(complex))
    return x


def prepare(case, seed):
    from paper_2512_18010_amd import binding
    x = _inputs(case, seed)
    st = SimpleNamespace(case=case, x=x)
    if case["kind"] == "serve":
        st.server = binding.Server(0, 0, 4)
        return st
    st.ctx = binding.Context(0)
    if case["kind"] in ("points", "fit", "lowq"):
        # a molecule that is loaded already; its precompute has run
        st.ctx.load_molecule(x.mol)
        st.ctx.load_transitions(x.T)
        st.ctx.set_options(EPS if case["kind"] != "fit" else 0.0, 1.0)
        st.ctx.query()
        return st
    ns = case["states"]
    st.T = torch.from_numpy(x.T).to("cuda:0")
    f32 = dict(dtype=torch.float32, device="cuda:0")
    if case["kind"] == "sph":
        shape = (ns, case["radii"], case["n_theta"], case["n_phi"])
        st.R = torch.empty((ns, case["radii"], (case["lmax"] + 1) ** 2, 2), dtype=torch.float64, device="cuda:0")
        st.avg = torch.empty((ns, case["radii"]), dtype=torch.float64, device="cuda:0")
    else:
        shape = (ns, case["nx"], case["ny"], case["nz"])
        if case["kind"] == "fft":
            st.phi = torch.empty(shape, **f32)
        elif case["sym"]:
            st.ctx.set_symmetry(True)
    st.f, st.f2 = torch.empty(shape + (2,), **f32), torch.empty(shape, **f32)
    return st


def run(st):
    case, x = st.case, st.x
    kind = case["kind"]
    if kind == "serve":
        tickets = [st.server.submit(m, T, _grid(r), precision=r["precision"], screen_eps=EPS)
                   for m, T, r in zip(x.mols, x.Ts, x.reqs)]
        done = [st.server.wait(t) for t in tickets]
        assert all(d[0] == 0 for d in done)
        return [(d[2], d[3]) for d in done]
    ctx = st.ctx
    if kind == "points":
        return ctx.eval_points(x.q)
    if kind == "lowq":
        mu, f0 = ctx.dipole(x.dE)
        return mu, f0, ctx.eval_separable(_grid(case), *x.w)
    if kind == "fit":
        return ctx.dipole_fit(case["qfit"], x.dE)
    ctx.load_molecule(x.mol)
    ctx.load_transitions_device(st.T)
    ctx.set_options(EPS, 1.0)
    if kind == "grid":
        ctx.eval_grid_device(_grid(case), st.f, st.f2, precision=case["precision"])
        return st.f, st.f2
    if kind == "fft":
        n, xmin, L = _box(x.mol, case)
        ctx.eval_fft_device(n, xmin, L, st.f, st.f2, st.phi, precision=case["precision"])
        return st.f, st.f2, st.phi
    ctx.eval_spherical_device(case["lmax"], x.qs, case["n_theta"], case["n_phi"], st.f, st.f2, st.R, st.avg)
    return st.f, st.f2, st.R, st.avg


# ------------------------------------------------------------------ the work

_counts = {}


def _pairs(case):
    """(component pairs, primitive terms, 1D-row values per grid value, primitive pairs) that a threshold of 1e-9 on the
    Gaussian product prefactor leaves, counted on one molecule of the case's class."""
    key = (case["heavy"], case["hyd"], case["d"])
    if key not in _counts:
        m = _molecule(case, np.random.Generator(np.random.PCG64(1)))
        nc = np.array([(l + 1) * (l + 2) // 2 for l in m.shell_l.tolist()])
        e = m.exps.reshape(-1, 3)
        X = m.xyz[m.shell_atom]
        K = R = rows = geo = 0
        for a in range(len(nc)):
            r2 = ((X[a] - X[a:]) ** 2).sum(axis=1)[:, None, None]
            mu = e[a][None, :, None] * e[a:][:, None, :] / (e[a][None, :, None] + e[a:][:, None, :])
            kept = (mu * r2 < math.log(1e9)).reshape(len(r2), -1).sum(axis=1)
            comps = nc[a] * nc[a:]
            comps[0] = nc[a] * (nc[a] + 1) // 2
            K += int((comps * (kept > 0)).sum())
            R += int((comps * kept).sum())
            geo += int(kept.sum())
            rows += int((3 * (m.shell_l[a] + 1) * (m.shell_l[a:] + 1) * kept).sum())
        _counts[key] = K, R, rows, geo, int(nc.sum())
    return _counts[key]


def work(case):
    kind = case["kind"]
    if kind == "serve":
        w = [work(r) for r in _requests(case)]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    K, R, rows, geo, nbf = _pairs(case)
    ns = case["states"]
    t_bytes = 8 * ns * nbf * nbf
    if kind == "grid":
        nq = case["nx"] * case["ny"] * case["nz"]
        half = 0.5 if case["sym"] else 1.0
        return {"bytes": t_bytes + 12 * ns * nq, "flops": half * nq * (8.0 * R + 4.0 * K * ns)}
    if kind == "points":
        # per point: three 1D values per row (about 40 operations each), one triple product per term, the contraction
        return {"bytes": (24 + 12 * ns) * case["points"], "flops": case["points"] * (40.0 * rows + 14.0 * R + 4.0 * K * ns)}
    if kind == "fft":
        nr = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": t_bytes + 16 * ns * nr,
                "flops": nr * ns * (nbf * (nbf + 1.0) + 2.5 * math.log2(max(nr, 2)))}
    if kind == "sph":
        nl = (case["lmax"] + 1) ** 2
        return {"bytes": t_bytes + ns * case["radii"] * (16 * nl + 8 + 12 * case["n_theta"] * case["n_phi"]),
                "flops": 8.0 * ns * geo * case["radii"] * nl}
    if kind == "lowq":
        n = case["nx"] + case["ny"] + case["nz"]
        return {"bytes": 16 * (rows + K * ns), "flops": 40.0 * rows * n / 3.0 + 12.0 * R + 10.0 * K * ns}
    return {"bytes": 16 * rows, "flops": 576 * (40.0 * rows + 14.0 * R + 4.0 * K * ns)}


# ------------------------------------------------------------------ the same in 64 bits

def _dev():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=_dev())


def _norm1d(a, i):
    """[int x^2i e^{-2 a x^2} dx]^{-1/2}"""
    return (np.array([1.0, 1.0, 3.0])[i] / (4.0 * a) ** i * np.sqrt(np.pi / (2.0 * a))) ** -0.5


def _functions(mol):
    """Per shell: its first function and, per component, the normalised contraction weights of its primitives."""
    out, first = [], 0
    for s, l in enumerate(mol.shell_l.tolist()):
        a, c = mol.exps[3 * s:3 * s + 3], mol.coefs[3 * s:3 * s + 3]
        ws = []
        for pw in CART[l]:
            w = c * np.prod([_norm1d(a, i) for i in pw], axis=0)
            p = a[:, None] + a[None, :]
            S = np.ones_like(p)
            for i in pw:
                S = S * np.sqrt(np.pi / p) * (np.array([1.0, 1.0, 3.0])[i] / (2.0 * p) ** i)
            ws.append(w / math.sqrt(w @ S @ w))
        out.append((first, np.array(ws)))
        first += len(ws)
    return out, first


def _geometries(mol, T):
    """Groups of primitive pairs by (l_A, l_B): centres P [g, 3], p [g], the powers (u, v, w) and the coefficients
    C [s, n_uvw, g] of f_s(q) = sum_g e^{-q^2/4p + i q.P} sum_uvw C (i q_x)^u (i q_y)^v (i q_z)^w."""
    fn, _ = _functions(mol)
    ls = mol.shell_l
    groups = []
    for la in range(3):
        for lb in range(3):
            A, B = np.where(ls == la)[0], np.where(ls == lb)[0]
            ab = np.array([(a, b) for a in A for b in B if a <= b], dtype=np.int64).reshape(-1, 2)
            if not len(ab):
                continue
            a, b = ab[:, 0], ab[:, 1]
            ea, eb = _t(mol.exps.reshape(-1, 3)[a])[:, :, None], _t(mol.exps.reshape(-1, 3)[b])[:, None, :]
            p = ea + eb
            XA, XB = _t(mol.xyz[mol.shell_atom[a]]), _t(mol.xyz[mol.shell_atom[b]])
            P = (ea[..., None] * XA[:, None, None] + eb[..., None] * XB[:, None, None]) / p[..., None]
            pre = torch.exp(-ea * eb / p * ((XA - XB) ** 2).sum(-1)[:, None, None]) * (math.pi / p) ** 1.5
            # 1D coefficients e[axis][i][j][u]: E[(y + PA + z)^i (y + PB + z)^j], y normal of variance 1/2p, z = iq/2p
            mom = [torch.ones_like(p), torch.zeros_like(p), 0.5 / p, torch.zeros_like(p), 0.75 / p ** 2]
            e1 = {}
            for ax in range(3):
                pa, pb = P[..., ax] - XA[:, None, None, ax], P[..., ax] - XB[:, None, None, ax]
                for i in range(la + 1):
                    for j in range(lb + 1):
                        bt = [torch.zeros_like(p) for _ in range(i + j + 1)]
                        for k in range(i + 1):
                            for m in range(j + 1):
                                bt[k + m] = bt[k + m] + math.comb(i, k) * math.comb(j, m) * pa ** (i - k) * pb ** (j - m)
                        for u in range(i + j + 1):
                            e1[ax, i, j, u] = sum(bt[t] * math.comb(t, u) * mom[t - u] for t in range(u, i + j + 1)) / (2 * p) ** u
            L = la + lb
            uvw = [(u, v, w) for u in range(L + 1) for v in range(L + 1 - u) for w in range(L + 1 - u - v)]
            C = torch.zeros((T.shape[0], len(uvw)) + tuple(p.shape), dtype=torch.float64, device=_dev())
            Td = _t(T)
            fa = torch.as_tensor([fn[k][0] for k in a], device=_dev())
            fb = torch.as_tensor([fn[k][0] for k in b], device=_dev())
            wa, wb = _t(np.array([fn[k][1] for k in a])), _t(np.array([fn[k][1] for k in b]))   # [pair, comp, prim]
            same = torch.as_tensor(a == b, device=_dev())
            for c1, pw1 in enumerate(CART[la]):
                for c2, pw2 in enumerate(CART[lb]):
                    Tp = Td[:, fa + c1, fb + c2]
                    Tp = Tp + torch.where(same, torch.zeros_like(Tp), Td[:, fb + c2, fa + c1])
                    k = pre * wa[:, c1, :, None] * wb[:, c2, None, :]
                    for n, pw in enumerate(uvw):
                        if all(pw[x] <= pw1[x] + pw2[x] for x in range(3)):
                            e = k
                            for x in range(3):
                                e = e * e1[x, pw1[x], pw2[x], pw[x]]
                            C[:, n] += Tp[:, :, None, None] * e
            g = p.numel()
            groups.append((P.reshape(g, 3), p.reshape(g), uvw, C.reshape(T.shape[0], len(uvw), g)))
    return groups


def _f_at(groups, q, ns):
    """f_s at points q [n, 3] -> complex128 [s, n]."""
    q = _t(q)
    f = torch.zeros((ns, len(q)), dtype=torch.complex128, device=_dev())
    for q0 in range(0, len(q), 32768):
        qc = q[q0:q0 + 32768]
        q2 = (qc ** 2).sum(1)
        for P, p, uvw, C in groups:
            F = torch.zeros((ns * len(uvw), 2 * len(qc)), dtype=torch.float64, device=_dev())
            for g0 in range(0, len(p), 4096):
                g = slice(g0, g0 + 4096)
                ga, ph = torch.exp(-q2[None, :] / (4.0 * p[g, None])), P[g] @ qc.T
                E = torch.cat([ga * torch.cos(ph), ga * torch.sin(ph)], dim=1)
                F += C[:, :, g].reshape(ns * len(uvw), -1) @ E
            F = torch.complex(F[:, :len(qc)], F[:, len(qc):]).reshape(ns, len(uvw), len(qc))
            for n, pw in enumerate(uvw):
                f[:, q0:q0 + 32768] += F[:, n] * (1j ** sum(pw)) * qc[:, 0] ** pw[0] * qc[:, 1] ** pw[1] * qc[:, 2] ** pw[2]
    return f


def _f_grid(mol, T, grid):
    """f_s on a Cartesian grid, e^{-q^2/4p + iq.P} as the product of its axes' factors -> complex128 [s, nx, ny, nz]."""
    ns = T.shape[0]
    ax = [_t(np.linspace(grid.qmin[a], grid.qmax[a], grid.n[a])) for a in range(3)]
    nyz = grid.n[1] * grid.n[2]
    f = torch.zeros((ns, grid.n[0], nyz), dtype=torch.complex128, device=_dev())
    qy, qz = ax[1].repeat_interleave(grid.n[2]), ax[2].repeat(grid.n[1])
    step = max(1, 65536 // nyz)
    for P, p, uvw, C in _geometries(mol, T):
        E = [torch.polar(torch.exp(-ax[a] ** 2 / (4.0 * p[:, None])), P[:, a, None] * ax[a]) for a in range(3)]
        mono = torch.stack([qy ** w[1] * qz ** w[2] for w in uvw])
        for x0 in range(0, grid.n[0], step):
            qx = ax[0][x0:x0 + step]
            F = torch.zeros((ns * len(uvw), 2 * len(qx) * nyz), dtype=torch.float64, device=_dev())
            for g0 in range(0, len(p), 4096):
                g = slice(g0, g0 + 4096)
                Eyz = (E[1][g][:, :, None] * E[2][g][:, None, :]).reshape(-1, 1, nyz)
                Exyz = torch.view_as_real(E[0][g][:, x0:x0 + step, None] * Eyz).reshape(Eyz.shape[0], -1)
                F += C[:, :, g].reshape(ns * len(uvw), -1) @ Exyz
            F = torch.view_as_complex(F.reshape(ns, len(uvw), len(qx), nyz, 2))
            for n, pw in enumerate(uvw):
                f[:, x0:x0 + step] += F[:, n] * (1j ** sum(pw)) * qx[:, None] ** pw[0] * mono[n]
    return f.reshape((ns,) + tuple(grid.n))


def _pair_of(f):
    """(f as [..., 2], |f|^2)"""
    return torch.view_as_real(f.contiguous()), f.real ** 2 + f.imag ** 2


def _exact_fft(mol, T, case):
    n, xmin, L = _box(mol, case)
    fn, nbf = _functions(mol)
    ax = [xmin[a] + np.arange(n[a]) * (L[a] / n[a]) for a in range(3)]
    pts = _t(np.stack(np.meshgrid(*ax, indexing="ij"), axis=-1).reshape(-1, 3))
    Ts = [_t(t + t.T) * 0.5 for t in T]
    phi = torch.empty((len(Ts), len(pts)), dtype=torch.float64, device=_dev())
    for i0 in range(0, len(pts), 1 << 17):
        x = pts[i0:i0 + (1 << 17)]
        ao = torch.empty((nbf, len(x)), dtype=torch.float64, device=_dev())
        for s, l in enumerate(mol.shell_l.tolist()):
            d = x - _t(mol.xyz[mol.shell_atom[s]])
            e = torch.exp(-_t(mol.exps[3 * s:3 * s + 3])[:, None] * (d ** 2).sum(1)[None, :])
            for c, pw in enumerate(CART[l]):
                ao[fn[s][0] + c] = (_t(fn[s][1][c]) @ e) * d[:, 0] ** pw[0] * d[:, 1] ** pw[1] * d[:, 2] ** pw[2]
        for k, t in enumerate(Ts):
            phi[k, i0:i0 + (1 << 17)] = ((t @ ao) * ao).sum(0)
    phi = phi.reshape((len(Ts),) + n)
    F = torch.fft.fftshift(torch.fft.fftn(phi.to(torch.complex128), dim=(1, 2, 3)), dim=(1, 2, 3)).conj()
    ph = [_t(2.0 * np.pi * (np.arange(n[a]) - n[a] // 2) / L[a] * xmin[a]) for a in range(3)]
    ang = ph[0][:, None, None] + ph[1][None, :, None] + ph[2][None, None, :]
    return _pair_of(F * torch.polar(torch.full_like(ang, float(np.prod(np.array(L) / np.array(n)))), ang)) + (phi,)


def _harmonics(lmax, theta, phi):
    """Orthonormal complex Y_l^m (Condon-Shortley), index l^2 + l + m -> complex128 [(lmax+1)^2, n]."""
    x, sx = np.cos(theta), np.sin(theta)
    out = np.zeros(((lmax + 1) ** 2, theta.size), np.complex128)
    pmm = np.full(theta.size, math.sqrt(0.25 / math.pi))
    for m in range(lmax + 1):
        if m:
            pmm = -math.sqrt((2 * m + 1) / (2 * m)) * sx * pmm
        below, cur = np.zeros_like(pmm), pmm
        for l in range(m, lmax + 1):
            out[l * l + l + m] = cur * np.exp(1j * m * phi)
            out[l * l + l - m] = (-1) ** m * np.conj(out[l * l + l + m])
            a = math.sqrt(((2 * l + 1) * (2 * l + 3)) / ((l + 1 - m) * (l + 1 + m)))
            b = math.sqrt(((2 * l + 3) * (l - m) * (l + m)) / ((2 * l - 1) * (l + 1 - m) * (l + 1 + m))) if l > m else 0.0
            below, cur = cur, a * x * cur - b * below
    return out


def _exact_sph(mol, T, case, qs):
    lmax, ns = case["lmax"], T.shape[0]
    r = float(np.linalg.norm(mol.xyz, axis=1).max()) + 3.0
    nt = int((lmax + math.e * qs.max() * r / 2 + 24) / 2) + 2
    xg, wg = np.polynomial.legendre.leggauss(nt)
    th, ph = np.meshgrid(np.arccos(xg), 2.0 * np.pi * np.arange(2 * nt) / (2 * nt), indexing="ij")
    th, ph = th.ravel(), ph.ravel()
    w = np.repeat(wg, 2 * nt) * (np.pi / nt)
    u = np.stack([np.sin(th) * np.cos(ph), np.sin(th) * np.sin(ph), np.cos(th)], axis=1)
    f = _f_at(_geometries(mol, T), (qs[:, None, None] * u[None]).reshape(-1, 3), ns).reshape(ns * len(qs), -1)
    Y = torch.as_tensor(_harmonics(lmax, th, ph), device=_dev())
    R = (f * _t(w)) @ Y.conj().T.contiguous()
    tg, pg = np.meshgrid(np.pi * np.arange(case["n_theta"]) / (case["n_theta"] - 1),
                         2.0 * np.pi * np.arange(case["n_phi"]) / case["n_phi"], indexing="ij")
    fg = (R @ torch.as_tensor(_harmonics(lmax, tg.ravel(), pg.ravel()), device=_dev()))
    fg = fg.reshape(ns, len(qs), case["n_theta"], case["n_phi"])
    R = R.reshape(ns, len(qs), -1)
    return _pair_of(fg) + (torch.view_as_real(R.contiguous()), (R.abs() ** 2).sum(-1) / (4.0 * math.pi))


def _exact_dipole(groups, dE):
    mu = 0.0
    for P, p, uvw, C in groups:
        for a in range(3):
            e = [0, 0, 0]
            e[a] = 1
            d = C[:, uvw.index((0, 0, 0))] @ P[:, a]
            if tuple(e) in uvw:
                d = d + C[:, uvw.index(tuple(e))].sum(-1)
            row = torch.zeros((C.shape[0], 3), dtype=torch.float64, device=_dev())
            row[:, a] = d
            mu = mu + row
    return mu, 2.0 / 3.0 * _t(dE) * (mu ** 2).sum(1)


def _exact_separable(groups, grid, ws, ns):
    out = torch.zeros(ns, dtype=torch.complex128, device=_dev())
    for P, p, uvw, C in groups:
        top = max(max(w) for w in uvw)
        S = []
        for a in range(3):
            q = _t(np.linspace(grid.qmin[a], grid.qmax[a], grid.n[a]))
            E = torch.polar(torch.exp(-q ** 2 / (4.0 * p[:, None])), P[:, a, None] * q)
            w = torch.as_tensor(ws[a], device=_dev())
            S.append([(E * (w * (1j * q) ** u)).sum(1) for u in range(top + 1)])
        for n, (u, v, w) in enumerate(uvw):
            out += C[:, n].to(torch.complex128) @ (S[0][u] * S[1][v] * S[2][w])
    return out


def _exact_fit(groups, q_fit, dE, ns):
    xt, wt = np.polynomial.legendre.leggauss(6)
    ph = 2.0 * np.pi * np.arange(12) / 12
    st = np.sqrt(1.0 - xt ** 2)
    u = np.stack([np.outer(st, np.cos(ph)), np.outer(st, np.sin(ph)), np.outer(xt, np.ones(12))], axis=-1).reshape(-1, 3)
    r = q_fit * np.arange(1, 9) / 8.0
    f = _f_at(groups, (r[:, None, None] * u[None]).reshape(-1, 3), ns).reshape(ns, 8, 72)
    avg = ((f.abs() ** 2) * _t(np.repeat(wt, 12) / 24.0)).sum(-1).cpu().numpy()
    x = (r / q_fit) ** 2
    c = np.linalg.lstsq(np.stack([np.ones(8), x, x * x], axis=1), avg.T, rcond=None)[0].T
    c = c / np.array([1.0, q_fit ** 2, q_fit ** 4])
    return c, 2.0 * dE * c[:, 1]


def exact(case, seed):
    x = _inputs(case, seed)
    kind = case["kind"]
    if kind == "serve":
        out = []
        for m, T, r in zip(x.mols, x.Ts, x.reqs):
            f = _f_grid(m, T, _grid(r))
            out.append((f.cpu().numpy(), (f.real ** 2 + f.imag ** 2).cpu().numpy()))
        return out
    if kind == "grid":
        return _pair_of(_f_grid(x.mol, x.T, _grid(case)))
    if kind == "fft":
        return _exact_fft(x.mol, x.T, case)
    if kind == "sph":
        return _exact_sph(x.mol, x.T, case, x.qs)
    groups = _geometries(x.mol, x.T)
    ns = case["states"]
    if kind == "points":
        f = _f_at(groups, x.q, ns).cpu().numpy()
        return f, np.abs(f) ** 2
    if kind == "lowq":
        mu, f0 = _exact_dipole(groups, x.dE)
        return mu, f0, _exact_separable(groups, _grid(case), x.w, ns)
    return _exact_fit(groups, case["qfit"], x.dE, ns)
