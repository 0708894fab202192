"""Grid kernel: values far below the peak keep their relative accuracy.

One centre and positive weights, so every term of f is positive and the error
of the sum is bounded relative to the sum itself, at every q.  A diffuse basis
(exponents up to 1) at |q_i| up to 12: f falls by more than twenty decades.
With a tight shell of small weight the tail is its contribution alone.
"""
import os

import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu

NTH = min(16, os.cpu_count() or 1)

# FP32: the roundings of a term (1D tables, W, weight, U's sum over at most 9
# terms, z operand: 16) and the additions of two k-steps of 32, each 2^-24.
# Split precision: what BF16 halves hold, 2^-16, and the additions of all k-steps
# (15 shell pairs of 9 rows: 160).
TOL = {"fp32": 80 * 2.0 ** -24, "bf16x3": 2.0 ** -16 + 176 * 2.0 ** -24}


def one_centre(weight):
    rng = np.random.Generator(np.random.PCG64(77))
    n = 5
    exps = np.exp(rng.uniform(np.log(0.1), np.log(1.0), size=(n, 3)))
    if weight:
        exps[-1] = [20.0, 30.0, 40.0]
    mol = wl.Molecule(Z=np.array([6]), xyz=np.zeros((1, 3)), shell_atom=np.zeros(n, np.int32),
                      shell_l=np.zeros(n, np.int32), shell_nprim=np.full(n, 3, np.int32), exps=exps.ravel(),
                      coefs=rng.uniform(0.2, 1.0, size=3 * n))
    T = rng.uniform(0.5, 1.0, size=(3, n, n))
    if weight:
        T[:, -1, :] *= weight
        T[:, :, -1] *= weight
    return mol, T


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("weight", [0.0, 1e-1, 1e-4, 1e-9], ids=lambda w: f"tight{w:g}")   # of the tight shell
@pytest.mark.parametrize("sym", [True, False])
def test_tail_relative(oracle_mod, sym, weight, precision):
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    mol, T = one_centre(weight)
    grid = wl.Grid(n=(7, 6, 35), qmin=(-12.0, -11.0, -12.0 if sym else -9.0), qmax=(12.0, 12.0, 12.0))
    print("case grid_range", sym, weight, precision, flush=True)
    with binding.Context(0) as ctx:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        f, _ = ctx.eval_grid_host(grid, precision)
    ref = oracle_mod.eval_grid(mol, T, grid, n_threads=NTH)
    a = np.abs(ref)
    err = (np.abs(f - ref) / a).max()
    print(f"  |f| from {a.max():.1e} down to {a.min():.1e}: relative error {err:.1e}", flush=True)
    assert err <= TOL[precision]


def diffuse(states):
    """Two centres, s, p and d shells, exponents up to 1: split precision takes its BF16 parts."""
    rng = np.random.Generator(np.random.PCG64(500 + states))
    l = np.array([0, 1, 2, 0, 1], np.int32)
    mol = wl.Molecule(Z=np.array([6, 6]), xyz=np.array([[0.0, 0.0, 0.0], [1.0, 1.5, -0.7]]),
                      shell_atom=np.array([0, 0, 0, 1, 1], np.int32), shell_l=l, shell_nprim=np.full(5, 2, np.int32),
                      exps=np.exp(rng.uniform(np.log(0.1), 0.0, size=10)), coefs=rng.uniform(0.2, 1.0, size=10))
    T = rng.normal(size=(states, mol.nbf, mol.nbf))
    return mol, T


# (states, nx, ny, nz, symmetric q_z): every width of a column tile and a remainder
@pytest.mark.parametrize("case", [(1, 3, 5, 33, True), (3, 6, 3, 65, False), (12, 2, 5, 64, True), (24, 2, 3, 47, False),
                                  (31, 2, 3, 130, False)],
                         ids=lambda c: f"s{c[0]}_{c[1]}x{c[2]}x{c[3]}{'sym' if c[4] else ''}")
def test_split_bf16_parts(oracle_mod, case):
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    from tests.metrics import TOL_F2, errors
    ns, nx, ny, nz, sym = case
    mol, T = diffuse(ns)
    grid = wl.Grid(n=(nx, ny, nz), qmin=(-10.0, -10.0, -10.0 if sym else -9.0), qmax=(10.0, 9.0, 10.0))
    print("case split_bf16_parts", case, flush=True)
    with binding.Context(0) as ctx:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        f, f2 = ctx.eval_grid_host(grid, "bf16x3")
    ref = oracle_mod.eval_grid(mol, T, grid, n_threads=NTH)
    e = errors(f, ref)["f2_peak_norm"].max()
    print(f"  max peak-normalised |f|^2 err {e:.2e}", flush=True)
    assert e <= TOL_F2["bf16x3"]
    with binding.Server(0, 0, 2) as srv:   # the batch kernel: the same tiles
        t = srv.submit(mol, T, grid, precision="bf16x3", screen_eps=0.0)
        status, _, fs, f2s = srv.wait(t)[:4]
    assert status == 0
    np.testing.assert_array_equal(fs.view(np.float32), f.view(np.float32))
    np.testing.assert_array_equal(f2s, f2)
