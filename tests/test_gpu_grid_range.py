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
TOL = {"fp32": 80 * 2.0 ** -24}


def one_centre(tight):
    rng = np.random.Generator(np.random.PCG64(77))
    n = 5
    exps = np.exp(rng.uniform(np.log(0.1), np.log(1.0), size=(n, 3)))
    if tight:
        exps[-1] = [20.0, 30.0, 40.0]
    mol = wl.Molecule(Z=np.array([6]), xyz=np.zeros((1, 3)), shell_atom=np.zeros(n, np.int32),
                      shell_l=np.zeros(n, np.int32), shell_nprim=np.full(n, 3, np.int32), exps=exps.ravel(),
                      coefs=rng.uniform(0.2, 1.0, size=3 * n))
    T = rng.uniform(0.5, 1.0, size=(3, n, n))
    if tight:
        T[:, -1, :] *= 1e-9
        T[:, :, -1] *= 1e-9
    return mol, T


@pytest.mark.parametrize("precision", ["fp32"])
@pytest.mark.parametrize("tight", [False, True])
@pytest.mark.parametrize("sym", [True, False])
def test_tail_relative(oracle_mod, sym, tight, precision):
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    mol, T = one_centre(tight)
    grid = wl.Grid(n=(7, 6, 35), qmin=(-12.0, -11.0, -12.0 if sym else -9.0), qmax=(12.0, 12.0, 12.0))
    print("case grid_range", sym, tight, precision, flush=True)
    with binding.Context(0) as ctx:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        f, _ = ctx.eval_grid_host(grid, precision)
    ref = oracle_mod.eval_grid(mol, T, grid, n_threads=NTH)
    a = np.abs(ref)
    err = (np.abs(f - ref) / a).max()
    print(f"  |f| from {a.max():.1e} down to {a.min():.1e}: relative error {err:.1e}", flush=True)
    assert a.min() < 1e-9 * a.max()
    assert err <= TOL[precision]
