"""FFT method: contraction coefficients of very different size.

With normalise the result does not depend on the scale of a shell's
coefficients (the contracted norm undoes it), however small or large they are
given: the transition density on a box against the oracle's for the same
molecule, and against the density of the molecule with coefficients of order 1.
"""
import dataclasses
import os

import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu

NTH = min(16, os.cpu_count() or 1)


def density(mol, T, n, xmin, L, precision):
    from paper_2512_18010_amd import binding
    with binding.Context(0) as ctx:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        return ctx.eval_fft_host(n, xmin, L, want_phi=True, precision=precision)[2]


# FP32: as the other density tests, FP32 roundings of sums over the basis with a
# decade of cancellation; split-BF16: 2^-16 a product
@pytest.mark.parametrize("precision,tol", [("fp32", 1e-6), ("bf16x3", 1e-4)])
@pytest.mark.parametrize("scale", [1e-12, 1e9])
def test_coefficient_scale(oracle_mod, scale, precision, tol):
    import torch  # noqa: F401
    rng = np.random.Generator(np.random.PCG64(31))
    mol = wl.make_molecule(rng, 2, 2, layout="box", box_A=3.0)
    T = wl.make_transitions(rng, mol.nbf, wl.n_occupied(mol.Z), 3)
    off = np.concatenate([[0], np.cumsum(mol.shell_nprim)])
    coefs = mol.coefs.copy()
    for s in range(0, mol.n_shells, 2):   # every other shell
        coefs[off[s]:off[s + 1]] *= scale
    scaled = dataclasses.replace(mol, coefs=coefs)
    n, L = (16, 8, 16), np.array([9.0, 8.0, 10.0])
    xmin = mol.xyz.mean(axis=0) - 0.5 * L
    print("case fft_coefs", scale, precision, flush=True)
    a, b = (density(m, T, n, xmin, L, precision) for m in (scaled, mol))
    _, ref = oracle_mod.fft_form_factor(mol, T, n, xmin, L, spin_factor=1.0, n_threads=NTH)
    peak = np.abs(ref).reshape(3, -1).max(axis=1).reshape(3, 1, 1, 1)
    ea, eb = (np.abs(x - ref).__truediv__(peak).max() for x in (a, b))
    print(f"  density error {ea:.1e}, coefficients of order 1 {eb:.1e}", flush=True)
    assert max(ea, eb) <= tol


# the last basis of every tile width and the first of the next: 64, 32 and 16 points, one workgroup per CU, the largest
@pytest.mark.parametrize("precision,tol", [("fp32", 1e-6), ("bf16x3", 1e-4)])
@pytest.mark.parametrize("nbf", [192, 193, 400, 401, 820, 1232])
def test_basis_sizes(oracle_mod, nbf, precision, tol):
    import torch  # noqa: F401
    rng = np.random.Generator(np.random.PCG64(nbf))
    mol = wl.Molecule(Z=np.full(20, 6), xyz=rng.uniform(-3.0, 3.0, size=(20, 3)),
                      shell_atom=rng.integers(0, 20, size=nbf).astype(np.int32), shell_l=np.zeros(nbf, np.int32),
                      shell_nprim=np.ones(nbf, np.int32), exps=np.exp(rng.uniform(np.log(0.2), np.log(20.0), size=nbf)),
                      coefs=np.ones(nbf))
    T = rng.normal(size=(2, nbf, nbf)) / nbf
    n, L = (8, 4, 8), np.array([8.0, 8.0, 8.0])
    xmin = np.array([-4.0, -4.0, -4.0])
    print("case fft_basis_sizes", nbf, precision, flush=True)
    phi = density(mol, T, n, xmin, L, precision)
    _, ref = oracle_mod.fft_form_factor(mol, T, n, xmin, L, spin_factor=1.0, n_threads=NTH)
    e = (np.abs(phi - ref).reshape(2, -1).max(axis=1) / np.abs(ref).reshape(2, -1).max(axis=1)).max()
    print(f"  density error {e:.1e}", flush=True)
    assert e <= tol


def test_basis_too_large():
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    mol = wl.Molecule(Z=np.array([6]), xyz=np.zeros((1, 3)), shell_atom=np.zeros(1233, np.int32),
                      shell_l=np.zeros(1233, np.int32), shell_nprim=np.ones(1233, np.int32), exps=np.ones(1233),
                      coefs=np.ones(1233))
    for precision in ("fp32", "bf16x3"):
        with pytest.raises(binding.ScffError) as ei:
            density(mol, np.zeros((1, 1233, 1233)), (8, 8, 8), (-4.0,) * 3, (8.0,) * 3, precision)
        assert ei.value.code == binding.SCFF_EINVAL
