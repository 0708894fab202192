"""FFT method, FP32 precision: the powers of two of the split operands.

Points far from the molecule (every AO value small), weights scaled by exact
powers of two (the result scales exactly: only exponents move), transitions
whose rows differ by many orders of magnitude, one basis per tile width (64, 32
and 16 points).
"""
import os

import numpy as np
import pytest

import workload as wl
from tests.test_gpu_fft import TOL_FFT

pytestmark = pytest.mark.gpu

NTH = min(16, os.cpu_count() or 1)


def evaluate(mol, T, n, xmin, L):
    from paper_2512_18010_amd import binding
    with binding.Context(0) as ctx:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        return ctx.eval_fft_host(n, xmin, L, want_phi=True)


def peak_error(x, ref):
    ns = ref.shape[0]
    return (np.abs(x - ref).reshape(ns, -1).max(axis=1) / np.abs(ref).reshape(ns, -1).max(axis=1)).max()


@pytest.mark.parametrize("heavy,hyd,shift,rows", [(2, 2, 0.0, False), (2, 2, 8.0, False), (3, 1, 0.0, True),
                                                  (16, 0, 0.0, False), (30, 24, 0.0, False)])
def test_scales(oracle_mod, heavy, hyd, shift, rows):
    import torch  # noqa: F401
    rng = np.random.Generator(np.random.PCG64(90 + heavy))
    mol = wl.make_molecule(rng, heavy, hyd, layout="box", box_A=3.0 if heavy < 10 else 8.0)
    T = wl.make_transitions(rng, mol.nbf, wl.n_occupied(mol.Z), 3)
    if rows:   # weights over 30 orders of magnitude, row by row
        T = T * (10.0 ** rng.uniform(-30.0, 0.0, mol.nbf))[None, :, None]
        T = 0.5 * (T + T.transpose(0, 2, 1))
    n = (16, 8, 16)
    L = np.array([9.0, 8.0, 10.0])
    xmin = mol.xyz.mean(axis=0) - 0.5 * L + shift
    print("case fft_scales", heavy, hyd, shift, rows, mol.nbf, flush=True)
    f, f2, phi, _ = evaluate(mol, T, n, xmin, L)
    f_ref, phi_ref = oracle_mod.fft_form_factor(mol, T, n, xmin, L, spin_factor=1.0, n_threads=NTH)
    e = peak_error(phi, phi_ref)
    print(f"  phi {e:.1e} f {peak_error(f, f_ref):.1e}", flush=True)
    # phi: operands within 2^-23 each, FP32 sums of 16-term products over the
    # basis, one rounding; cancellation in the sum costs a decade at most here
    assert e <= 1e-6
    assert np.abs(np.abs(f) ** 2 - np.abs(f_ref) ** 2).max() <= TOL_FFT * (np.abs(f_ref) ** 2).max()
    for k in (-20, 30):
        fk, _, phik, _ = evaluate(mol, T * 2.0 ** k, n, xmin, L)
        for a, b in ((phik, phi), (fk, f)):
            m = np.abs(b) > 1e-25   # scaled values stay normal numbers
            np.testing.assert_array_equal(a[m], b[m] * np.float32(2.0 ** k))
