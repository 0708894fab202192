"""Separable integrals: each weighted value is as accurate as its own phase.

One s function far from the origin; with weights that pick a single grid value
the integral is one 1D value, e^{-q^2/4p} e^{iqP} times constants, against the
same in 120 bits.  The axis has exactly representable values.
"""
import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [129, 128])   # symmetric about 0 (n odd: q = 0 once) and not
def test_single_values(n):
    import torch  # noqa: F401
    from mpmath import exp, mp, mpf, pi
    from paper_2512_18010_amd import binding
    mp.prec = 120
    P, alpha = np.array([9.7, 11.3, -8.7]), 3.0
    mol = wl.Molecule(Z=np.array([6]), xyz=P[None], shell_atom=np.zeros(1, np.int32), shell_l=np.zeros(1, np.int32),
                      shell_nprim=np.ones(1, np.int32), exps=np.array([alpha]), coefs=np.ones(1))
    q = -8.0 + 0.125 * np.arange(n)
    grid = wl.Grid(n=(n, n, n), qmin=(-8.0,) * 3, qmax=(q[-1],) * 3)
    zero = np.zeros(n, complex)
    zero[64] = 1.0   # q = 0: a phase of 0 on the other axes
    print("case separable_phase", n, flush=True)
    with binding.Context(0) as ctx:
        ctx.load_molecule(mol)
        ctx.load_transitions(np.ones((1, 1, 1)))
        ctx.set_options(0.0, 1.0)
        for axis in range(3):
            for i in range(n):
                w = [zero, zero, zero]
                w[axis] = np.zeros(n, complex)
                w[axis][i] = 1.0
                v = ctx.eval_separable(grid, *w)[0]
                # a normalised s function: f(q) = e^{-q^2/4p} e^{iqP}, p = 2 alpha
                ref = exp(-mpf(q[i]) ** 2 / (8 * mpf(alpha))) * exp(1j * mpf(q[i]) * mpf(P[axis]))
                # three roundings of qP / 2 pi in the phase; sine, cosine, exponential,
                # norms and products: 20 roundings; one of the exponent
                tol = 2.0 ** -53 * (4 * abs(q[i] * P[axis]) + 24 + q[i] ** 2 / (8 * alpha))
                assert abs(mpf(v.real) + 1j * mpf(v.imag) - ref) <= tol * abs(ref), (axis, i, q[i])
