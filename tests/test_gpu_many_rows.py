"""A molecule whose precompute has more than 2^31 flags of rows and of weights.

485 s shells of 32 primitives: 362 million 1D rows, 121 million terms; with 32
states the grid kernel's weights exceed 2^31 values.  The shells are 97 copies of
five, so f is that of five shells with the transition densities summed over the
copies: points and transition dipoles against the FP64 oracle (the dipole as
the slope of f at q = 0).
"""
import numpy as np
import pytest

import workload as wl
from tests.metrics import errors

pytestmark = pytest.mark.gpu

def test_points_of_many_terms(oracle_mod):
    import torch
    from paper_2512_18010_amd import binding
    if torch.cuda.get_device_properties(0).total_memory < 200e9:
        pytest.skip("needs 110 GB of device memory")
    kinds, copies, ns = 5, 97, 32
    n = kinds * copies
    rng = np.random.Generator(np.random.PCG64(485))
    exps = np.exp(rng.uniform(np.log(0.1), np.log(50.0), size=(kinds, 32)))
    coefs = rng.uniform(0.1, 1.0, size=(kinds, 32))

    def molecule(m):
        return wl.Molecule(Z=np.full(kinds, 6), xyz=np.linspace(-2.0, 2.0, 3 * kinds).reshape(kinds, 3) ** 2 - 1.0,
                           shell_atom=np.tile(np.arange(kinds, dtype=np.int32), m), shell_l=np.zeros(kinds * m, np.int32),
                           shell_nprim=np.full(kinds * m, 32, np.int32), exps=np.tile(exps, (m, 1)).ravel(),
                           coefs=np.tile(coefs, (m, 1)).ravel())

    mol = molecule(copies)
    T = rng.normal(size=(ns, n, n)) / n
    T5 = T.reshape(ns, copies, kinds, copies, kinds).sum(axis=(1, 3))
    h = 1e-3
    q = np.array([[0.3, -0.2, 0.5], [h, 0, 0], [-h, 0, 0]])
    print("case many_rows", flush=True)
    with binding.Context(0) as ctx:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        f, f2 = ctx.eval_points(q)
        mu, _ = ctx.dipole(None)
        info = ctx.query()
    print(f"  {info['device_bytes'] / 1e9:.0f} GB", flush=True)
    assert info["prim_comp_pairs_kept"] == n * (n + 1) // 2 * 1024
    ref = oracle_mod.eval_points(molecule(1), T5, q, n_threads=1)
    assert errors(f, ref)["f2_peak_norm"].max() <= 1e-6
    slope = (ref[:, 1] - ref[:, 2]).imag / (2 * h)   # error h^2/6 times the third moment
    assert np.abs(mu[:, 0] - slope).max() <= 1e-4 * np.abs(slope).max()
