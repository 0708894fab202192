"""Spherical contraction: row tiles of 32 (two blocks of 16 rows with extents of
their own), column tiles of 128, radii in fours, segments of the geometries, no
geometry with d functions, against the oracle's R_lm; with and without room for
the segments' partial sums.  All FP64: the spherical method's own tolerance.
"""
import numpy as np
import pytest

import workload as wl
from tests.test_gpu_sph import TOL_R, oracle_R, r_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nq,lmax,with_d", [(1, 1, 0, True), (2, 6, 11, False), (13, 5, 7, True), (32, 3, 8, True)])
def test_contraction_tiles(oracle_mod, ns, nq, lmax, with_d):
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    rng = np.random.Generator(np.random.PCG64(40 + ns))
    mol = wl.make_molecule(rng, 2, 2, layout="box", box_A=2.0, with_d=with_d)
    T = wl.make_transitions(rng, mol.nbf, wl.n_occupied(mol.Z), ns)
    qs = np.linspace(0.0, 2.5, nq) if nq > 1 else np.array([1.3])
    print("case sph_tiles", ns, nq, lmax, with_d, flush=True)
    out, full = [], 0
    for less in (0, 1):
        with binding.Context(0, hbm_budget_bytes=full - 1 if less else 0) as ctx:
            ctx.load_molecule(mol)
            ctx.load_transitions(T)
            ctx.set_options(0.0, 1.0)
            R, _, _, avg = ctx.eval_spherical_host(lmax, qs)
            full = full or ctx.query()["device_bytes"]
            out.append(R)
    ref = oracle_R(oracle_mod, mol, T, qs, lmax)
    e = r_error(out[0], ref).max()
    print(f"  R relative {e:.1e}", flush=True)
    assert e <= TOL_R
    assert r_error(out[1], ref).max() <= TOL_R
    np.testing.assert_allclose(avg, oracle_mod.angular_average_from_R(out[0]), rtol=1e-12)
