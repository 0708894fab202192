"""Column tiles of the grid kernel on wide q_z axes against the FP64 oracle.

A tile takes 1 to 3 (FP32) or 4 (split-BF16) groups of 16 columns, with at most
one group of padding in all; the widths put the choice on each side of that:
4, 7, 8 and 13 groups, full and with a remainder.  Every element is compared;
tolerance: the precision's own peak-normalised |f|^2 limit.
"""
import os

import numpy as np
import pytest

import workload as wl
from tests.metrics import TOL_F2, errors

pytestmark = pytest.mark.gpu

NTH = min(16, os.cpu_count() or 1)


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("nz", [64, 101, 112, 128, 195, 208])
def test_column_tiles(oracle_mod, nz, precision):
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    rng = np.random.Generator(np.random.PCG64(nz))
    mol = wl.make_molecule(rng, 3, 3, layout="box", box_A=3.0)
    T = wl.make_transitions(rng, mol.nbf, wl.n_occupied(mol.Z), 6)
    grid = wl.Grid(n=(2, 5, nz), qmin=(-3.0, -4.0, -5.0), qmax=(4.0, 3.5, 4.25))
    print("case column_tiles", nz, precision, flush=True)
    ctx = binding.Context(0)
    try:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        f, f2 = ctx.eval_grid_host(grid, precision)
    finally:
        ctx.close()
    ref = oracle_mod.eval_grid(mol, T, grid, n_threads=NTH)
    np.testing.assert_allclose(f2, np.abs(f) ** 2, rtol=2e-6, atol=1e-12 * np.abs(f).max() ** 2)
    e = errors(f, ref)["f2_peak_norm"].max()
    print(f"  max peak-normalised |f|^2 err {e:.2e}", flush=True)
    assert e <= TOL_F2[precision]
