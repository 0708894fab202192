"""Tile edges of the grid kernel against the FP64 oracle, every element.

A tile is 64 rows (row = line * states + state, lines in pairs of one q_x) by
16 to 64 columns (the upper half of a q_z axis symmetric about 0), z rows come
in steps of 32, terms in steps of one or two.  The cases put a remainder on
each of them.  Tolerance: the precision's own peak-normalised |f|^2 limit.
"""
import os

import numpy as np
import pytest

import workload as wl
from tests.metrics import TOL_F2, errors

pytestmark = pytest.mark.gpu

NTH = min(16, os.cpu_count() or 1)

# (states, nx, ny, nz, symmetric q_z)
CASES = [
    (1, 1, 1, 1, False),      # one output value
    (1, 7, 19, 33, True),     # most line pairs per tile, 17 columns
    (1, 4, 16, 128, True),    # few states: one term per step, 4 column groups do not fit
    (2, 5, 13, 16, False),    # one full column group
    (3, 6, 11, 65, False),    # 5 groups: two column tiles, odd number of lines
    (5, 3, 9, 97, True),      # 49 columns: 4 groups with one column in the last
    (7, 2, 7, 17, False),
    (12, 4, 8, 64, True),     # 2 column groups
    (13, 3, 5, 31, True),
    (16, 2, 6, 96, True),     # rows of a tile end with a line, 3 groups
    (24, 2, 3, 47, False),
    (31, 2, 5, 130, False),   # 9 groups: column tiles of 3
    (32, 3, 1, 66, True),     # single line per q_x
]


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"s{c[0]}_{c[1]}x{c[2]}x{c[3]}{'sym' if c[4] else ''}")
def test_tile_edges(oracle_mod, case, precision):
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    ns, nx, ny, nz, sym = case
    rng = np.random.Generator(np.random.PCG64(1000 * ns + nz))
    mol = wl.make_molecule(rng, 3, 3, layout="box", box_A=3.0)
    T = wl.make_transitions(rng, mol.nbf, wl.n_occupied(mol.Z), ns)
    grid = wl.Grid(n=(nx, ny, nz), qmin=(-3.0, -4.0, -5.0), qmax=(4.0, 3.5, 5.0 if sym else 4.25))
    print("case tile_edges", case, precision, flush=True)
    ctx = binding.Context(0)
    try:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        f, f2 = ctx.eval_grid_host(grid, precision)
    finally:
        ctx.close()
    ref = oracle_mod.eval_grid(mol, T, grid, n_threads=NTH)
    assert np.isfinite(f.view(np.float32)).all()
    np.testing.assert_allclose(f2, np.abs(f) ** 2, rtol=2e-6, atol=1e-12 * np.abs(f).max() ** 2)
    e = errors(f, ref)["f2_peak_norm"].max()
    print(f"  max peak-normalised |f|^2 err {e:.2e}", flush=True)
    assert e <= TOL_F2[precision]
