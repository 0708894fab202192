"""Partial sums that one call keeps do not take the budget from another.

Point evaluations, the spherical method and split grids keep buffers of partial
sums with the context; they can do with less, so a later call that needs the
memory gets it: a grid that fits the budget on a fresh context fits after any
other call, and the other way round.
"""
import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu


def test_grid_fits_after_points():
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    W = wl.make_config(0)
    rng = np.random.Generator(np.random.PCG64(3))
    T = wl.make_transitions(rng, W.mol.nbf, wl.n_occupied(W.mol.Z), 12)
    grid = wl.Grid(n=(40, 40, 40), qmin=(-5.0,) * 3, qmax=(5.0,) * 3)
    q = rng.uniform(-4.0, 4.0, size=(6000, 3))
    print("case budget_partials", flush=True)

    def context(budget):
        ctx = binding.Context(0, budget)
        ctx.load_molecule(W.mol)
        ctx.load_transitions(T)
        return ctx

    with context(0) as ctx:
        p_ref, _ = ctx.eval_points(q)
        points = ctx.query()["device_bytes"]
    with context(0) as ctx:
        f_ref, _ = ctx.eval_grid_host(grid, "fp32")
        held = ctx.query()["device_bytes"]
    print(f"  grid {held} bytes, points {points}", flush=True)
    assert points > 30e6   # the partial sums are in it
    # room for the grid and a little: the points take what is free, then the grid what it needs
    with context(held + q.size * 8 + 6000 * 12 * 12 + (1 << 20)) as ctx:
        for _ in range(2):
            p, _ = ctx.eval_points(q)
            assert np.abs(p - p_ref).max() <= 1e-6 * np.abs(p_ref).max()
            f, _ = ctx.eval_grid_host(grid, "fp32")
            assert np.abs(f - f_ref).max() <= 1e-6 * np.abs(f_ref).max()
