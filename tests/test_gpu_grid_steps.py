"""Grid kernel: column tiles of a grid off centre on every axis, and the k-steps
(32 z rows each) of a tile, whole and split over workgroups.

Off centre no mirror values are computed and a tile takes up to six column
groups; from four on it keeps one V block, awaited inside a k-step of one or two
terms and between the steps of a longer one.
"""
import os

import numpy as np
import pytest

import workload as wl
from tests.metrics import TOL_F2, errors

pytestmark = pytest.mark.gpu

NTH = min(16, os.cpu_count() or 1)


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
# (states, nz): 1 to 6 groups a tile, whole and with a remainder, and two tiles
@pytest.mark.parametrize("case", [(3, 16), (24, 31), (5, 48), (12, 49), (24, 64), (1, 64), (7, 80), (32, 96), (2, 81), (24, 112)],
                         ids=lambda c: f"s{c[0]}_{c[1]}")
def test_off_centre_widths(oracle_mod, case, precision):
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    ns, nz = case
    rng = np.random.Generator(np.random.PCG64(100 * ns + nz))
    mol = wl.make_molecule(rng, 3, 3, layout="box", box_A=3.0)
    T = wl.make_transitions(rng, mol.nbf, wl.n_occupied(mol.Z), ns)
    grid = wl.Grid(n=(2, 3, nz), qmin=(-3.0, -4.0, -5.0), qmax=(4.0, 3.5, 4.25))
    print("case off_centre_widths", case, precision, flush=True)
    with binding.Context(0) as ctx:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        f, f2 = ctx.eval_grid_host(grid, precision)
    ref = oracle_mod.eval_grid(mol, T, grid, n_threads=NTH)
    np.testing.assert_allclose(f2, np.abs(f) ** 2, rtol=2e-6, atol=1e-12 * np.abs(f).max() ** 2)
    e = errors(f, ref)["f2_peak_norm"].max()
    print(f"  max peak-normalised |f|^2 err {e:.2e}", flush=True)
    assert e <= TOL_F2[precision]


def s_shells(n):
    """n s shells of one primitive: n (n + 1) / 2 z rows of one term each."""
    rng = np.random.Generator(np.random.PCG64(n))
    mol = wl.Molecule(Z=np.full(n, 6), xyz=rng.uniform(-2.0, 2.0, size=(n, 3)), shell_atom=np.arange(n, dtype=np.int32),
                      shell_l=np.zeros(n, np.int32), shell_nprim=np.ones(n, np.int32),
                      exps=np.exp(rng.uniform(np.log(0.3), np.log(5.0), size=n)), coefs=np.ones(n))
    return mol, rng.normal(size=(4, n, n))


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("sym", [True, False])
@pytest.mark.parametrize("n,ksteps", [(7, 1), (8, 2), (11, 3), (14, 4), (18, 6), (20, 7)])
def test_ksteps_whole_and_split(oracle_mod, n, ksteps, sym, precision):
    """Odd and even numbers of k-steps, whole and one or a few per workgroup: the
    split must have taken place (its partial sums are in the context's memory), and
    a budget that has no room for them gives the whole sum."""
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    mol, T = s_shells(n)
    assert (n * (n + 1) // 2 + 31) // 32 == ksteps
    grid = wl.Grid(n=(3, 4, 70), qmin=(-3.0, -4.0, -5.0 if sym else -4.0), qmax=(4.0, 3.5, 5.0))
    print("case ksteps", n, sym, precision, flush=True)
    held, out = [], []
    for budget in (0, None):
        with binding.Context(0, held[0] - (ksteps > 1) if budget is None else 0) as ctx:
            ctx.load_molecule(mol)
            ctx.load_transitions(T)
            ctx.set_options(0.0, 1.0)
            f, _ = ctx.eval_grid_host(grid, precision)
            held.append(ctx.query()["device_bytes"])
            out.append(f)
    splits = (held[0] - held[1]) // (16 * out[0].size)
    print(f"  {splits} ranges of {ksteps} k-steps", flush=True)
    assert splits == 0 if ksteps == 1 else 2 <= splits <= ksteps
    ref = oracle_mod.eval_grid(mol, T, grid, n_threads=NTH)
    for f in out:
        assert errors(f, ref)["f2_peak_norm"].max() <= TOL_F2[precision]
    # the same products; only the order of the sums over k-steps differs
    assert np.abs(out[0] - out[1]).max() <= {"fp32": 1e-6, "bf16x3": 2e-6}[precision] * np.abs(ref).max()
