"""Point evaluation: point blocks of 64, state blocks of 8, 4 and 1, shares of
the shell pairs, screened terms, against the FP64 oracle.

Everything is summed in FP64 and rounded once to FP32, so |f|^2 is within 2
FP32 roundings of f (2 x 2^-24 relative) and one of its own: 2e-7 of the peak.
Screening at eps moves f by at most eps of the sum of the term bounds, which
is some hundred times the peak here: 1e-6 at eps = 1e-9.
"""
import os

import numpy as np
import pytest

import workload as wl
from tests.metrics import errors

pytestmark = pytest.mark.gpu

NTH = min(16, os.cpu_count() or 1)


@pytest.mark.parametrize("ns,nq,eps", [(1, 1, 0.0), (3, 63, 0.0), (4, 64, 1e-9), (8, 65, 0.0), (12, 130, 1e-9),
                                       (13, 7, 0.0), (15, 200, 0.0), (32, 129, 1e-9)])
def test_points_blocks(oracle_mod, ns, nq, eps):
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    rng = np.random.Generator(np.random.PCG64(70 + ns))
    mol = wl.make_molecule(rng, 3, 2, layout="box", box_A=4.0)
    T = wl.make_transitions(rng, mol.nbf, wl.n_occupied(mol.Z), ns)
    q = rng.uniform(-4.0, 4.0, (nq, 3))
    q[0] = 0.3   # near the peak, so that few points still carry a scale
    print("case points_blocks", ns, nq, eps, flush=True)
    ctx = binding.Context(0)
    try:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(eps, 1.0)
        f, f2 = ctx.eval_points(q)
    finally:
        ctx.close()
    ref = oracle_mod.eval_points(mol, T, q, n_threads=NTH)
    np.testing.assert_allclose(f2, np.abs(f) ** 2, rtol=2e-6, atol=1e-12 * np.abs(f).max() ** 2)
    e = errors(f, ref)["f2_peak_norm"].max()
    print(f"  max peak-normalised |f|^2 err {e:.2e}", flush=True)
    assert e <= (1e-6 if eps else 2e-7)


def test_points_shares_under_budget():
    """Where the memory budget does not hold the shares' partial sums there are
    fewer of them: the same values up to the order of the FP64 sums."""
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    W = wl.make_config(0)
    q = np.random.Generator(np.random.PCG64(5)).uniform(-3.0, 3.0, (700, 3))
    print("case points_shares_under_budget", flush=True)
    out, full = [], 0
    for less in (0, 1, 1 << 16):
        with binding.Context(0, hbm_budget_bytes=full - less if less else 0) as ctx:
            ctx.load_molecule(W.mol)
            ctx.load_transitions(W.T)
            ctx.set_options(0.0, 1.0)
            out.append(ctx.eval_points(q)[0])
            held = ctx.query()["device_bytes"]
            assert not less or held <= full - less
            full = full or held
    scale = np.abs(out[0]).max()
    for o in out[1:]:
        assert np.abs(out[0] - o).max() <= 2.0 ** -23 * scale
