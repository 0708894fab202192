"""Grid kernel contracted along each axis, against the FP64 oracle.

A grid that is short along z, or symmetric about 0 along another axis only, is
contracted along that one where this saves more than the layout takes: columns then
lie apart in the output, lines run over the other two axes, and the term layout
changes with the axis.
"""
import functools
import os

import numpy as np
import pytest

import workload as wl
from tests.metrics import TOL_F2, errors

pytestmark = pytest.mark.gpu

NTH = min(16, os.cpu_count() or 1)

# (states, n, qmin, qmax, symmetric mode)
S = (-4.0, -4.5, -5.0), (4.0, 4.5, 5.0)
CASES = {
    "x_long": (3, (40, 5, 3), (-4.0, -3.0, 0.5), (4.0, 3.5, 1.0), False),
    "x_off_centre": (24, (37, 3, 2), (-4.0, -3.0, 0.5), (3.0, 3.5, 1.0), False),
    "y_long": (12, (4, 50, 1), (-4.0, -3.0, 0.5), (4.0, 3.0, 1.0), False),
    "y_symmetric": (13, (20, 21, 22), (-4.0, -3.0, -1.0), (3.0, 3.0, 5.0), False),
    "x_line": (1, (129, 1, 1), (-4.0, 1.0, 0.5), (4.0, 1.0, 0.5), False),
    "mode_x": (5, (34, 6, 3), *S, True),
    "mode_y": (24, (6, 47, 4), *S, True),
    "mode_z": (5, (9, 6, 33), *S, True),
    # long enough that another axis than z pays
    "x_contracted": (3, (300, 70, 1), (-4.0, -3.0, 0.5), (4.0, 3.5, 1.0), False),
    "x_contracted_off_centre": (24, (150, 23, 1), (-4.0, -3.0, 0.5), (3.0, 3.5, 1.0), False),
    "y_contracted": (12, (75, 95, 1), (-4.0, -3.0, 0.5), (3.0, 3.0, 1.0), False),
    "y_contracted_off_centre": (13, (39, 70, 3), (-4.0, -3.0, -1.0), (3.0, 3.5, 2.0), False),
    "x_contracted_line": (32, (4000, 1, 1), (-4.0, 1.0, 0.5), (4.0, 1.0, 0.5), False),
    "mode_x_contracted": (12, (600, 21, 1), (-4.0, -4.5, 0.0), (4.0, 4.5, 0.0), True),
    "mode_y_contracted": (24, (61, 95, 2), *S, True),
}


def workload_of(case):
    ns, n, qmin, qmax, _ = CASES[case]
    rng = np.random.Generator(np.random.PCG64(31 * ns + n[0]))
    mol = wl.make_molecule(rng, 3, 3, layout="box", box_A=3.0)
    return mol, wl.make_transitions(rng, mol.nbf, wl.n_occupied(mol.Z), ns), wl.Grid(n=n, qmin=qmin, qmax=qmax)


@functools.lru_cache(maxsize=1)
def reference(case):
    import oracle
    return oracle.eval_grid(*workload_of(case), n_threads=NTH)


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("case", list(CASES))
def test_axes(oracle_mod, case, precision):
    import torch  # noqa: F401
    from paper_2512_18010_amd import binding
    mol, T, grid = workload_of(case)
    print("case grid_axes", case, precision, flush=True)
    with binding.Context(0) as ctx:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        ctx.set_symmetry(CASES[case][4])
        f, f2 = ctx.eval_grid_host(grid, precision)
    ref = reference(case)
    np.testing.assert_allclose(f2, np.abs(f) ** 2, rtol=2e-6, atol=1e-12 * np.abs(f).max() ** 2)
    e = errors(f, ref)["f2_peak_norm"].max()
    print(f"  max peak-normalised |f|^2 err {e:.2e}", flush=True)
    assert e <= TOL_F2[precision]


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("n", [(600, 21, 1), (601, 20, 1), (21, 600, 1), (6, 3, 40)], ids=str)
def test_symmetric_mode_conjugates(n, precision):
    """In the symmetric mode the planes ix >= ceil(nx / 2) are the conjugates of their mirror points bit
    for bit, whichever axis is contracted."""
    from paper_2512_18010_amd import binding
    mol, T, _ = workload_of("mode_x_contracted")
    a = [q if m > 1 else 0.0 for q, m in zip(S[1], n)]
    grid = wl.Grid(n=n, qmin=tuple(-x for x in a), qmax=tuple(a))
    print("case symmetric_mode_conjugates", n, precision, flush=True)
    with binding.Context(0) as ctx:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        ctx.set_symmetry(True)
        f, f2 = ctx.eval_grid_host(grid, precision)
    h = (n[0] + 1) // 2
    np.testing.assert_array_equal(f[:, h:], np.conj(f[:, ::-1, ::-1, ::-1][:, h:]))
    np.testing.assert_array_equal(f2[:, h:], f2[:, ::-1, ::-1, ::-1][:, h:])


def test_axes_in_turn(oracle_mod):
    """One context, grids of different axes in turn, points and the allocation-free call between them."""
    import ctypes

    import torch
    from paper_2512_18010_amd import binding
    mol, T, gx = workload_of("mode_y_contracted")
    ns = T.shape[0]
    grids = [wl.Grid(n=(90, 31, 1), qmin=gx.qmin, qmax=gx.qmax), wl.Grid(n=(5, 3, 40), qmin=gx.qmin, qmax=gx.qmax),
             wl.Grid(n=(31, 90, 1), qmin=gx.qmin, qmax=gx.qmax)]
    refs = [oracle_mod.eval_grid(mol, T, g, n_threads=NTH) for g in grids]
    stream = torch.cuda.current_stream()
    with binding.Context(0) as ctx:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        seen = {}
        for i in (0, 1, 0, 2, 1, 2):
            f, _ = ctx.eval_grid_host(grids[i], "fp32")
            assert errors(f, refs[i])["f2_peak_norm"].max() <= TOL_F2["fp32"]
            np.testing.assert_array_equal(seen.setdefault(i, f), f)
            p, _ = ctx.eval_points(grids[i].points()[::7])
            e = np.abs(p - refs[i].reshape(ns, -1)[:, ::7]).max() / np.abs(refs[i]).max()
            assert e <= 1e-6
            for j in range(3):   # on the layout at hand
                o = torch.empty((ns,) + grids[j].n + (2,), dtype=torch.float32, device="cuda")
                g = binding.make_grid(grids[j].n, grids[j].qmin, grids[j].qmax)
                assert binding.scff_eval_grid_noalloc(ctx._h, ctypes.byref(g), 0, o.data_ptr(), None,
                                                      ctypes.c_void_p(stream.cuda_stream)) == binding.SCFF_OK
                torch.cuda.synchronize()
                a = o.cpu().numpy()
                assert errors(a[..., 0] + 1j * a[..., 1], refs[j])["f2_peak_norm"].max() <= TOL_F2["fp32"]
                if j == i:
                    np.testing.assert_array_equal(a[..., 0] + 1j * a[..., 1], f)


def test_capture_after_other_axes(oracle_mod):
    """Grids evaluated before, of different axes, in one captured graph: the graph takes the layout at
    hand and no memory."""
    import torch
    from paper_2512_18010_amd import binding
    mol, T, gx = workload_of("mode_y_contracted")
    ns = T.shape[0]
    grids = [wl.Grid(n=(90, 31, 1), qmin=gx.qmin, qmax=gx.qmax), wl.Grid(n=(31, 90, 1), qmin=gx.qmin, qmax=gx.qmax),
             wl.Grid(n=(5, 3, 40), qmin=gx.qmin, qmax=gx.qmax)]
    refs = [oracle_mod.eval_grid(mol, T, g, n_threads=NTH) for g in grids]
    outs = [torch.empty((ns,) + g.n + (2,), dtype=torch.float32, device="cuda") for g in grids]
    print("case capture_after_other_axes", flush=True)
    with binding.Context(0) as ctx:
        ctx.load_molecule(mol)
        ctx.load_transitions(T)
        ctx.set_options(0.0, 1.0)
        for g, o in zip(grids, outs):
            ctx.eval_grid_device(g, o, None)
        torch.cuda.synchronize()
        held = ctx.query()["device_bytes"]
        graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            for g, o in zip(grids, outs):
                ctx.eval_grid_device(g, o, None, stream=stream)
        assert ctx.query()["device_bytes"] == held
        for _ in range(3):
            for o in outs:
                o.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            for o, ref in zip(outs, refs):
                a = o.cpu().numpy()
                assert errors(a[..., 0] + 1j * a[..., 1], ref)["f2_peak_norm"].max() <= TOL_F2["fp32"]
