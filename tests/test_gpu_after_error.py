"""A call that fails leaves the context usable as before, under stream capture too.

The next allocation-free evaluation may be captured into a graph: no call that
a capture forbids (a device-wide wait for the failed call's work) is made then.
"""
import ctypes

import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu


def fail_dipole(ctx, W):
    ctx.dipole(np.full(W.T.shape[0], np.nan))


def fail_memory(ctx, W):   # host outputs beyond the context's budget
    ctx.eval_grid_host(wl.Grid(n=(64, 64, 64), qmin=(-5.0,) * 3, qmax=(5.0,) * 3), "fp32")


def fail_radii(ctx, W):   # tables of a spherical evaluation beyond the budget
    ctx.eval_spherical_host(24, np.linspace(0.1, 5.0, 64), 16, 16)


@pytest.mark.parametrize("failing", [fail_dipole, fail_memory, fail_radii])
def test_capture_after_error(failing):
    import torch
    from paper_2512_18010_amd import binding
    W = wl.make_config(0)
    W.grid = wl.Grid(n=(9, 8, 19), qmin=(-5.0,) * 3, qmax=(5.0,) * 3)
    shape = (W.T.shape[0],) + tuple(W.grid.n)
    g = binding.make_grid(W.grid.n, W.grid.qmin, W.grid.qmax)
    f_ref = torch.empty(shape + (2,), dtype=torch.float32, device="cuda")
    with binding.Context(0) as big:
        big.load_molecule(W.mol)
        big.load_transitions(W.T)
        big.eval_grid_device(W.grid, f_ref, None)
        torch.cuda.synchronize()
        held = big.query()["device_bytes"]
    print("case capture_after_error", failing.__name__, flush=True)
    with binding.Context(0, held + (1 << 20)) as ctx:
        ctx.load_molecule(W.mol)
        ctx.load_transitions(W.T)
        ctx.query()
        with pytest.raises(binding.ScffError) as ei:
            failing(ctx, W)
        assert ei.value.code in (binding.SCFF_EINVAL, binding.SCFF_ENOMEM) and str(ei.value)
        f = torch.full(shape + (2,), float("nan"), dtype=torch.float32, device="cuda")
        graph = torch.cuda.CUDAGraph()
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            rc = binding.scff_eval_grid_noalloc(ctx._h, ctypes.byref(g), 0, f.data_ptr(), None,
                                                ctypes.c_void_p(stream.cuda_stream))
        assert rc == binding.SCFF_OK
        for _ in range(3):
            f.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(f, f_ref)
