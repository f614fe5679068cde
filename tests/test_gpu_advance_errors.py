"""A one-call advance whose input set-up refuses returns that error (not one
the steps would add) and leaves its outputs as they were."""
import ctypes as ct

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import gpu_box, to_dev  # noqa: E402


@pytest.mark.parametrize("ndim", [2, 3])
@pytest.mark.parametrize("what,code", [("x_nan", "ENONFINITE"), ("x_far", "ERANGE"), ("v_inf", "ENONFINITE"),
                                       ("m_large", "ERANGE")])
def test_refused_input_leaves_outputs(what, code, ndim):
    from paper_1412_1087_amd import mhdpic as M
    wl = W.gyro2d(nx=16, ny=12, ppc=3, seed=441) if ndim == 2 else W.bell3d(n=(8, 6, 5), ppc=3, seed=442)
    x, v, m = wl.x.copy(), wl.v.copy(), wl.m.copy()
    if what == "x_nan":
        x[0, 5] = np.nan
    elif what == "x_far":
        x[1, 5] = 1e12
    elif what == "v_inf":
        v[2, 5] = np.inf
    else:
        m[5] = 1e5
    d = [to_dev(a) for a in (x, v, m, wl.qm, wl.B, wl.vg, wl.rho)]
    boxes = [gpu_box(wl.box)]
    arr, npart, dts = M._boxes_array(boxes), (ct.c_int64 * 1)(wl.N), (ct.c_double * 1)(wl.dt)
    outs = [torch.full((3, wl.N), 7.0, dtype=torch.float64, device="cuda") for _ in range(2)]
    D = torch.full((8, wl.box.n_cells), 7, dtype=torch.int64, device="cuda")
    ws = torch.zeros(M.workspace_size(boxes, [wl.N]), dtype=torch.uint8, device="cuda")
    for n_steps in (0, 2):
        rc = M.lib().mhdpic_advance(arr, 1, npart, 0, *[M._ptr(t) for t in d], dts, n_steps, 1,
                                    M._ptr(outs[0]), M._ptr(outs[1]), M._ptr(D), M._ptr(ws), ws.numel(),
                                    M._stream(None))
        assert rc == getattr(M, code)
        assert all(bool((t == 7.0).all()) for t in outs) and bool((D == 7).all())
