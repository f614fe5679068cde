"""Errors of a one-call advance by where they arise: what set-up refuses leaves
the outputs as they were (binary32 form), what only a step finds is returned
with the outputs of a context's same calls written."""
import ctypes as ct

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import gpu_box, to_dev  # noqa: E402


def _workload(ndim):
    return W.gyro2d(nx=16, ny=12, ppc=3, seed=443) if ndim == 2 else W.bell3d(n=(8, 6, 5), ppc=3, seed=444)


def _advance(wl, arrays, precision, n_steps, n_sub=1):
    from paper_1412_1087_amd import mhdpic as M
    boxes = [gpu_box(wl.box)]
    outs = [torch.full((3, wl.N), 7.0, dtype=torch.float64, device="cuda") for _ in range(2)]
    outs.append(torch.full((8, wl.box.n_cells), 7, dtype=torch.int64, device="cuda"))
    ws = torch.zeros(M.workspace_size(boxes, [wl.N], precision), dtype=torch.uint8, device="cuda")
    rc = M.lib().mhdpic_advance(M._boxes_array(boxes), 1, (ct.c_int64 * 1)(wl.N), precision,
                                *[M._ptr(t) for t in arrays], (ct.c_double * 1)(wl.dt), n_steps, n_sub,
                                *[M._ptr(t) for t in outs], M._ptr(ws), ws.numel(), M._stream(None))
    return rc, outs


@pytest.mark.parametrize("ndim", [2, 3])
@pytest.mark.parametrize("what,code", [("x_nan", "ENONFINITE"), ("x_far", "ERANGE"), ("v_inf", "ENONFINITE"),
                                       ("m_large", "ERANGE")])
def test_refused_input_in_binary32_leaves_outputs(what, code, ndim):
    from paper_1412_1087_amd import mhdpic as M
    wl = _workload(ndim)
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
    for n_steps in (0, 2):
        rc, outs = _advance(wl, d, M.FP32_MIXED, n_steps)
        assert rc == getattr(M, code)
        assert all(bool((t == 7).all()) for t in outs)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ndim", [2, 3])
def test_error_of_a_step_writes_outputs(ndim, precision):
    from paper_1412_1087_amd import mhdpic as M
    wl = _workload(ndim)
    # a gas velocity of 10^9: the momentum of the first kick passes 2^51 quanta
    d = [to_dev(a) for a in (wl.x, wl.v, wl.m, wl.qm, wl.B, wl.vg + 1e9, wl.rho)]
    for n_steps, n_sub in ((1, 1), (2, 3)):
        rc, (x, v, D) = _advance(wl, d, precision, n_steps, n_sub)
        assert rc == M.ERANGE
        ctx = M.Context([gpu_box(wl.box)], [wl.N], *d[:4], precision=precision)
        ctx.step(*d[4:], [wl.dt], n_steps, n_sub=n_sub)
        xc, vc = ctx.particles_read()
        assert torch.equal(x, xc) and torch.equal(v, vc) and torch.equal(D, ctx.deposit_read())
        with pytest.raises(M.MhdpicError) as e:
            ctx.check()
        assert e.value.code == M.ERANGE
