"""A one-call advance whose input set-up refuses does not run its steps."""
import ctypes as ct
import time

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import gpu_box, to_dev  # noqa: E402


def test_refused_run_ends_at_its_first_binning():
    from paper_1412_1087_amd import mhdpic as M
    wl = W.bell3d(n=(48, 48, 48), ppc=16, seed=445)
    boxes = [gpu_box(wl.box)]
    d = [to_dev(a) for a in (wl.x, wl.v, wl.m, wl.qm, wl.B, wl.vg, wl.rho)]
    outs = [torch.empty((3, wl.N), dtype=torch.float64, device="cuda") for _ in range(2)]
    outs.append(torch.empty((8, wl.box.n_cells), dtype=torch.int64, device="cuda"))
    ws = torch.zeros(M.workspace_size(boxes, [wl.N]), dtype=torch.uint8, device="cuda")

    def advance():
        torch.cuda.synchronize()
        t = time.perf_counter()
        rc = M.lib().mhdpic_advance(M._boxes_array(boxes), 1, (ct.c_int64 * 1)(wl.N), 0,
                                    *[M._ptr(a) for a in d], (ct.c_double * 1)(wl.dt), 60, 1,
                                    *[M._ptr(a) for a in outs], M._ptr(ws), ws.numel(), M._stream(None))
        return rc, time.perf_counter() - t

    runs = [advance() for _ in range(3)]
    assert all(rc == M.OK for rc, _ in runs)
    accepted = min(t for _, t in runs)
    d[2][5] = 1e5  # a mass whose n_CR passes 2^51 quanta
    runs = [advance() for _ in range(3)]
    assert all(rc == M.ERANGE for rc, _ in runs)
    refused = min(t for _, t in runs)
    # 60 steps of 1.8 million particles against 60 times three launches of empty lists
    assert refused < accepted / 2, (refused, accepted)
    d[2][5] = float(wl.m[5])
    assert advance()[0] == M.OK
