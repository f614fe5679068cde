"""Set-up of contexts whose box records fit one launch's arguments (8) and of
larger ones, one-call and kept, over workspaces full of old data: against the
oracle, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import assert_states_exact, gpu_box, oracle_run, to_dev  # noqa: E402


@pytest.mark.parametrize("nb", [1, 8, 9, 17])
def test_setup_over_old_data(nb):
    from paper_1412_1087_amd import mhdpic as M
    wls = [W.gyro2d(nx=6 + 3 * b, ny=5 + 2 * b, ppc=4, seed=431 + b) for b in range(nb)]
    boxes, counts = [gpu_box(w.box) for w in wls], [w.N for w in wls]
    part = [to_dev(np.concatenate([getattr(w, n) for w in wls], axis=-1)) for n in ("x", "v", "m", "qm")]
    f = [to_dev(np.concatenate([getattr(w, n) for w in wls], axis=-1)) for n in ("B", "vg", "rho")]
    dts = [w.dt for w in wls]
    ws = torch.full((M.workspace_size(boxes, counts),), 0xA5, dtype=torch.uint8, device="cuda")
    for _ in range(2):  # fresh garbage, then a used workspace
        x, v, D = (t.cpu().numpy() for t in M.advance(boxes, counts, *part, *f, dts, 2, workspace=ws))
        ctx = M.Context(boxes, counts, *part)
        ctx.step(*f, dts, 2)
        assert np.array_equal(ctx.deposit_read().cpu().numpy(), D)
        p0 = c0 = 0
        for w in wls:
            o = oracle_run(w)
            o.step(w.B, w.vg, w.rho, w.dt, 2)
            c1, p1 = c0 + w.box.n_cells, p0 + w.N
            assert (D[:, c0:c1] == o.D).all()
            assert_states_exact(x[:, p0:p1], v[:, p0:p1], o.positions(), o.v, "setup")
            c0, p0 = c1, p1
