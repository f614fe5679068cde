"""Work items of less than 4096 particles (small contexts): tiles split into
several items, one-pass items and a workspace that only holds the layout with
the largest items, against the oracle, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import DeviceRun, assert_states_exact, gpu_box, oracle_run, to_dev  # noqa: E402


@pytest.mark.parametrize("make,n_steps", [
    (lambda: W.gyro2d(nx=8, ny=8, ppc=8, seed=301), 3),        # one item of 512
    (lambda: W.gyro2d(nx=9, ny=9, ppc=19, seed=302), 3),       # a tile in four items
    (lambda: W.gyro2d(nx=33, ny=40, ppc=30, seed=303), 2),     # ragged tiles of many items
    (lambda: W.bell3d(n=(9, 5, 4), ppc=23, seed=304), 3),      # 3D, 513 and more per tile
    (lambda: W.bell3d(n=(16, 8, 8), ppc=9, seed=305), 2),
])
def test_small_items_match_oracle(make, n_steps):
    wl = make()
    g = DeviceRun(wl)
    g.step(n_steps)
    o = oracle_run(wl)
    o.step(wl.B, wl.vg, wl.rho, wl.dt, n_steps)
    assert (g.deposits()[0] == o.D).all()
    x, v = g.particles()[0]
    assert_states_exact(x, v, o.positions(), o.v, "small items")


def test_workspace_of_the_largest_items_still_serves():
    from paper_1412_1087_amd import mhdpic as M
    wl = W.gyro2d(nx=32, ny=32, ppc=16, seed=306)
    box, args = gpu_box(wl.box), [to_dev(a) for a in (wl.x, wl.v, wl.m, wl.qm, wl.B, wl.vg, wl.rho)]
    size = M.workspace_size([box], [wl.N])
    out = []
    for less in (0, 256):  # 256 bytes less no longer hold the 32 items of 512
        ws = torch.zeros(size - less, dtype=torch.uint8, device="cuda")
        out.append([t.cpu().numpy() for t in M.advance([box], [wl.N], *args, wl.dt, 2, workspace=ws)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    with pytest.raises(M.MhdpicError) as e:
        M.advance([box], [wl.N], *args, wl.dt, 2,
                  workspace=torch.zeros(size // 2, dtype=torch.uint8, device="cuda"))
    assert e.value.code == M.ENOMEM
