"""The default tiles of small contexts, below, at and above the tile counts at
which the shape changes, and the large contexts' shapes that a smaller
workspace gets: against the oracle, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import assert_states_exact, gpu_box, oracle_run, to_dev  # noqa: E402


@pytest.mark.parametrize("n", [
    (2, 2, 1), (9, 17, 1),                    # one and a few 8x8
    (128, 128, 1), (129, 128, 1),             # 256 tiles of 8x8; more: 16x16
    (256, 256, 1), (257, 256, 1),             # 256 tiles of 16x16; more: 32x16
    (32, 16, 16), (33, 16, 16),               # 128 tiles of 4x4x4; more: 8x4x4
    (3, 2, 5),
])
def test_default_tiles_match_oracle(n):
    from paper_1412_1087_amd import mhdpic as M
    ppc = 1 if n[0] * n[1] > 1000 else 6
    wl = W.gyro2d(nx=n[0], ny=n[1], ppc=ppc, seed=451) if n[2] == 1 else W.bell3d(n=n, ppc=ppc, seed=452)
    box = gpu_box(wl.box)
    d = [to_dev(a) for a in (wl.x, wl.v, wl.m, wl.qm, wl.B, wl.vg, wl.rho)]
    o = oracle_run(wl)
    o.step(wl.B, wl.vg, wl.rho, wl.dt, 2)
    size = M.workspace_size([box], [wl.N])
    for less in (0, 256):
        ws = torch.zeros(size - less, dtype=torch.uint8, device="cuda")
        try:
            x, v, D = (t.cpu().numpy() for t in M.advance([box], [wl.N], *d, wl.dt, 2, workspace=ws))
        except M.MhdpicError as e:  # (already the largest layout)
            assert less and e.code == M.ENOMEM
            continue
        assert np.array_equal(D, o.D)
        assert_states_exact(x, v, o.positions(), o.v, "default tiles")
