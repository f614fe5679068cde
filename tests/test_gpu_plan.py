"""The binning's plan over one, few and many blocks (16 tiles each; more than
64 blocks read their predecessors in several windows) and the field
preparation beside the scatter, against the oracle, bit for bit."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import DeviceRun, assert_states_exact, oracle_run  # noqa: E402


@pytest.mark.parametrize("timed", [False, True])  # timed: the fields in their own launch
@pytest.mark.parametrize("n,tile,ppc", [
    ((8, 8, 1), (8, 8, 1), 4),        # one tile
    ((128, 8, 1), (8, 8, 1), 3),      # 16 tiles: one block
    ((136, 8, 1), (8, 8, 1), 3),      # 17
    ((256, 257, 1), (8, 8, 1), 1),    # 1056 tiles: 66 blocks
    ((64, 68, 16), (4, 4, 4), 1),     # 1088 tiles in 3D, two rows of groups
])
def test_plan_matches_oracle(n, tile, ppc, timed):
    if n[2] == 1:
        wl = W.gyro2d(nx=n[0], ny=n[1], ppc=ppc, seed=401)
    else:
        wl = W.bell3d(n=n, ppc=ppc, seed=402)
    g = DeviceRun(wl, tile=tile)
    o = oracle_run(wl)
    if timed:
        g.ctx.timing(True)
    for k in (1, 2):
        g.step(k)
        o.step(wl.B, wl.vg, wl.rho, wl.dt, k)
        assert (g.deposits()[0] == o.D).all()
    x, v = g.particles()[0]
    assert_states_exact(x, v, o.positions(), o.v, "plan")
