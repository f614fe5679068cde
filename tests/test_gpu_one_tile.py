"""All particles in one tile of many: its work items' bounds at and beside
multiples of their number, at set-up and after steps, against the oracle, bit
for bit."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import DeviceRun, assert_states_exact, oracle_run  # noqa: E402


# one-pass items of 512: one, just two, remainders of 1 and of all but 1, and
# more items than a wave has lanes
@pytest.mark.parametrize("N", [1, 512, 513, 1025, 1535, 1536, 40001])
def test_particles_of_one_tile_match_oracle(N):
    nx = 24
    wl = W.gyro2d(nx=nx, ny=nx, ppc=-(-N // (nx * nx)), seed=471)
    wl.x, wl.v, wl.m, wl.qm = (a[..., :N].copy() for a in (wl.x, wl.v, wl.m, wl.qm))
    wl.x[:2] = 9.0 + wl.x[:2] * (6.0 / nx)  # inside the middle tile of 8x8
    g, o = DeviceRun(wl, tile=(8, 8, 1)), oracle_run(wl)
    assert (g.deposits()[0] == o.D).all()
    for _ in range(2):
        g.step(1)
        o.step(wl.B, wl.vg, wl.rho, wl.dt, 1)
        assert (g.deposits()[0] == o.D).all()
    assert_states_exact(*g.particles()[0], o.positions(), o.v, f"{N} in one tile")
