"""The deposits' read-out, with and without clearing, into an output aligned to
16 bytes and one aligned to 8 only, for cell counts with and without a
remainder against the kernel's blocks: exact."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import DeviceRun, oracle_run  # noqa: E402


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n", [(2, 2), (16, 16), (33, 31)])
def test_deposit_read_alignment_and_clear(n, shift):
    wl = W.gyro2d(nx=n[0], ny=n[1], ppc=5, seed=411)
    g = DeviceRun(wl)
    g.step(1)
    o = oracle_run(wl)
    o.step(wl.B, wl.vg, wl.rho, wl.dt, 1)
    nc = n[0] * n[1]
    buf = torch.full((8 * nc + 2,), -7, dtype=torch.int64, device="cuda")
    out = buf[shift:shift + 8 * nc].view(8, nc)
    for reset in (False, True):
        g.ctx.deposit_read(reset, out=out)
        assert (out.cpu().numpy() == o.D).all()
    rest = torch.cat((buf[:shift], buf[shift + 8 * nc:]))
    assert (rest == -7).all()
    D = g.ctx.deposit_read(False, out=out).cpu().numpy()
    assert (D[:4] == o.D[:4]).all() and (D[4:] == 0).all()
