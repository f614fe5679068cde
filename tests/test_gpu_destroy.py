"""A context destroyed while its read-out waits on a busy stream: the workspace
is the caller's to overwrite when the call returns."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import DeviceRun  # noqa: E402


@pytest.mark.parametrize("precision", [0, 1])
def test_workspace_is_free_after_destroy(precision):
    busy = DeviceRun(W.bell3d(n=(48, 48, 48), ppc=16, seed=433))
    busy.step(1)
    g = DeviceRun(W.gyro2d(nx=128, ny=128, ppc=32, seed=434), precision=precision)
    g.step(3)
    before = [t.cpu().numpy() for t in g.ctx.particles_read()]
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    busy.ctx.step(busy.B, busy.vg, busy.rho, [busy.wls[0].dt], 60, stream=s1)
    read = g.ctx.particles_read(stream=s1)
    g.ctx.destroy()
    with torch.cuda.stream(s2):
        g.ctx.workspace.zero_()
    s2.synchronize()
    torch.cuda.synchronize()
    assert not bool(g.ctx.workspace.any())
    for a, b in zip(read, before):
        assert np.array_equal(a.cpu().numpy(), b)
