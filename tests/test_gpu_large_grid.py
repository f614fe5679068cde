"""A step of so many tiles and cells that the binning's blocks and the field
preparation's no longer fit one launch (2^32 threads): the fields then have a
launch of their own.  Against a context of the boxes that hold particles."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import DeviceRun, assert_states_exact, oracle_run  # noqa: E402


def test_columns_one_cell_wide_match_oracle():
    wl = W.gyro2d(nx=1, ny=40, ppc=20, seed=460)
    g, o = DeviceRun(wl, tile=(8, 8, 1)), oracle_run(wl)
    g.step(3)
    o.step(wl.B, wl.vg, wl.rho, wl.dt, 3)
    assert (g.deposits()[0] == o.D).all()
    assert_states_exact(*g.particles()[0], o.positions(), o.v, "columns")


def test_step_beyond_one_launch_of_binning_and_fields():
    from paper_1412_1087_amd import mhdpic as M
    nb, ny, N = 1015, 65536, 3000  # columns of 1 x 65536 cells in tiles of 8x8: eight cells a tile
    NT, NC = nb * (ny // 8), nb * ny
    assert NT * 512 + 4096 < 2**32 < NT * 512 + NC
    held = [0, 500, nb - 1]
    g = torch.Generator(device="cuda")
    g.manual_seed(461)

    def rand(*shape):
        return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=g)

    x = rand(3, 3 * N)
    x[1] *= ny
    x[2] = 0.0
    v = 4.0 * rand(3, 3 * N) - 2.0
    m = torch.full((3 * N,), 1e-3, dtype=torch.float64, device="cuda")
    qm = torch.ones_like(m)
    B, vg = rand(3, NC), 0.1 * rand(3, NC)
    rho = torch.ones(NC, dtype=torch.float64, device="cuda")

    def run(boxes, counts, f):
        ctx = M.Context([M.Box(ndim=2, n=(1, ny), hall=1, tile=(8, 8)) for _ in range(boxes)], counts, x, v, m, qm)
        ctx.step(*f, 0.05, 2)
        out = [t.cpu().numpy() for t in ctx.particles_read()], ctx.deposit_read()
        ctx.check()
        return out

    counts = [N if b in held else 0 for b in range(nb)]
    (xl, vl), D = run(nb, counts, (B, vg, rho))
    cells = torch.cat([torch.arange(b * ny, (b + 1) * ny, device="cuda") for b in held])
    (xs, vs), Ds = run(3, [N] * 3, [t.index_select(t.dim() - 1, cells) for t in (B, vg, rho)])
    assert np.array_equal(xl, xs) and np.array_equal(vl, vs)
    assert torch.equal(D[:, cells], Ds)
    D[:, cells] = 0
    assert not bool(D.any())
