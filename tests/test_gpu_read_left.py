"""Read-outs of contexts that particles have left, at the particle numbers where
their route changes: bytes or a fill tell the written records (2^20), straight
to the columns or through records (binary64, 1.5 to 2.8 million in 2D).  Equal,
bit for bit, to the read-out that a captured call takes."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N", [1, 3, 1021, 2**20 - 1, 2**20, 2**20 + 1, 1_500_000, 1_520_000, 2_790_000, 2_800_000])
def test_read_outs_of_left_contexts(N, precision):
    from paper_1412_1087_amd import mhdpic as M
    nx, ny = 300, 40
    g = torch.Generator(device="cuda")
    g.manual_seed(481)

    def rand(*shape):
        return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=g)

    x, v = rand(3, N), 10.0 * rand(3, N) - 5.0
    x[0] *= nx
    x[1] *= ny
    x[2] = 0.0
    m = torch.full((N,), 1e-6, dtype=torch.float64, device="cuda")
    box = M.Box(ndim=2, n=(nx, ny), boundary=((M.ABSORB, M.ABSORB), (0, 0), (0, 0)))
    ctx = M.Context([box], [N], x, v, m, torch.ones_like(m), precision=precision)
    B, vg = 0.1 * rand(3, nx * ny), torch.zeros(3, nx * ny, dtype=torch.float64, device="cuda")
    ctx.step(B, vg, None, 0.09, 8)
    xr, vr = ctx.particles_read()
    live = sum(ctx.counts())
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        xd, vd = ctx.particles_read(stream=s)
    graph.replay()
    torch.cuda.synchronize()
    for a, b in ((xr, xd), (vr, vd)):
        assert torch.equal(a.view(torch.int64), b.view(torch.int64))
    assert int((~torch.isnan(xr[0])).sum()) == live and (N < 1000 or live < N)
    ctx.check()
