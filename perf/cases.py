"""Timing cases of the cosmic-ray particle step, through its public entry points.

A case is one pass of a program that uses the library: the coupled loop of an
MHD code (feedback of the predictor, one particle step, deposits read and
reset), several steps through fixed fields, sub-cycled steps, a batch of
independent boxes as one graph launch, the shock set-up with injection and
removal, and the one-call form without a context.  The sizes are those of the
repository's workloads and benchmark legs, or generic odd ones between them.

Inputs are drawn on the GPU from the seed alone, with the distributions of
``paper_1412_1087_amd.workloads``: a drifting beam (Bell-instability box), an
isotropic population in a weakly perturbed field (gyration test), the power-law
band of the shock strip, and the shock wall's precursor.
"""
import math
import random

import torch

from paper_1412_1087_amd import mhdpic as M

DEV = "cuda:0"
C_LIGHT = 20.0
FRAC_BITS = 40


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------

def _case(name, call, pop, n, ppc, precision="fp64", hall=0, steps=1, sub=1, **more):
    n = tuple(n) + (1,) * (3 - len(n))
    c = dict(call=call, pop=pop, ndim=3 if pop in ("beam", "iso3d") else 2, nx=n[0], ny=n[1],
             nz=n[2], ppc=float(ppc), precision=precision, hall=int(hall), steps=int(steps),
             sub=int(sub))
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the gyration test's box, one coupled step: a small 2D run, bound by launches
        _case("gyro32_step", "step", "gyro", (32, 32), 16),
        # a serving-style call on a small odd 2D box: no context, no allocation, particles back
        _case("advance_2d_small", "advance_noalloc", "gyro", (37, 29), 11, steps=2),
        # the same without a context in 3D: ragged tiles, Hall term, two sub-steps per step
        _case("advance_3d_hall", "advance", "beam", (40, 33, 27), 9, hall=1, steps=4, sub=2),
        # the headline box in the loop of an MHD code: feedback, one step, deposits read and reset
        _case("beam64_coupled", "coupled", "beam", (64, 64, 64), 16, hall=1),
        # the headline box as the benchmark runs it: many steps through fixed fields
        _case("beam64_run", "step", "beam", (64, 64, 64), 16, hall=1, steps=20),
        # sub-cycling in a ragged box (five particle steps per field update)
        _case("beam_subcycled", "step", "beam", (61, 50, 47), 13, hall=1, sub=5),
        # isotropic CRs in 3D: particles change cells in every direction
        _case("iso3d", "step", "iso3d", (80, 72, 66), 10),
        # the precision form on the large beam box
        _case("beam128_fp32", "step", "beam", (128, 128, 128), 32, precision="fp32", hall=1),
        # the shock strip: a dense band and a thin rest
        _case("strip", "step", "strip", (8192, 32), 64),
        # a smaller strip in the precision form, particles read out for a spectrum after the step
        _case("strip_fp32_read", "read", "strip", (4099, 30), 25, precision="fp32"),
        # the batch of independent boxes, ten steps per graph launch
        _case("batch_graph", "graph", "batch", (16, 128), 16, steps=10, boxes=256),
        # the shock set-up: wall, inflow, injection at the front every step, removal by tag
        _case("shock_wall", "shock", "wall", (8192, 256), 1),
    ]


MOST_UPDATES = 60e6  # particle updates of a drawn pass, below the largest listed one's


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["step3d", "step3d", "coupled", "iso3d", "step2d", "strip", "read", "advance",
                       "advance_small", "graph", "shock"])
    prec = rng.choice(["fp64", "fp64", "fp32"])
    if kind == "advance_small":
        # at most what the library's static scratch holds
        n = (round(_log(rng, 8, 90)), round(_log(rng, 8, 90)))
        return _case(None, "advance_noalloc", "gyro", n, round(_log(rng, 2, 40), 2), prec,
                     steps=rng.randint(1, 3), sub=rng.choice([1, 1, 2]))
    if kind == "graph":
        return _case(None, "graph", "batch", (16, rng.randint(24, 128)), round(_log(rng, 4, 32), 2),
                     prec, steps=2 * rng.randint(1, 5), boxes=round(_log(rng, 8, 256)))
    if kind == "shock":
        return _case(None, "shock", "wall", (round(_log(rng, 512, 8192)), round(_log(rng, 16, 256))),
                     round(_log(rng, 0.5, 8), 2), prec)
    steps = rng.choice([1, 1, 1, 2, 5])
    sub = rng.choice([1, 1, 1, 2, 5])
    if kind in ("strip", "read"):
        nx, ny = round(_log(rng, 512, 8192)), round(_log(rng, 17, 64))
        ppc = min(_log(rng, 6, 100), 2 ** 24 / (nx * ny))
        return _case(None, "read" if kind == "read" else "step", "strip", (nx, ny), round(ppc, 2), prec,
                     steps=steps if kind == "strip" else 1, sub=1)
    if kind == "step2d":
        n = (round(_log(rng, 16, 1500)), round(_log(rng, 16, 1500)))
        ppc = min(_log(rng, 2, 60), MOST_UPDATES / (n[0] * n[1] * steps * sub))
        return _case(None, "step", "gyro", n, round(ppc, 2), prec, steps=steps, sub=sub)
    n = tuple(round(_log(rng, 12, 120)) for _ in range(3))
    most = MOST_UPDATES / (n[0] * n[1] * n[2] * steps * sub)
    ppc = round(max(0.5, min(_log(rng, 2, 40), most)), 2)
    if kind == "iso3d":
        return _case(None, "step", "iso3d", n, ppc, prec, hall=rng.randint(0, 1), steps=steps, sub=sub)
    call = {"coupled": "coupled", "advance": "advance"}.get(kind, "step")
    if call == "advance":
        n = tuple(min(k, 64) for k in n)
        ppc = min(ppc, 16.0)
    return _case(None, call, "beam", n, ppc, prec, hall=rng.choice([1, 1, 0]), steps=steps, sub=sub)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(g, *shape):
    return torch.rand(*shape, dtype=torch.float64, device=DEV, generator=g)


def _normal(g, *shape):
    return torch.randn(*shape, dtype=torch.float64, device=DEV, generator=g)


def _centres(n):
    """Cell-centre coordinates [3][cells] of a box of unit cells, x fastest."""
    ax = [torch.arange(k, dtype=torch.float64, device=DEV) + 0.5 for k in n]
    z, y, x = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    return torch.stack([x.reshape(-1), y.reshape(-1), z.reshape(-1)])


def _perturbation(g, xc, length, ndim, m_max, rms, n_modes=12):
    """A divergence-free field: the curl of a few modes of a random potential.
    length [3] or [3][cells]: the box a cell belongs to."""
    f = torch.zeros_like(xc)
    for _ in range(n_modes):
        m = torch.zeros(3, dtype=torch.float64, device=DEV)
        m[:ndim] = torch.randint(-m_max, m_max + 1, (ndim,), device=DEV, generator=g).to(torch.float64)
        m[0] += (m.abs().sum() == 0).to(torch.float64)
        k = 2.0 * math.pi * m.reshape(3, *([1] * (length.dim() - 1))) / length
        if length.dim() == 1:
            k = k[:, None]
        a, phi = _normal(g, 3, 1), 2.0 * math.pi * _uniform(g, 1)
        amp = torch.stack([k[1] * a[2] - k[2] * a[1], k[2] * a[0] - k[0] * a[2],
                           k[0] * a[1] - k[1] * a[0]])
        f += amp * torch.cos((k * xc).sum(0) + phi)
    return f * (rms / f.square().sum(0).mean().sqrt().clamp_min(1e-300))


def _isotropic(g, mag):
    mu = 2.0 * _uniform(g, mag.numel()) - 1.0
    ph = 2.0 * math.pi * _uniform(g, mag.numel())
    s = (1.0 - mu * mu).sqrt()
    return torch.stack([mag * s * ph.cos(), mag * s * ph.sin(), mag * mu])


def _dt(v, B, C, dx=1.0, phase=0.05):
    """The Larmor-time rule, capped by the move limit of two cells per step."""
    gam = (1.0 + v.square().sum(0) / (C * C)).sqrt().min()
    return min(phase * float(gam) / float(B.square().sum(0).max().sqrt()), 0.98 * 2.0 * dx / C)


def _box(case, n, dx=(1.0, 1.0, 1.0), C=C_LIGHT, **more):
    return M.Box(ndim=case["ndim"], n=n, dx=dx, C=C, qomc_gas=1.0, hall=case["hall"],
                 frac_bits=FRAC_BITS, max_move_cells=2, **more)


def _single(case, g):
    """One box: beam, iso3d, gyro or strip."""
    n, nd, pop = (case["nx"], case["ny"], case["nz"]), case["ndim"], case["pop"]
    nc = n[0] * n[1] * n[2]
    N = max(1, round(nc * case["ppc"]))
    length = torch.tensor([float(k) for k in n], dtype=torch.float64, device=DEV)
    x = _uniform(g, 3, N) * length[:, None]
    if nd == 2:
        x[2] = 0.0
    rho = torch.ones(nc, dtype=torch.float64, device=DEV)
    vg = torch.zeros(3, nc, dtype=torch.float64, device=DEV)
    if pop == "strip":
        # 80 % in a band about the front at 0.3 L; dN/dp ~ p^-2 on [1, 1000]
        L = float(n[0])
        nb = round(0.8 * N)
        r = _uniform(g, N)
        x[0, :nb] = (0.25 + 0.1 * r[:nb]) * L
        t = 0.9 * L * r[nb:]
        x[0, nb:] = torch.where(t < 0.25 * L, t, t + 0.1 * L)
        x = x[:, torch.randperm(N, device=DEV, generator=g)].contiguous()
        p = 1.0 / (1.0 - _uniform(g, N) * 0.999)
        v = _isotropic(g, p * C_LIGHT)
        up = (torch.arange(n[0], device=DEV) + 0.5 < 0.3 * L).repeat(n[1])
        rho = torch.where(up, 1.0, 4.0).to(torch.float64)
        vg[0] = torch.where(up, 4.0, 1.0)
        B = torch.zeros(3, nc, dtype=torch.float64, device=DEV)
        B[:2] = math.sqrt(0.5)
        B = B + _perturbation(g, _centres(n), length, nd, 8, 0.01)
        m = 2e-3 * nc / N
    else:
        beam = pop == "beam"
        B0 = (1.0, 0.0, 0.0) if beam else (1.0, 0.5, 0.0)
        B = torch.tensor(B0, dtype=torch.float64, device=DEV)[:, None]
        B = B + _perturbation(g, _centres(n), length, nd, 8 if beam else 4, 0.01 if beam else 0.11)
        if beam:
            v = 0.1 * C_LIGHT * _normal(g, 3, N)
            v[0] += 0.8 * C_LIGHT / math.sqrt(1.0 - 0.64)
            m = 0.05 * nc / N
        else:
            u = 1.0 + 9.0 * _uniform(g, N)
            v = _isotropic(g, u / (1.0 - (u / C_LIGHT).square()).sqrt())
            vg[0] = 0.1
            m = 2e-3 * nc / N
    m = torch.full((N,), m, dtype=torch.float64, device=DEV)
    # the particle step's dt; a sub-cycled step is n_sub of them
    dt = _dt(v, B, C_LIGHT) * case["sub"]
    return dict(boxes=[_box(case, n)], counts=[N], x=x, v=v, m=m, qm=torch.ones_like(m), B=B, vg=vg,
                rho=rho, dt=[dt])


def _batch_shapes(case):
    """(nx, ny, particles per cell) of each box: the case's geometry, sides
    log-uniform in [nx, ny], particles per cell log-uniform in [ppc/4, 4 ppc]."""
    rng = random.Random(1000 * case["boxes"] + case["ny"])
    out = []
    for _ in range(case["boxes"]):
        a, b = (round(_log(rng, case["nx"], case["ny"])) for _ in range(2))
        out.append((a, b, max(1, round(_log(rng, case["ppc"] / 4.0, case["ppc"] * 4.0)))))
    return out


def _batch(case, g):
    """Independent gyration boxes in one context (_batch_shapes)."""
    nb = case["boxes"]
    shapes = torch.tensor(_batch_shapes(case), device=DEV).T
    sides, ppc = shapes[:2], shapes[2]
    cells = sides[0] * sides[1]
    counts = cells * ppc
    sx, sy = (s.tolist() for s in sides)
    cb = torch.repeat_interleave(torch.arange(nb, device=DEV), cells)  # box of each cell
    loc = torch.arange(cb.numel(), device=DEV) - (cells.cumsum(0) - cells)[cb]
    xc = torch.stack([(loc % sides[0][cb]) + 0.5, (loc // sides[0][cb]) + 0.5,
                      torch.full_like(loc, 0) + 0.5]).to(torch.float64)
    length = torch.stack([sides[0][cb], sides[1][cb], torch.ones_like(cb)]).to(torch.float64)
    B = torch.tensor((1.0, 0.5, 0.0), dtype=torch.float64, device=DEV)[:, None]
    B = B + _perturbation(g, xc, length, 2, 4, 0.11)
    vg = torch.zeros_like(B)
    vg[0] = 0.1
    pb = torch.repeat_interleave(torch.arange(nb, device=DEV), counts)
    N = pb.numel()
    x = torch.zeros(3, N, dtype=torch.float64, device=DEV)
    for d in (0, 1):
        x[d] = _uniform(g, N) * sides[d][pb]
    u = 1.0 + 9.0 * _uniform(g, N)
    v = _isotropic(g, u / (1.0 - (u / C_LIGHT).square()).sqrt())
    m = (2e-3 / ppc.to(torch.float64))[pb].contiguous()
    return dict(boxes=[_box(case, (a, b, 1)) for a, b in zip(sx, sy)], counts=counts.tolist(), x=x, v=v,
                m=m, qm=torch.ones_like(m), B=B, vg=vg, rho=torch.ones(B.shape[1], dtype=torch.float64,
                                                                      device=DEV), dt=[_dt(v, B, C_LIGHT)] * nb)


WALL_DX, WALL_V0, WALL_ETA = 12.0, 30.0, 2e-3
WALL_POOL = 64  # injected batches that a pass takes in turn


def _wall_front(case):
    return case["nx"] // 4


def _wall_velocities(g, N, lo, hi):
    C = 10.0 * math.sqrt(2.0) * WALL_V0
    gam = 1.0 + 10.0 * 0.5 * WALL_V0 ** 2 / (C * C)
    vinj = C * math.sqrt(gam * gam - 1.0)
    return _isotropic(g, vinj * (math.log(lo) + (math.log(hi) - math.log(lo)) * _uniform(g, N)).exp())


def _wall(case, g):
    """The shock set-up: a reflecting wall at x = 0, an absorbing inflow face,
    CRs about the front, four injected per cell of swept gas."""
    nx, ny = case["nx"], case["ny"]
    nc = nx * ny
    C = 10.0 * math.sqrt(2.0) * WALL_V0
    N = max(1, round(nc * case["ppc"]))
    fc = _wall_front(case)
    width = min(170.0, 0.2 * nx)
    x = torch.zeros(3, N, dtype=torch.float64, device=DEV)
    x[0] = (fc + width * (2.0 * _uniform(g, N) - 1.0)) * WALL_DX
    x[1] = _uniform(g, N) * (ny * WALL_DX)
    v = _wall_velocities(g, N, 1.0, 20.0)
    up = (torch.arange(nx, device=DEV) >= fc).repeat(ny)
    rho = torch.where(up, 1.0, 4.0).to(torch.float64)
    vg = torch.zeros(3, nc, dtype=torch.float64, device=DEV)
    vg[0] = torch.where(up, -WALL_V0, 0.0)
    B = 0.05 * _normal(g, 3, nc)
    B[0] = 1.0
    mass = WALL_ETA * WALL_DX * WALL_DX / 4.0
    m = torch.full((N,), mass, dtype=torch.float64, device=DEV)
    dt = 0.9 * 2.0 * WALL_DX / C
    per = max(1, round(4 * ny * (WALL_V0 / 3.0) * dt / WALL_DX))
    pool = []
    for _ in range(WALL_POOL):
        px = torch.zeros(3, per, dtype=torch.float64, device=DEV)
        px[0] = (fc - _uniform(g, per)) * WALL_DX
        px[1] = _uniform(g, per) * (ny * WALL_DX)
        pm = torch.full((per,), mass, dtype=torch.float64, device=DEV)
        pool.append((px, _wall_velocities(g, per, 1.0, 1.0001), pm, torch.ones_like(pm),
                     torch.empty_like(pm)))
    box = _box(case, (nx, ny, 1), dx=(WALL_DX, WALL_DX, 1.0), C=C, capacity=N + (1 << 20),
               boundary=((M.REFLECT, M.ABSORB), (0, 0), (0, 0)))
    return dict(boxes=[box], counts=[N], x=x, v=v, m=m, qm=torch.ones_like(m), B=B, vg=vg, rho=rho,
                dt=[dt], pool=pool, per=per, t=0.0, k=0)


def _inputs(case, seed):
    g = _gen(seed)
    if case["pop"] == "batch":
        return _batch(case, g)
    return _wall(case, g) if case["pop"] == "wall" else _single(case, g)


def prepare(case, seed):
    s = _inputs(case, seed)
    prec = M.FP64 if case["precision"] == "fp64" else M.FP32_MIXED
    s.update(call=case["call"], prec=prec, steps=case["steps"], sub=case["sub"])
    if case["call"] == "advance":
        size = M.workspace_size(s["boxes"], s["counts"], prec)
        s["ws"] = torch.empty(size, dtype=torch.uint8, device=DEV)
    elif case["call"] != "advance_noalloc":
        s["ctx"] = M.Context(s["boxes"], s["counts"], s.pop("x"), s.pop("v"), s.pop("m"), s.pop("qm"),
                             precision=prec)
        nc = s["ctx"].n_cells
        s["D"] = torch.empty(8, nc, dtype=torch.int64, device=DEV)
        if case["call"] == "coupled":
            s["fb"] = torch.empty(10, nc, dtype=torch.float64, device=DEV)
        if case["call"] == "graph":
            s["stream"] = torch.cuda.Stream()
            torch.cuda.synchronize()
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def run(s):
    call = s["call"]
    if call.startswith("advance"):
        x, v, D = M.advance(s["boxes"], s["counts"], s["x"], s["v"], s["m"], s["qm"], s["B"], s["vg"],
                            s["rho"], s["dt"], s["steps"], n_sub=s["sub"], precision=s["prec"],
                            workspace=s.get("ws"), noalloc=call == "advance_noalloc")
        return {"x": x, "v": v, "D": D}
    ctx = s["ctx"]
    if call == "graph":
        ctx.step_graph(s["B"], s["vg"], s["rho"], s["dt"], s["steps"], s["stream"], n_sub=s["sub"])
        return {"D": ctx.deposit_read(True, out=s["D"], stream=s["stream"])}
    out = {}
    if call == "coupled":
        out["fb"] = ctx.feedback(s["B"], s["vg"], s["rho"], out=s["fb"])
    if call == "shock":
        x, v, m, qm, tags = s["pool"][s["k"] % WALL_POOL]
        s["k"] += 1
        s["t"] += 1.0
        tags.fill_(s["t"])
        ctx.inject([s["per"]], x, v, m, qm, tags)
        if s["k"] % 8 == 0:
            ctx.remove_tagged(0.5 * s["t"], s["t"])
    ctx.step(s["B"], s["vg"], s["rho"], s["dt"], s["steps"], n_sub=s["sub"])
    out["D"] = ctx.deposit_read(True, out=s["D"])
    if call == "read":
        out["x"], out["v"] = ctx.particles_read()
    return out


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------

def work(case):
    nd, fp64 = case["ndim"], case["precision"] == "fp64"
    if case["pop"] == "batch":
        shapes = _batch_shapes(case)
        nc = sum(a * b for a, b, _ in shapes)
        N = sum(a * b * p for a, b, p in shapes)
    else:
        nc = case["nx"] * case["ny"] * case["nz"]
        N = max(1, round(nc * case["ppc"]))
    w = 8 if fp64 else 4
    updates = N * case["steps"] * case["sub"]
    # per particle update: cell, offsets, four-velocity, m, q/m read; cell,
    # offsets, four-velocity written
    p_bytes = 8 + w * (2 * nd + 6 + 2)
    # per step: B, v_g, rho and the n, J before it read, n, J after it written,
    # -dM, -dE_k read and written
    c_bytes = 56 + 32 + 32 + 64
    byts = updates * p_bytes + nc * case["steps"] * c_bytes
    k = 27 if nd == 3 else 9
    # gather of six components, eight deposit channels (a product, its rounding and a sum each),
    # and the push itself
    flops = updates * (k * (2 * 6 + 3 * 8 + 4) + 200)
    if case["call"] in ("step", "coupled", "graph", "read", "shock"):
        byts += nc * 8 * 8  # deposits handed out
    if case["call"] == "coupled":
        byts += nc * 168  # the feedback: 11 values in, 10 out
        flops += nc * 80
    if case["call"].startswith("advance"):
        byts += N * (8 * 8 + 6 * 8) + nc * 8 * 8
    if case["call"] == "read":
        byts += N * 6 * 8
    return {"bytes": byts, "flops": flops}


# --------------------------------------------------------------------------
# 64-bit reference
# --------------------------------------------------------------------------

def _tsc(d):
    return [0.5 * (0.5 - d) ** 2, 0.75 - d * d, 0.5 * (0.5 + d) ** 2]


def _stencil(X, n, nd):
    """Cells and weights of the TSC stencil at positions X (cell units)."""
    i = torch.floor(X)
    ws = [_tsc(X[d] - i[d] - 0.5) for d in range(nd)]
    i = i.to(torch.int64)
    idx, wts = [], []
    for oz in range(3 if nd == 3 else 1):
        for oy in range(3):
            for ox in range(3):
                z = torch.remainder(i[2] + oz - 1, n[2]) if nd == 3 else 0
                c = (z * n[1] + torch.remainder(i[1] + oy - 1, n[1])) * n[0] + torch.remainder(
                    i[0] + ox - 1, n[0])
                idx.append(c)
                wts.append(ws[0][ox] * ws[1][oy] * (ws[2][oz] if nd == 3 else 1.0))
    return idx, wts


def _cross(a, b):
    return torch.stack([a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]])


def _current(X, v, m, qm, n, nd, C, nc):
    """n_CR and J_CR per cell (unit cells)."""
    u = v * (C / (C * C + v.square().sum(0)).sqrt())
    amounts = torch.cat([(qm * m)[None], qm * m * u])
    nj = torch.zeros(4, nc, dtype=torch.float64, device=X.device)
    for c, w in zip(*_stencil(X, n, nd)):
        nj.index_add_(1, c, amounts * w)
    return nj[0], nj[1:]


def _hall(ncr, J, B, E0, rho):
    R = ncr / (rho + ncr)
    return (1.0 - R) * (ncr * E0 + _cross(J, B))


def exact(case, seed):
    if case["call"] not in ("advance", "advance_noalloc", "coupled", "read"):
        return None  # deposits only: whole numbers
    s = _inputs(case, seed)
    n, nd, C = (case["nx"], case["ny"], case["nz"]), case["ndim"], C_LIGHT
    if len(s["counts"]) != 1 or case["pop"] == "wall":
        return None
    nc = n[0] * n[1] * n[2]
    x, v, m, qm, B, rho = s["x"], s["v"], s["m"], s["qm"], s["B"], s["rho"]
    E0 = -_cross(s["vg"], B)
    if case["call"] == "coupled":
        ncr, J = _current(x, v, m, qm, n, nd, C, nc)
        R = ncr / (rho + ncr)
        F = _hall(ncr, J, B, E0, rho)
        Rs = R if case["hall"] else torch.zeros_like(R)
        if not case["hall"]:
            F = ncr * E0 + _cross(J, B)
        dE = -F / rho if case["hall"] else torch.zeros_like(F)
        vA = (B.square().sum(0) / rho).sqrt()
        lam = torch.where(ncr > 0, R * (J / ncr.clamp_min(1e-300) - s["vg"]) / vA, torch.zeros_like(J))
        fb = torch.cat([-F, -((1.0 - Rs) * (J * E0).sum(0))[None], _cross(dE, B), lam])
        return {"fb": fb, "D": None}
    L = torch.tensor([float(k) for k in n], dtype=torch.float64, device=x.device)[:nd, None]
    dts = s["dt"][0] / case["sub"]

    def drift(x, v):
        u = v * (C / (C * C + v.square().sum(0)).sqrt())
        x = x.clone()
        x[:nd] = torch.remainder(x[:nd] + 0.5 * dts * u[:nd], L)
        return x

    for _ in range(case["steps"]):
        E = E0
        if case["hall"]:
            ncr, J = _current(x, v, m, qm, n, nd, C, nc)
            E = E0 - _hall(ncr, J, B, E0, rho) / rho
        for _ in range(case["sub"]):
            x = drift(x, v)
            Ep, Bp = torch.zeros_like(v), torch.zeros_like(v)
            for c, w in zip(*_stencil(x, n, nd)):
                Ep += w * E[:, c]
                Bp += w * B[:, c]
            Ep = Ep - (Ep * Bp).sum(0) / Bp.square().sum(0) * Bp
            h = 0.5 * dts * qm
            w0 = v + h * Ep
            t = h * (C / (C * C + w0.square().sum(0)).sqrt()) * Bp
            p = w0 + _cross(w0, t)
            v = w0 + _cross(2.0 / (1.0 + t.square().sum(0)) * p, t) + h * Ep
            x = drift(x, v)
    return {"x": x, "v": v, "D": None}
