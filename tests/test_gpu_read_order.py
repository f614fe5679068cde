"""A read-out that has not run yet, and calls after it that use the same part
of the workspace: on another thread's per-thread stream (one handle for both),
and on a third stream after a call that was refused on a second."""
import threading
from types import SimpleNamespace

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import DeviceRun  # noqa: E402

PER_THREAD = SimpleNamespace(cuda_stream=2)  # hipStreamPerThread


def _same_bits(a, b):
    return all(np.array_equal(p.cpu().numpy().view(np.uint64), q.cpu().numpy().view(np.uint64))
               for p, q in zip(a, b))


def _busy():
    """A context whose steps keep a stream busy for some tens of ms."""
    g = DeviceRun(W.bell3d(n=(48, 48, 48), ppc=16, seed=431))
    g.step(1)
    return lambda stream: g.ctx.step(g.B, g.vg, g.rho, [g.wls[0].dt], 60, stream=stream)


def _contexts():
    wl = W.gyro2d(nx=128, ny=128, ppc=32, seed=432)
    g, h = DeviceRun(wl), DeviceRun(wl)
    g.step(2)
    h.step(2)
    before = [t.clone() for t in h.ctx.particles_read()]
    h.step(1)
    after = [t.clone() for t in h.ctx.particles_read()]
    torch.cuda.synchronize()
    return g, [wl.dt], before, after


def test_per_thread_streams_of_two_threads():
    busy = _busy()
    g, dt, before, after = _contexts()
    out, errors = {}, []
    enqueued, done = threading.Event(), threading.Event()

    def reader():
        try:
            busy(PER_THREAD)
            out["read"] = g.ctx.particles_read(stream=PER_THREAD)
        except Exception as e:  # noqa: BLE001
            errors.append(e)
        enqueued.set()
        done.wait(60)  # (the thread's stream lives as long as the thread)

    def stepper():
        try:
            g.ctx.step(g.B, g.vg, g.rho, dt, 1, stream=PER_THREAD)
            out["after"] = g.ctx.particles_read(stream=PER_THREAD)
            torch.cuda.synchronize()
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    a, b = threading.Thread(target=reader), threading.Thread(target=stepper)
    a.start()
    assert enqueued.wait(60)
    b.start()
    b.join(60)
    done.set()
    a.join(60)
    assert not errors and not a.is_alive() and not b.is_alive()
    torch.cuda.synchronize()
    assert _same_bits(out["read"], before) and _same_bits(out["after"], after)


def test_refused_call_between():
    from paper_1412_1087_amd import mhdpic as M
    busy = _busy()
    g, dt, before, after = _contexts()
    s1, s2, s3 = (torch.cuda.Stream() for _ in range(3))
    busy(s1)
    read = g.ctx.particles_read(stream=s1)
    with pytest.raises(M.MhdpicError):
        g.ctx.inject([-1], None, None, None, None, stream=s2)
    g.ctx.step(g.B, g.vg, g.rho, dt, 1, stream=s3)
    end = g.ctx.particles_read(stream=s3)
    torch.cuda.synchronize()
    assert _same_bits(read, before) and _same_bits(end, after)
