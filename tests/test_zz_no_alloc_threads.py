"""mhdpic_advance_noalloc from several threads at once, each on a stream and with
boxes of its own, and with input that one of them has refused: the results of
the same calls one after another."""
import threading

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1412_1087_amd import workloads as W  # noqa: E402

from gpu_helpers import gpu_box, to_dev  # noqa: E402


def test_calls_of_several_threads_take_turns():
    from paper_1412_1087_amd import mhdpic as M
    wls = [W.gyro2d(nx=40, ny=30, ppc=20, seed=501), W.bell3d(n=(16, 12, 10), ppc=9, seed=502),
           W.gyro2d(nx=9, ny=120, ppc=5, seed=503), W.bell3d(n=(7, 21, 8), ppc=12, seed=504)]
    args = [[to_dev(a) for a in (w.x, w.v, w.m, w.qm, w.B, w.vg, w.rho)] for w in wls]
    args[2][2][3] = 1e6  # a mass that set-up refuses
    torch.cuda.synchronize()

    def call(k, stream):
        try:
            return M.advance([gpu_box(wls[k].box)], [wls[k].N], *args[k], wls[k].dt, 3, noalloc=True,
                             stream=stream)
        except M.MhdpicError as e:
            return e.code

    ref = [call(k, None) for k in range(4)]
    assert ref[2] == M.ERANGE
    got = [[] for _ in wls]

    def work(k):
        s = torch.cuda.Stream()
        for _ in range(25):
            got[k].append(call(k, s))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
    assert not any(t.is_alive() for t in threads)
    for k in range(4):
        assert len(got[k]) == 25
        for out in got[k]:
            if k == 2:
                assert out == ref[2]
            else:
                assert all(torch.equal(a, b) for a, b in zip(out, ref[k]))
