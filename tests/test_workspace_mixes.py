"""The class autotuner's workspace holds every mix of one tile shape per box-size
class, in the layout that a context of that mix gets."""
import ctypes as ct
import itertools
import random

import pytest

SHAPES = {2: [(16, 16, 1), (32, 16, 1), (8, 8, 1), (32, 32, 1), (64, 16, 1)],
          3: [(8, 4, 4), (8, 8, 4), (4, 4, 4), (8, 8, 8), (16, 4, 4)]}


def _size_class(n):
    return ((n[0] * n[1] * n[2]).bit_length() - 1) // 2


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ndim", [2, 3])
def test_class_workspace_holds_every_mix(ndim, precision):
    from paper_1412_1087_amd import mhdpic as M
    rng = random.Random(491)
    lo, hi = (4, 200) if ndim == 2 else (3, 60)
    for _ in range(60):
        ns = [tuple(rng.randint(lo, hi) for _ in range(ndim)) + (1,) * (3 - ndim)
              for _ in range(rng.choice([2, 3, 8]))]
        counts = [int(n[0] * n[1] * n[2] * rng.uniform(1.0, 40.0)) for n in ns]
        arr = M._boxes_array([M.Box(ndim=ndim, n=n) for n in ns])
        size = ct.c_size_t()
        M._check(M.lib().mhdpic_autotune_classes_workspace_size(arr, len(ns), (ct.c_int64 * len(ns))(*counts),
                                                                precision, ct.byref(size)))
        classes = sorted({_size_class(n) for n in ns})
        for mix in itertools.product(SHAPES[ndim], repeat=min(len(classes), 3)):
            tile = {c: mix[k % len(mix)] for k, c in enumerate(classes)}
            try:
                need = M.workspace_size([M.Box(ndim=ndim, n=n, tile=tile[_size_class(n)]) for n in ns], counts,
                                        precision)
            except M.MhdpicError as e:  # a shape beyond the LDS in this precision
                assert e.code == M.ENOTSUP
                continue
            assert need <= size.value, (ns, counts, tile)
