"""lr_workspace_size is part of the interface: a program that keeps a workspace of a
fixed size fits the batches it always fitted.

The sizes are counted in tiles of TILE vectors, one table of n_fft x n_fft
entries on the non-separable path, two work fields, the masks and regions and
one set of dphi partials per group of samples, each part rounded up to 256
bytes.
"""

import ctypes
import os

import pytest

from paper_2306_11268_amd import binding as lb

pytestmark = pytest.mark.skipif(not os.path.exists(lb.LIB_PATH), reason="liblr.so not built")

TILE = {64: 16, 100: 16, 128: 16, 200: 32, 256: 8, 350: 32, 400: 8, 500: 16, 512: 8, 1000: 8, 1024: 8}


def expected(approx, n, m, layers, regions, batch, op):
    up = lambda x: -(-x // 256) * 256  # noqa: E731
    tiles = -(-n // TILE[m])
    nn = n * n
    total = 2 * up(8 * m) if approx == lb.LR_FRESNEL else up(8 * m * m)
    total += 2 * up(8 * batch * (nn if approx == lb.LR_FRESNEL else n * m))
    if op == lb.LR_OP_PROPAGATE:
        return total
    total += up(8 * layers * nn)
    if regions:
        total += up(8 * regions) + 2 * up(8 * n) + 2 * up(4 * n)
    if op == lb.LR_OP_FORWARD:
        return total + (up(4 * batch * tiles * regions) if regions else 0)
    if regions:
        total += up(4 * batch * regions)
    per = max(1, min(batch, -(-batch * tiles // 2048)))
    groups = -(-batch // per) if batch else 1
    return total + up(4 * layers * groups * nn)


@pytest.mark.parametrize("m", sorted(TILE))
def test_sizes(m):
    lib = lb.load()
    coords = (ctypes.c_int32 * 64)(*([0] * 64))
    p = ctypes.cast(coords, ctypes.POINTER(ctypes.c_int32))
    for approx in (lb.LR_FRESNEL, lb.LR_ANGULAR_SPECTRUM, lb.LR_RS_IR, lb.LR_FRAUNHOFER):
        for n in sorted({m, m - 2, m // 2 - (m // 2 - m) % 2, 2 + m % 2}):
            for layers, regions in ((1, 0), (2, 10), (5, 64)):
                net = lb.LrDonn(532e-9, 36e-6, 0.3, approx, n, m, layers, 1.0, lb.LrDetector(regions, 1, p, p),
                                ctypes.c_void_p(0x1000))
                for batch in (0, 1, 3, 33, 64, 255, 500, 4097):
                    for op in (lb.LR_OP_PROPAGATE, lb.LR_OP_FORWARD, lb.LR_OP_BACKWARD):
                        if approx == lb.LR_FRAUNHOFER and op != lb.LR_OP_PROPAGATE:
                            continue
                        got = lib.lr_workspace_size(ctypes.byref(net), batch, op)
                        assert got == expected(approx, n, m, layers, regions, batch, op), (approx, n, layers, regions,
                                                                                          batch, op)
