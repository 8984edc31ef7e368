"""The streaming quantize kernel's projection sums round no more often than the
chunked kernel's, which they replace (host rule only, no GPU)."""
import ctypes
import math
import os
import random

import pytest

from paper_2607_05711_amd import _lib

pytestmark = pytest.mark.skipif(not os.path.exists(_lib.LIB_PATH), reason="libfourtune.so not built")


def chains(rows, cols, R, layout):
    f = _lib.load().ftx_quant_chain
    f.argtypes, f.restype = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int32, ctypes.c_int] + [ctypes.POINTER(ctypes.c_int32)] * 2, None
    s, c = ctypes.c_int32(), ctypes.c_int32()
    f(rows, cols, R, layout, s, c)
    return s.value, c.value


@pytest.mark.parametrize("layout", [0, 1])
def test_projection_sums_round_no_more_often(layout):
    rng = random.Random(layout)
    sizes = [(32768, 21504, 96), (8709, 13568, 96), (13938, 13312, 64), (18432, 21504, 96), (1, 32, 16), (4608, 12288, 64)]
    sizes += [(int(math.exp(rng.uniform(0, 11))), 32 * rng.randint(1, 1000), 16 * rng.randint(1, 8)) for _ in range(3000)]
    for s in sizes:
        streaming, chunked = chains(*s, layout)
        assert streaming <= max(chunked, 6), s      # six: one step, the sums of its sets, one partial
