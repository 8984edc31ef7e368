"""Which kernel a product takes (host rule only, no GPU): shapes on both sides
of the rule whose times differ by more than a tenth either way."""
import ctypes
import os

import pytest

from paper_2607_05711_amd import _lib

pytestmark = pytest.mark.skipif(not os.path.exists(_lib.LIB_PATH), reason="libfourtune.so not built")


def gemm_kernel(bwd, M, N, K, R=0, out_f32=False):
    f = _lib.load().ftx_gemm_kernel
    f.argtypes, f.restype = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int32, ctypes.c_int], ctypes.c_int
    return f(int(bwd), M, N, K, R, int(out_f32))


@pytest.mark.parametrize("bwd,M,N,K,R,want", [
    # long reductions, whose scales leave a CU room for one 128x128 workgroup only (us on 256, 128, 64 rows)
    (False, 1252, 5376, 8448, 32, 256),     # 49, 67, 55
    (False, 14590, 384, 7680, 16, 256),     # 45, 86, 73
    (False, 1750, 4224, 9728, 0, 256),      # 52, 84, 77
    (False, 9390, 1664, 13952, 0, 256),     # 172, 225, 190
    (True, 9106, 4480, 512, 64, 256),       # 32, 38, 36
    (False, 228, 17536, 6144, 0, 256),      # 34, 42, 40
    # few large tiles
    (False, 512, 3072, 3072, 64, 64),       # 22.5 on 256, 12.3 on 64
    (False, 512, 3072, 12288, 64, 64),      # 65, 31
    (True, 1678, 12928, 256, 32, 64),       # 60, 52, 28
    (False, 3344, 2048, 640, 64, 128),      # 14.3, 12.0, 15.8
    # the benchmark's layers
    (False, 4608, 9216, 3072, 64, 256),
    (True, 4608, 9216, 3072, 64, 256),
    (False, 18432, 3072, 15360, 96, 256),
    # widths that only the small tiles take, and a reduction too long for their scales
    (False, 1111, 3168, 2080, 32, 64),
    (False, 33, 96, 66080, 16, 0),
])
def test_kernel_of_a_product(bwd, M, N, K, R, want):
    assert gemm_kernel(bwd, M, N, K, R) == want


def mlp_fused(bwd, M, N, K, R, R2):
    f = _lib.load().ftx_mlp_fused
    f.argtypes, f.restype = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int32] * 2, ctypes.c_int
    return bool(f(int(bwd), M, N, K, R, R2))


@pytest.mark.parametrize("bwd,M,D,W,R2,want", [
    # us in the GEMM's epilogue and as a pass of its own
    (False, 4608, 3072, 12288, 0, True),    # 145, 166
    (True, 4608, 3072, 12288, 0, True),     # 154, 172
    (False, 4608, 3072, 12288, 64, True),   # 167, 174
    (True, 4608, 3072, 12288, 64, True),    # 178, 184
    (False, 18432, 3072, 12288, 0, True),   # 529, 683
    (False, 1500, 2432, 9728, 0, True),     # 36, 51
    (False, 2000, 1024, 4096, 0, True),     # 24, 30
    (False, 839, 1920, 7680, 0, True),      # 28, 32
    (True, 2000, 1024, 4096, 0, False),     # 27, 25
    (False, 512, 3072, 12288, 64, False),   # 42, 39
    (True, 512, 3072, 12288, 64, False),    # 46, 41
    (False, 321, 512, 2048, 0, False),      # 21, 16
    (True, 321, 512, 2048, 64, False),      # 29, 18
])
def test_form_of_the_mlp_calls(bwd, M, D, W, R2, want):
    N, K = (D, W) if bwd else (W, D)
    assert mlp_fused(bwd, M, N, K, 64, R2) == want
