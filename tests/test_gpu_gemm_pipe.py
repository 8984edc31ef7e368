"""The MLP pair's calls on either side of their rule, with the 256x256 GEMM's
GELU and dGELU epilogues at the edges of its tiles.  Every case first asserts
the form that the rule gives it; oracle and bounds are those of the MLP tests."""
import pytest

from tests import test_gpu_mlp as mlp
from tests.test_gemm_rule import gemm_kernel, mlp_fused

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,R,R2,fused", [
    (1030, 384, 8480, 32, 32, True),     # ragged rows and columns, a half last stage
    (1030, 1024, 8480, 0, 64, True),     # paired A scales
    (1030, 640, 8480, 48, 0, True),      # no projection
    (2000, 1024, 4096, 32, 0, True),     # 128x128 tiles would gain less than the pass over z costs
    (1202, 640, 2528, 16, 0, False),     # small tiles, a pass of several chunks and row blocks without a projection
    (520, 1024, 9216, 32, 48, False),    # 128x128 tiles
])
def test_fc1_either_side_of_the_rule(M, K, N, R, R2, fused):
    assert mlp_fused(False, M, N, K, R, R2) == fused
    mlp.test_fc1_forward_gelu_quantize_project(M, K, N, R, R2)


@pytest.mark.parametrize("M,N,K,R,R1,fused", [
    (1030, 384, 8576, 32, 32, True),
    (1030, 1024, 8576, 0, 16, True),
    (1030, 640, 8576, 48, 0, True),
    (520, 1024, 9216, 32, 48, False),    # dGELU on 128x128 tiles
    (1202, 640, 2560, 16, 0, False),
])
def test_fc2_either_side_of_the_rule(M, N, K, R, R1, fused):
    assert mlp_fused(True, M, N, K, R, R1) == fused
    if not fused and K == 9216:
        assert gemm_kernel(True, M, N, K, R) == 128
    mlp.test_fc2_backward_dgelu_quantize_project(M, N, K, R, R1)
