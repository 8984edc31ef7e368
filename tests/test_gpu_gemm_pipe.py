"""The 256x256 FP4 GEMM at the edges of its tiles, and the MLP pair's calls on
either side of their rule.  Every case first asserts the kernel that the rule
gives it: ragged rows and columns, a half last stage (reduction an odd multiple
of 128), paired and unpaired A scales (reduction a multiple of 512 or not), low-
rank widths with a half last chunk, none and four, both output types, and the
fused GELU and dGELU epilogues.  Oracle and bounds are those of the parity and
MLP tests."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2607_05711_amd import _lib, gen
from tests import test_gpu_mlp as mlp
from tests.test_gemm_rule import gemm_kernel, mlp_fused
from tests.test_gpu_parity import check_gemm, dev_bf16, dev_u8, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bwd,M,KR,NO,R", [
    (False, 1030, 128, 9376, 16),    # one half stage; ragged last row and column tile
    (False, 1030, 384, 8480, 48),    # a stage and a half; half a last low-rank chunk
    (False, 1281, 896, 7008, 0),     # one row past a tile; no low-rank stage
    (False, 1030, 768, 8480, 128),   # whole stages, an odd number of them
    (False, 1030, 512, 8480, 80),    # paired A scales
    (False, 1027, 1536, 8224, 64),
    (True, 1030, 128, 9344, 16),
    (True, 1030, 384, 8576, 48),
    (True, 1281, 896, 6784, 0),
    (True, 1030, 768, 8576, 128),
    (True, 1030, 512, 8576, 80),
    (True, 1027, 1536, 8320, 64),
])
def test_gemm_on_large_tiles(bwd, M, KR, NO, R):
    N, K = (KR, NO) if bwd else (NO, KR)
    assert gemm_kernel(bwd, M, N, K, R, True) == gemm_kernel(bwd, M, N, K, R, False) == 256
    rng = np.random.default_rng(M + KR + NO + R)
    aq = rng.integers(0, 256, (M, KR // 2)).astype(np.uint8)
    asc = rng.integers(110, 140, (M, KR // 32)).astype(np.uint8)
    wq = rng.integers(0, 256, (N, K // 2)).astype(np.uint8)
    ws = rng.integers(110, 140, (N // 32, K // 32)).astype(np.uint8)
    P = LR = Pt = Lt = None
    if R:
        P = rng.standard_normal((M, R)).astype(np.float32)
        LR = gen.f32_to_bf16_bits(rng.standard_normal((K, R) if bwd else (R, N)).astype(np.float32))
        Pt, Lt = torch.from_numpy(P).to("cuda:0"), dev_bf16(LR)
        P = P.astype(np.float64)
    args = (dev_u8(aq), dev_u8(asc), dev_u8(wq), dev_u8(ws), K, Pt, Lt)
    if bwd:
        o32, o16 = (_lib.ft_linear_bwd_input(*args, out_dtype=t) for t in (torch.float32, torch.bfloat16))
        want, S = ref.linear_bwd_input(aq, asc, wq, ws, K, P, LR)
    else:
        bias = gen.f32_to_bf16_bits(rng.standard_normal(N).astype(np.float32))
        o32, o16 = (_lib.ft_linear_fwd(*args, dev_bf16(bias), out_dtype=t) for t in (torch.float32, torch.bfloat16))
        want, S = ref.linear_fwd(aq, asc, wq, ws, K, P, LR, bias)
    torch.cuda.synchronize()
    check_gemm(host(o32), host(o16), want, S, "backward-input" if bwd else "forward")


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
