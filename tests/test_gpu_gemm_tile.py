"""The FP4 GEMM on small output tiles (64x128 and 128x128) and the shapes on
the other side of its rule, against the oracle: every output in fp32 mode
within 1e-5 of the sum of magnitudes, bf16 as its exact rounding."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2607_05711_amd import _lib, gen
from tests.test_gpu_parity import check_layer, dev_bf16, dev_u8, host, make_case, run_gpu_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,r,rs", [
    (64, 256, 128, 16, 16),      # exactly one tile of 64x128
    (65, 288, 160, 8, 8),        # one row, one 32-column block and one scale byte past it
    (129, 3072, 3072, 96, 32),   # R = 128: four low-rank stages, the ring's five slots
    (63, 3104, 416, 0, 0),       # no low-rank stage; KR/32 = 97: scale bytes at any alignment
    (1111, 2080, 3168, 24, 8),   # two 64-row workgroups on a CU; 65 and 99 scale bytes per row
    (520, 1024, 9216, 32, 32),   # 128x128 tiles, two slots and two workgroups on a CU
    (1500, 1056, 1312, 8, 24),   # 128x128 or 64x128 tiles with a ragged last row and column tile
    (2300, 512, 4736, 16, 32),   # forward on 256x256 tiles with ragged edges, backward on small ones
])
def test_layer_on_small_tiles(M, K, N, r, rs):
    shape = gen.custom_shape(M, K, N, r=r, r_s=rs, n_outliers=3, outlier_scale=30.0, dy_kind="student_t3")
    d = make_case(shape, M)
    check_layer(d, shape, run_gpu_layer(d, shape, with_bias=(M % 2 == 1)), with_bias=(M % 2 == 1))


@pytest.mark.parametrize("M,KR,NO,R", [
    (70, 21504, 96, 32),         # fewer ring slots beside the scales of a long reduction
    (40, 49184, 64, 16),         # two slots
    (33, 66080, 96, 16),         # too long for the scales to stay in LDS: the register-staged kernel
])
def test_long_reductions(M, KR, NO, R):
    """Random codes, both directions.  The fp32 chain rounds once per
    64-element step, so at these lengths the bound is the chain's own:
    KR / 64 roundings of 2^-24 of the sum of magnitudes."""
    rng = np.random.default_rng(KR)
    aq = rng.integers(0, 256, (M, KR // 2)).astype(np.uint8)
    asc = rng.integers(110, 130, (M, KR // 32)).astype(np.uint8)
    P = rng.standard_normal((M, R)).astype(np.float32)
    LR = gen.f32_to_bf16_bits(rng.standard_normal((R, NO)).astype(np.float32))
    tol = max(1e-5, (KR / 64 + 2 * R / 16 + 1) * 2.0 ** -24)
    Pg = torch.from_numpy(P).to("cuda:0")
    wq = rng.integers(0, 256, (NO, KR // 2)).astype(np.uint8)
    ws = rng.integers(110, 130, (NO // 32, KR // 32)).astype(np.uint8)
    y = _lib.ft_linear_fwd(dev_u8(aq), dev_u8(asc), dev_u8(wq), dev_u8(ws), KR, Pg, dev_bf16(LR), None,
                           out_dtype=torch.float32)
    torch.cuda.synchronize()
    yr, S = ref.linear_fwd(aq, asc, wq, ws, KR, P.astype(np.float64), LR, None)
    assert np.all(np.abs(host(y) - yr) <= tol * S)
    wq = rng.integers(0, 256, (KR, NO // 2)).astype(np.uint8)
    ws = rng.integers(110, 130, (KR // 32, NO // 32)).astype(np.uint8)
    D = np.ascontiguousarray(LR.T)
    dx = _lib.ft_linear_bwd_input(dev_u8(aq), dev_u8(asc), dev_u8(wq), dev_u8(ws), NO, Pg, dev_bf16(D),
                                  out_dtype=torch.float32)
    torch.cuda.synchronize()
    dxr, S = ref.linear_bwd_input(aq, asc, wq, ws, NO, P.astype(np.float64), D)
    assert np.all(np.abs(host(dx) - dxr) <= tol * S)
