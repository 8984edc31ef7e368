"""The streaming quantize + projection kernel at the edges of its tiles: rows
around a workgroup's 128, widths that end within a 64-column step, runs of
every length, every tile count of the projection, both layouts and both scale
rules.  Codes and scales bit for bit against the oracle, the projection within
the fp32 bound of its sums."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2607_05711_amd import _lib, gen
from tests._helpers import adversarial_rows
from tests.test_gpu_parity import dev_bf16, host, proj_bound

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,R,layout", [
    (1, 32, 16, 0), (1, 32, 16, 1),          # half a step
    (127, 96, 48, 0), (129, 96, 48, 1),      # a step and a half; R no multiple of 32
    (128, 2080, 64, 0), (300, 2080, 64, 1),  # 65 scale bytes per row
    (33, 1312, 96, 0), (200, 1312, 80, 1),   # three projection tiles
    (257, 1056, 128, 0), (130, 1056, 112, 1),  # four
    (16, 4160, 32, 1),                       # 65 steps: a last run of one step
])
@pytest.mark.parametrize("no_clip", [False, True])
def test_streaming_quantize_project(rows, cols, R, layout, no_clip):
    g = np.random.default_rng(rows + cols + R)
    x = gen.f32_to_bf16_bits((g.standard_normal((rows, cols)) * np.exp2(g.integers(-3, 4, (rows, cols)))).astype(np.float32))
    a = adversarial_rows(cols, seed=1)
    finite = [r for r in a if np.all((r & 0x7FFF) < 0x6000)]      # keep the projection's sums in fp32's range
    x[:min(rows, len(finite))] = np.stack(finite)[:rows]
    p = gen.f32_to_bf16_bits(g.standard_normal((cols, R) if layout == 0 else (R, cols)).astype(np.float32))
    mode = dict(scale_rule=_lib.FT_SCALE_NO_CLIP) if no_clip else {}
    codes, scales, out = _lib.ft_quantize_blockwise_mode(dev_bf16(x), proj=dev_bf16(p), proj_layout=layout, **mode)
    torch.cuda.synchronize()
    want = ref.quantize_ex(x, 1, scale_rule=1) if no_clip else ref.quantize(x, 1)
    assert np.array_equal(host(codes), want[0]) and np.array_equal(host(scales), want[1])
    P, Pabs = ref.proj(x, p, layout)
    assert np.all(np.abs(host(out) - P) <= proj_bound(cols, Pabs))


@pytest.mark.parametrize("layout", [0, 1])
def test_rows_too_wide_for_the_streaming_kernel(layout):
    """From 2^23 columns on, 128 rows pass its 32-bit offsets and the chunked
    kernel takes the call: codes and scales are those of the call without a
    projection, the projection within the bound of its chains (at most 256
    products in a partial, and one partial per 256 columns or more)."""
    rows, cols, R = 3, (1 << 23) + 32, 16
    g = torch.Generator(device="cuda:0").manual_seed(layout)
    x = torch.randn((rows, cols), generator=g, device="cuda:0").to(torch.bfloat16)
    p = torch.randn((cols, R) if layout == 0 else (R, cols), generator=g, device="cuda:0").to(torch.bfloat16)
    codes, scales, out = _lib.ft_quantize_blockwise(x, proj=p, proj_layout=layout)
    codes0, scales0, _ = _lib.ft_quantize_blockwise(x)
    torch.cuda.synchronize()
    assert torch.equal(codes, codes0) and torch.equal(scales, scales0)
    want, mag = torch.zeros((2, rows, R), dtype=torch.float64, device="cuda:0")
    for c in range(0, cols, 1 << 20):
        a = x[:, c:c + (1 << 20)].double()
        b = (p[c:c + (1 << 20)] if layout == 0 else p[:, c:c + (1 << 20)].T.contiguous()).double()
        want += a @ b
        mag += a.abs() @ b.abs()
    bound = (256 + cols / 256) * 2.0 ** -24 * mag
    assert bool(((out.double() - want).abs() <= bound).all())
