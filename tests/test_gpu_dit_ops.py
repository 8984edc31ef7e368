"""The fused DiT kernels (LayerNorm + modulation, q/k RMSNorm + rotary
embedding, GELU, gated residual), forward and backward, against the same
formulas in 64 bits; the calls that must run as torch operations instead."""
import pytest
import torch

from paper_2607_05711_amd import _dit_ops as ops

BF = torch.bfloat16
DEV = "cuda:0"
gpu = pytest.mark.gpu


def rnd(shape, seed, std=1.0, dev=DEV):
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    return (torch.randn(shape, generator=g, device=dev) * std).to(BF)


def tables(rows, hd, dev=DEV):
    a = torch.arange(rows * (hd // 2), device=dev, dtype=torch.float32).reshape(rows, 1, hd // 2) * 0.37
    return torch.cos(a), torch.sin(a)


def relerr(a, b):
    return ((a.double() - b.double()).norm() / b.double().norm()).item()


def norm64(x):
    return torch.nn.functional.layer_norm(x, (x.shape[-1],), eps=1e-6)


def rms64(x, w, cos, sin):
    y = x * torch.rsqrt(x.pow(2).mean(-1, keepdim=True) + 1e-6) * w.double()
    y = (y + (y.to(BF).double() - y).detach()).unflatten(-1, (-1, 2))      # stored in bf16
    c, s = cos.double(), sin.double()
    return torch.stack([y[..., 0] * c - y[..., 1] * s, y[..., 0] * s + y[..., 1] * c], -1).flatten(-2)


# A bf16 result is half a unit (2^-9) off at most; the rounding errors of many
# elements are uniform, so their 2-norm is near 2^-9 / sqrt(3) / (the mean
# mantissa's spread), below 2^-8.5.  Twice that where a bf16 value is rounded
# again on the way (q, k and their gradients).
TOL, TOL2 = 2.0 ** -8.5, 2.0 ** -7.5


@gpu
@pytest.mark.parametrize("rows,H", [(1, 8), (3, 136), (5, 520), (257, 1024), (130, 3072), (6, 4096)])
def test_modulate(rows, H):
    x, sh, sc, dy = rnd((rows, H), 1) + 0.5, rnd((1, 3 * H), 2)[:, H:2 * H], rnd((1, H), 3, 0.3), rnd((rows, H), 4)
    if H * 2 % 16:
        pytest.skip("chunk not aligned")
    x.requires_grad_(True)
    y = ops.modulate(x, sh, sc)
    assert type(y.grad_fn).__name__ == "_ModulateBackward"
    y.backward(dy)
    xd = x.detach().double().requires_grad_(True)
    yd = norm64(xd) * (1.0 + sc.double()) + sh.double()
    yd.backward(dy.double())
    assert relerr(y.detach(), yd.detach()) < TOL
    assert relerr(x.grad, xd.grad) < TOL


@gpu
@pytest.mark.parametrize("rows,H", [(1, 8), (257, 136), (33, 3072)])
def test_gated_residual(rows, H):
    x, y, g, d = (rnd((rows, H), 1).requires_grad_(True), rnd((rows, H), 2).requires_grad_(True), rnd((1, H), 3),
                  rnd((rows, H), 4))
    out = ops.gated_residual(x, g, y)
    assert type(out.grad_fn).__name__ == "_GateBackward"
    out.backward(d)
    assert torch.equal(out, x + g * y) and torch.equal(x.grad, d) and torch.equal(y.grad, d * g)


@gpu
@pytest.mark.parametrize("K,N", [(1, 8), (7, 128), (128, 136), (129, 8), (1000, 3072), (3072, 9216), (2056, 18440), (5000, 65544)])
def test_modulation(K, N):
    """Edges of the 128 columns and rows of a step, one and several steps a part."""
    v, w = rnd((1, K), 1, 2.0), rnd((K, N), 2)
    y = ops.modulation(v, w)
    assert y.shape == (1, N) and torch.equal(y[0], ops.modulation(v[0], w))
    s = torch.nn.functional.silu(v.double()).to(BF).double()
    assert relerr(y, s @ w.double()) < TOL
    for stays in (rnd((2, K), 1), rnd((1, 2 * K), 1)[:, ::2], v.clone().requires_grad_(True)):
        assert relerr(ops.modulation(stays, w).detach(), torch.nn.functional.silu(stays.detach()) @ w) < TOL2


@gpu
@pytest.mark.parametrize("T1,T2,heads,hd", [(1, 1, 1, 8), (7, 30, 3, 16), (5, 12, 2, 512), (64, 200, 24, 128)])
def test_joint_qkv(T1, T2, heads, hd):
    H = heads * hd
    txt, img = (rnd((t, 3 * H), 5 + t).requires_grad_(True) for t in (T1, T2))
    norms = [(rnd((hd,), 10 + i) + 1.0, rnd((hd,), 20 + i) + 1.0) for i in range(2)]
    cos, sin = tables(T1 + T2, hd)
    q, k, v = ops.joint_qkv(txt, img, norms, cos, sin, heads, hd)
    assert type(q.grad_fn).__name__ == "_JointQkvBackward"
    # gradients with heads before tokens in memory, as an attention backward returns them
    dq, dk, dv = (rnd((heads, T1 + T2, hd), 30 + i).transpose(0, 1) for i in range(3))
    torch.autograd.backward((q, k, v), (dq, dk, dv))
    t, m = txt.detach().double().requires_grad_(True), img.detach().double().requires_grad_(True)
    got = []
    for x, n, c, s in ((t, norms[0], cos[:T1], sin[:T1]), (m, norms[1], cos[T1:], sin[T1:])):
        a, b, w = x.view(-1, 3, heads, hd).unbind(1)
        got.append((rms64(a, n[0], c, s), rms64(b, n[1], c, s), w))
    ref = [torch.cat([got[0][i], got[1][i]], 0) for i in range(3)]
    torch.autograd.backward(ref, [d.double() for d in (dq, dk, dv)])
    for a, b in zip((q, k, v), ref):
        assert relerr(a.detach(), b.detach()) < TOL2
    assert relerr(txt.grad, t.grad) < TOL2 and relerr(img.grad, m.grad) < TOL2
    assert torch.equal(v.detach(), torch.cat([txt.detach(), img.detach()], 0).view(-1, 3, heads, hd)[:, 2])


@gpu
@pytest.mark.parametrize("T,heads,hd,Fm", [(1, 1, 8, 8), (37, 3, 32, 200), (130, 24, 128, 12288)])
def test_single_stream_mix(T, heads, hd, Fm):
    H = heads * hd
    h = (rnd((T, 3 * H + Fm), 7, 1.5)).requires_grad_(True)
    qn, kn = rnd((hd,), 8) + 1.0, rnd((hd,), 9) + 1.0
    cos, sin = tables(T, hd)
    mix = lambda q, k, v: (2.0 * q - k + 0.5 * v).reshape(q.shape[0], -1)   # in the attention's place
    c = ops.single_stream_mix(h, qn, kn, cos, sin, heads, hd, H, mix)
    assert type(c.grad_fn).__name__ == "_FillLeftBackward"
    dc = rnd((T, H + Fm), 11)
    c.backward(dc)
    x = h.detach().double().requires_grad_(True)
    q, k, v = x[:, :3 * H].reshape(-1, 3, heads, hd).unbind(1)
    ref = torch.cat([mix(rms64(q, qn, cos, sin), rms64(k, kn, cos, sin), v),
                     torch.nn.functional.gelu(x[:, 3 * H:], approximate="tanh")], -1)
    ref.backward(dc.double())
    assert relerr(c.detach()[:, H:], ref.detach()[:, H:]) < TOL
    assert relerr(c.detach()[:, :H], ref.detach()[:, :H]) < 2 * TOL2      # three more bf16 steps in the mix
    for a, b in ((0, 2 * H), (2 * H, 3 * H), (3 * H, 3 * H + Fm)):
        assert relerr(h.grad[:, a:b], x.grad[:, a:b]) < 2 * TOL2
    with torch.no_grad():
        assert torch.equal(ops.single_stream_mix(h, qn, kn, cos, sin, heads, hd, H, mix), c)


@gpu
@pytest.mark.parametrize("L,heads,gain", [(1, 2, 1.0), (64, 1, 1.0), (65, 3, 1.0), (300, 8, 4.0), (1000, 2, 1.0),
                                          (1300, 24, 1.0)])    # the last with two key tiles per wave
def test_attention(L, heads, gain):
    q, k = (rnd((L, heads, 128), 1 + i, gain).requires_grad_(True) for i in range(2))
    h = rnd((L, 4 * heads * 128), 3)
    v = h[:, heads * 128:2 * heads * 128].view(L, heads, 128).detach().requires_grad_(True)    # strided, as in a block
    g = rnd((L, 3 * heads * 128), 4, 1e-3)[:, :heads * 128]
    runs = []
    for _ in range(2):
        q.grad = k.grad = v.grad = None
        o = ops.attention(q, k, v)
        assert type(o.grad_fn).__name__ == "_AttentionBackward"
        o.backward(g)
        runs.append([o.detach().clone(), q.grad, k.grad, v.grad])
    assert all(torch.equal(a, b) for a, b in zip(*runs))       # fixed summation orders
    Q, K, V = (t.detach().double().requires_grad_(True) for t in (q, k, v))
    ref = torch.cat([torch.softmax(Q[:, i] @ K[:, i].T * 128 ** -0.5, -1) @ V[:, i] for i in range(heads)], -1)
    ref.backward(g.double())
    # p and ds are rounded to bf16 once before their products, and the result once; ds = p (dp - delta) cancels where
    # the scores are sharp (gain 4), which the bf16 rounding of the result o in delta sees
    tol = TOL2 * (1.0 if gain == 1.0 else 4.0)
    assert relerr(runs[0][0], ref.detach()) < TOL2
    for got, want in zip(runs[0][1:], (Q.grad, K.grad, V.grad)):
        # (one token: dq and dk are exactly zero in the reference)
        assert got.double().norm() < 1e-5 if L == 1 and want.norm() < 1e-9 else relerr(got, want) < tol


@gpu
def test_attention_where_every_score_is_far_below_zero():
    """Scores near -300: the stage's rows past the last key (whose score is 0) must not reach dq."""
    a = rnd((1, 2, 128), 1).float() * 5.2
    q, k = ((s * a + rnd((70, 2, 128), 2 + i).float()).to(BF).requires_grad_(True) for i, s in enumerate((1.0, -1.0)))
    v, g = rnd((70, 2, 128), 4).requires_grad_(True), rnd((70, 256), 5)
    o = ops.attention(q, k, v)
    o.backward(g)
    Q, K, V = (t.detach().double().requires_grad_(True) for t in (q, k, v))
    s = Q[:, 0] @ K[:, 0].T * 128 ** -0.5
    assert s.max() < -150
    ref = torch.cat([torch.softmax(Q[:, i] @ K[:, i].T * 128 ** -0.5, -1) @ V[:, i] for i in range(2)], -1)
    ref.backward(g.double())
    for got, want in ((o.detach(), ref.detach()), (q.grad, Q.grad), (k.grad, K.grad), (v.grad, V.grad)):
        assert bool(torch.isfinite(got).all()) and relerr(got, want) < 8 * TOL2


@gpu
def test_attention_of_other_shapes_is_the_library_s():
    q, k, v = (rnd((40, 2, 64), 1 + i) for i in range(3))
    assert torch.equal(ops.attention(q, k, v), ops.torch_attention(q, k, v))


@gpu
def test_attention_under_autocast_is_the_library_s():
    """Autocast to another type converts q, k and v; to bf16 it changes nothing."""
    q, k, v = (rnd((40, 2, 128), 1 + i) for i in range(3))
    with torch.autocast("cuda", dtype=torch.float16):
        o = ops.attention(q, k, v)
        assert o.dtype == torch.float16 and torch.equal(o, ops.torch_attention(q, k, v))
    want = ops.attention(q, k, v)
    with torch.autocast("cuda", dtype=BF):
        assert torch.equal(ops.attention(q, k, v), want)
    h, n, (cos, sin) = rnd((40, 3 * 256 + 64), 4), torch.ones(128, dtype=BF, device=DEV), tables(40, 128)
    with torch.autocast("cuda", dtype=torch.float16):      # the MLP part stays bf16: the two meet in fp32
        assert ops.single_stream_mix(h, n, n, cos, sin, 2, 128, 256).dtype == torch.float32


@gpu
def test_attention_gradient_of_far_rows():
    """A gradient whose rows lie further apart than the kernels' 32-bit offsets reach; q, k and v whose contiguous
    gradients would."""
    q, k, v = (rnd((64, 1, 128), 1 + i).requires_grad_(True) for i in range(3))
    far = torch.empty((64, 8460000), dtype=BF, device=DEV)[:, :128]
    far.copy_(rnd((64, 128), 4))
    o = ops.attention(q, k, v)
    assert type(o.grad_fn).__name__ == "_AttentionBackward"
    got = torch.autograd.grad(o, (q, k, v), far, retain_graph=True)
    want = torch.autograd.grad(o, (q, k, v), far.contiguous())
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    del far
    big = torch.empty((64, 131072, 128), dtype=BF, device=DEV).transpose(0, 1)
    assert not ops._attention_ok(big, big, big)


@gpu
def test_calls_that_stay_torch_operations():
    """Gradients of the modulation, other types and layouts, widths past the
    kernel's, functional transforms and a differentiated backward."""
    x, sh, sc, dy = rnd((6, 64), 1), rnd((1, 64), 2), rnd((1, 64), 3), rnd((6, 64), 4)
    a, b = sh.clone().requires_grad_(True), sc.clone().requires_grad_(True)
    ops.modulate(x, a, b).backward(dy)
    assert torch.allclose(a.grad.float(), dy.float().sum(0, keepdim=True), atol=0.05) and b.grad is not None
    want = ops.torch_modulate(x, sh, sc)
    xt = x.t().contiguous().t()
    assert torch.equal(ops.modulate(xt, sh, sc), want)
    assert torch.equal(ops.modulate(x.float(), sh, sc), ops.torch_modulate(x.float(), sh, sc))
    wide = rnd((2, 4104), 5)
    assert torch.equal(ops.modulate(wide, wide[:1], wide[1:]), ops.torch_modulate(wide, wide[:1], wide[1:]))
    assert torch.equal(torch.func.vmap(lambda r: ops.modulate(r, sh, sc))(x[None].contiguous())[0], want)
    _, tangent = torch.func.jvp(lambda r: ops.modulate(r, sh, sc), (x,), (dy,))
    assert tangent.shape == x.shape
    assert ops.gated_residual(x, sc[:, :1], x).shape == x.shape
    x1 = x.clone().requires_grad_(True)
    g, = torch.autograd.grad(ops.modulate(x1, sh, sc), x1, dy, create_graph=True)
    gg, = torch.autograd.grad(g.float().pow(2).sum(), x1)
    x2 = x.clone().requires_grad_(True)
    g2, = torch.autograd.grad(ops.torch_modulate(x2, sh, sc), x2, dy, create_graph=True)
    gg2, = torch.autograd.grad(g2.float().pow(2).sum(), x2)
    assert torch.equal(gg, gg2)


def test_cpu_tensors_run_as_torch_operations():
    x, sh, y = rnd((5, 48), 1, dev="cpu"), rnd((1, 48), 2, dev="cpu"), rnd((5, 48), 3, dev="cpu")
    assert torch.equal(ops.modulate(x, sh, sh), ops.torch_modulate(x, sh, sh))
    assert torch.equal(ops.gated_residual(x, sh, y), x + sh * y)
    cos, sin = tables(5, 16, "cpu")
    qn = torch.ones(16, dtype=BF)
    q, k, v = ops.joint_qkv(x[:2], x[2:], [(qn, qn), (qn, qn)], cos, sin, 1, 16)
    assert q.shape == k.shape == v.shape == (5, 1, 16)
    c = ops.single_stream_mix(rnd((5, 48 + 24), 4, dev="cpu"), qn, qn, cos, sin, 1, 16, 16, lambda q, k, v: v.reshape(5, 16))
    assert c.shape == (5, 16 + 24)
