"""The DiT block's work between its linears on kernels of the library
(csrc/dit_ops.hip, csrc/attention.hip), as autograd functions, and the torch operations they stand for.

Each public function here takes the fused path when its inputs are what the
kernels hold (contiguous bf16 on one GPU, widths in range, modulation, norm
weights and rotary tables without gradients) and nothing traces or transforms
the call; every other call, on any device or type, runs the torch operations.
A backward that is itself differentiated runs them too.
"""
import ctypes

import torch
import torch.nn.functional as F

from . import _lib

BF = torch.bfloat16
EPS = 1e-6

_P, _I = ctypes.c_void_p, ctypes.c_int64
_SIGNATURES = {
    "ftdit_modulate": [_P, _P, _P, _P, _I, _I, _P],
    "ftdit_modulate_bwd": [_P, _P, _P, _P, _I, _I, _P],
    "ftdit_qkv": [_P] + [_I] * 6 + [_P] * 8 + [_P],
    "ftdit_qkv_bwd": [_P] + [_I] * 6 + [_P] * 4 + [_P, _I, _I] * 3 + [_P, _P, _P],
    "ftdit_mod": [_P, _P, _P, _P, _I, _I, _P],
    "ftdit_gate": [_P, _P, _P, _P, _I, _I, _P],
    "ftdit_attn_fwd": [_I, _I] + [_P, _I, _I] * 3 + [_P, _I, _P, _P],
    "ftdit_attn_bwd": [_I, _I] + [_P, _I, _I] * 4 + [_P, _I] + [_P] * 6,
}
_ready = None


def _load():
    global _ready
    if _ready is None:
        L = _lib.load()
        for n, sig in _SIGNATURES.items():
            getattr(L, n).argtypes = sig
            getattr(L, n).restype = ctypes.c_int
        L.ftdit_mod_parts.argtypes, L.ftdit_mod_parts.restype = [_I, _I], _I
        _ready = L
    return _ready


def _call(name, dev, *args):
    f = getattr(_load(), name)
    args = [a.data_ptr() if isinstance(a, torch.Tensor) else a for a in args]
    if torch.cuda.current_device() != dev.index:
        with torch.cuda.device(dev):
            status = f(*args, _lib._stream(dev))
    else:
        status = f(*args, _lib._stream(dev))
    if status != _lib.FT_OK:
        raise _lib.FourTuneError(status, name)


# --------------------------------------------------------- which calls fuse
def _untraced():
    """No compiler, functional transform, forward-mode level or dispatch mode sees this call."""
    return not (torch.compiler.is_compiling() or torch.jit.is_tracing() or
                torch._C._functorch.peek_interpreter_stack() is not None or
                torch.autograd.forward_ad._current_level >= 0 or
                torch._C._len_torch_dispatch_stack() > 0 or torch._C._len_torch_function_stack() > 0)


def _plain(dtype, dev, *tensors):
    """Ordinary contiguous, 16-byte aligned tensors of this type on this GPU."""
    for t in tensors:
        if type(t) not in (torch.Tensor, torch.nn.Parameter) or t.dtype != dtype or t.device != dev or \
                not t.is_contiguous() or t.data_ptr() % 16:
            return False
    return True


def _constant(*tensors):
    return not (torch.is_grad_enabled() and any(t.requires_grad for t in tensors))


def _row(t, x):
    """A [H] or [1, H] vector that broadcasts over the rows of x without changing its shape."""
    return t.numel() == x.shape[-1] == t.shape[-1] and t.dim() <= x.dim()


# ---------------------------------------------------------- torch operations
def layer_norm(x):
    return F.layer_norm(x.float(), (x.shape[-1],), eps=EPS)


def torch_modulate(x, shift, scale):
    return (layer_norm(x) * (1.0 + scale.float()) + shift.float()).to(BF)


def rms_norm(x, w):
    xf = x.float()
    return (xf * torch.rsqrt(xf.pow(2).mean(-1, keepdim=True) + EPS) * w.float()).to(BF)


def rope(x, cos, sin):
    """Rotary embedding on consecutive pairs of the head dimension:
    x [tokens, heads, head_dim]; cos, sin [tokens, 1, head_dim / 2]."""
    xf = x.float().unflatten(-1, (-1, 2))
    x0, x1 = xf[..., 0], xf[..., 1]
    return torch.stack([x0 * cos - x1 * sin, x0 * sin + x1 * cos], -1).flatten(-2).to(BF)


def torch_joint_qkv(txt, img, norms, cos, sin, heads, hd):
    parts = []
    for x, (qn, kn) in ((txt, norms[0]), (img, norms[1])):
        q, k, v = x.view(-1, 3, heads, hd).unbind(1)
        parts.append((rms_norm(q, qn), rms_norm(k, kn), v))
    q, k, v = (torch.cat([parts[0][i], parts[1][i]], 0) for i in range(3))
    return rope(q, cos, sin), rope(k, cos, sin), v


def torch_qkv_gelu(h, qn, kn, cos, sin, heads, hd, hidden):
    qkv, mlp = h.split([3 * hidden, h.shape[-1] - 3 * hidden], -1)
    q, k, v = qkv.reshape(-1, 3, heads, hd).unbind(1)
    return rope(rms_norm(q, qn), cos, sin), rope(rms_norm(k, kn), cos, sin), v, F.gelu(mlp, approximate="tanh")


# ------------------------------------------------------ LayerNorm + modulation
class _Modulate(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, shift, scale):
        out = torch.empty_like(x)
        H = x.shape[-1]
        _call("ftdit_modulate", x.device, x, shift, scale, out, x.numel() // H, H)
        ctx.save_for_backward(x, scale)
        return out

    @staticmethod
    def backward(ctx, dy):
        x, scale = ctx.saved_tensors
        if torch.is_grad_enabled():
            return torch.autograd.grad(torch_modulate(x, torch.zeros_like(scale), scale), x, dy, create_graph=True)[0], None, None
        dy = _aligned(dy)
        dx = torch.empty_like(x)
        H = x.shape[-1]
        _call("ftdit_modulate_bwd", x.device, x, scale, dy, dx, x.numel() // H, H)
        return dx, None, None


def _aligned(t):
    t = t.contiguous()
    return t if t.data_ptr() % 16 == 0 else t.clone()


def modulate(x, shift, scale):
    """bf16(LayerNorm(x) (1 + scale) + shift) over the last dimension, no affine weights."""
    if _untraced() and x.is_cuda and x.numel() and x.shape[-1] % 8 == 0 and x.shape[-1] <= 4096 and \
            _plain(BF, x.device, x, shift, scale) and _row(shift, x) and _row(scale, x) and _constant(shift, scale):
        return _Modulate.apply(x, shift, scale)
    return torch_modulate(x, shift, scale)


# ----------------------------------------------------------- modulation vector
def modulation(vec, w):
    """silu(vec) @ w: the block's shift, scale and gate vectors."""
    if vec.is_cuda and _untraced() and vec.dim() > 0 and w.dim() == 2 and 0 < vec.numel() == vec.shape[-1] == w.shape[0] < 1 << 20 and \
            0 < w.shape[1] < 1 << 24 and w.shape[1] % 8 == 0 and _plain(BF, vec.device, vec, w) and _constant(vec, w) and \
            not torch.is_autocast_enabled("cuda"):
        out = torch.empty(vec.shape[:-1] + w.shape[1:], dtype=BF, device=vec.device)
        K, N = w.shape
        parts = torch.empty((_load().ftdit_mod_parts(K, N), N), dtype=torch.float32, device=vec.device)
        _call("ftdit_mod", vec.device, vec, w, out, parts, K, N)
        return out
    return F.silu(vec) @ w


# ------------------------------------------------------------- gated residual
def _gate(x, gate, y):
    out = torch.empty_like(y)
    H = y.shape[-1]
    _call("ftdit_gate", y.device, x, gate, y, out, y.numel() // H, H)
    return out


class _Gate(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, gate, y):
        ctx.save_for_backward(gate)
        return _gate(x, gate, y)

    @staticmethod
    def backward(ctx, dout):
        gate, = ctx.saved_tensors
        if torch.is_grad_enabled():
            return dout, None, dout * gate
        return dout, None, _gate(None, gate, _aligned(dout)) if ctx.needs_input_grad[2] else None


def gated_residual(x, gate, y):
    """x + gate * y, the product rounded to bf16 before the sum."""
    if _untraced() and x.is_cuda and x.numel() and x.shape == y.shape and x.shape[-1] % 8 == 0 and \
            x.shape[-1] < 1 << 24 and _plain(BF, x.device, x, gate, y) and _row(gate, x) and _constant(gate):
        # (without gradients an autograd function is 4 us of a small call's time)
        return _gate(x, gate, y) if _constant(x, y) else _Gate.apply(x, gate, y)
    return x + gate * y


# --------------------------------------------------------------- q, k, v, GELU
def _in_reach(rows, stride):
    """Whether the kernels' 32-bit offsets hold this many rows (and a stage past them) of this stride."""
    return (rows + 63) * stride * 2 + 256 < 1 << 31


def _strided(t):
    """A [rows, heads, head_dim] gradient the backward kernels can read (unit stride within a head)."""
    if t.stride(-1) != 1 or t.stride(0) % 8 or t.stride(1) % 8 or t.data_ptr() % 16 or not _in_reach(t.shape[0], t.stride(0)):
        t = t.clone(memory_format=torch.contiguous_format)
    return t


def _qkv_bwd(h, row0, heads, F_, qn, kn, cos, sin, dq, dk, dv, dc, dh):
    args = []
    for t in (dq, dk, dv):
        args += [t, t.stride(0), t.stride(1)]
    _call("ftdit_qkv_bwd", h.device, h, h.shape[0], h.shape[1], row0, heads, qn.numel(), F_, qn, kn, cos, sin, *args, dc, dh)


class _JointQkv(torch.autograd.Function):
    """q, k, v [txt + img tokens, heads, head_dim] of the two streams' fused projections."""

    @staticmethod
    def forward(ctx, txt, img, qn_t, kn_t, qn_i, kn_i, cos, sin, heads):
        T, hd, H = txt.shape[0] + img.shape[0], qn_t.numel(), txt.shape[1] // 3
        q, k, v = (torch.empty((T, heads, hd), dtype=BF, device=txt.device) for _ in range(3))
        for x, row0, qn, kn in ((txt, 0, qn_t, kn_t), (img, txt.shape[0], qn_i, kn_i)):
            _call("ftdit_qkv", x.device, x, x.shape[0], 3 * H, row0, heads, hd, 0, qn, kn, cos, sin, q, k, v, None)
        ctx.save_for_backward(txt, img, qn_t, kn_t, qn_i, kn_i, cos, sin)
        ctx.heads = heads
        return q, k, v

    @staticmethod
    def backward(ctx, dq, dk, dv):
        txt, img, qn_t, kn_t, qn_i, kn_i, cos, sin = ctx.saved_tensors
        if torch.is_grad_enabled():
            out = torch_joint_qkv(txt, img, ((qn_t, kn_t), (qn_i, kn_i)), cos, sin, ctx.heads, qn_t.numel())
            need = [t for t, n in zip((txt, img), ctx.needs_input_grad) if n]
            d = list(torch.autograd.grad(out, need, (dq, dk, dv), create_graph=True))
            return tuple(d.pop(0) if n else None for n in ctx.needs_input_grad[:2]) + (None,) * 7
        dq, dk, dv = _strided(dq), _strided(dk), _strided(dv)
        got = []
        for x, row0, qn, kn, need in ((txt, 0, qn_t, kn_t, ctx.needs_input_grad[0]),
                                      (img, txt.shape[0], qn_i, kn_i, ctx.needs_input_grad[1])):
            dx = torch.empty_like(x) if need else None
            if need:
                _qkv_bwd(x, row0, ctx.heads, 0, qn, kn, cos, sin, dq, dk, dv, None, dx)
            got.append(dx)
        return (*got, None, None, None, None, None, None, None)


def _heads_ok(hd, rows, cos, sin, norms, dev):
    return 8 <= hd <= 512 and hd & (hd - 1) == 0 and _plain(BF, dev, *norms) and all(n.shape == (hd,) for n in norms) and \
        _plain(torch.float32, dev, cos, sin) and cos.shape == sin.shape == (rows, 1, hd // 2)


def joint_qkv(txt, img, norms, cos, sin, heads, hd):
    """The joint attention's q, k (normalized and rotated) and v [txt + img tokens, heads, head_dim] from the streams'
    projections [tokens, 3 hidden]; norms: (q, k) weights of text and image."""
    (qn_t, kn_t), (qn_i, kn_i) = norms
    if _untraced() and txt.is_cuda and txt.dim() == img.dim() == 2 and txt.shape[0] and img.shape[0] and \
            txt.shape[1] == img.shape[1] == 3 * heads * hd and 0 < heads * hd < 1 << 20 and \
            _plain(BF, txt.device, txt, img) and \
            _heads_ok(hd, txt.shape[0] + img.shape[0], cos, sin, (qn_t, kn_t, qn_i, kn_i), txt.device) and \
            _constant(qn_t, kn_t, qn_i, kn_i, cos, sin):
        return _JointQkv.apply(txt, img, qn_t, kn_t, qn_i, kn_i, cos, sin, heads)
    return torch_joint_qkv(txt, img, norms, cos, sin, heads, hd)


class _QkvGelu(torch.autograd.Function):
    """q, k, v of the single-stream block's fused projection h [T, 3H + F], and the output linear's input [T, H + F]
    with GELU of the MLP part in its place (its first H columns are written later)."""

    @staticmethod
    def forward(ctx, h, qn, kn, cos, sin, heads, H):
        T, hd, F_ = h.shape[0], H // heads, h.shape[1] - 3 * H
        q, k = (torch.empty((T, heads, hd), dtype=BF, device=h.device) for _ in range(2))
        c = torch.empty((T, H + F_), dtype=BF, device=h.device)
        _call("ftdit_qkv", h.device, h, T, h.shape[1], 0, heads, hd, F_, qn, kn, cos, sin, q, k, None, c)
        ctx.save_for_backward(h, qn, kn, cos, sin)
        ctx.heads, ctx.H = heads, H
        return q, k, h.detach()[:, 2 * H:3 * H].view(T, heads, hd), c

    @staticmethod
    def backward(ctx, dq, dk, dv, dc):
        h, qn, kn, cos, sin = ctx.saved_tensors
        H = ctx.H
        if torch.is_grad_enabled():
            out = torch_qkv_gelu(h, qn, kn, cos, sin, ctx.heads, qn.numel(), H)
            return (torch.autograd.grad(out, h, (dq, dk, dv, dc[:, H:]), create_graph=True)[0],) + (None,) * 6
        dh = torch.empty_like(h)
        _qkv_bwd(h, 0, ctx.heads, h.shape[1] - 3 * H, qn, kn, cos, sin, _strided(dq), _strided(dk), _strided(dv),
                 _aligned(dc), dh)
        return (dh,) + (None,) * 6


# ------------------------------------------------------------------- attention
def _rows(t):
    """(pointer, token stride, head stride) of a [tokens, heads, 128] tensor."""
    return t, t.stride(0), t.stride(1)


def _attention_ok(*qkv):
    q = qkv[0]
    # contiguous gradients are in reach too; autocast to another type would convert q, k and v
    if not (_untraced() and q.is_cuda and q.dim() == 3 and q.numel() and q.shape[2] == 128 and
            q.shape[0] * q.shape[1] < 1 << 27 and _in_reach(q.shape[0], q.shape[1] * 128) and
            not (torch.is_autocast_enabled("cuda") and torch.get_autocast_dtype("cuda") is not BF)):
        return False
    for t in qkv:
        if type(t) is not torch.Tensor or t.dtype != BF or t.device != q.device or t.shape != q.shape or \
                t.stride(2) != 1 or t.stride(0) % 8 or t.stride(1) % 8 or t.data_ptr() % 16 or \
                not _in_reach(q.shape[0], t.stride(0)):
            return False
    return True


class _Attention(torch.autograd.Function):
    """softmax(q k^T / sqrt(128)) v over all tokens into the first columns of c [tokens, >= heads * 128]."""

    @staticmethod
    def forward(ctx, c, q, k, v):
        L, heads, _ = q.shape
        lse = torch.empty((heads, L), dtype=torch.float32, device=q.device)
        _call("ftdit_attn_fwd", q.device, L, heads, *_rows(q), *_rows(k), *_rows(v), c, c.stride(0), lse)
        ctx.mark_dirty(c)
        ctx.save_for_backward(c, q, k, v, lse)
        return c

    @staticmethod
    @torch.autograd.function.once_differentiable
    def backward(ctx, dc):
        c, q, k, v, lse = ctx.saved_tensors
        L, heads, hd = q.shape
        g = dc[:, :heads * hd].view(L, heads, hd) if dc.stride(1) == 1 else dc[:, :heads * hd].reshape(L, heads, hd)
        g = _strided(g)
        dq, dk, dv = (torch.empty((L, heads, hd), dtype=BF, device=q.device) for _ in range(3))
        delta = torch.empty_like(lse)
        _call("ftdit_attn_bwd", q.device, L, heads, *_rows(q), *_rows(k), *_rows(v), *_rows(g), c, c.stride(0), lse, delta,
              dq, dk, dv)
        return dc if ctx.needs_input_grad[0] else None, dq, dk, dv


def torch_attention(q, k, v):
    """Fused attention kernels only (no unfused matmul fallback)."""
    from torch.nn.attention import SDPBackend, sdpa_kernel
    q, k, v = (t.transpose(0, 1).unsqueeze(0) for t in (q, k, v))     # [1, heads, L, hd]
    with sdpa_kernel([SDPBackend.FLASH_ATTENTION, SDPBackend.EFFICIENT_ATTENTION]):
        o = F.scaled_dot_product_attention(q, k, v)
    return o.squeeze(0).transpose(0, 1).reshape(q.shape[2], -1)


def attention(q, k, v):
    """Joint attention over all tokens; q, k, v [L, heads, head_dim] bf16; returns [L, heads * head_dim]."""
    if _attention_ok(q, k, v):
        c = torch.empty((q.shape[0], q.shape[1] * q.shape[2]), dtype=BF, device=q.device)
        return _Attention.apply(c, q, k, v)
    return torch_attention(q, k, v)


class _FillLeft(torch.autograd.Function):
    """c with o in its first columns (in place: they held nothing)."""

    @staticmethod
    def forward(ctx, c, o):
        ctx.width = o.shape[1]
        c[:, :ctx.width].copy_(o)
        ctx.mark_dirty(c)
        return c

    @staticmethod
    def backward(ctx, dc):
        return dc, dc[:, :ctx.width]


def single_stream_mix(h, qn, kn, cos, sin, heads, hd, hidden, mix=attention):
    """The single-stream block between its linears: [mix(q, k, v) | GELU(mlp)] of h [T, 3 hidden + mlp]."""
    if _untraced() and h.is_cuda and h.dim() == 2 and h.shape[0] and 3 * hidden < h.shape[1] < 1 << 24 and \
            h.shape[1] % 8 == 0 and hidden == heads * hd < 1 << 20 and _plain(BF, h.device, h) and \
            _heads_ok(hd, h.shape[0], cos, sin, (qn, kn), h.device) and _constant(qn, kn, cos, sin):
        q, k, v, c = _QkvGelu.apply(h, qn, kn, cos, sin, heads, hidden)
        if mix is attention and _attention_ok(q, k, v):
            return _Attention.apply(c, q, k, v)
        o = mix(q, k, v)
        return _FillLeft.apply(c, o) if o.dtype == BF else torch.cat([o, c[:, hidden:]], -1)
    q, k, v, m = torch_qkv_gelu(h, qn, kn, cos, sin, heads, hd, hidden)
    return torch.cat([mix(q, k, v), m], -1)
