"""Performance cases of the W4A4G4 triple-branch layer on one MI355X.

Each case is one pass that a program built on this package makes, through its
public entry points: the C ABI's binding (`paper_2607_05711_amd._lib`) with
buffers and workspaces that the program keeps, or the modules of
`paper_2607_05711_amd.dit` through autograd.

Kinds:
  linear  one triple-branch linear through the ft_* calls: a training step
          (forward, input gradient, adapter gradients) or the forward alone
  mlp     the MLP pair with the fused GELU / dGELU epilogues, one training step
  quant   the gradient's quantization with a numerics variant
  block   one DiT block: single-stream forward and backward, or the forward
          alone of either kind

`exact` gives the same outputs in 64 bits from plain torch: the quantized
operands are inputs of the products as the method defines them, and the
values that the layer stores in bf16 are rounded to bf16 where it stores them.
"""
import math

import torch
import torch.nn.functional as F

from paper_2607_05711_amd import _lib, dit

DEV = "cuda:0"
BF, F32, F64, U8 = torch.bfloat16, torch.float32, torch.float64, torch.uint8


def _linear(name, M, K, N, r, rs, out="bf16", train=True):
    c = {"kind": "linear", "M": M, "K": K, "N": N, "r": r, "rs": rs, "out": out, "train": train}
    return dict(c, name=name) if name else c


def _mlp(name, M, D, W, r, rs):
    c = {"kind": "mlp", "M": M, "D": D, "W": W, "r": r, "rs": rs}
    return dict(c, name=name) if name else c


def _quant(name, M, N, R, stochastic, no_clip):
    c = {"kind": "quant", "M": M, "N": N, "R": R, "stochastic": stochastic, "no_clip": no_clip}
    return dict(c, name=name) if name else c


def _block(name, single, heads, img, txt, r, rs, train=True):
    c = {"kind": "block", "single": single, "heads": heads, "img": img, "txt": txt, "r": r, "rs": rs, "train": train}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest layer of the tests: adapter fine-tuning of a small layer, where launches and latency are all
        _linear("layer_tiny", 128, 256, 256, 16, 16),
        # FLUX.1-dev attention output projection over the 512 text tokens of a double block
        _linear("layer_text", 512, 3072, 3072, 32, 32),
        # FLUX.1-dev QKV projection, 4096 image + 512 text tokens: the headline layer
        _linear("layer_qkv", 4608, 3072, 9216, 32, 32),
        # single-stream block linears at batch 4, the largest layers
        _linear("layer_single_in", 18432, 3072, 21504, 64, 32),
        _linear("layer_single_out", 18432, 15360, 3072, 64, 32),
        # sampling with the tuned model: the forward alone, one single-stream input linear
        _linear("sample_single_in", 4608, 3072, 21504, 32, 32, train=False),
        # a layer of another model: odd token count, widths that are multiples of 32 only, results in 32 bits
        _linear("layer_ragged_f32", 1111, 2080, 3168, 24, 8, out="f32"),
        # FLUX.1-dev MLP pair over image and text tokens, and over the text tokens
        _mlp("mlp_image", 4608, 3072, 12288, 32, 32),
        _mlp("mlp_text", 512, 3072, 12288, 32, 32),
        # gradient quantization with stochastic rounding and the no-clip scale rule
        _quant("quant_stochastic", 4608, 9216, 64, True, True),
        # whole DiT blocks at 1024 x 1024: a single-stream block in training (38 of the model's 57), forward and
        # backward through autograd, and a double-stream block in sampling
        _block("block_single", True, 24, 4096, 512, 32, 32),
        _block("sample_block_double", False, 24, 4096, 512, 32, 32, train=False),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _width(rng, lo, hi):
    """A layer width: a multiple of 128 mostly (what models have), else of 32."""
    m = 128 if rng.random() < 0.7 else 32
    return max(m, int(round(_log(rng, lo, hi) / m)) * m)


def _ranks(rng, most):
    """(r, rs) with r + rs a multiple of 16, at most `most`."""
    R = 16 * rng.randint(2, most // 16)
    r = min(R - 8, rng.choice([8, 16, 24, 32, 64]))
    return r, R - r


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "sample", "mlp", "mlp", "quant", "block"])
    if kind in ("linear", "sample"):
        while True:
            M, K, N = int(_log(rng, 100, 18433)), _width(rng, 256, 15360), _width(rng, 256, 21504)
            if M * K * N <= 18432 * 3072 * 21504:
                break
        r, rs = _ranks(rng, 96)
        return _linear(None, M, K, N, r, rs, "f32" if rng.random() < 0.25 else "bf16", kind == "linear")
    if kind == "mlp":
        D = 128 * rng.randint(4, 24)
        r, rs = _ranks(rng, 64)
        return _mlp(None, int(_log(rng, 100, 4609)), D, 4 * D, r, rs)
    if kind == "quant":
        s, n = rng.choice([(True, True), (True, False), (False, True)])
        return _quant(None, int(_log(rng, 100, 4609)), _width(rng, 256, 12288), 16 * rng.randint(1, 6), s, n)
    r, rs = _ranks(rng, 64)
    single = rng.random() < 0.7
    return _block(None, single, rng.choice([8, 16, 24]), rng.randint(16, 64) ** 2, rng.randint(33, 512), r, rs,
                  single and rng.random() < 0.7)


# ------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 11)
    return g


def _normal(g, shape, std):
    return (torch.randn(shape, generator=g, device=DEV) * std).to(BF)


def _activations(g, M, K):
    """N(0, 1) with 0.5 % outlier channels x30."""
    x = torch.randn((M, K), generator=g, device=DEV)
    x[:, torch.randperm(K, generator=g, device=DEV)[:max(1, round(0.005 * K))]] *= 30.0
    return x.to(BF)


def _gradient(g, M, N):
    """Heavy-tailed: 1e-3 * Student-t with three degrees of freedom."""
    z = torch.randn((M, N), generator=g, device=DEV)
    chi = torch.zeros((M, N), device=DEV)
    for _ in range(3):
        chi += torch.randn((M, N), generator=g, device=DEV) ** 2
    return (1e-3 * z / torch.sqrt(chi / 3.0)).to(BF)


def _layer(g, K, N, R):
    """One layer's frozen weight (bf16, before its quantization), D = [L1 | A], U = [L2 ; B] and bias."""
    return {"W": _normal(g, (N, K), 0.02), "D": _normal(g, (K, R), 0.01), "U": _normal(g, (R, N), 0.01),
            "b": _normal(g, (N,), 0.02)}


def _draws(case, seed):
    g = _gen(seed)
    if case["kind"] == "linear":
        M, K, N, R = case["M"], case["K"], case["N"], case["r"] + case["rs"]
        d = {"l": _layer(g, K, N, R), "X": _activations(g, M, K)}
        if case["train"]:
            d["dY"] = _gradient(g, M, N)
        return d
    if case["kind"] == "mlp":
        M, D, W, R = case["M"], case["D"], case["W"], case["r"] + case["rs"]
        return {"l1": _layer(g, D, W, R), "l2": _layer(g, W, D, R), "X": _activations(g, M, D),
                "dY": _gradient(g, M, D)}
    return {"dY": _gradient(g, case["M"], case["N"]), "U": _normal(g, (case["R"], case["N"]), 0.01)}


def _quantized(l):
    """The layer as a program keeps it: weight codes and scales, factors, bias."""
    wq, ws, _ = _lib.ft_quantize_blockwise(l["W"], block_rows=32)
    return {"wq": wq, "ws": ws, "D": l["D"], "U": l["U"], "b": l["b"]}


def _buf(shape, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV)


def _space(n):
    return _buf((max(16, n),), U8)


def prepare(case, seed):
    if case["kind"] == "block":
        return _prepare_block(case, seed)
    s = dict(_draws(case, seed), case=case)
    if case["kind"] == "linear":
        M, K, N, r = case["M"], case["K"], case["N"], case["r"]
        R = r + case["rs"]
        y_t = F32 if case["out"] == "f32" else BF
        s["l"] = _quantized(s["l"])
        s.update(xq=_buf((M, K // 2), U8), xs=_buf((M, K // 32), U8), P=_buf((M, R), F32), y=_buf((M, N), y_t),
                 wx=_space(_lib.ft_quantize_workspace_size(M, K, 1, R, _lib.FT_PROJ_COLS_BY_R)))
        if case["train"]:
            s.update(gq=_buf((M, N // 2), U8), gs=_buf((M, N // 32), U8), Qp=_buf((M, R), F32), dx=_buf((M, K), y_t),
                     dA=_buf((K, r), F32), dB=_buf((r, N), F32),
                     wg=_space(_lib.ft_quantize_workspace_size(M, N, 1, R, _lib.FT_PROJ_R_BY_COLS)),
                     wl=_space(_lib.ft_lora_grads_workspace_size(M, K, N, R, r)))
    elif case["kind"] == "mlp":
        M, D, W, r = case["M"], case["D"], case["W"], case["r"]
        R = r + case["rs"]
        s["l1"], s["l2"] = _quantized(s["l1"]), _quantized(s["l2"])
        s.update(xq=_buf((M, D // 2), U8), xs=_buf((M, D // 32), U8), P1=_buf((M, R), F32), P2=_buf((M, R), F32),
                 z=_buf((M, W), BF), h=_buf((M, W), BF), hq=_buf((M, W // 2), U8), hs=_buf((M, W // 32), U8),
                 y=_buf((M, D), BF), gq=_buf((M, D // 2), U8), gs=_buf((M, D // 32), U8), Qp2=_buf((M, R), F32),
                 Qp1=_buf((M, R), F32), dz=_buf((M, W), BF), dzq=_buf((M, W // 2), U8), dzs=_buf((M, W // 32), U8),
                 dx=_buf((M, D), BF), dA1=_buf((D, r), F32), dB1=_buf((r, W), F32), dA2=_buf((W, r), F32),
                 dB2=_buf((r, D), F32),
                 wx=_space(_lib.ft_quantize_workspace_size(M, D, 1, R, _lib.FT_PROJ_COLS_BY_R)),
                 wg=_space(_lib.ft_quantize_workspace_size(M, D, 1, R, _lib.FT_PROJ_R_BY_COLS)),
                 wf=_space(_lib.ft_linear_fwd_gelu_workspace_size(M, W, R)),
                 wb=_space(_lib.ft_linear_bwd_input_dgelu_workspace_size(M, W, R)),
                 wl1=_space(_lib.ft_lora_grads_workspace_size(M, D, W, R, r)),
                 wl2=_space(_lib.ft_lora_grads_workspace_size(M, W, D, R, r)))
    else:
        M, N, R = case["M"], case["N"], case["R"]
        s.update(gq=_buf((M, N // 2), U8), gs=_buf((M, N // 32), U8), Qp=_buf((M, R), F32), seed=int(seed),
                 wg=_space(_lib.ft_quantize_workspace_size(M, N, 1, R, _lib.FT_PROJ_R_BY_COLS)))
    return s


def _config(case):
    H = 128 * case["heads"]
    return dit.DiTConfig(hidden=H, heads=case["heads"], mlp=4 * H, double_blocks=1, single_blocks=1,
                         img_tokens=case["img"], txt_tokens=case["txt"], lora_rank=case["r"], stab_rank=case["rs"])


def _linears(blk):
    return [(n, m) for n, m in blk.named_modules() if isinstance(m, dit.FourTuneLinear)]


def _prepare_block(case, seed):
    """A block in the middle of training or after it (its B factors are not zero), and what reaches it from both sides."""
    g, cfg = _gen(seed), _config(case)
    if case["single"]:
        blk = dit.SingleBlock(cfg, dit.FourTuneLinear, g, DEV)
    else:
        blk = dit.DoubleBlock(cfg, dit.FourTuneLinear, dit.FourTuneMLP, g, DEV)
    with torch.no_grad():
        for _, m in _linears(blk):
            m.B.normal_(0.0, 0.01, generator=g)
            m.sync()
    n = (cfg.txt_tokens + cfg.img_tokens,) if case["single"] else (cfg.img_tokens, cfg.txt_tokens)
    return {"case": case, "blk": blk, "rope": dit.rope_tables(cfg, DEV), "vec": _normal(g, (1, cfg.hidden), 1.0),
            "x": [_normal(g, (t, cfg.hidden), 1.0) for t in n],
            "dy": [_gradient(g, t, cfg.hidden) for t in n] if case["train"] else None}


# --------------------------------------------------------------------- pass
def run(s):
    return {"linear": _run_linear, "mlp": _run_mlp, "quant": _run_quant, "block": _run_block}[s["case"]["kind"]](s)


def _run_linear(s):
    c, l, L = s["case"], s["l"], _lib
    K = c["K"]
    L.ft_quantize_blockwise(s["X"], proj=l["D"], codes=s["xq"], scales=s["xs"], proj_out=s["P"], workspace=s["wx"])
    L.ft_linear_fwd(s["xq"], s["xs"], l["wq"], l["ws"], K, s["P"], l["U"], l["b"], y=s["y"])
    out = {k: s[k] for k in ("xq", "xs", "P", "y")}
    if c["train"]:
        L.ft_quantize_blockwise(s["dY"], proj=l["U"], proj_layout=L.FT_PROJ_R_BY_COLS, codes=s["gq"], scales=s["gs"],
                                proj_out=s["Qp"], workspace=s["wg"])
        L.ft_linear_bwd_input(s["gq"], s["gs"], l["wq"], l["ws"], K, s["Qp"], l["D"], dx=s["dx"])
        L.ft_lora_grads(s["X"], s["dY"], s["P"], s["Qp"], c["r"], col0=c["rs"], dA=s["dA"], dB=s["dB"],
                        workspace=s["wl"])
        out.update((k, s[k]) for k in ("gq", "gs", "Qp", "dx", "dA", "dB"))
    return out


def _run_mlp(s):
    c, l1, l2, L = s["case"], s["l1"], s["l2"], _lib
    D, W, r, rs = c["D"], c["W"], c["r"], c["rs"]
    L.ft_quantize_blockwise(s["X"], proj=l1["D"], codes=s["xq"], scales=s["xs"], proj_out=s["P1"], workspace=s["wx"])
    L.ft_linear_fwd_gelu(s["xq"], s["xs"], l1["wq"], l1["ws"], D, s["P1"], l1["U"], l1["b"], D2=l2["D"], z=s["z"],
                         h=s["h"], hq=s["hq"], hs=s["hs"], P2=s["P2"], workspace=s["wf"])
    L.ft_linear_fwd(s["hq"], s["hs"], l2["wq"], l2["ws"], W, s["P2"], l2["U"], l2["b"], y=s["y"])
    L.ft_quantize_blockwise(s["dY"], proj=l2["U"], proj_layout=L.FT_PROJ_R_BY_COLS, codes=s["gq"], scales=s["gs"],
                            proj_out=s["Qp2"], workspace=s["wg"])
    L.ft_linear_bwd_input_dgelu(s["gq"], s["gs"], l2["wq"], l2["ws"], W, s["z"], s["Qp2"], l2["D"], U1=l1["U"],
                                dz=s["dz"], dzq=s["dzq"], dzs=s["dzs"], Qp1=s["Qp1"], workspace=s["wb"])
    L.ft_linear_bwd_input(s["dzq"], s["dzs"], l1["wq"], l1["ws"], D, s["Qp1"], l1["D"], dx=s["dx"])
    L.ft_lora_grads(s["h"], s["dY"], s["P2"], s["Qp2"], r, col0=rs, dA=s["dA2"], dB=s["dB2"], workspace=s["wl2"])
    L.ft_lora_grads(s["X"], s["dz"], s["P1"], s["Qp1"], r, col0=rs, dA=s["dA1"], dB=s["dB1"], workspace=s["wl1"])
    return {k: s[k] for k in _MLP_OUT}


_MLP_OUT = ("xq", "xs", "P1", "z", "h", "hq", "hs", "P2", "y", "gq", "gs", "Qp2", "dz", "dzq", "dzs", "Qp1", "dx",
            "dA1", "dB1", "dA2", "dB2")


def _run_quant(s):
    c = s["case"]
    _lib.ft_quantize_blockwise_mode(
        s["dY"], proj=s["U"], proj_layout=_lib.FT_PROJ_R_BY_COLS, codes=s["gq"], scales=s["gs"], proj_out=s["Qp"],
        workspace=s["wg"], scale_rule=_lib.FT_SCALE_NO_CLIP if c["no_clip"] else _lib.FT_SCALE_FLOOR,
        rounding=_lib.FT_ROUND_STOCHASTIC if c["stochastic"] else _lib.FT_ROUND_NEAREST_EVEN, seed=s["seed"], stream=3)
    return {k: s[k] for k in ("gq", "gs", "Qp")}


def _run_block(s):
    blk, single = s["blk"], s["case"]["single"]
    if not s["case"]["train"]:
        with torch.no_grad():
            out = blk(*s["x"], s["vec"], s["rope"])
        return {"out": [out] if single else list(out)}
    for p in blk.parameters():
        p.grad = None
    x = [t.detach().requires_grad_(True) for t in s["x"]]
    out = blk(*x, s["vec"], s["rope"])
    out = [out] if single else list(out)
    torch.autograd.backward(out, s["dy"])
    return {"out": [t.detach() for t in out], "dx": [t.grad for t in x],
            "lora": {n: [m.A.grad, m.B.grad] for n, m in _linears(blk)}}


# --------------------------------------------------------------- what it takes
def work(case):
    if case["kind"] == "quant":
        M, N, R = case["M"], case["N"], case["R"]
        return {"bytes": M * N * (2 + 0.5 + 1 / 32) + 2 * R * N + 4 * M * R, "flops": 2.0 * M * N * R}
    if case["kind"] == "linear":
        M, K, N, r = case["M"], case["K"], case["N"], case["r"]
        R, o = r + case["rs"], 4 if case["out"] == "f32" else 2
        q = 0.5 + 1 / 32
        b = N * K * (0.5 + 1 / 1024) + 2 * R * (K + N) + 2 * N + M * K * (2 + q) + 4 * M * R + o * M * N
        f = 2.0 * M * N * K + 2.0 * M * R * (K + N)
        if case["train"]:
            b += M * N * (2 + q) + 4 * M * R + o * M * K + 4 * r * (K + N)
            f += 2.0 * M * N * K + 2.0 * M * R * (K + N) + 2.0 * r * M * (K + N)
        return {"bytes": b, "flops": f}
    if case["kind"] == "mlp":
        return _mlp_work(case["M"], case["D"], case["W"], case["r"], case["rs"])
    H, r, rs, L = 128 * case["heads"], case["r"], case["rs"], case["img"] + case["txt"]
    lin = [(H, 7 * H), (5 * H, H)] if case["single"] else [(H, 3 * H), (H, H), (H, 4 * H), (4 * H, H)]
    t = 1 if case["train"] else 0
    f = sum(2.0 * (1 + t) * L * K * N + (2.0 * (1 + t) * (r + rs) + 2.0 * t * r) * L * (K + N) for K, N in lin)
    f += (4.0 + 8.0 * t) * L * L * H                          # attention, forward and backward
    copies = 1 if case["single"] else 2                       # image and text weights
    b = copies * sum(K * N * (0.5 + 1 / 1024) + (2 * (r + rs) + 4 * t * r) * (K + N) for K, N in lin)
    b += (1 + t) * 2 * 2 * L * H
    return {"bytes": b, "flops": f}


def _mlp_work(M, D, W, r, rs):
    R, q = r + rs, 0.5 + 1 / 32
    b = 2 * D * W * (0.5 + 1 / 1024) + 2 * 2 * R * (D + W) + 2 * (D + W)
    b += M * D * (2 + q) + M * W * (2 + 2 + q) + 2 * M * D + 8 * M * R        # X, xq; z, h, hq; y; P1, P2
    b += M * D * (2 + q) + M * W * (2 + q) + 2 * M * D + 8 * M * R + 8 * r * (D + W)
    return {"bytes": b, "flops": 8.0 * M * D * W + 8.0 * M * R * (D + W) + 4.0 * r * M * (D + W)}


def tolerance(case):
    # Measured against exact() and against the same path with its sums in another order, times four: fp32 results
    # differ by their accumulation, the adapter gradients by the two-term split of their factors; bf16 results by
    # their rounding; codes of computed values by ties; a block's results by codes that move with a rounding before
    # (norms evaluated in 64 bits move a single-stream block's by 1.1e-3 and a double-stream block's, which is the
    # longer chain, by 1.1e-2).
    if case["kind"] == "quant":
        return {"rel": 2e-6, "max": 8e-5}
    if case["kind"] == "linear":
        return {"rel": 1e-5, "max": 4e-4} if case["out"] == "f32" else {"rel": 6e-3, "max": 3e-2}
    if case["kind"] == "mlp":
        return {"rel": 6e-3, "max": 0.3, "differ": 1e-3}
    return {"rel": 5e-3, "max": 0.6} if case["single"] else {"rel": 3e-2, "max": 0.9}


# -------------------------------------------------------------------- 64 bits
class _Rounded(torch.autograd.Function):
    """A value (and, on the way back, its gradient) stored in bf16."""

    @staticmethod
    def forward(ctx, x):
        return x.to(BF).to(F64)

    @staticmethod
    def backward(ctx, g):
        return g.to(BF).to(F64)


_bf = _Rounded.apply


def _pow2(e):
    return ((e.long() + 1023) << 52).view(F64)


def _mx(x):
    """MXFP4 values of x [rows, cols] in 1x32 blocks: a power-of-two scale from the block's largest magnitude and the
    nearest E2M1 value, ties to the even code, saturating."""
    return _mx_grid(x.to(F64).unflatten(1, (-1, 32)), (-1,)).flatten(1)


def _mx_tiles(w):
    t = w.to(F64).unflatten(1, (-1, 32)).unflatten(0, (-1, 32))          # [nb, 32, kb, 32]
    return _mx_grid(t, (1, 3)).flatten(2).flatten(0, 1)


def _mx_grid(t, dims):
    a = t.abs()
    _, e = torch.frexp(a.amax(dim=dims, keepdim=True))
    s = _pow2((e - 3).clamp(min=-127))
    a = a / s
    v = torch.zeros_like(a)
    for at, step, even in ((0.25, 0.5, 0), (0.75, 0.5, 1), (1.25, 0.5, 0), (1.75, 0.5, 1), (2.5, 1.0, 0), (3.5, 1.0, 1),
                           (5.0, 2.0, 0)):
        v += step * ((a >= at) if even else (a > at))
    return torch.copysign(v * s, t)


def _gelu(z):
    return F.gelu(z, approximate="tanh")


def _dgelu(z):
    with torch.enable_grad():
        z = z.detach().requires_grad_(True)
        return torch.autograd.grad(_gelu(z).sum(), z)[0]


def exact(case, seed):
    if case["kind"] == "block":
        return _exact_block(case, seed)
    d = _draws(case, seed)
    if case["kind"] == "quant":
        return {"gq": None, "gs": None, "Qp": d["dY"].to(F64) @ d["U"].to(F64).T}
    rs = case["rs"]
    if case["kind"] == "linear":
        l, X = {k: v.to(F64) for k, v in d["l"].items()}, d["X"].to(F64)
        W = _mx_tiles(l["W"])
        P = X @ l["D"]
        out = {"xq": None, "xs": None, "P": P, "y": _mx(X) @ W.T + P @ l["U"] + l["b"]}
        if case["train"]:
            dY = d["dY"].to(F64)
            Qp = dY @ l["U"].T
            out.update(gq=None, gs=None, Qp=Qp, dx=_mx(dY) @ W + Qp @ l["D"].T, dA=X.T @ Qp[:, rs:], dB=P[:, rs:].T @ dY)
        return out
    l1, l2 = ({k: v.to(F64) for k, v in d[n].items()} for n in ("l1", "l2"))
    W1, W2, X, dY = _mx_tiles(l1["W"]), _mx_tiles(l2["W"]), d["X"].to(F64), d["dY"].to(F64)
    P1 = X @ l1["D"]
    z = _bf(_mx(X) @ W1.T + P1 @ l1["U"] + l1["b"])
    h = _bf(_gelu(z))
    P2 = h @ l2["D"]
    Qp2 = dY @ l2["U"].T
    dz = _bf((_mx(dY) @ W2 + Qp2 @ l2["D"].T) * _dgelu(z))
    Qp1 = dz @ l1["U"].T
    got = {"P1": P1, "z": z, "h": h, "P2": P2, "y": _mx(h) @ W2.T + P2 @ l2["U"] + l2["b"], "Qp2": Qp2, "dz": dz,
           "Qp1": Qp1, "dx": _mx(dz) @ W1 + Qp1 @ l1["D"].T, "dA1": X.T @ Qp1[:, rs:], "dB1": P1[:, rs:].T @ dz,
           "dA2": h.T @ Qp2[:, rs:], "dB2": P2[:, rs:].T @ dY}
    return {k: got.get(k) for k in _MLP_OUT}


def _stored_weight(m):
    """The layer's frozen weight from its stored codes and 32x32 scales."""
    mag = torch.tensor([0, 0.5, 1, 1.5, 2, 3, 4, 6], dtype=F64, device=DEV)
    c = torch.stack([m.wq & 15, m.wq >> 4], -1).flatten(1).long()
    s = _pow2(m.ws.reshape(m.N // 32, m.K // 32).int() - 127).repeat_interleave(32, 0).repeat_interleave(32, 1)
    return torch.where(c >= 8, -mag[c & 7], mag[c & 7]) * s


class _Linear64(torch.autograd.Function):
    """The triple-branch linear in 64 bits: quantized operands, adapter gradients from the unquantized ones."""

    @staticmethod
    def forward(ctx, x, A, B, W, D, U, b, rs):
        ctx.save_for_backward(x, W, D, U)
        ctx.rs = rs
        return _mx(x) @ W.T + (x @ D) @ U + b

    @staticmethod
    def backward(ctx, dy):
        x, W, D, U = ctx.saved_tensors
        Qp, rs = dy @ U.T, ctx.rs
        return _mx(dy) @ W + Qp @ D.T, x.T @ Qp[:, rs:], (x @ D)[:, rs:].T @ dy, None, None, None, None, None


def _norm64(x):
    return F.layer_norm(x, (x.shape[-1],), eps=1e-6)


def _heads64(x, w, rope):
    x = _bf(x * torch.rsqrt(x.pow(2).mean(-1, keepdim=True) + 1e-6) * w.to(F64))
    x = x.unflatten(-1, (-1, 2))
    cos, sin = (t.to(F64) for t in rope)
    return _bf(torch.stack([x[..., 0] * cos - x[..., 1] * sin, x[..., 0] * sin + x[..., 1] * cos], -1).flatten(-2))


def _attention64(q, k, v):
    return _bf(torch.cat([torch.softmax(q[:, i] @ k[:, i].T * q.shape[-1] ** -0.5, -1) @ v[:, i]
                          for i in range(q.shape[1])], -1))


def _exact_block(case, seed):
    s = _prepare_block(case, seed)
    blk, cfg = s["blk"], _config(case)
    H, hd = cfg.heads, cfg.head_dim
    leaves = {}

    def linear(name, x):
        m = dict(_linears(blk))[name]
        leaves[name] = [m.A.detach().to(F64).requires_grad_(True), m.B.detach().to(F64).requires_grad_(True)]
        return _bf(_Linear64.apply(x, *leaves[name], _stored_weight(m), m.D.to(F64), m.U.to(F64), m.bias.to(F64), m.rs))

    x = [t.to(F64).requires_grad_(True) for t in s["x"]]
    if case["single"]:
        sh, sc, gate = _bf(_bf(F.silu(s["vec"].to(F64))) @ blk.mod.to(F64)).chunk(3, -1)
        a = linear("linear1", _bf(_norm64(x[0]) * (1.0 + sc) + sh))
        q, k, v = a[:, :3 * cfg.hidden].reshape(-1, 3, H, hd).unbind(1)
        o = _attention64(_heads64(q, blk.qn, s["rope"]), _heads64(k, blk.kn, s["rope"]), v)
        y = linear("linear2", torch.cat([o, _bf(_gelu(a[:, 3 * cfg.hidden:]))], -1))
        out = [_bf(x[0] + _bf(gate * y))]
    else:
        mods, qkv, out, T = {}, {}, {}, cfg.txt_tokens
        cos, sin = s["rope"]
        part = {"txt": (cos[:T], sin[:T]), "img": (cos[T:], sin[T:])}
        for n, t in (("img", x[0]), ("txt", x[1])):
            mods[n] = _bf(_bf(F.silu(s["vec"].to(F64))) @ blk.mod[n].to(F64)).chunk(6, -1)
            a = linear("qkv." + n, _bf(_norm64(t) * (1.0 + mods[n][1]) + mods[n][0]))
            q, k, v = a.reshape(-1, 3, H, hd).unbind(1)
            qkv[n] = _heads64(q, blk.qn[n], part[n]), _heads64(k, blk.kn[n], part[n]), v
        o = _attention64(*(torch.cat([qkv["txt"][i], qkv["img"][i]], 0) for i in range(3)))
        for n, t, att in (("img", x[0], o[T:]), ("txt", x[1], o[:T])):
            _, _, g1, sh2, sc2, g2 = mods[n]
            t = _bf(t + _bf(g1 * linear("out." + n, att)))
            h = _bf(_gelu(linear("mlp.%s.fc1" % n, _bf(_norm64(t) * (1.0 + sc2) + sh2))))
            out[n] = _bf(t + _bf(g2 * linear("mlp.%s.fc2" % n, h)))
        out = [out["img"], out["txt"]]
    if not case["train"]:
        return {"out": [t.detach() for t in out]}
    torch.autograd.backward(out, [t.to(F64) for t in s["dy"]])
    return {"out": [t.detach() for t in out], "dx": [t.grad for t in x],
            "lora": {n: [t.grad for t in leaves[n]] for n, _ in _linears(blk)}}
