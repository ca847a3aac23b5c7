"""Performance cases: the calls a program makes into this framework, with
their inputs, their cost and their 64-bit reference.

A case is one call of a public entry point (a linear layer, its GEMM or its
quantizer, in NVFP4 or MXFP4) or one denoiser block of the synthetic rollout
loop.  Sizes are those of the synthetic layers in ``workloads`` (one
1152-wide layer, SANA-, FLUX.1- and SD3.5-Large-like denoisers) plus generic
ragged ones.  ``draw`` gives further cases over the same ranges: 1 to 26574
tokens, layers 16 to 12288 wide, every block-aligned reduction length.
"""
import math

import torch

import paper_2604_06916_amd as sol
from paper_2604_06916_amd import stage1

DEV = "cuda"
MAX_TOKENS = 26574


def listed():
    return [
        # the smallest layer: 128 tokens through one 1152-wide linear, outputs
        # allocated by the call; its time is launches and latency
        dict(name="linear-128", call="linear", fmt="nvfp4", M=128, N=1152, K=1152,
             dist="outlier", bias=True, kept=False),
        # the same layer in MXFP4, with the output and workspace that a
        # sampling loop keeps
        dict(name="linear-128-mx", call="linear", fmt="mxfp4", M=128, N=1152, K=1152,
             dist="outlier", bias=True, kept=True),
        # the text stream of one SD3.5-like image: 333 tokens through QKV
        dict(name="text-333-qkv", call="linear", fmt="nvfp4", M=333, N=7296, K=2432,
             dist="rowscale", bias=True, kept=False),
        # sizes that are no multiple of any tile: odd token count and width,
        # a reduction length that is only a multiple of the 16-element block
        dict(name="ragged-777", call="linear", fmt="nvfp4", M=777, N=1235, K=1040,
             dist="normal", bias=True, kept=False),
        # one SANA-like 1024-token image through the MLP-up layer
        dict(name="image-1024-up", call="linear", fmt="nvfp4", M=1024, N=5600, K=2240,
             dist="heavy", bias=True, kept=True),
        # a group of 8 SANA-like rollouts through QKV (K % 128 == 64)
        dict(name="sana-qkv", call="linear", fmt="nvfp4", M=8192, N=6720, K=2240,
             dist="heavy", bias=True, kept=True),
        # the same group through the MXFP4 MLP-down layer (K % 128 == 96)
        dict(name="sana-down-mx", call="linear", fmt="mxfp4", M=8192, N=2240, K=5600,
             dist="heavy", bias=True, kept=True),
        # the largest GEMMs: 4 FLUX.1-like rollouts (18432 tokens) through QKV
        # in NVFP4 and through MLP-up in MXFP4, operands already packed
        dict(name="flux-qkv-gemm", call="gemm", fmt="nvfp4", M=18432, N=9216, K=3072,
             dist="normal", bias=True, kept=True),
        dict(name="flux-up-gemm-mx", call="gemm", fmt="mxfp4", M=18432, N=12288, K=3072,
             dist="normal", bias=True, kept=True),
        # activations quantized on the fly, as in front of every linear: the
        # FLUX.1-like hidden state (113 MB) in NVFP4, the SD3.5-like one in MXFP4
        dict(name="flux-quantize", call="quantize", fmt="nvfp4", M=18432, N=0, K=3072,
             dist="normal", bias=False, kept=True),
        dict(name="sd35-quantize-mx", call="quantize", fmt="mxfp4", M=MAX_TOKENS, N=0, K=2432,
             dist="rowscale", bias=False, kept=False),
        # one whole denoiser block (norms, four NVFP4 linears, BF16 attention,
        # GELU, residuals) on 2 rollouts of 4608 tokens, hidden 3072
        dict(name="block-nvfp4", call="block", fmt="nvfp4", M=2 * 4608, N=12288, K=3072,
             dist="normal", bias=True, kept=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


#: reduction lengths of the denoisers' layers
WIDTHS = (1152, 2240, 2432, 3072, 5600, 9728, 12288)


def draw(rng):
    fmt = rng.choice(("nvfp4", "nvfp4", "mxfp4"))
    call = rng.choice(("linear", "linear", "gemm", "quantize"))
    block = 16 if fmt == "nvfp4" else 32
    M = _log_uniform(rng, 1, MAX_TOKENS)
    K = rng.choice(WIDTHS) if rng.random() < 0.5 else \
        block * _log_uniform(rng, 64 // block, 12288 // block)
    N = 0
    if call != "quantize":
        N = _log_uniform(rng, 16, 12288) if rng.random() < 0.5 else rng.choice(WIDTHS)
        # no more work than the largest listed GEMM of the format
        most = 18432 * 3072 * (9216 if fmt == "nvfp4" else 12288)
        M = max(1, min(M, most // (N * K)))
    else:
        M = max(1, min(M, MAX_TOKENS * 2432 // K))
    return dict(call=call, fmt=fmt, M=M, N=N, K=K,
                dist=rng.choice(("normal", "outlier", "heavy", "rowscale", "gelu")),
                bias=call != "quantize" and rng.random() < 0.75, kept=rng.random() < 0.5)


# ---- inputs ---------------------------------------------------------------

def _generator(seed, role):
    return torch.Generator(device=DEV).manual_seed(1000 * int(seed) + role)


def _activations(case, seed):
    """BF16 activations with the denoisers' value distributions."""
    M, K, dist = case["M"], case["K"], case["dist"]
    g = _generator(seed, 1)
    x = torch.randn(M, K, device=DEV, generator=g)
    if dist == "outlier":            # 4 channels 20 times larger
        cols = torch.randperm(K, device=DEV, generator=g)[:4]
        x[:, cols] *= 20.0
    elif dist == "heavy":            # 1% of elements Student-t with 3 degrees of freedom
        pick = torch.rand(M, K, device=DEV, generator=g) < 0.01
        n = int(pick.sum())
        z = torch.randn(4, n, device=DEV, generator=g)
        x[pick] = z[0] / (z[1:].square().sum(0) / 3).sqrt()
    elif dist == "rowscale":         # per-token scale 10^U(-1, 1)
        x *= 10.0 ** (2.0 * torch.rand(M, 1, device=DEV, generator=g) - 1.0)
    elif dist == "gelu":             # the MLP-down layer's input
        x = torch.nn.functional.gelu(x)
    return x.to(torch.bfloat16)


def _weight(N, K, seed, role):
    g = _generator(seed, role)
    w = (0.02 * torch.randn(N, K, device=DEV, generator=g)).to(torch.bfloat16)
    b = (0.02 * torch.randn(N, device=DEV, generator=g)).to(torch.bfloat16)
    return w, b


def _block_model(case, seed):
    cfg = stage1.Stage1Config(blocks=1, hidden=case["K"], heads=case["K"] // 128, mlp=case["N"],
                              rollouts=case["M"] // 4608, tokens=4608, steps=1)
    model = [{name: _weight(N, K, seed, 10 + j)
              for j, (name, N, K) in enumerate(stage1.layer_shapes(cfg))}]
    return cfg, model


def prepare(case, seed):
    M, N, K, call, nv = case["M"], case["N"], case["K"], case["call"], case["fmt"] == "nvfp4"
    s = dict(case=case, x=_activations(case, seed))
    u8 = dict(dtype=torch.uint8, device=DEV)
    if call == "block":
        cfg, model = _block_model(case, seed)
        s["runner"] = stage1.Runner(cfg, model, case["fmt"], torch.device(DEV))
        return s
    if call == "quantize":
        # a program that quantizes into buffers it keeps
        s["out"] = {}
        if case["kept"]:
            s["out"] = dict(codes=torch.empty(M, K // 2, **u8),
                            scales=torch.empty(M, K // (16 if nv else 32), **u8))
            if nv:
                s["out"]["global_scale"] = torch.empty(1, device=DEV)
                s["out"]["workspace"] = torch.empty(sol.nvfp4_quantize_workspace_bytes(M, K), **u8)
        return s
    w, b = _weight(N, K, seed, 2)
    s["bias"] = b if case["bias"] else None
    s["w"] = sol.nvfp4_quantize(w) if nv else sol.mxfp4_quantize(w)
    s["out"] = {}
    if case["kept"]:
        s["out"]["out"] = torch.empty(M, N, dtype=torch.bfloat16, device=DEV)
    if call == "linear":
        if case["kept"]:
            need = sol.nvfp4_linear_workspace_bytes(M, N, K) if nv else \
                sol.mxfp4_linear_workspace_bytes(M, K)
            s["out"]["workspace"] = torch.empty(need, **u8)
    else:
        s["x"] = sol.nvfp4_quantize(s["x"]) if nv else sol.mxfp4_quantize(s["x"])
        if case["kept"] and nv:
            need = sol.nvfp4_gemm_workspace_bytes(M, N, K)
            if need:
                s["out"]["workspace"] = torch.empty(need, **u8)
    return s


def run(state):
    case = state["case"]
    call, nv = case["call"], case["fmt"] == "nvfp4"
    if call == "block":
        return state["runner"].blocks(state["x"])
    if call == "quantize":
        return (sol.nvfp4_quantize if nv else sol.mxfp4_quantize)(state["x"], **state["out"])
    if call == "linear":
        return (sol.nvfp4_linear if nv else sol.mxfp4_linear)(state["x"], *state["w"], state["bias"],
                                                             **state["out"])
    return (sol.nvfp4_gemm if nv else sol.mxfp4_gemm)(*state["x"], *state["w"], state["bias"],
                                                      **state["out"])


# ---- cost and tolerance ---------------------------------------------------

def _packed(rows, K, fmt):
    """Bytes of a packed [rows, K] operand: codes and block scales."""
    return rows * K * (0.5 + (1 / 16 if fmt == "nvfp4" else 1 / 32))


def work(case):
    M, N, K, fmt, call = case["M"], case["N"], case["K"], case["fmt"], case["call"]
    if call == "quantize":
        return {"bytes": 2 * M * K + _packed(M, K, fmt), "flops": 0}
    if call == "block":
        hidden, mlp = K, N
        shapes = ((3 * hidden, hidden), (hidden, hidden), (mlp, hidden), (hidden, mlp))
        flops = sum(2 * M * n * k for n, k in shapes) + 4 * M * 4608 * hidden
        return {"bytes": sum(_packed(n, k, fmt) for n, k in shapes) + 4 * M * hidden, "flops": flops}
    x = 2 * M * K if call == "linear" else _packed(M, K, fmt)
    return {"bytes": x + _packed(N, K, fmt) + 2 * M * N + (2 * N if case["bias"] else 0),
            "flops": 2 * M * N * K}


def tolerance(case):
    # codes, scales and alpha are defined bit for bit
    if case["call"] == "quantize":
        return "exact"
    # one block: a BF16 rounding that differs flips FP4 codes of every later
    # layer.  The block with its linears' FP32 sums in another order (two K
    # halves through torch) is 2.3e-3 away, single elements 0.22; the 64-bit
    # form, whose attention rounds elsewhere, 5.8e-2.
    if case["call"] == "block":
        return {"rel": 1e-2, "max": 0.9}
    # FP32 sums of exact products, one BF16 rounding: 1.66e-3 from the
    # 64-bit result, single elements 3.9e-3 (half a BF16 step)
    return {"rel": 6.6e-3, "max": 0.016}


# ---- the same in 64 bits --------------------------------------------------

def _f32(x):
    return x.float().double()


def _e2m1(y):
    """Magnitude nearest to |y| among 0, .5, 1, 1.5, 2, 3, 4, 6 with ties to
    the even code, and that code with the sign of y in bit 3."""
    a = y.abs()
    code = ((a > 0.25).to(torch.uint8) + (a >= 0.75) + (a > 1.25) + (a >= 1.75) + (a > 2.5)
            + (a >= 3.5) + (a > 5.0))
    table = torch.tensor([0, 0.5, 1, 1.5, 2, 3, 4, 6], dtype=torch.float64, device=y.device)
    value = table[code.long()]
    sign = torch.signbit(y)
    return torch.where(sign, -value, value), code + 8 * sign.to(torch.uint8)


def _nvfp4(x):
    """Decoded values (without alpha), codes, scale bytes and alpha of a BF16
    matrix: every step rounded to binary32, formed from 64-bit operations."""
    rows, K = x.shape
    b = x.double().view(rows, K // 16, 16)
    amax = b.abs().amax(-1)
    alpha = _f32(amax.max() / 2688.0)
    t = _f32(alpha * 6.0)
    s = _f32(amax / t) if alpha > 0 else torch.zeros_like(amax)
    s8 = s.clamp(max=448.0).float().to(torch.float8_e4m3fn)
    s = s8.double()
    d = _f32(s * alpha)
    r = torch.where(s > 0, _f32(1.0 / d), torch.zeros_like(d))
    q, codes = _e2m1(_f32(b * r.unsqueeze(-1)))
    return (q * s.unsqueeze(-1)).view(rows, K), codes.view(rows, K), s8.view(torch.uint8), alpha


def _mxfp4(x):
    rows, K = x.shape
    b = x.double().view(rows, K // 32, 32)
    amax = b.abs().amax(-1).to(torch.bfloat16)
    field = (amax.view(torch.int16).int() & 0x7FFF) >> 7
    byte = (field - 2).clamp(min=0)
    scale = ((byte.long() + (1023 - 127)) << 52).view(torch.float64)   # 2^(byte - 127)
    q, codes = _e2m1(b / scale.unsqueeze(-1))
    return (q * scale.unsqueeze(-1)).view(rows, K), codes.view(rows, K), byte.to(torch.uint8)


def _decoded(x, fmt):
    if fmt == "nvfp4":
        v, _, _, alpha = _nvfp4(x)
        return v, alpha
    return _mxfp4(x)[0], 1.0


def _linear(x, w, bias, fmt):
    (xv, xa), (wv, wa) = _decoded(x, fmt), _decoded(w, fmt)
    scale = xa * wa if fmt == "nvfp4" else 1.0
    out = torch.empty(x.shape[0], w.shape[0], dtype=torch.float64, device=x.device)
    for r in range(0, x.shape[0], 4096):
        out[r:r + 4096] = xv[r:r + 4096] @ wv.t() * scale
    return out if bias is None else out + bias.double()


def _block(case, seed):
    """The denoiser block, each stored tensor rounded to BF16."""
    cfg, model = _block_model(case, seed)
    L, bf = model[0], torch.bfloat16
    lin = lambda x, name: _linear(x, *L[name], case["fmt"]).to(bf)  # noqa: E731
    norm = lambda x: (x.double() / (x.double().square().mean(-1, keepdim=True) + 1e-6).sqrt()).to(bf)  # noqa: E731
    x = _activations(case, seed)
    qkv = lin(norm(x), "qkv").view(cfg.rollouts, cfg.tokens, 3, cfg.heads, 128)
    a = torch.empty(cfg.rollouts, cfg.tokens, cfg.heads, 128, dtype=bf, device=DEV)
    for r in range(cfg.rollouts):
        for h in range(cfg.heads):
            q, k, v = (qkv[r, :, i, h].double() for i in range(3))
            a[r, :, h] = (torch.softmax(q @ k.t().contiguous() / math.sqrt(128), -1) @ v).to(bf)
    x = (x.double() + lin(a.reshape(case["M"], cfg.hidden), "out").double()).to(bf)
    u = lin(norm(x), "up").double()
    u = (0.5 * u * (1 + torch.tanh(math.sqrt(2 / math.pi) * (u + 0.044715 * u ** 3)))).to(bf)
    return x.double() + lin(u, "down").double()


def exact(case, seed):
    if case["call"] == "block":
        return _block(case, seed)
    x = _activations(case, seed)
    if case["call"] == "quantize":
        if case["fmt"] == "nvfp4":
            _, codes, scales, alpha = _nvfp4(x)
        else:
            _, codes, scales = _mxfp4(x)
        packed = codes[:, 0::2] | (codes[:, 1::2] << 4)
        return (packed, scales, alpha.view(1)) if case["fmt"] == "nvfp4" else (packed, scales)
    w, b = _weight(case["N"], case["K"], seed, 2)
    return _linear(x, w, b if case["bias"] else None, case["fmt"])
