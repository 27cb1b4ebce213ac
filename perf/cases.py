"""The work a user of this framework has it do, as cases that can be timed and compared.

Each case is one pass through the public binding (``paper_2608_27370_amd.puro``)
as a training or serving program makes it: buffers that such a program keeps
(workspaces, saved state, outputs of a training step) are made in ``prepare``,
everything the call itself does is in ``run``. Kinds:

* ``gemm``    -- serving: quantise an activation of any number of rows and
  multiply it by a weight quantised once, with bias and/or residual.
* ``linear``  -- the FP8 linear layer, forward and (``bwd``) backward, per-tensor
  or blockwise, with kept buffers.
* ``module``  -- ``puro.Linear`` under autograd, gradient into ``main_grad``.
* ``rmsnorm`` -- RMSNorm fused with the quantisation of the projection's input.
* ``swiglu``  -- SwiGLU fused with the down projection's input quantisation, and
  its backward fused with the gate/up projection's gradient quantisation.
* ``lm_head`` -- LM head with cross-entropy, forward and backward.
* ``muonh``   -- one MuonH optimiser step of a batch of matrices.

Values follow the distributions the framework's own workloads state: N(0, 1)
activations with 1% outlier channels x20, N(0, 0.02^2) weights, N(0, 1e-3^2)
gradients, Student-t(3) hidden states at the LM head.
"""

import math

import torch

from paper_2608_27370_amd import puro

G = 128


def listed():
    return [
        # a short batch of decode-time tokens through the QKV projection (its
        # weight quantised once), with the bias: the smallest call, an odd
        # number of rows
        dict(name="serve_qkv_77", kind="gemm", M=77, N=2048, K=1536, bias=True, residual=False),
        # the single forward of the Qwen2-1.5B hidden size, per-tensor
        dict(name="linear_fwd_256", kind="linear", M=256, N=1536, K=1536, blockwise=False, dy="e5m2", bwd=False),
        # a torch module in a small training step, blockwise, ragged against
        # every tile
        dict(name="module_step_1152", kind="module", M=1152, N=2944, K=1664),
        # per-tensor QKV projection of one 8192-token micro-batch, E5M2 gradients
        dict(name="qkv_tensor_8192", kind="linear", M=8192, N=2048, K=1536, blockwise=False, dy="e5m2", bwd=True),
        # the paper's blockwise recipe at two micro-batches: the widest and the
        # deepest linear of a Qwen2-1.5B layer
        dict(name="gate_up_block_16384", kind="linear", M=16384, N=17920, K=1536, blockwise=True, dy="e4m3", bwd=True),
        dict(name="down_block_16384", kind="linear", M=16384, N=1536, K=8960, blockwise=True, dy="e4m3", bwd=True),
        # prefill of an odd-length prompt through the O projection, into the
        # residual stream
        dict(name="serve_o_3001", kind="gemm", M=3001, N=2056, K=2064, bias=False, residual=True),
        # the memory-bound ops around the linears
        dict(name="rmsnorm_block_8192", kind="rmsnorm", M=8192, K=1536, blockwise=True),
        dict(name="swiglu_block_8192", kind="swiglu", M=8192, K=8960, blockwise=True),
        # the LM head: the full Qwen2 vocabulary in BF16, and a smaller
        # vocabulary with ragged tiles in blockwise FP8
        dict(name="lm_head_bf16_8192", kind="lm_head", M=8192, V=151936, K=1536, fp8=False),
        dict(name="lm_head_fp8_3968", kind="lm_head", M=3968, V=50304, K=2048, fp8=True),
        # the optimiser step of the 28 layers' QKV matrices
        dict(name="muonh_qkv_28", kind="muonh", count=28, rows=2048, cols=1536),
    ]


def _log(rng, lo, hi, step=1):
    """A size between lo and hi, even over its logarithm, a multiple of step."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(-(-lo // step) * step, min(hi // step * step, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choice(["gemm", "linear", "linear", "module", "rmsnorm", "swiglu", "lm_head", "muonh"])
    if kind == "gemm":
        bias = rng.random() < 0.5
        return dict(kind=kind, M=_log(rng, 16, 8192), N=_log(rng, 512, 8192, 8), K=_log(rng, 512, 8192, 16),
                    bias=bias, residual=not bias or rng.random() < 0.3)
    if kind == "linear":
        block = rng.random() < 0.6
        s = G if block else 16
        return dict(kind=kind, M=_log(rng, 256, 16384, s), N=_log(rng, 1024, 18432, s), K=_log(rng, 1024, 9216, s),
                    blockwise=block, dy="e4m3" if block or rng.random() < 0.3 else "e5m2", bwd=rng.random() < 0.75)
    if kind == "module":
        return dict(kind=kind, M=_log(rng, 256, 8192, G), N=_log(rng, 1024, 8192, G), K=_log(rng, 1024, 8192, G))
    if kind == "rmsnorm":
        return dict(kind=kind, M=_log(rng, 256, 32768, G), K=_log(rng, 1024, 4096, G), blockwise=rng.random() < 0.7)
    if kind == "swiglu":
        return dict(kind=kind, M=_log(rng, 256, 16384, G), K=_log(rng, 1024, 9216, G), blockwise=rng.random() < 0.7)
    if kind == "lm_head":
        return dict(kind=kind, M=_log(rng, 512, 8192, G), V=_log(rng, 16384, 151936, G), K=_log(rng, 1024, 1536, G),
                    fp8=rng.random() < 0.5)
    return dict(kind=kind, count=rng.randint(1, 28), rows=_log(rng, 1024, 4096, G), cols=_log(rng, 1024, 2048, G))


# ------------------------------------------------------------------- inputs
def _gen(seed, t):
    return torch.Generator(device="cuda").manual_seed(seed * 16 + t)


def _normal(seed, t, shape, std=1.0, dtype=torch.bfloat16):
    return (torch.randn(shape, generator=_gen(seed, t), device="cuda") * std).to(dtype)


def _activations(seed, t, shape):
    """N(0, 1) with 1% of the channels x20."""
    g = _gen(seed, t)
    x = torch.randn(shape, generator=g, device="cuda")
    cols = torch.randperm(shape[1], generator=g, device="cuda")[:max(1, shape[1] // 100)]
    x[:, cols] *= 20.0
    return x.to(torch.bfloat16)


def _student_t3(seed, t, shape):
    g = _gen(seed, t)
    z = torch.randn(shape, generator=g, device="cuda")
    c = torch.zeros(shape, device="cuda")
    for _ in range(3):
        c += torch.randn(shape, generator=g, device="cuda").square_()
    return (z / (c / 3.0).sqrt()).to(torch.bfloat16)


def _inputs(case, seed):
    """The tensors of a case, from the seed alone."""
    k = case["kind"]
    if k == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return dict(X=_activations(seed, 0, (M, K)), W=_normal(seed, 1, (N, K), 0.02),
                    bias=_normal(seed, 2, (N,)) if case["bias"] else None,
                    residual=_normal(seed, 3, (M, N)) if case["residual"] else None)
    if k in ("linear", "module"):
        M, N, K = case["M"], case["N"], case["K"]
        return dict(X=_activations(seed, 0, (M, K)), W=_normal(seed, 1, (N, K), 0.02),
                    dY=_normal(seed, 2, (M, N), 1e-3))
    if k == "rmsnorm":
        return dict(x=_activations(seed, 0, (case["M"], case["K"])),
                    gamma=(1.0 + 0.1 * _normal(seed, 1, (case["K"],), dtype=torch.float32)).to(torch.bfloat16))
    if k == "swiglu":
        return dict(gu=_normal(seed, 0, (case["M"], 2 * case["K"]), 1.7), dh=_normal(seed, 1, (case["M"], case["K"]), 1e-3))
    if k == "lm_head":
        M, V, K = case["M"], case["V"], case["K"]
        return dict(X=_student_t3(seed, 0, (M, K)), W=_normal(seed, 1, (V, K), 0.02),
                    targets=torch.randint(V, (M,), generator=_gen(seed, 2), device="cuda", dtype=torch.int32))
    shape = (case["count"], case["rows"], case["cols"])
    W = _normal(seed, 0, shape, 0.02, torch.float32)
    return dict(W=W, G=_normal(seed, 1, shape, 1e-3, torch.float32), buf=_normal(seed, 2, shape, 1e-3, torch.float32),
                radius=W.flatten(1).norm(dim=1))


def _recipe(case):
    dy = puro.E4M3 if case["dy"] == "e4m3" else puro.E5M2
    if case["blockwise"]:
        return puro.LinearRecipe(puro.E4M3, puro.E4M3, dy, 1, puro.SCALE_POW2)
    return puro.LinearRecipe(puro.E4M3, puro.E4M3, dy, 0, puro.SCALE_FP32)


def _bytes(n):
    return torch.empty(max(1, n), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case)
    k = case["kind"]
    if k == "gemm":
        w = puro.quantize_fp8(s.pop("W"), puro.E4M3)
        s["w"] = puro.operand(w["q"], puro.E4M3, puro.SCALE_TENSOR, w["scale"])
    elif k == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        r = s["recipe"] = _recipe(case)
        s["saved"] = puro.linear_saved(M, N, K, r, "cuda")
        s["ws"] = _bytes(max(puro.linear_fwd_workspace_size(M, N, K, r),
                             puro.linear_bwd_workspace_size(M, N, K, r) if case["bwd"] else 0))
        s["Y"] = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
        if case["bwd"]:
            s["dX"] = torch.empty(M, K, dtype=torch.bfloat16, device="cuda")
            s["dW"] = torch.empty(N, K, dtype=torch.float32, device="cuda")
    elif k == "module":
        layer = puro.Linear(case["K"], case["N"], device="cuda")
        with torch.no_grad():
            layer.weight.copy_(s.pop("W"))
        s["layer"] = layer
        s["X"].requires_grad_(True)
    elif k == "lm_head":
        M, V, K = case["M"], case["V"], case["K"]
        r = s["recipe"] = puro.LM_HEAD_FP8 if case["fp8"] else puro.LM_HEAD_BF16
        s["ws"] = _bytes(max(puro.lm_head_ce_workspace_size(M, V, K, r, b) for b in (False, True)))
        s["dX"] = torch.empty(M, K, dtype=torch.bfloat16, device="cuda")
        s["dW"] = torch.empty(V, K, dtype=torch.float32, device="cuda")
    elif k == "muonh":
        s["w_bf16"] = torch.empty(s["W"].shape, dtype=torch.bfloat16, device="cuda")
        s["ws"] = _bytes(puro.lib().puro_muonh_workspace_size(case["count"], case["rows"], case["cols"]))
    return s


_ETA = 0.02     # MuonH's weight learning rate (a step turns W by this angle)


def run(s):
    case = s["case"]
    k = case["kind"]
    if k == "gemm":
        x = puro.quantize_fp8(s["X"], puro.E4M3)
        a = puro.operand(x["q"], puro.E4M3, puro.SCALE_TENSOR, x["scale"])
        return puro.fp8_gemm_epilogue(a, case["M"], s["w"], case["N"], case["K"], bias=s["bias"], residual=s["residual"])
    if k == "linear":
        Y, saved = puro.linear_fwd(s["X"], s["W"], s["recipe"], Y=s["Y"], saved=s["saved"], ws=s["ws"])
        if not case["bwd"]:
            return dict(Y=Y)
        dX, dW = puro.linear_bwd(s["dY"], saved, s["recipe"], case["K"], dX=s["dX"], dW=s["dW"], ws=s["ws"])
        return dict(Y=Y, dX=dX, dW=dW)
    if k == "module":
        layer, X = s["layer"], s["X"]
        layer.weight.main_grad.zero_()
        X.grad = None
        Y = layer(X)
        Y.backward(s["dY"])
        return dict(Y=Y.detach(), dX=X.grad, dW=layer.weight.main_grad)
    mode = puro.SCALE_ROW_1x128 if case.get("blockwise") else puro.SCALE_TENSOR
    rnd = puro.SCALE_POW2 if case.get("blockwise") else puro.SCALE_FP32
    if k == "rmsnorm":
        return _present(puro.rmsnorm_quantize_fp8(s["x"], s["gamma"], 1e-6, puro.E4M3, mode, rnd, want_qT=True))
    if k == "swiglu":
        h = puro.swiglu_quantize_fp8(s["gu"], case["K"], puro.E4M3, mode, rnd, want_qT=True)
        dgu = puro.swiglu_bwd_quantize_fp8(s["dh"], s["gu"], puro.E4M3, mode, rnd, want_qT=True)
        return dict(h=_present(h), dgu=_present(dgu))
    if k == "lm_head":
        lse, loss = puro.lm_head_ce_fwd(s["X"], s["W"], s["targets"], s["recipe"], ws=s["ws"])
        dX, dW = puro.lm_head_ce_bwd(s["X"], s["W"], s["targets"], lse, s["recipe"], 1.0 / case["M"],
                                     dX=s["dX"], dW=s["dW"], ws=s["ws"])
        return dict(lse=lse, loss=loss, dX=dX, dW=dW)
    puro.muonh_step(s["W"], s["G"], s["buf"], s["radius"], _ETA, w_bf16=s["w_bf16"], ws=s["ws"])
    return dict(W=s["W"], buf=s["buf"], w_bf16=s["w_bf16"])


def _present(d):
    return {k: v for k, v in d.items() if v is not None}


# ------------------------------------------------------- what a pass has to do
def work(case):
    k = case["kind"]
    if k == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return dict(bytes=2 * M * K + N * K + 2 * M * N + (2 * N if case["bias"] else 0)
                    + (2 * M * N if case["residual"] else 0), flops=2 * M * N * K)
    if k in ("linear", "module"):
        M, N, K = case["M"], case["N"], case["K"]
        saved = M * K + N * K
        fwd, bwd = 2 * (M * K + N * K + M * N) + saved, saved + 2 * M * N + 2 * M * K + 4 * N * K
        both = k == "module" or case["bwd"]
        return dict(bytes=fwd + (bwd if both else 0), flops=(6 if both else 2) * M * N * K)
    if k == "rmsnorm":
        e = case["M"] * case["K"]
        return dict(bytes=4 * e + 4 * case["M"] + 2 * case["K"] + (8 * e // G if case["blockwise"] else 4), flops=4 * e)
    if k == "swiglu":
        # forward: gate and up in, H twice out; backward: dH, gate and up in, dgu twice out
        e = case["M"] * case["K"]
        return dict(bytes=(4 + 2) * e + (2 + 4 + 4) * e + (8 * 3 * e // G if case["blockwise"] else 8), flops=30 * e)
    if k == "lm_head":
        M, V, K = case["M"], case["V"], case["K"]
        # logits, dX and dW: three products
        return dict(bytes=2 * (2 * M * K + 2 * V * K) + 2 * M * K + 4 * V * K + 16 * M, flops=6 * M * V * K)
    n, r, c = case["count"], *sorted((case["rows"], case["cols"]))
    # five steps of A = XX^T (symmetric), AA^T (symmetric) and BX
    return dict(bytes=n * r * c * (4 * 5 + 2), flops=n * 5 * (r * r * c + r * r * r + 2 * r * r * c))


def tolerance(case):
    k = case["kind"]
    if k in ("gemm", "linear", "module"):
        # BF16 outputs: one rounding (2^-9 at most, 1.7e-3 in the 2-norm of two
        # that differ everywhere) of a binary32 sum of the same FP8 products
        return {"rel": 2e-3, "max": 2e-2}
    if k in ("rmsnorm", "swiglu"):
        # the last BF16 bit of the value that is quantised may differ (another
        # order of the norm's sum, another exp), and a code or, rarely, a
        # group's power-of-two scale with it
        return {"rel": 1e-2, "max": 0.9, "differ": 1e-3}
    if k == "lm_head":
        # dz is rounded to BF16 (and, in FP8, quantised from that); dX is BF16
        return {"rel": 4e-3, "max": 0.1} if not case["fp8"] else {"rel": 1e-2, "max": 0.2}
    # Newton-Schulz in BF16: the direction moves by its roundings, W by eta
    # times that, and W's BF16 copy by its one rounding
    return {"rel": 2e-3, "max": 5e-2}


# --------------------------------------------------------- the same in 64 bits
_FMAX = {"e4m3": 448.0, "e5m2": 57344.0}
_EMAX = {"e4m3": 8, "e5m2": 15}
_F8 = {"e4m3": torch.float8_e4m3fn, "e5m2": torch.float8_e5m2}


def _q(x, fmt, rows, cols):
    """x (BF16) quantised in groups of rows x cols (0: one scale for all), as
    float64 values; the scales of the groups beside them."""
    if not rows:
        amax = x.abs().max().float()
        if amax == 0:
            return x.double(), torch.ones(1, device=x.device)
        top = torch.full_like(amax, _FMAX[fmt])       # tensor by tensor: one correctly rounded division
        v = (x.float() * (top / amax)).clamp(-_FMAX[fmt], _FMAX[fmt])
        s = amax / top
        return v.to(_F8[fmt]).double() * s.double(), s.reshape(1)
    R, C = x.shape
    g = x.reshape(R // rows, rows, C // cols, cols)
    amax = g.abs().amax(dim=(1, 3), keepdim=True).float()
    m, e = torch.frexp(amax)
    e = e - 1 - _EMAX[fmt] + (m > 0.875).to(e.dtype)
    e = torch.where(amax == 0, torch.zeros_like(e), e).clamp(-127, 127)
    s = torch.ldexp(torch.ones_like(amax), e)
    q = (g.float() / s).to(_F8[fmt])
    return (q.double() * s.double()).reshape(R, C), s.reshape(R // rows, C // cols)


def _rms_y(x, gamma, eps):
    x = x.double()
    rstd = 1.0 / (x.square().mean(dim=1) + eps).sqrt()
    return (x * rstd[:, None] * gamma.double()).to(torch.bfloat16), rstd


def _scales(y, blockwise):
    """The scale outputs of a quantisation of y with a transposed copy."""
    if not blockwise:
        return dict(q=None, qT=None, scale=_q(y, "e4m3", 0, 0)[1].double())
    return dict(q=None, qT=None, scale=_q(y, "e4m3", 1, G)[1].double(),
                scaleT=_q(y, "e4m3", G, 1)[1].t().contiguous().double())


def exact(case, seed):
    s = _inputs(case, seed)
    k = case["kind"]
    if k == "gemm":
        y = _q(s["X"], "e4m3", 0, 0)[0] @ _q(s["W"], "e4m3", 0, 0)[0].t()
        if s["bias"] is not None:
            y += s["bias"].double()
        return y if s["residual"] is None else y + s["residual"].double()
    if k in ("linear", "module"):
        block = k == "module" or case["blockwise"]
        dy = case.get("dy", "e4m3")
        row, col, blk = ((1, G), (G, 1), (G, G)) if block else ((0, 0),) * 3
        W = _q(s["W"], "e4m3", *blk)[0]
        r = dict(Y=_q(s["X"], "e4m3", *row)[0] @ W.t())
        if k == "module" or case["bwd"]:
            r["dX"] = _q(s["dY"], dy, *row)[0] @ W
            r["dW"] = _q(s["dY"], dy, *col)[0].t().contiguous() @ _q(s["X"], "e4m3", *col)[0]
        return r
    if k == "rmsnorm":
        y, rstd = _rms_y(s["x"], s["gamma"], 1e-6)
        return dict(_scales(y, case["blockwise"]), rstd=rstd)
    if k == "swiglu":
        g, u, dh = s["gu"][:, :case["K"]].double(), s["gu"][:, case["K"]:].double(), s["dh"].double()
        sg = torch.sigmoid(g)
        h = (g * sg * u).to(torch.bfloat16)
        dgu = torch.cat([dh * u * sg * (1 + g * (1 - sg)), dh * g * sg], dim=1).to(torch.bfloat16)
        return dict(h=_scales(h, case["blockwise"]), dgu=_scales(dgu, case["blockwise"]))
    if k == "lm_head":
        return _exact_lm_head(case, s)
    return _exact_muonh(case, s)


def _exact_lm_head(case, s):
    M, V, K = case["M"], case["V"], case["K"]
    X, W, t = s["X"], s["W"], s["targets"].long()
    Xl, Xw, Wl = ((_q(X, "e4m3", 1, G)[0], _q(X, "e4m3", G, 1)[0], _q(W, "e4m3", G, G)[0]) if case["fp8"]
                  else (X.double(), X.double(), W.double()))
    step = 16384
    lse = torch.full((M,), -math.inf, dtype=torch.float64, device="cuda")
    for v in range(0, V, step):
        lse = torch.logaddexp(lse, torch.logsumexp(Xl @ Wl[v:v + step].t(), dim=1))
    loss = lse - (Xl * Wl[t]).sum(dim=1)
    dX = torch.zeros(M, K, dtype=torch.float64, device="cuda")
    dW = torch.empty(V, K, dtype=torch.float64, device="cuda")
    for v in range(0, V, step):
        w = Wl[v:v + step]
        dz = torch.exp(Xl @ w.t() - lse[:, None])
        hit = (t >= v) & (t < v + w.shape[0])
        dz[hit.nonzero()[:, 0], t[hit] - v] -= 1.0
        dz /= M
        if case["fp8"]:
            b = dz.to(torch.bfloat16)
            dX += _q(b, "e4m3", 1, G)[0] @ w
            dW[v:v + step] = _q(b, "e4m3", G, 1)[0].t().contiguous() @ Xw
        else:
            dX += dz @ w
            dW[v:v + step] = dz.t().contiguous() @ Xw
    return dict(lse=lse, loss=loss, dX=dX, dW=dW)


def _exact_muonh(case, s):
    mu = 0.95
    W, Gr = s["W"].double(), s["G"].double()
    buf = mu * s["buf"].double() + (1 - mu) * Gr
    V = (1 - mu) * Gr + mu * buf
    out = torch.empty_like(W)
    for i in range(case["count"]):
        x = V[i] / (V[i].norm() + 1e-7)
        tall = x.shape[0] > x.shape[1]
        x = x.t().contiguous() if tall else x
        for _ in range(5):
            a = x @ x.t()
            b = -4.7750 * a + 2.0315 * (a @ a)
            x = 3.4445 * x + b @ x
        u = x.t() if tall else x
        w = W[i] - _ETA * s["radius"][i].double() * u / u.norm()
        out[i] = s["radius"][i].double() * w / w.norm()
    return dict(W=out, buf=buf, w_bf16=out)
