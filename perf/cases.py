"""The work that is timed: MXFP4 linear layers through the public calls, over the sizes and recipes they are used at.

A case names the calls (`calls`), the layer (M tokens, K in-features, N out-features) and the recipe.  The calls are

  fwd      mxfp4_linear_fwd: both operands quantised, one GEMM (evaluation, or a forward pass that saves nothing)
  kept     mxfp4_quantize of the tokens and mxfp4_gemm against weights that stay quantised (generation, evaluation)
  step     mxfp4_linear_fwd_save and mxfp4_linear_bwd_saved: one training step of the layer, each tensor read once
  plain    mxfp4_linear_fwd and mxfp4_linear_bwd: the same step without a saved buffer
  wgrad    mxfp4_linear_bwd for the weight gradient alone (the input of the first layer needs none)

Outputs, workspace and saved buffer are the caller's and are kept between passes, as in a training loop.
"""
import torch

import paper_2605_09825_amd as mx

HADAMARD = {"none": mx.HAD_NONE, "h32": mx.HAD_DET, "sign32": mx.HAD_RANDSIGN, "h16": mx.HAD_DET16,
            "sign16": mx.HAD_RANDSIGN16}
ROUNDING = {"rne": mx.RNE, "sr": mx.SR}
FORMATS = {"4": mx.FMT_E2M1, "8": mx.FMT_E4M3}


def _case(name, calls, M, N, K, had="h32", rnd="rne", out="bf16", geometry="1d", stages="444", accumulate=False,
          x="normal", dy="normal"):
    """stages: bits of the operands of Fprop, Dgrad and Wgrad; out: element type of Y and dX (dW is fp32)."""
    case = dict(calls=calls, M=M, N=N, K=K, had=had, rnd=rnd, out=out, geometry=geometry, stages=stages,
                accumulate=accumulate, x=x, dy=dy)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest call: one small Fprop with fp32 output, where launches and latency are all there is
        _case("fwd_small", "fwd", 256, 512, 512, had="none", out="fp32"),
        # a handful of tokens against kept 8B QKV weights: one generation step of a small batch
        _case("kept_few_tokens", "kept", 24, 6144, 4096),
        # a short evaluation batch: the tokens are few and ragged, the weights are quantised on the way
        _case("fwd_short_batch", "fwd", 200, 4096, 4096),
        # a long sequence whose token count fits no tile
        _case("fwd_ragged_tokens", "fwd", 4010, 6144, 4096),
        # a small model's MLP up projection (768 -> 3072), randomised H16, one training step
        _case("step_small_model", "step", 2048, 3072, 768, had="sign16"),
        # a layer whose widths are multiples of 32 only, gradients accumulated over microbatches
        _case("plain_odd_widths", "plain", 2080, 4320, 1440, had="h16", accumulate=True),
        # the k or v projection of an 8B model: few output tiles
        _case("step_kv", "step", 8192, 1024, 4096),
        # the fused QKV projection of an 8B model, the benchmark's headline layer
        _case("step_qkv", "step", 8192, 6144, 4096),
        # the attention output projection with Fprop in MXFP4 and both gradient GEMMs in MXFP8
        _case("step_o_gradients_in_8_bits", "step", 8192, 4096, 4096, stages="488"),
        # the MLP down projection with 32 x 32 scale regions and no rotation
        _case("step_down_2d", "step", 4096, 4096, 14336, had="none", geometry="2d"),
        # weight gradient under stochastic rounding, heavy-tailed output gradients
        _case("wgrad_stochastic", "wgrad", 16384, 4096, 4096, had="none", rnd="sr", dy="heavy"),
        # the largest: the fused gate and up projections of an 8B model, activations with outlier channels
        _case("step_gate_up", "step", 8192, 28672, 4096, x="outliers"),
    ]


def _flops(case):
    gemms = {"fwd": 1, "kept": 1, "step": 3, "plain": 3, "wgrad": 1}[case["calls"]]
    return 2.0 * case["M"] * case["N"] * case["K"] * gemms


_LARGEST = 8192 * 28672 * 4096 * 6.0


def draw(rng):
    def size(lo, hi, multiple):
        v = lo * (hi / lo) ** rng.random()
        step = multiple if rng.random() < 0.6 else max(multiple, 256)  # ragged widths, and the usual ones
        return max(multiple, int(v / step) * step)

    while True:
        calls = rng.choice(["fwd", "fwd", "kept", "step", "step", "plain", "wgrad"])
        forward = calls in ("fwd", "kept")
        M = size(1, 16384, 1) if forward else size(64, 16384, 32)
        N = size(256, 28672, 8 if forward else 32)
        K = size(128, 14336, 32)
        had = rng.choice(list(HADAMARD))
        rnd = rng.choice(["rne", "rne", "rne", "sr"])
        square = rnd == "rne" and not forward and rng.random() < 0.2
        stages = "444" if square or calls == "kept" or rng.random() < 0.7 else rng.choice(["488", "448", "484", "888"])
        case = _case(None, calls, M, N, K, had=had, rnd=rnd, out=rng.choice(["bf16", "bf16", "fp32"]),
                     geometry="2d" if square else "1d", stages=stages,
                     accumulate=calls in ("step", "plain", "wgrad") and rng.random() < 0.3,
                     x=rng.choice(["normal", "outliers"]), dy=rng.choice(["normal", "heavy"]))
        eight_bit = 2.0 if "8" in stages else 1.0
        if M * N < 2**28 and M * K < 2**28 and eight_bit * _flops(case) <= 0.5 * _LARGEST:
            return case


def _normal(gen, rows, cols, std):
    return (torch.randn((rows, cols), generator=gen, device="cuda", dtype=torch.float32) * std).to(torch.bfloat16)


def _activations(gen, rows, cols, kind):
    x = torch.randn((rows, cols), generator=gen, device="cuda", dtype=torch.float32)
    if kind == "outliers":  # 0.1 % of the channels, a hundred times as large
        channels = torch.randperm(cols, generator=gen, device="cuda")[:max(1, cols // 1000)]
        x[:, channels] *= 100.0
    return x.to(torch.bfloat16)


def _gradients(gen, rows, cols, kind):
    if kind == "normal":
        return _normal(gen, rows, cols, 1e-3)
    g = torch.randn((rows, cols), generator=gen, device="cuda", dtype=torch.float32)  # Student t, 3 degrees of freedom
    chi = torch.zeros_like(g)
    for _ in range(3):
        chi += torch.randn((rows, cols), generator=gen, device="cuda", dtype=torch.float32).square_()
    return (g / (chi / 3.0).sqrt_() * 1e-3).to(torch.bfloat16)


def _tensors(case, seed):
    """X, W and, where the case has a backward call, dY and the dW it starts from."""
    M, N, K = case["M"], case["N"], case["K"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    x, w, dy, dw = _activations(gen, M, K, case["x"]), _normal(gen, N, K, 0.02), None, None
    if case["calls"] not in ("fwd", "kept"):
        dy = _gradients(gen, M, N, case["dy"])
        # (with accumulation: the gradient of the microbatches before this one)
        dw = torch.randn((N, K), generator=gen, device="cuda") * 1e-2
    return x, w, dy, dw


def prepare(case, seed):
    M, N, K, calls = case["M"], case["N"], case["K"], case["calls"]
    out = mx.OUT_FP32 if case["out"] == "fp32" else mx.OUT_BF16
    dtype = torch.float32 if case["out"] == "fp32" else torch.bfloat16
    fprop, dgrad, wgrad = (FORMATS[c] for c in case["stages"])
    cfg = mx.make_cfg(HADAMARD[case["had"]], ROUNDING[case["rnd"]], seed, y_dtype=out, dx_dtype=out,
                      dw_dtype=mx.OUT_FP32, dw_accumulate=case["accumulate"],
                      geometry=mx.GEOM_2D if case["geometry"] == "2d" else mx.GEOM_1D,
                      fprop_format=fprop, dgrad_format=dgrad, wgrad_format=wgrad)
    x, w, dy, dw = _tensors(case, seed)
    s = {"calls": calls, "cfg": cfg, "K": K, "out": out, "x": x, "w": w}
    bytes_of = dict(dtype=torch.uint8, device="cuda")
    if calls != "wgrad":
        s["y"] = torch.empty((M, N), dtype=dtype, device="cuda")
    if calls == "kept":
        s["wq"], s["ws"] = mx.mxfp4_quantize(s.pop("w"), mx.AXIS_LAST, cfg.hadamard, cfg.rounding, seed ^ (1 << 48))
        s["xq"], s["xs"] = torch.empty((M, K // 2), **bytes_of), torch.empty((M, K // 32), **bytes_of)
        return s
    if calls != "wgrad":
        s["ws_f"] = torch.empty(mx.mxfp4_linear_workspace_bytes(M, N, K, cfg, False), **bytes_of)
    if calls != "fwd":
        s["dy"], s["dw"] = dy, dw
        s["ws_b"] = torch.empty(mx.mxfp4_linear_workspace_bytes(M, N, K, cfg, True), **bytes_of)
        if calls != "wgrad":
            s["dx"] = torch.empty((M, K), dtype=dtype, device="cuda")
    if calls == "step":
        s["saved"] = torch.empty(mx.mxfp4_linear_saved_bytes(M, N, K, cfg), **bytes_of)
    return s


def run(s):
    calls, cfg = s["calls"], s["cfg"]
    if calls == "kept":
        mx.mxfp4_quantize(s["x"], mx.AXIS_LAST, cfg.hadamard, cfg.rounding, cfg.seed, q=s["xq"], s=s["xs"])
        return mx.mxfp4_gemm(s["xq"], s["xs"], s["wq"], s["ws"], out=s["y"], out_dtype=s["out"])
    if calls == "fwd":
        return mx.mxfp4_linear_fwd(s["x"], s["w"], cfg, y=s["y"], workspace=s["ws_f"])[0]
    if calls == "wgrad":
        return mx.mxfp4_linear_bwd(s["dy"], s["x"], None, cfg, dw=s["dw"], need_dx=False, workspace=s["ws_b"])[1]
    if calls == "step":
        y, _, saved = mx.mxfp4_linear_fwd_save(s["x"], s["w"], cfg, y=s["y"], workspace=s["ws_f"], saved=s["saved"])
        dx, dw, _ = mx.mxfp4_linear_bwd_saved(s["dy"], saved, s["K"], cfg, dx=s["dx"], dw=s["dw"],
                                              workspace=s["ws_b"])
    else:
        y, _ = mx.mxfp4_linear_fwd(s["x"], s["w"], cfg, y=s["y"], workspace=s["ws_f"])
        dx, dw, _ = mx.mxfp4_linear_bwd(s["dy"], s["x"], s["w"], cfg, dx=s["dx"], dw=s["dw"], workspace=s["ws_b"])
    return {"y": y, "dx": dx, "dw": dw}


def work(case):
    M, N, K, calls = case["M"], case["N"], case["K"], case["calls"]
    e = 4 if case["out"] == "fp32" else 2
    x, y = M * K, M * N
    if calls == "kept":
        return {"bytes": 2 * x + N * K * (0.5 + 1 / 32) + e * y, "flops": _flops(case)}
    dw = N * K * (8 if case["accumulate"] else 4)
    if calls == "wgrad":
        return {"bytes": 2 * x + 2 * y + dw, "flops": _flops(case)}
    nbytes = 2 * x + 2 * N * K + e * y
    if calls != "fwd":
        nbytes += 2 * y + e * x + dw
    return {"bytes": nbytes, "flops": _flops(case)}


def tolerance(case):
    # Quantisation is exact.  Against products of the same operands in 64 bits the MXFP4 outputs measured 0 to 6e-8;
    # fp32 sums in another order may also round a bf16 output the other way (2^-7 of its value, rarely).  The matrix
    # unit aligns groups of MXFP8 products and drops their low bits: 2.3e-4 measured in bf16, 1.5e-5 in fp32.
    if "8" in case["stages"]:
        return {"rel": 1e-3, "max": 1.6e-2}
    if case["out"] == "fp32":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 1e-4, "max": 8e-3}


# ---- the same results in plain torch: operands quantised by their definition, products summed in 64 bits ----------

def _mix(v):
    v = (v ^ (v >> 16)) * 0x9E3779B9 & 0xFFFFFFFF
    v = (v ^ (v >> 15)) * 0xBB67AE85 & 0xFFFFFFFF
    return v ^ (v >> 16)


def _rand32(seed, low, high):
    key = _mix((seed >> 32 & 0xFFFFFFFF) ^ 0x6A09E667)
    return _mix(_mix((low + (seed & 0xFFFFFFFF) * 0x9E3779B9) & 0xFFFFFFFF) ^ high ^ key)


def _rotate(v, had, seed):
    """Blocks of 32 along the last axis: sign diagonal, butterflies and one multiply, every operation in fp32."""
    if had.startswith("sign"):
        mask = _rand32(seed & 0xFFFFFFFFFFFF, 0xFFFFFFFF, 0xFFFFFFFF)
        v = v * torch.tensor([1.0 - 2.0 * (mask >> i & 1) for i in range(32)], device=v.device)
    if had == "none":
        return v
    points = 32 if had.endswith("32") else 16
    h = 1
    while h < points:
        p = v.view(v.shape[:-1] + (32 // (2 * h), 2, h))
        v = torch.stack((p[..., 0, :] + p[..., 1, :], p[..., 0, :] - p[..., 1, :]), dim=-2).reshape(v.shape)
        h *= 2
    return v * torch.tensor(32.0 ** -0.5 if points == 32 else 0.25, dtype=torch.float32, device=v.device)


def _quantised(case, x, stream, bits, seed):
    """The values that x [R][C] has as a quantised operand with blocks of 32 along its last axis, in 64 bits."""
    R, C = x.shape
    seed = (seed & (2**64 - 1)) ^ (stream << 48)
    out = torch.empty((R, C), dtype=torch.float64, device=x.device)
    step = max(32, (1 << 25) // C // 32 * 32)
    for r in range(0, R, step):
        v = x[r:r + step].float().reshape(-1, C // 32, 32)
        if bits == "4":
            v = _rotate(v, case["had"], seed)
        amax = v.abs().amax(dim=-1)
        if case["geometry"] == "2d":
            amax = amax.view(-1, 32, C // 32).amax(dim=1).repeat_interleave(32, dim=0)
        exponent = ((amax.view(torch.int32) >> 23) - (2 if bits == "4" else 8)).clamp(min=0) - 127
        scale = ((exponent.long() + 1023) << 52).view(torch.float64).unsqueeze(-1)  # 2^exponent
        t = v.double() / scale
        if bits == "8":
            t = t.clamp(-448.0, 448.0).float().to(torch.float8_e4m3fn).double()
        else:
            a = t.abs().clamp(max=6.0)
            grid = torch.where(a < 2.0, 0.5, torch.where(a < 4.0, 1.0, 2.0))
            a = a / grid
            if case["rnd"] == "sr":
                index = torch.arange(r * C, r * C + a.numel(), device=x.device).view(a.shape)
                u = (2 * (_rand32(seed, index & 0xFFFFFFFF, index >> 32) >> 9) + 1).double() * 2.0**-24
                a = a.floor() + (u < a - a.floor()).double()
            else:
                a = a.round()
            t = torch.copysign(a * grid, t)
        out[r:r + step] = (t * scale).view(-1, C)
    return out


def exact(case, seed):
    x, w, dy, dw0 = _tensors(case, seed)
    calls, (fprop, dgrad, wgrad) = case["calls"], case["stages"]
    X, W, DY, WT, DYT, XT = range(6)
    if calls != "wgrad":
        y = _quantised(case, x, X, fprop, seed) @ _quantised(case, w, W, fprop, seed).T
        if calls in ("fwd", "kept"):
            return y
    dw = (_quantised(case, dy.T.contiguous(), DYT, wgrad, seed) @
          _quantised(case, x.T.contiguous(), XT, wgrad, seed).T)
    if case["accumulate"]:
        dw += dw0
    if calls == "wgrad":
        return dw
    dx = _quantised(case, dy, DY, dgrad, seed) @ _quantised(case, w.T.contiguous(), WT, dgrad, seed).T
    return {"y": y, "dx": dx, "dw": dw}
