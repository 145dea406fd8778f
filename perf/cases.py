"""The calls this library is timed on: per-layer DP weight gradients as training programs make them.

A case names an entry point and a problem:
  entry   "linear"    flashdp_linear_dp_grad, the one-layer call with the thread's context and the library's workspace
          "block"     flashdp_block_dp_grad over the layers of a block, workspace owned by the caller
          "micro"     flashdp_block_dp_grad_micro once per micro-batch of an accumulated batch, noise with the last
          "static"    flashdp_linear_dp_grad_static, the call that allocates nothing
          "dplinear"  forward and backward of a chain of DPLinear modules through torch's autograd
          "deferred"  the same inside deferred_weight_grads (one library call per block)
  dtype   storage of X and dY: "bf16", "f16" or "fp32"
  B, T    samples per call and tokens per sample; micro = micro-batches per pass ("micro" only)
  dims    the layers, "d_inxd_out" separated by blanks
  park    0, or the number of samples the caller's workspace holds parked at a time ("block" only)
  C, sigma  clipping threshold and noise multiplier

The sizes are those of this repository's workloads (GPT-2 and Llama linear layers, the tiny fp32 layer), the other
linear layers of a GPT-2 block, and generic ones: rows without a sequence, short sequences, sizes no tile divides.
Values follow the recipe of workloads/: X standard normal, dY normal with a small variance times a per-sample scale
10^U(-1, 1), so that norms spread over two decades and most samples clip.
"""
from __future__ import annotations

import math

import torch

import paper_2507_01154_amd as F
from paper_2507_01154_amd.autograd import DPLinear, deferred_weight_grads

DEVICE = "cuda:0"
_TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "fp32": torch.float32}
_CODE = {"bf16": F.BF16, "f16": F.F16, "fp32": F.F32}
_BYTES = {"bf16": 2, "f16": 2, "fp32": 4}

GPT2_BLOCK = "768x2304 768x768 768x3072 3072x768"
LLAMA13B_BLOCK = "5120x5120 5120x5120 5120x5120 5120x5120 5120x13824 5120x13824 13824x5120"


def _case(name, entry, dtype, B, T, dims, sigma=1.0, C=1.0, micro=1, park=0):
    return dict(name=name, entry=entry, dtype=dtype, B=B, T=T, dims=dims, C=C, sigma=sigma, micro=micro, park=park)


def listed():
    return [
        # the tiny fp32 layer of the workloads: nothing but call, launch and latency costs
        _case("tiny_fp32", "linear", "fp32", 4, 16, "32x32"),
        # classifier on rows without a sequence (T = 1), the many-small-samples end of DP-SGD; ten classes: a size no
        # vector width divides
        _case("mlp_rows_fp32", "dplinear", "fp32", 256, 1, "784x512 512x10"),
        # fine-tuning on short sequences: many samples of few tokens, the linear layers of a GPT-2 block, fp16
        _case("gpt2_short_f16", "block", "f16", 32, 128, GPT2_BLOCK, sigma=0.6),
        # micro-batches of one sample, four per optimizer step
        _case("gpt2_micro_bf16", "micro", "bf16", 1, 1024, GPT2_BLOCK, micro=4),
        # the MLP of a GPT-2 block as a training loop runs it: forward, input gradients, DP weight gradients
        _case("gpt2_mlp_train", "deferred", "bf16", 4, 1024, "768x3072 3072x768"),
        # a single GPT-2 layer through the entry point for callers that cannot allocate
        _case("gpt2_c_fc_static", "static", "bf16", 8, 1024, "768x3072"),
        # multiples of 8 that no tile divides, a token count that no k-tile divides
        _case("ragged_bf16", "linear", "bf16", 5, 333, "1096x2312", sigma=0.5),
        # an odd number of output features: the output layer over GPT-2's vocabulary
        _case("vocab_odd_bf16", "block", "bf16", 2, 1024, "768x50257"),
        # the Llama-7B attention projection in single precision, and in bf16
        _case("llama7b_q_proj_fp32", "block", "fp32", 4, 2048, "4096x4096", sigma=0.8),
        _case("llama7b_q_proj_bf16", "linear", "bf16", 4, 2048, "4096x4096", sigma=0.8),
        # a Llama-13B MLP projection with memory for two parked samples only; clipping without noise
        _case("llama13b_up_bounded", "block", "bf16", 4, 2048, "5120x13824", sigma=0.0, park=2),
        # the benchmark: all seven linear layers of a Llama-13B decoder block
        _case("llama13b_block", "block", "bf16", 8, 2048, LLAMA13B_BLOCK),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _feature(rng, lo, hi, align):
    return max(align, _log_int(rng, lo, hi) // align * align)


def draw(rng):
    """One more case: entry, type and sizes independent of each other, sizes log-uniform, cut down until it costs no
    more than the Llama-13B block."""
    entry = rng.choice(["linear", "block", "block", "micro", "static", "dplinear", "deferred"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f16", "fp32"])
    align = rng.choice([1, 8, 8, 8, 64, 128])
    n_layers = rng.choice([2, 3, 4]) if entry in ("block", "micro", "dplinear", "deferred") else 1
    if entry == "block" and rng.random() < 0.4:
        n_layers = 1
    T = rng.choice([_log_int(rng, 1, 64), _log_int(rng, 64, 512), _log_int(rng, 512, 2048), 1024, 2048])
    B = _log_int(rng, 1, 256 if T <= 16 else 64 if T <= 256 else 16)
    micro = rng.choice([2, 3, 4]) if entry == "micro" else 1
    feats = [_feature(rng, 24, 13824, align) for _ in range(n_layers + 1)]
    sigma = rng.choice([0.0, 0.5, 0.8, 1.0])
    C = rng.choice([0.1, 1.0, 1.0, 10.0])

    def dims():
        return list(zip(feats[:-1], feats[1:]))

    def seconds():
        # rough rates of the three families of shapes, to keep a drawn case below the largest listed one
        t = 0.0
        for p, d in dims():
            rate = 7e12 if (p % 8 or d % 8) and dtype != "fp32" or (p % 4 or d % 4) else 1.0e14 if dtype == "fp32" else 6e14
            n = 3 if entry in ("dplinear", "deferred") else 1
            t += micro * (n * 2.0 * B * T * p * d / rate + 16.0 * B * p * d / 4e12 + 20.0 * p * d / 4e12)
        return t

    while seconds() > 6e-3:
        k = max(range(n_layers + 1), key=lambda i: feats[i])
        if feats[k] > 4 * max(align, 128):
            feats[k] = max(align, int(feats[k] * 0.7) // align * align)
        elif B > 1:
            B = max(1, B * 2 // 3)
        else:
            T = max(1, T * 2 // 3)
    if entry == "static":
        while B * feats[0] * feats[1] * _BYTES[dtype] > 60 << 20:    # what the static workspace holds
            k = 0 if feats[0] >= feats[1] else 1
            feats[k] = max(align, int(feats[k] * 0.7) // align * align)
    park = 0
    if entry == "block" and n_layers == 1 and B >= 2 and rng.random() < 0.4:
        park = rng.randint(1, B - 1)
    return _drop_name(_case("", entry, dtype, B, T, " ".join(f"{p}x{d}" for p, d in dims()), sigma, C, micro, park))


def _drop_name(c):
    c.pop("name")
    return c


def _layers(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["dims"].split()]


def _x(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32).to(dtype)


def _dy(gen, B, T, d, dtype, variance):
    scale = math.sqrt(variance) * 10.0 ** (2.0 * torch.rand((B, 1, 1), generator=gen, device=DEVICE) - 1.0)
    out = torch.empty((B, T, d), dtype=dtype, device=DEVICE)
    step = max(1, (1 << 26) // max(1, T * d))          # the fp32 draw is transient
    for i in range(0, B, step):
        n = min(step, B - i)
        out[i:i + n] = (torch.randn((n, T, d), generator=gen, device=DEVICE) * scale[i:i + n]).to(dtype)
    return out


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    dtype, B, T = _TORCH[case["dtype"]], case["B"], case["T"]
    layers = _layers(case)
    variance = 1e-4 if T > 1024 else 1e-3
    s = dict(entry=case["entry"], B=B, T=T, code=_CODE[case["dtype"]], C=case["C"], sigma=case["sigma"], seed=1 + seed % (1 << 30))

    if case["entry"] in ("dplinear", "deferred"):
        torch.manual_seed(seed)
        s["modules"] = [DPLinear(p, d, C=case["C"], sigma=case["sigma"], seed=s["seed"], layer=l, dtype=dtype, device=DEVICE,
                                 auto_step=False) for l, (p, d) in enumerate(layers)]
        shape = (B, layers[0][0]) if T == 1 else (B, T, layers[0][0])
        s["x"] = _x(gen, shape, dtype).requires_grad_(True)
        dy = _dy(gen, B, T, layers[-1][1], dtype, variance)
        s["dy"] = dy.reshape(B, -1) if T == 1 else dy
        return s

    n_micro = case["micro"]
    outs = [torch.empty((d, p), dtype=torch.float32, device=DEVICE) for p, d in layers]
    norms = [[torch.empty((B,), dtype=torch.float32, device=DEVICE) for _ in layers] for _ in range(n_micro)]
    batches = []
    for m in range(n_micro):
        batches.append([dict(X=_x(gen, (B, T, p), dtype), dY=_dy(gen, B, T, d, dtype, variance), d_in=p, d_out=d,
                             C=case["C"], sigma=case["sigma"], seed=s["seed"] + l, layer=l, out_grad=outs[l], out_norms=norms[m][l])
                        for l, (p, d) in enumerate(layers)])
    s.update(batches=batches, arrays=[F.make_layers(b) for b in batches], outs=outs, norms=norms)
    if case["entry"] in ("block", "micro"):
        if case["park"]:
            need = F.flashdp_workspace_bytes_chunked(s["arrays"][0], B, T, s["code"], case["park"], 1)
        else:
            need = F.flashdp_workspace_bytes(s["arrays"][0], B, T, s["code"], "overlap" if len(layers) > 1 else "scratch")
        s["workspace"] = torch.empty((need,), dtype=torch.uint8, device=DEVICE)
    if case["entry"] == "linear":
        F.flashdp_set_stream()
        F.flashdp_set_dtype(s["code"])
        F.flashdp_set_layer(0)
        F.flashdp_set_schedule("auto")
        F.flashdp_set_workspace(None)
    return s


def _train(s):
    modules, x = s["modules"], s["x"]
    x.grad = None
    for m in modules:
        m.weight.grad = None
    y = x
    for k, m in enumerate(modules):
        y = m(torch.nn.functional.gelu(y) if k else y)
    y.backward(s["dy"])
    return y, x


def run(s):
    entry = s["entry"]
    if entry == "linear":
        L = s["batches"][0][0]
        F.flashdp_linear_dp_grad(L["X"], L["dY"], s["B"], s["T"], L["d_in"], L["d_out"], s["C"], s["sigma"], L["seed"],
                                 L["out_grad"], L["out_norms"])
    elif entry == "static":
        L = s["batches"][0][0]
        F.flashdp_linear_dp_grad_static(L["X"], L["dY"], s["B"], s["T"], L["d_in"], L["d_out"], s["code"], s["C"], s["sigma"],
                                        L["seed"], L["layer"], L["out_grad"], L["out_norms"])
    elif entry == "block":
        F.flashdp_block_dp_grad(s["arrays"][0], s["B"], s["T"], s["code"], "auto", s["workspace"])
    elif entry == "micro":
        last = len(s["arrays"]) - 1
        for m, arr in enumerate(s["arrays"]):
            F.flashdp_block_dp_grad_micro(arr, s["B"], s["T"], s["code"], "auto", s["workspace"], accumulate=m > 0, add_noise=m == last)
    else:
        if entry == "deferred":
            with deferred_weight_grads():
                y, x = _train(s)
        else:
            y, x = _train(s)
        return dict(y=y.detach(), dx=x.grad, grads=[m.weight.grad for m in s["modules"]], norms=[m.last_norms for m in s["modules"]])
    return dict(grads=s["outs"], norms=s["norms"])


def work(case):
    """Every operand read once and every result written once; one contraction per layer and micro-batch (DPLinear: the
    forward product and the input gradient as well)."""
    B, T, m, e = case["B"], case["T"], case["micro"], _BYTES[case["dtype"]]
    flops = bytes_ = 0.0
    for p, d in _layers(case):
        if case["entry"] in ("dplinear", "deferred"):
            flops += 3 * 2.0 * B * T * p * d
            # X, W and dY in; Y, dX and the weight gradient out
            bytes_ += e * (B * T * (2.0 * p + 2.0 * d) + 2.0 * p * d) + 4.0 * B
        else:
            flops += m * 2.0 * B * T * p * d
            bytes_ += m * (e * B * T * (p + d) + 4.0 * B) + 4.0 * p * d
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """Relative 2-norm error between two correct forms of the same sums.

    16-bit types: a per-sample gradient may be rounded to bfloat16 once on its way (as parked by the library; 1.7e-3
    of the gradient, measured) or not at all.  fp32: other orders of addition, 2e-6 of the gradient.  The noise field
    is prescribed value by value (6e-7 at most, measured; 2e-7 in norm), so where noise is added the gradient's error counts by
    the gradient's share of the output: at least one clipped sample of norm C against sigma C sqrt(elements), at most
    all samples aligned.  Norms taken before or after that rounding differ by 1.2e-3 / sqrt(elements).  DPLinear rounds its
    results to the storage type and passes gradients on through 16-bit tensors."""
    worst = 0.0
    total = case["B"] * case["micro"]
    for p, d in _layers(case):
        share = 1.0
        if case["sigma"] > 0.0:
            share = total / math.sqrt(total * total + case["sigma"] ** 2 * p * d)
        rel = (4 * 1.7e-3 * share + 4 * 1.2e-3 / math.sqrt(p * d)) if case["dtype"] != "fp32" else 1e-5 * share
        worst = max(worst, rel + 2e-6)
    if case["entry"] in ("dplinear", "deferred"):
        worst = max(worst, 1e-5 if case["dtype"] == "fp32" else 4e-3)
    return {"rel": worst, "max": 12 * worst}    # single values stray up to 10 times as far as the norm (measured)
