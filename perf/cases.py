"""Performance cases of the NVFP4 W4A4 linear layer: what a program that
serves a model through ``paper_2609_04098_amd.linear`` calls, from one decode
token to a whole prefill batch.

A case names a module (the projections of ``synth.CONFIGS`` and their column or
row shards), a token count, an entry point and its options.  Inputs have the
distributions of ``synth`` (residual stream with outlier channels, heavy-tailed
MLP activations, one weight scale per fused segment), drawn on the GPU.
"""

import math

import torch

from paper_2609_04098_amd import linear as L
from paper_2609_04098_amd import synth

BLOCK = 16
EPS = 1e-6

# Weight scale of each fused segment, and the kind of activation, per module.
SIGMA = {"gdn_qkv": (0.02, 0.03, 0.014), "mlp_gate_up": (0.015, 0.0195), "mlp_down": (0.01,),
         "ab_gates": (0.05, 0.05), "ragged": (0.02, 0.03)}
X_KIND = {"gdn_qkv": "residual", "mlp_gate_up": "residual", "mlp_down": "student_t", "ab_gates": "residual",
          "ragged": "residual"}


def listed():
    return [
        # One token of a single-user chat: latency of the widest projection.
        dict(name="decode_1_gate_up", call="quantize_gemm", module="mlp_gate_up", shard=1, m=1, g="dynamic", out="bf16"),
        # A few concurrent users (or drafted tokens), calibrated scale, long reduction, narrow output.
        dict(name="decode_4_down", call="quantize_gemm", module="mlp_down", shard=1, m=4, g="static", out="bf16"),
        # A small decode batch on the fused GDN q/k/v projection.
        dict(name="decode_32_qkv", call="quantize_gemm", module="gdn_qkv", shard=1, m=32, g="dynamic", out="bf16"),
        # A continuous-batching decode step: around a hundred sequences, never a round number.
        dict(name="batch_100_gate_up", call="linear", module="mlp_gate_up", shard=1, m=100, g="dynamic", out="bf16"),
        # The same server under load, or a short prompt, on the long reduction.
        dict(name="batch_200_down", call="linear", module="mlp_down", shard=1, m=200, g="dynamic", out="bf16"),
        # A prefill chunk through a GDN block's input side: norm, q/k/v and the b|a gates.
        dict(name="chunk_1000_gdn_block", call="gdn_block", module="gdn_qkv", shard=1, m=1000, g="static", out="bf16"),
        # A long prompt through the down projection, length as it comes.
        dict(name="prefill_5000_down", call="linear", module="mlp_down", shard=1, m=5000, g="dynamic", out="bf16"),
        # The largest ordinary prefill batch, the widest projection (the bench workload).
        dict(name="prefill_8192_gate_up", call="linear", module="mlp_gate_up", shard=1, m=8192, g="dynamic", out="bf16"),
        # The tall-skinny gate projection over a long context.
        dict(name="prefill_32768_gates", call="quantize_gemm", module="ab_gates", shard=1, m=32768, g="dynamic", out="bf16"),
        # A model whose sizes are no multiples of anything but the block; FP32 output for a caller that adds in FP32.
        dict(name="ragged_777", call="linear", module="ragged", n=1300, k=1040, m=777, g="dynamic", out="f32"),
        # Norm in front of the projections of a prefill batch, calibrated scale, normalized output kept.
        dict(name="norm_quant_8192", call="rmsnorm_quantize_act", module="mlp_gate_up", shard=1, m=8192, g="static", out="bf16"),
        # Quantizer alone (one activation serving several projections), ragged length.
        dict(name="quantize_2047_down", call="quantize_act", module="mlp_down", shard=1, m=2047, g="dynamic", out="bf16"),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    call = rng.choice(["quantize_gemm", "quantize_gemm", "linear", "linear", "linear", "gates", "gdn_block", "ragged",
                       "rmsnorm_quantize_act", "quantize_act"])
    module = rng.choice(["gdn_qkv", "mlp_gate_up", "mlp_down"])
    shard = rng.choice([1, 1, 2, 4, 8])
    g = rng.choice(["dynamic", "static"])
    out = rng.choice(["bf16", "bf16", "bf16", "f32"])
    if call == "quantize_gemm":
        return dict(call=call, module=module, shard=shard, m=_log_uniform(rng, 1, 32), g=g, out=out)
    if call == "linear":
        return dict(call=call, module=module, shard=shard, m=_log_uniform(rng, 33, 8000), g="dynamic", out=out)
    if call == "gates":
        return dict(call="quantize_gemm", module="ab_gates", shard=1, m=_log_uniform(rng, 33, 32768), g=g, out=out)
    if call == "gdn_block":
        return dict(call=call, module="gdn_qkv", shard=shard, m=_log_uniform(rng, 1, 8000), g="static", out="bf16")
    if call == "ragged":
        return dict(call="linear", module="ragged", n=_log_uniform(rng, 129, 4000), k=16 * _log_uniform(rng, 8, 400),
                    m=_log_uniform(rng, 1, 3000), g="dynamic", out=out)
    return dict(call=call, module=rng.choice(["mlp_gate_up", "mlp_down"]), shard=1, m=_log_uniform(rng, 1, 8000),
                g="static" if call == "rmsnorm_quantize_act" else g, out="bf16")


def _segments(case):
    """Rows of each fused segment, K."""
    if case["module"] == "ragged":
        return [case["n"] // 3, case["n"] - case["n"] // 3], case["k"]
    cfg = synth.CONFIGS[case["module"]]
    s = case["shard"]
    if case["module"] == "mlp_down":               # row parallel: K is cut
        return list(cfg.segments), cfg.k // s
    return [n // s for n in cfg.segments], cfg.k   # column parallel: every segment is cut


def _offsets(segments):
    offs = [0]
    for n in segments:
        offs.append(offs[-1] + n)
    return offs


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    segments, k = _segments(case)
    m = case["m"]

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)

    def uniform(n, lo, hi):
        return torch.rand(n, generator=gen, device="cuda", dtype=torch.float32) * (hi - lo) + lo

    factor = None
    if X_KIND[case["module"]] == "residual":
        hot = torch.randperm(k, generator=gen, device="cuda")[:max(1, int(round(0.005 * k)))]
        factor = torch.ones(k, device="cuda", dtype=torch.float32)
        factor[hot] = uniform(hot.numel(), 50.0, 200.0)
    x = torch.empty((m, k), device="cuda", dtype=torch.bfloat16)
    for r in range(0, m, 8192):
        v = normal(min(8192, m - r), k)
        if factor is None:                         # Student-t with 3 degrees of freedom
            chi = sum(normal(*v.shape).square() for _ in range(3))
            v = v / (chi / 3.0).sqrt() * 0.5
        else:
            v = v * factor
        x[r:r + v.shape[0]] = v.to(torch.bfloat16)

    def weight(segs, sigmas, k_):
        return torch.cat([(normal(n, k_) * s).to(torch.bfloat16) for n, s in zip(segs, sigmas)])

    w = dict(x=x)
    call = case["call"]
    if call not in ("rmsnorm_quantize_act", "quantize_act"):
        w["w"] = weight(segments, SIGMA[case["module"]], k)
        w["offs"] = _offsets(segments)
    if call in ("rmsnorm_quantize_act", "gdn_block"):
        w["gamma"] = uniform(k, 0.5, 1.5).to(torch.bfloat16)
    if call == "gdn_block":
        w["w_ab"] = weight((48, 48), SIGMA["ab_gates"], k)
        w["a_log"] = uniform(48, 1.0, 16.0).log()
        w["dt_bias"] = uniform(48, -4.0, 2.0)
    if case["g"] == "static":                      # calibrated: the range of such activations
        v = x.float()
        if "gamma" in w:
            v = v * torch.rsqrt(v.square().mean(1, keepdim=True) + EPS) * w["gamma"].float()
        w["g"] = 2688.0 / (1.05 * float(v.abs().max()))
    return w


def prepare(case, seed):
    """Packed weights, parameters and activations on the GPU."""
    s = _inputs(case, seed)
    s["case"] = dict(case)
    s["out"] = torch.float32 if case["out"] == "f32" else torch.bfloat16
    if "w" in s:
        s["pw"] = L.pack_weight(s.pop("w"), s.pop("offs"))
    if "w_ab" in s:
        s["pab"] = L.pack_weight(s.pop("w_ab"), [0, 48, 96])
    if "gamma" in s:
        s["g"] = torch.tensor([s["g"]], dtype=torch.float32, device="cuda")
    return s


def run(s):
    call = s["case"]["call"]
    if call == "quantize_gemm":
        y, g = L.quantize_gemm(s["x"], s["pw"], s.get("g"), s["out"])
        return {"y": y, "g": g}
    if call == "linear":
        return {"y": L.linear(s["x"], s["pw"], s["out"])}
    if call == "gdn_block":
        aq = L.rmsnorm_quantize_act(s["x"], s["gamma"], EPS, s["g"])
        return {"qkv": L.gemm(aq, s["pw"], s["out"]),
                "gates": L.gemm_gdn_gates(aq, s["pab"], s["a_log"], s["dt_bias"], s["out"])}
    if call == "rmsnorm_quantize_act":
        y = torch.empty_like(s["x"])
        aq = L.rmsnorm_quantize_act(s["x"], s["gamma"], EPS, s["g"], y=y)
        return {"y": y, "codes": aq.codes, "scales": aq.scales}
    aq = L.quantize_act(s["x"], s.get("g"))
    return {"codes": aq.codes, "scales": aq.scales, "g": aq.g}


def work(case):
    segments, k = _segments(case)
    n, m = sum(segments), case["m"]
    out = 4 if case["out"] == "f32" else 2
    packed = 0.5625 * k                            # bytes of a quantized row: 4 bits a value, a byte a block
    call = case["call"]
    if call == "quantize_act":
        return {"bytes": m * (2 * k + packed) + 4, "flops": 0}
    if call == "rmsnorm_quantize_act":
        return {"bytes": m * (4 * k + packed) + 2 * k, "flops": 4 * m * k}
    total = {"bytes": 2 * m * k + n * packed + out * m * n, "flops": 2 * m * n * k}
    if call == "gdn_block":
        total["bytes"] += 96 * packed + out * m * 96 + 2 * k
        total["flops"] += 2 * m * 96 * k + 4 * m * k
    return total


def tolerance(case):
    """FP32 output: FP32 sums in another order.  BF16 output: the same, with a
    rounding to bf16 that can then go the other way.  The norm's binary32 sum
    in another order moves an occasional normalized value, and with it a code,
    by one step; quantizing is exact."""
    call = case["call"]
    if call == "quantize_act":
        return "exact"
    if call == "rmsnorm_quantize_act":
        return {"rel": 5e-4, "max": 8e-3, "differ": 1e-4}
    if call == "gdn_block":
        return {"rel": 3e-4, "max": 3e-2}
    if case["out"] == "f32":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 2e-4, "max": 8e-3}


# ------------------------------------------------------------ 64-bit reference


def _quantize64(v, g):
    """Dequantized values times G of a float64 [rows, K] tensor (exact: every
    product below has far fewer than 53 significant bits, and no quotient is
    nearer to a rounding midpoint than float64 resolves)."""
    rows, k = v.shape
    b = v.view(rows, k // BLOCK, BLOCK)
    u = b.abs().amax(2) * g / 6.0
    e = torch.frexp(u.clamp(min=2.0 ** -6))[1].double() - 1.0
    step = torch.exp2(e - 3.0)
    s = (torch.round(u / step) * step).clamp(max=448.0).unsqueeze(2)
    q = torch.where(s > 0, b.abs() * g / s.clamp(min=2.0 ** -9), torch.zeros_like(b))
    step = torch.where(q < 2.0, 0.5, torch.where(q < 4.0, 1.0, 2.0)).double()
    mag = (torch.round(q / step) * step).clamp(max=6.0)
    return (torch.copysign(mag, b) * s).view(rows, k)


def _scale64(v):
    """fl32(2688 / amax) of a tensor, as a float."""
    return float((torch.tensor(2688.0, dtype=torch.float32) / v.abs().max().float().cpu()))


def _matmul64(a, ga, w, offs):
    """dq(A) dq(W)^T in float64; a: quantized values times G_A."""
    y = torch.empty((a.shape[0], w.shape[0]), dtype=torch.float64, device=a.device)
    for lo, hi in zip(offs[:-1], offs[1:]):
        gw = _scale64(w[lo:hi])
        for c in range(lo, hi, 4096):
            d = min(hi, c + 4096)
            y[:, c:d] = a @ _quantize64(w[c:d].double(), gw).t() / (ga * gw)
    return y


def exact(case, seed):
    s = _inputs(case, seed)
    call = case["call"]
    x = s["x"].double()
    if "gamma" in s:
        x = x * torch.rsqrt(x.square().mean(1, keepdim=True) + EPS) * s["gamma"].double()
        if call == "rmsnorm_quantize_act":
            return {"y": x, "codes": None, "scales": None}
        x = x.float().to(torch.bfloat16).double()
    g = float(torch.tensor(s["g"], dtype=torch.float32)) if "g" in s else _scale64(s["x"])
    gt = torch.tensor([g], dtype=torch.float64)
    if call == "quantize_act":
        return {"codes": None, "scales": None, "g": gt}
    a = torch.cat([_quantize64(x[r:r + 2048], g) for r in range(0, x.shape[0], 2048)])
    del x
    y = _matmul64(a, g, s["w"], s["offs"])
    if call == "quantize_gemm":
        return {"y": y, "g": gt}
    if call == "linear":
        return {"y": y}
    v = _matmul64(a, g, s["w_ab"], [0, 48, 96])
    t = torch.nn.functional.softplus(v[:, 48:] + s["dt_bias"].double())
    return {"qkv": y, "gates": torch.cat([torch.sigmoid(v[:, :48]), torch.exp(-s["a_log"].double().exp() * t)], 1)}
