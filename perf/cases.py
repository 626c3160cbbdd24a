"""Performance cases of the MoE layer: what a program that owns one GPU's share of an MoE layer has it do.

A case is one call (or one chain of staged calls) of the public entry points on device-resident tensors:
  forward   moe_forward: gate, routing, expert FFNs, combine;
  staged    moe_gate, moe_dispatch (which also packs the rows), moe_expert_ffn, moe_combine one by one, as a program
            with an exchange of its own between the stages calls them;
  backward  moe_backward under the routing that the forward's gate chose.
Inputs are drawn on the GPU with the distributions of the layer's synthetic workloads: x ~ N(0, 1), weights scaled by
1 / sqrt(fan-in), biases N(0, 0.5^2), Zipf-skewed gate biases where a case asks for them, dout ~ N(0, 1).
"""
import math

import torch

from paper_2506_04667_amd import binding as moe

_ITEM = {"f32": 4, "bf16": 2, "f16": 2}


def _case(name, path, dtype, T, H, I, E, k, cf=1.0, act="gelu_erf", bias=False, zipf=0.0, layout=False, choice_major=False):
    return {"name": name, "path": path, "dtype": dtype, "T": T, "H": H, "I": I, "E": E, "k": k, "capacity_factor": cf, "act": act,
            "bias": bias, "zipf_s": zipf, "capacity_mode": "layout" if layout else "per_choice",
            "drop_policy": "choice_major" if choice_major else "token_major"}


def listed():
    return [
        # the smallest configuration of the benchmark: a few tokens through a small layer, launches and latency only
        _case("fwd_tiny_f32", "forward", "f32", 128, 64, 128, 4, 1, cf=2.0, act="relu"),
        # a decode step: 64 tokens over 128 experts, so that the call is a read of the experts' weights
        _case("fwd_decode_bf16", "forward", "bf16", 64, 2048, 2048, 128, 2),
        # sizes that are multiples of 8 and nothing more, biases, tanh-GELU: an odd layer with an odd number of tokens
        _case("fwd_ragged_bf16", "forward", "bf16", 757, 328, 840, 8, 2, act="gelu_tanh", bias=True),
        # the small fp32 configuration: fewer tiles than the chip has CUs
        _case("fwd_small_f32", "forward", "f32", 2048, 1024, 4096, 16, 2, cf=1.25, act="gelu_tanh"),
        # Zipf-skewed routing in fp16: a few experts full to capacity, most with few rows or none
        _case("fwd_skew_f16_e128", "forward", "f16", 16384, 2048, 2048, 128, 2, cf=1.25, zipf=1.2),
        # the headline: 16K tokens, 128 local experts, top-2
        _case("fwd_paper_bf16_e128", "forward", "bf16", 16384, 2048, 2048, 128, 2),
        # one GPU's share of a 128-expert layer on eight GPUs: as many rows, an eighth of the weights
        _case("fwd_share_bf16_e16", "forward", "bf16", 16384, 2048, 2048, 16, 2),
        # many choices per token and wide rows
        _case("fwd_topk8_bf16_e32", "forward", "bf16", 4096, 7168, 2048, 32, 8),
        # the headline's layer in fp32 with 64 experts
        _case("fwd_paper_f32_e64", "forward", "f32", 16384, 2048, 2048, 64, 2),
        # the stages one by one with packed rows, as around an exchange between GPUs; prefill of 4096 tokens
        _case("staged_bf16_e16", "staged", "bf16", 4096, 2048, 2048, 16, 2),
        # training: gradients of the small layer in fp32 and of the headline's layer in bf16
        _case("bwd_small_f32", "backward", "f32", 2048, 1024, 4096, 16, 2, cf=1.25, act="gelu_tanh"),
        _case("bwd_paper_bf16_e128", "backward", "bf16", 16384, 2048, 2048, 128, 2),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# bounds of a drawn case: the listed cases' own largest figures
_MOST_WEIGHTS = 128 * 2048 * 2048                  # elements of W1 (and of W2)
_MOST_GFLOP = {"f32": 275.0, "bf16": 1000.0, "f16": 1000.0}


def draw(rng):
    while True:
        path = rng.choice(["forward"] * 6 + ["staged"] * 2 + ["backward"] * 3)
        dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
        T = _log_uniform(rng, 16, 16384)
        step = rng.choice([8, 64, 64, 256])        # layer widths: multiples of 8, of 64, and round ones
        if path == "backward":
            step = max(step, 64)                   # layers that are trained have round widths
        H = max(step, _log_uniform(rng, 64, 7168) // step * step)
        I = max(step, _log_uniform(rng, max(64, H // 4), min(14336, 4 * H)) // step * step)
        E = rng.choice([4, 8, 16, 24, 32, 48, 64, 96, 128])
        k = rng.choice([1, 2, 2, 2, 4, 8])
        cf = rng.choice([1.0, 1.0, 1.25, 2.0])
        if k > E or E * H * I > _MOST_WEIGHTS:
            continue
        gflop = 4e-9 * T * k * H * I * (3 if path == "backward" else 1)
        if gflop > _MOST_GFLOP[dtype] or gflop < 0.004 or T * k * max(H, I) > 4096 * 8 * 7168:
            continue
        c = _case(None, path, dtype, T, H, I, E, k, cf=cf, act=rng.choice(["gelu_erf", "gelu_erf", "gelu_tanh", "relu"]),
                  bias=rng.random() < 0.3, zipf=rng.choice([0.0, 0.0, 0.0, 1.2]), layout=rng.random() < 0.15,
                  choice_major=rng.random() < 0.15)
        del c["name"]
        return c


def _config(case):
    return moe.make_config(case["T"], case["H"], case["I"], case["E"], case["k"], case["capacity_factor"], case["act"], case["dtype"],
                           drop_policy=case["drop_policy"], capacity_mode=case["capacity_mode"])


def prepare(case, seed):
    """Weights, inputs, the output buffers and the workspace of one layer."""
    T, H, I, E, k = (case[n] for n in ("T", "H", "I", "E", "k"))
    td = moe.TORCH_DTYPE[case["dtype"]]
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(scale, *shape, dtype=td):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, scale, generator=gen)

    moe.moe_init()
    cfg = _config(case)
    s = {"path": case["path"], "cfg": cfg, "buffers": moe.Buffers(cfg), "x": normal(1.0, T, H), "Wg": normal(1 / math.sqrt(H), H, E),
         "W1": normal(1 / math.sqrt(H), E, H, I), "W2": normal(1 / math.sqrt(I), E, I, H), "b1": None, "b2": None, "gate_bias": None}
    if case["bias"]:
        s["b1"], s["b2"] = normal(0.5, E, I), normal(0.5, E, H)
    if case["zipf_s"] > 0.0:
        rank = torch.randperm(E, generator=gen, device="cuda") + 1
        s["gate_bias"] = (-case["zipf_s"] * rank.double().log()).float()
    b = s["buffers"]
    if case["path"] == "staged":
        b.alloc_staged()
    if case["path"] == "backward":
        s["dout"] = normal(1.0, T, H)
        s["workspace"] = torch.empty(moe.moe_backward_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
        s["grads"] = {n: torch.empty(shape, dtype=torch.float32, device="cuda")
                      for n, shape in (("dx", (T, H)), ("dWg", (H, E)), ("dgate_bias", (E,)), ("dW1", (E, H, I)), ("db1", (E, I)),
                                       ("dW2", (E, I, H)), ("db2", (E, H)))}
        moe.moe_gate(cfg, b.workspace, s["x"], s["Wg"], s["gate_bias"], b.gate_logits, b.topk_expert, b.topk_weight)
        b.workspace = None
    return s


def run(s):
    cfg, b = s["cfg"], s["buffers"]
    if s["path"] == "backward":
        g = s["grads"]
        moe.moe_backward(cfg, s["workspace"], s["x"], s["Wg"], s["W1"], s["b1"], s["W2"], s["b2"], b.topk_expert, b.topk_weight, s["dout"],
                         g["dx"], g["dWg"], g["dgate_bias"], g["dW1"], g["db1"], g["dW2"], g["db2"])
        return g
    if s["path"] == "staged":
        moe.moe_gate(cfg, b.workspace, s["x"], s["Wg"], s["gate_bias"], b.gate_logits, b.topk_expert, b.topk_weight)
        moe.moe_dispatch(cfg, b.workspace, s["x"], b.topk_expert, b.topk_weight, b.slot, b.expert_demand, b.slot_token, b.slot_weight, b.xe)
        moe.moe_expert_ffn(cfg, b.workspace, b.xe, b.expert_demand, s["W1"], s["b1"], s["W2"], s["b2"], b.y)
        moe.moe_combine(cfg, b.y, b.topk_expert, b.topk_weight, b.slot, b.out)
    else:
        moe.moe_forward(cfg, b.workspace, s["x"], s["Wg"], s["gate_bias"], s["W1"], s["b1"], s["W2"], s["b2"], b.out, b.gate_logits,
                        b.topk_expert, b.topk_weight, b.slot, b.expert_demand)
    outputs = {"out": b.out, "gate_logits": b.gate_logits, "topk_expert": b.topk_expert, "topk_weight": b.topk_weight, "slot": b.slot,
               "expert_demand": b.expert_demand}
    if s["path"] == "staged":                      # rows of xe and y beyond an expert's live rows are not written: zero since prepare()
        outputs.update(xe=b.xe, y=b.y, slot_token=b.slot_token, slot_weight=b.slot_weight)
    return outputs


def _expected_rows(case):
    """Expected (kept rows over all experts, experts with a row): the binomial demand of each expert, cut at the capacity."""
    T, E, k, s = case["T"], case["E"], case["k"], case["zipf_s"]
    C, _ = moe.moe_capacity(_config(case))
    if s > 0.0:
        # logits are N(0, 1) - s ln(rank): how often each rank is among the k largest, from a fixed sample of tokens
        sample = 8192
        logits = torch.randn(sample, E, generator=torch.Generator().manual_seed(1)) - s * torch.arange(1, E + 1).log()
        p = (torch.bincount(logits.topk(k).indices.flatten(), minlength=E) / sample).tolist()
    else:
        p = [k / E] * E
    rows = live = 0.0
    for q in p:
        mean, sd = T * q, math.sqrt(max(T * q * (1.0 - q), 1e-12))
        z = (C - mean) / sd
        pdf, cdf = math.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi), 0.5 * (1.0 + math.erf(z / math.sqrt(2.0)))
        rows += min(mean, max(0.0, mean - ((mean - C) * (1.0 - cdf) + sd * pdf)))
        live += 1.0 - (1.0 - q) ** T
    return rows, live


def work(case):
    """What the path cannot do without: every input (weights of experts with rows) read once, every output written once."""
    T, H, I, E, k = (case[n] for n in ("T", "H", "I", "E", "k"))
    el = _ITEM[case["dtype"]]
    rows, live = _expected_rows(case)
    weights = live * 2.0 * H * I * el + (live * (H + I) * el if case["bias"] else 0.0)
    gate = 2.0 * T * H * E
    if case["path"] == "backward":
        # in: x, dout, Wg, W1, W2, routing; out: dx, dWg, dW1, dW2 and the bias gradients, fp32.  Products: the first FFN
        # product again, the two data gradients, the two weight gradients; the gate's two
        moved = 2.0 * T * H * el + H * E * el + weights + T * k * 8.0 + 4.0 * (T * H + H * E + E + E * (2.0 * H * I + H + I))
        return {"bytes": moved, "flops": 5 * 2.0 * rows * H * I + 2.0 * H * T * k * 2}
    moved = T * H * el + H * E * el + weights + T * H * el + T * E * 4.0 + T * k * 12.0 + E * 4.0
    if case["path"] == "staged":
        C, _ = moe.moe_capacity(_config(case))
        moved += 4.0 * rows * H * el + E * C * 8.0  # xe and y are written by one call and read by the next
    return {"bytes": moved, "flops": 4.0 * rows * H * I + gate + 2.0 * rows * H}


def tolerance(case):
    """About four times what the path differs by from the same layer in float64 under the same routing, measured over the listed cases
    and thirty drawn ones (largest relative 2-norm; largest element): forward f32 1.2e-6, 8.6e-6; bf16 2.9e-3, 1.8e-2; f16 3.6e-4,
    5.5e-3; gradients f32 2.1e-6, 1.1e-5; bf16 3.6e-3, 6e-2; f16 4.1e-4, 2.8e-3.  The routing's whole values differ only where two logits
    tie to within the rounding of a sum, which moves the later slots of two experts."""
    if case["path"] == "backward":
        rel, most = {"f32": (8e-6, 5e-5), "bf16": (1.4e-2, 0.25), "f16": (1.6e-3, 0.012)}[case["dtype"]]
    else:
        rel, most = {"f32": (5e-6, 3.5e-5), "bf16": (1.2e-2, 0.072), "f16": (1.5e-3, 0.022)}[case["dtype"]]
    return {"rel": rel, "max": most, "differ": 2e-3}
