"""GPU parity of the backward pass: moe_backward, called through the C ABI, against oracle_backward under the
routing the GPU's own forward pass chose, on the same seeded inputs.

Tolerances (derived from the arithmetic: the HIP path keeps xe, a, h = w phi(a), da and dL in the storage dtype
between kernels, because they are matrix-core operands, takes dout as it is and accumulates in fp32; the oracle is double
throughout): |gpu - ref| <= tol |ref| + tol rms(ref) with
  tol = 3e-2 for bf16 storage: a weight gradient is a sum over an expert's rows of products with a factor that was rounded
        to storage (h, after a; or da); a CPU emulation of those roundings against the oracle
        (tests/test_oracle_backward_pins.py) reaches 1.8e-2 of the rms at H = 328, I = 840 for the worst of 2 M elements;
        half as much again for larger tensors.  fp16 rounds at an eighth of that: 5e-3;
  tol = 1e-4 for fp32 storage (fp32 accumulation over up to a few thousand terms, three chained contractions, the
        approximate erf/tanh in the activation's derivative)."""
import numpy as np
import pytest
import torch

from paper_2506_04667_amd import binding as moe
from paper_2506_04667_amd.inputs import WORKLOADS, make_inputs, scaled

import parity

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 3e-2, "f16": 5e-3}
NAMES = ["dx", "dWg", "dgate_bias", "dW1", "db1", "dW2", "db2"]


def _backward(w, dev, host, dout):
    cfg = moe.config_of(w)
    T, H, I, E = w.T, w.H, w.I, w.E
    f = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device="cuda")   # every element must be written
    g = {"dx": f(T, H), "dWg": f(H, E), "dgate_bias": f(E), "dW1": f(E, H, I), "db1": f(E, I), "dW2": f(E, I, H), "db2": f(E, H)}
    ws = torch.empty(moe.moe_backward_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    te = torch.from_numpy(host["topk_expert"]).cuda()
    tw = torch.from_numpy(host["topk_weight"]).cuda()
    moe.moe_backward(cfg, ws, dev["x"], dev["Wg"], dev["W1"], dev["b1"], dev["W2"], dev["b2"], te, tw, dout,
                     g["dx"], g["dWg"], g["dgate_bias"], g["dW1"], g["db1"], g["dW2"], g["db2"])
    torch.cuda.synchronize()
    return g


@pytest.mark.parametrize("case", [
    # fp32: ragged shapes, drops, biases, gate bias
    dict(T=300, H=64, I=72, E=6, k=2, capacity_factor=0.8, dtype="f32", with_bias=True, act="gelu_tanh", gate_bias=True),
    dict(T=257, H=40, I=136, E=3, k=3, capacity_factor=1.0, dtype="f32", with_bias=False, act="gelu_erf"),
    dict(T=130, H=72, I=64, E=5, k=1, capacity_factor=0.5, dtype="f32", with_bias=True, act="relu"),
    # 16-bit in tiles of 128 x 128, with K no multiple of 64 and with whole K-tiles
    dict(T=757, H=328, I=840, E=8, k=2, capacity_factor=1.0, dtype="bf16", with_bias=True, act="gelu_tanh"),
    dict(T=1500, H=256, I=512, E=8, k=2, capacity_factor=1.0, dtype="bf16", with_bias=True, act="gelu_erf", gate_bias=True),
    dict(T=900, H=256, I=256, E=12, k=3, capacity_factor=0.7, dtype="f16", with_bias=False, act="identity",
         drop_policy="choice_major"),
    # experts nobody picks and tokens that lose every choice
    dict(T=400, H=64, I=64, E=8, k=2, capacity_factor=0.25, dtype="f32", with_bias=True, act="gelu_erf", empty=(2, 5)),
    # more than 2048 tokens: the gate-weight gradient is a sum of partial products over token slices (here 2 slices of
    # 1088 tokens: the last one runs 76 rows past T into the zero padding)
    dict(T=2100, H=64, I=72, E=8, k=2, capacity_factor=1.0, dtype="f32", with_bias=False, act="relu", gate_bias=True),
    dict(T=3333, H=128, I=64, E=12, k=3, capacity_factor=1.0, dtype="bf16", with_bias=True, act="gelu_tanh"),
    # the paper's layer shape per expert (H = I = 2048, 256 slots, top-2, erf-GELU, bf16) with 16 experts: the tile
    # shapes, K = 256 weight-gradient GEMMs and weight-streaming kernels of the full-size backward pass
    dict(T=2048, H=2048, I=2048, E=16, k=2, capacity_factor=1.0, dtype="bf16", with_bias=False, act="gelu_erf"),
])
def test_backward_matches_the_oracle(oracle, case):
    case = dict(case)
    empty = case.pop("empty", ())
    use_gate_bias = case.pop("gate_bias", False)
    w = scaled(WORKLOADS["paper_bf16_e128"], name="backward", seed=51, **case)
    print("case", w, flush=True)
    cpu = make_inputs(w)
    gb = None
    if use_gate_bias or empty:
        gb = torch.from_numpy(np.random.default_rng(7).standard_normal(w.E).astype(np.float32) * 0.5)
        gb[list(empty)] = -1.0e4
        cpu["gate_bias"] = gb
    dev = parity.to_device(cpu)
    b, host = parity.gpu_forward(w, dev)
    for e in empty:
        assert host["expert_demand"][e] == 0
    dout_cpu = torch.from_numpy(np.random.default_rng(8).standard_normal((w.T, w.H)).astype(np.float32)).to(parity_dtype(w.dtype))
    g = _backward(w, dev, host, dout_cpu.cuda())
    ref = oracle.backward(cpu["x"], cpu["Wg"], None if gb is None else gb.numpy(), cpu["W1"], cpu["b1"], cpu["W2"], cpu["b2"],
                          host["topk_expert"], host["slot"], dout_cpu.double().numpy(), w.T, w.H, w.I, w.E, w.act, w.dtype)
    rep = {}
    for n in NAMES:
        if n in ("db1", "db2") and not w.with_bias:
            pass                                              # the bias gradients are defined (and checked) with or without biases
        rep[n] = parity.assert_close(g[n].double().cpu().numpy(), ref[n], TOL[w.dtype], n)
    print("  ", {n: "%.2e" % v for n, v in rep.items()}, flush=True)
    for e in empty:                                           # an expert without kept rows gets exact zeros
        assert float(g["dW1"][e].abs().max()) == 0.0 and float(g["dW2"][e].abs().max()) == 0.0
    all_dropped = (host["slot"] < 0).all(axis=1)
    if all_dropped.any():                                     # a token with no kept pair reaches nothing
        assert float(g["dx"][torch.from_numpy(all_dropped).cuda()].abs().max()) == 0.0
    # determinism: a second call gives the same bits
    g2 = _backward(w, dev, host, dout_cpu.cuda())
    for n in NAMES:
        assert torch.equal(g[n], g2[n]), n


def test_bf16_gradients_are_rounded_no_more_often_than_they_have_to_be(oracle):
    # relative 2-norms against the oracle: what the emulated roundings give (a, h, da), and a tenth for the fp32 sums and the
    # approximate activation; one more rounding of any of these operands would add 40 % to da's or h's error
    from test_oracle_backward_pins import emulated_gradients
    w = scaled(WORKLOADS["paper_bf16_e128"], name="roundings", seed=51, T=757, H=328, I=840, E=8, k=2, with_bias=True, act="gelu_tanh")
    cpu = make_inputs(w)
    dev = parity.to_device(cpu)
    _, host = parity.gpu_forward(w, dev)
    dout = torch.from_numpy(np.random.default_rng(8).standard_normal((w.T, w.H)).astype(np.float32)).to(torch.bfloat16)
    g = _backward(w, dev, host, dout.cuda())
    ref = oracle.backward(cpu["x"], cpu["Wg"], None, cpu["W1"], cpu["b1"], cpu["W2"], cpu["b2"], host["topk_expert"], host["slot"],
                          dout.double().numpy(), w.T, w.H, w.I, w.E, w.act, w.dtype)
    emulated = emulated_gradients(cpu, host["topk_expert"], host["topk_weight"], host["slot"], dout, w.E)
    for n, v in emulated.items():
        err = np.linalg.norm(g[n].double().cpu().numpy() - ref[n])
        assert err < 1.1 * np.linalg.norm(v - ref[n]), (n, err / np.linalg.norm(ref[n]), np.linalg.norm(v - ref[n]) / np.linalg.norm(ref[n]))


def parity_dtype(name):
    return {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[name]


def test_backward_argument_checks():
    cfg = moe.make_config(128, 64, 128, 4, 1, 2.0, "relu", "f32")
    n = moe.moe_backward_workspace_bytes(cfg)
    assert n > 0
    t = torch.zeros(64, device="cuda")
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    with pytest.raises(moe.MoeError) as e:
        moe.moe_backward(cfg, small, t, t, t, None, t, None, t, t, t, t, t, t, t, t, t, t)
    assert e.value.code == -3
    with pytest.raises(moe.MoeError) as e:
        moe.moe_backward_workspace_bytes(moe.make_config(128, 64, 128, 128, 65, 2.0, "relu", "f32"))
    assert e.value.code == -2                                 # more than 64 choices per token
