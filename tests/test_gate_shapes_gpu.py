"""The fused gate where rows of x end inside a K-tile, where rows of Wg do not start on 16-byte chunks (E a multiple of 4 but not of 8 in
16-bit storage) and where the sums over H are made in slices by several workgroups, against the oracle: logits within the bar of the storage
type, selection exact under the GPU's logits, and the staged call and the single-launch layer with the same bits as the forward call."""
import numpy as np
import pytest
import torch

from paper_2506_04667_amd import binding as moe
from paper_2506_04667_amd.inputs import WORKLOADS, make_inputs, scaled

import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,E,k,dtype,bias", [
    (65, 8, 8, 2, "bf16", True), (64, 72, 16, 1, "f16", False), (100, 1000, 24, 3, "bf16", True),        # 8 and 40 k in the last K-tile
    (33, 40, 4, 2, "f32", False), (130, 328, 136, 4, "f32", True),
    (70, 64, 4, 1, "bf16", True), (129, 200, 12, 3, "f16", True), (64, 128, 124, 5, "bf16", False), (50, 72, 132, 2, "f16", False),
    (10, 256, 252, 9, "bf16", True),
    (64, 1536, 128, 2, "bf16", True), (1, 7168, 32, 8, "f16", False), (200, 4440, 4, 2, "bf16", True),     # slices of 4 to 7 K-tiles
    (1000, 2048, 64, 2, "f32", True), (5000, 1640, 200, 3, "bf16", False), (17, 552, 8, 2, "f32", False),
])
def test_gate_shapes(oracle, T, H, E, k, dtype, bias):
    w = scaled(WORKLOADS["paper_bf16_e128"], name="gate", T=T, H=H, I=8, E=E, k=k, dtype=dtype, seed=37)
    cpu = make_inputs(w)
    gb = torch.from_numpy(np.random.default_rng(5).standard_normal(E).astype(np.float32)) if bias else None
    cfg = moe.config_of(w)
    b = moe.Buffers(cfg)
    b.workspace.fill_(255)
    b.gate_logits.fill_(float("nan"))
    moe.moe_gate(cfg, b.workspace, cpu["x"].cuda(), cpu["Wg"].cuda(), None if gb is None else gb.cuda(), b.gate_logits, b.topk_expert, b.topk_weight)
    got = b.gate_logits.cpu().numpy()
    ref = oracle.gate_logits(cpu["x"], cpu["Wg"], None if gb is None else gb.numpy(), T, H, E, dtype)
    parity.assert_close(got, ref, parity.TOL[dtype] if dtype == "f32" else 1e-4, "gate_logits")    # fp32 sums of exact products
    te, tw = oracle.topk(got, k)
    np.testing.assert_array_equal(b.topk_expert.cpu().numpy(), te)
    np.testing.assert_allclose(b.topk_weight.cpu().numpy(), tw, rtol=1e-5, atol=1e-7)


@pytest.mark.parametrize("case", [
    dict(T=200, H=2048, I=256, E=16, k=2, dtype="bf16"), dict(T=90, H=1536, I=512, E=40, k=1, dtype="f16"),
])
def test_sliced_gate_has_the_same_bits_in_every_call(case):
    w = scaled(WORKLOADS["paper_bf16_e128"], name="slices", seed=62, act="relu", **case)
    dev = parity.to_device(make_inputs(w))
    b0, host0 = parity.gpu_forward(w, dev)
    b1, host1 = parity.gpu_forward(w, dev, staged=True)
    b2, host2 = parity.gpu_forward(scaled(w, flags=moe.FLAG_LAYER_SINGLE_LAUNCH), dev)
    for b, host in ((b1, host1), (b2, host2)):
        for n in host0:
            np.testing.assert_array_equal(host0[n], host[n], err_msg=n)
        assert torch.equal(b0.out, b.out)


def test_infinity_beyond_the_last_k_stays_out():
    # the K-tile that ends beyond H must not read the next token's row or the next rows of memory: here those are infinite
    T, H, E = 3, 72, 8
    for dtype in ("bf16", "f32"):
        cfg = moe.make_config(T, H, 8, E, 1, 4.0, "relu", dtype)
        td = moe.TORCH_DTYPE[dtype]
        x = torch.ones(T, H, dtype=td, device="cuda")
        x[1] = float("inf")
        b = moe.Buffers(cfg)
        big = torch.full((H + 64, E), float("inf"), dtype=td, device="cuda")
        big[:H] = 1.0
        moe.moe_gate(cfg, b.workspace, x, big[:H], None, b.gate_logits, b.topk_expert, b.topk_weight)
        got = b.gate_logits.cpu()
        assert bool((got[0] == H).all()) and bool((got[2] == H).all()) and bool(torch.isinf(got[1]).all())
