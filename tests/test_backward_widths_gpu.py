"""moe_backward at row widths whose last pass over a row leaves most lanes of a wavefront idle (H / 8 or H / 4 chunks of 16
bytes, one to k more than a multiple of 64) and at expert counts just above a multiple of 64 with many choices per token:
every gradient against the oracle, with the tolerances derived in test_backward_gpu.py."""
import numpy as np
import pytest
import torch

from paper_2506_04667_amd.inputs import WORKLOADS, make_inputs, scaled

import parity
from test_backward_gpu import NAMES, TOL, _backward, parity_dtype

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    dict(T=150, H=520, I=64, E=4, k=2, dtype="bf16"),        # 65 chunks
    dict(T=150, H=528, I=72, E=12, k=8, dtype="f16"),        # 66 chunks, eight choices
    dict(T=90, H=264, I=64, E=72, k=12, dtype="f32"),        # 66 chunks; 72 experts, twelve choices
])
def test_gradients_at_widths_with_a_short_last_pass(oracle, case):
    w = scaled(WORKLOADS["paper_bf16_e128"], name="widths", seed=81, capacity_factor=1.25, with_bias=True, act="gelu_tanh", **case)
    print("case", w, flush=True)
    cpu = make_inputs(w)
    dev = parity.to_device(cpu)
    b, host = parity.gpu_forward(w, dev)
    dout = torch.from_numpy(np.random.default_rng(8).standard_normal((w.T, w.H)).astype(np.float32)).to(parity_dtype(w.dtype))
    g = _backward(w, dev, host, dout.cuda())
    ref = oracle.backward(cpu["x"], cpu["Wg"], None, cpu["W1"], cpu["b1"], cpu["W2"], cpu["b2"], host["topk_expert"], host["slot"],
                          dout.double().numpy(), w.T, w.H, w.I, w.E, w.act, w.dtype)
    for n in NAMES:
        parity.assert_close(g[n].double().cpu().numpy(), ref[n], TOL[w.dtype], n)
