"""moe_backward in 16-bit layers of few tasks, where the 128 x 128 tiles read weights [n][k] as they are stored (the data gradients) and the
weight gradients' kernel activations [slot][m].  Ragged columns and rows of both, experts with one row up to several row tiles; every
gradient against the oracle with the tolerances derived in test_backward_gpu.py, and bit-identical when the call is repeated.  (The
weight-streaming kernel's forms of the same products: test_backward_streaming_gpu.py.)"""
import numpy as np
import pytest
import torch

from paper_2506_04667_amd import binding as moe
from paper_2506_04667_amd.inputs import WORKLOADS, make_inputs, scaled

import parity
from test_backward_gpu import NAMES, TOL, _backward, parity_dtype

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    dict(T=1000, H=320, I=456, E=8, k=2, dtype="bf16"),                 # dh: K = 320, ragged N; dW2 456 ragged rows, dW1 ragged columns
    dict(T=1000, H=264, I=384, E=8, k=2, dtype="f16"),                  # dxe: K = 384, N = 264; dW1 264 rows
    dict(T=800, H=256, I=256, E=8, k=2, dtype="bf16"),                  # the shortest K the streaming kernel takes of [n][k] weights
    dict(T=800, H=192, I=512, E=8, k=2, dtype="bf16"),                  # too few for dh there, not for dxe
    dict(T=2000, H=256, I=512, E=12, k=2, dtype="f16", zipf_s=1.4, capacity_factor=3.0),    # one row up to four row tiles
])
def test_gradients_with_operands_as_stored(oracle, case):
    w = scaled(WORKLOADS["paper_bf16_e128"], name="layouts", seed=83, **{"capacity_factor": 1.0, "with_bias": True, "act": "gelu_tanh", **case})
    print("case", w, flush=True)
    cfg, cus = moe.config_of(w), torch.cuda.get_device_properties(0).multi_processor_count
    assert [moe.moe_gemm16_kernel(cfg, p, cus) for p in ("dh", "dxe", "dw")] == ["128", "128", "wgrad"]
    cpu = make_inputs(w)
    dev = parity.to_device(cpu)
    b, host = parity.gpu_forward(w, dev)
    dout = torch.from_numpy(np.random.default_rng(8).standard_normal((w.T, w.H)).astype(np.float32)).to(parity_dtype(w.dtype))
    g = _backward(w, dev, host, dout.cuda())
    gb = cpu.get("gate_bias")
    ref = oracle.backward(cpu["x"], cpu["Wg"], None if gb is None else gb.numpy(), cpu["W1"], cpu["b1"], cpu["W2"], cpu["b2"],
                          host["topk_expert"], host["slot"], dout.double().numpy(), w.T, w.H, w.I, w.E, w.act, w.dtype)
    again = _backward(w, dev, host, dout.cuda())
    for n in NAMES:
        parity.assert_close(g[n].double().cpu().numpy(), ref[n], TOL[w.dtype], n)
        assert torch.equal(g[n], again[n]), n
