"""The erf-GELU of 16-bit layers whose shapes the weight-streaming kernel's whole K-tiles do not take: within the rounding to storage of the
exact function over [-10, 10], also far below zero, where the streaming kernel's clamped polynomial is off by more than the value."""
import math

import pytest
import torch

from paper_2506_04667_amd import binding as moe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("E,H,I", [
    (2, 264, 264), (2, 256, 200), (2, 128, 128),         # few tasks: K no multiple of 64; columns; K below the streaming kernel's
    (64, 264, 264),                                      # the streaming kernel with a last pair of K-tiles that is filled up
])
def test_tail(E, H, I, dtype):
    # row r of every expert is the unit vector of h = r, so x W1 is row r of W1 exactly; W2 is the identity, so y = phi(W1)
    td = moe.TORCH_DTYPE[dtype]
    W1 = torch.linspace(-10.0, 10.0, E * H * I, dtype=torch.float64)[torch.randperm(E * H * I, generator=torch.Generator().manual_seed(1))]
    W1 = W1.to(td).reshape(E, H, I)
    cfg = moe.make_config(E * H, H, I, E, 1, 1.0, "gelu_erf", dtype)
    b = moe.Buffers(cfg).alloc_staged()
    assert b.C == H
    b.xe.zero_()
    b.xe[:, :H] = torch.eye(H, dtype=td)
    b.expert_demand.fill_(H)
    W2 = torch.eye(I, H, dtype=td).repeat(E, 1, 1)
    moe.moe_expert_ffn(cfg, b.workspace, b.xe, b.expert_demand, W1.cuda(), None, W2.cuda(), None, b.y)
    v = W1.double()
    want = 0.5 * v * torch.erfc(-v / math.sqrt(2))
    # two roundings to storage (fp16: to 2^-25 at least), and 0.75e-7 |v| of the erf with an fp32 sum and product on top
    bound = 2 * 2.0 ** (-8 if dtype == "bf16" else -11) * want.abs() + 1.5e-7 * v.abs() + (0.0 if dtype == "bf16" else 2 * 2.0 ** -25)
    err = (b.y[:, :H, :I].double().cpu() - want).abs()
    i = int((err - bound).argmax())
    assert bool((err <= bound).all()), (float(v.flatten()[i]), float(want.flatten()[i]), float(err.flatten()[i]))
