"""dWg = x^T dL over token counts that the slices of the sum divide well, badly or not at all, against float64 from the operands as stored."""
import pytest
import torch

from paper_2506_04667_amd import binding as moe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("T", [511, 512, 513, 700, 768, 1000, 1023, 1087, 2049, 4097, 5000])
def test_slices(T, dtype):
    H, I, E, k = 72, 64, 8, 2
    print("case", T, dtype, flush=True)
    cfg = moe.make_config(T, H, I, E, k, 8.0, "identity", dtype)          # nothing is dropped
    td = moe.TORCH_DTYPE[dtype]
    g = torch.Generator().manual_seed(T)
    n = lambda scale, *s: (torch.randn(*s, generator=g) * scale).to(td)
    x, Wg, W1, W2, dout = n(1, T, H), n(H ** -0.5, H, E), n(H ** -0.5, E, H, I), n(I ** -0.5, E, I, H), n(1, T, H)
    ex = torch.rand(T, E, generator=g).argsort(1)[:, :k].int().contiguous()
    w = torch.softmax(torch.randn(T, k, generator=g), 1)
    dx, dWg, dgb, dW1, db1, dW2, db2 = (torch.full(s, float("nan"), device="cuda") for s in
                                        ((T, H), (H, E), (E,), (E, H, I), (E, I), (E, I, H), (E, H)))
    ws = torch.full((moe.moe_backward_workspace_bytes(cfg),), 0xff, dtype=torch.uint8, device="cuda")    # NaNs wherever nothing is written
    c = lambda t: t.cuda()
    moe.moe_backward(cfg, ws, c(x), c(Wg), c(W1), None, c(W2), None, c(ex), c(w), c(dout), dx, dWg, dgb, dW1, db1, dW2, db2)
    X, D = x.double(), dout.double()
    a = torch.einsum("th,ehi->tei", X, W1.double())
    dh = torch.einsum("th,eih->tei", D, W2.double())
    p = w.double() * (a * dh).sum(2).gather(1, ex.long())
    dl = p - w.double() * p.sum(1, keepdim=True)
    dL = torch.zeros(T, E).double().scatter_(1, ex.long(), dl)
    want = X.T @ dL
    # 16-bit: a and dL are rounded to storage, each by 2^-8 (bf16) or 2^-11 (f16) of its value at most; f32: sums over at most 72 terms
    # and 256 or 1024 tokens, a few roundings of 2^-24 in the norm
    tol = {"f32": 2e-6, "bf16": 2.0 ** -7, "f16": 2.0 ** -10}[dtype]
    assert float((dWg.double().cpu() - want).norm() / want.norm()) < tol
