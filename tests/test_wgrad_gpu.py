"""Weight gradients over a workspace full of NaNs.  In 16-bit storage at the edges of the kernel that makes them: remainders of its 128 x 256 tiles, sums that end inside a
32-slot step, long sums in slices, experts without rows, expert counts that do not divide by the 8 XCDs.  Against float64 on the CPU
under the routing tables, from the 16-bit operands the sums are made of: the roundings of h and da to storage (2^-9 in bf16, 2^-12 in f16,
relative to each term; independent, so the sum's 2-norm error stays below that of one operand), and of a before phi (as much again).  In fp32
the sums end with the 32-slot step of the last live slot, up to which alone their transposed operands are written."""
import numpy as np
import pytest
import torch

from paper_2506_04667_amd import binding as moe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("T,H,I,E,k,C", [
    (70, 64, 64, 3, 1, 0), (33, 8, 16, 5, 2, 0),     # far below one tile; 13 or 14 slots a sum
    (300, 136, 264, 12, 2, 0),                       # one tile and 8 columns / rows more; odd expert count
    (2600, 64, 72, 4, 2, 0),                         # slices: 1300 slots in few tiles
    (500, 256, 512, 2, 2, 97),                       # every expert full at 97 slots of 128
    (40, 64, 320, 16, 1, 0), (1, 64, 64, 8, 1, 0),   # experts without rows; a single slot in all
])
def test_weight_gradients(T, H, I, E, k, C, dtype):
    cfg = moe.make_config(T, H, I, E, k, 1.0, "identity", dtype, capacity_override=C)
    td = moe.TORCH_DTYPE[dtype]
    g = torch.Generator().manual_seed(T + H + I + E)
    n = lambda scale, *s: (torch.randn(*s, generator=g) * scale).to(td)
    x, Wg, W1, W2, dout = n(1, T, H), n(H ** -0.5, H, E), n(H ** -0.5, E, H, I), n(I ** -0.5, E, I, H), n(1, T, H)
    order = torch.rand(T, E, generator=g).argsort(1)[:, :k].int().contiguous()
    if E >= 8:
        order[order == 3] = 2 if k == 1 else 3       # an expert that nobody names
    w = torch.rand(T, k, generator=g) + 0.1
    w = (w / w.sum(1, keepdim=True)).float()
    grads = {m: torch.full(s, float("nan"), device="cuda") for m, s in
             (("dx", (T, H)), ("dWg", (H, E)), ("dgb", (E,)), ("dW1", (E, H, I)), ("db1", (E, I)), ("dW2", (E, I, H)), ("db2", (E, H)))}
    ws = torch.full((moe.moe_backward_workspace_bytes(cfg),), 0xff, dtype=torch.uint8, device="cuda")    # NaNs wherever nothing is written
    c = lambda t: t.cuda()
    moe.moe_backward(cfg, ws, c(x), c(Wg), c(W1), None, c(W2), None, c(order), c(w), c(dout), grads["dx"], grads["dWg"], grads["dgb"],
                     grads["dW1"], grads["db1"], grads["dW2"], grads["db2"])
    cap, _ = moe.moe_capacity(cfg)
    used = [0] * E
    want1, want2, dwg = torch.zeros(E, H, I).double(), torch.zeros(E, I, H).double(), torch.zeros(H, E).double()
    X, D = x.double(), dout.double()
    p = torch.zeros(T, k).double()
    for t in range(T):
        for j in range(k):
            e = int(order[t, j])
            used[e] += 1
            if used[e] > cap:
                continue
            a, dh = X[t] @ W1[e].double(), W2[e].double() @ D[t]
            want2[e] += torch.outer(a, D[t]) * float(w[t, j])
            want1[e] += torch.outer(X[t], dh) * float(w[t, j])
            p[t, j] = float(w[t, j]) * (a @ dh)
    dl = p - w.double() * p.sum(1, keepdim=True)
    for t in range(T):
        for j in range(k):
            dwg[:, int(order[t, j])] += X[t] * dl[t, j]
    # f32: a and dh are sums of at most 256 products, the gradients of at most 2600 more, an addition of two roundings for every
    # 32 / 6 products: sqrt((256 + 2600) / 16) 2^-24 = 8e-7
    tol = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11, "f32": 2e-6}[dtype]
    for name, want in (("dW1", want1), ("dW2", want2), ("dWg", dwg)):
        got = grads[name].double().cpu()
        assert torch.isfinite(got).all(), name
        # dWg of a token's one choice is zero (the softmax over one logit): sums of rounding, against the size of its terms
        size = max(float(want.norm()), float((X.norm() * p.abs().max())) * 1e-3 if name == "dWg" else 0.0)
        assert float((got - want).norm()) <= tol * size, (name, float((got - want).norm()) / size)
    for e in range(E):
        if used[e] == 0:
            assert float(grads["dW1"][e].abs().max()) == 0.0 and float(grads["dW2"][e].abs().max()) == 0.0


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_infinity_in_the_last_token_enters_the_gate_gradient_once(dtype):
    # 33 tokens: the sum over the tokens ends one k into a K-tile of 32, and the last token's x is infinite.  Its activations are all
    # below zero or -inf, so that after ReLU its logit gradients come from b2 alone and are finite: dWg is infinite where it chose
    # an expert, NaN (infinity times no gradient) elsewhere, and untouched in the other rows
    T, H, I, E, k = 33, 8, 8, 4, 2
    td = moe.TORCH_DTYPE[dtype]
    g = torch.Generator().manual_seed(3)
    n = lambda *s: torch.randn(*s, generator=g).to(td)
    x, Wg, W1, W2, dout, b2 = n(T, H), n(H, E), -n(E, H, I).abs(), n(E, I, H), n(T, H), n(E, H)
    x[T - 1] = 1.0
    x[T - 1, 0] = float("inf")
    order = torch.stack([torch.arange(T) % E, (torch.arange(T) + 1) % E], 1).int()
    w = torch.full((T, k), 0.5)
    out = [torch.full(s, 7.0, device="cuda") for s in ((T, H), (H, E), (E,), (E, H, I), (E, I), (E, I, H), (E, H))]
    cfg = moe.make_config(T, H, I, E, k, 4.0, "relu", dtype)
    ws = torch.full((moe.moe_backward_workspace_bytes(cfg),), 0xff, dtype=torch.uint8, device="cuda")
    c = lambda t: t.cuda()
    moe.moe_backward(cfg, ws, c(x), c(Wg), c(W1), None, c(W2), c(b2), c(order), c(w), c(dout), *out)
    dWg = out[1].cpu()
    assert order[T - 1].tolist() == [0, 1]
    p = [float(dout[T - 1].double() @ b2[e].double()) for e in (0, 1)]
    sign = 1.0 if p[0] > p[1] else -1.0                # of dl of the first choice; the second's is the opposite
    assert float(dWg[0, 0]) == sign * float("inf") and float(dWg[0, 1]) == -sign * float("inf"), dWg[0]
    assert bool(torch.isnan(dWg[0, 2:]).all()) and bool(torch.isfinite(dWg[1:]).all())
