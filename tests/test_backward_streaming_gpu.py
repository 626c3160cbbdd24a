"""moe_backward on the kernels of large layers, over a workspace full of NaNs, against float64 under the same routing: the weight-streaming
kernel's forms for weights [n][k] (the data gradients: K a multiple of 64 from 256 on) and activations [slot][m] (the weight gradients), with
ragged rows and columns, the shortest K of each, capacities below the padded one, experts with no rows, few or all; and in fp32 weight gradients
whose sums end far below the padded capacity, in each body of the fp32 tiles and in spans.

Bounds (relative 2-norms).  16-bit: a, h, da, dxe and dL are rounded to storage, each by at most 2^-9 (bf16) or 2^-12 (f16) in the norm, the
identity for phi; dW1, dW2, db1 and dx hold two such roundings at most, dWg two and their difference: 2^-8 and 2^-7.  fp32: an addition
of two roundings for every 32 / 6 products, counted with partial sums as large as the whole: sqrt(n / 8) 2^-24 for n products."""
import math

import pytest
import torch

from paper_2506_04667_amd import binding as moe

pytestmark = pytest.mark.gpu


def run(T, H, I, E, k, C, act, dtype, empty=()):
    """The gradients and, in float64, what they should be; the experts' kept rows; the configuration."""
    cfg = moe.make_config(T, H, I, E, k, 1.0, act, dtype, capacity_override=C)
    td = moe.TORCH_DTYPE[dtype]
    gen = torch.Generator(device="cuda").manual_seed(T + H + I + E)
    n = lambda scale, *s: (torch.empty(s, device="cuda").normal_(generator=gen) * scale).to(td)
    x, Wg, W1, W2, dout = n(1, T, H), n(H ** -0.5, H, E), n(H ** -0.5, E, H, I), n(I ** -0.5, E, I, H), n(1, T, H)
    score = torch.empty(T, E, device="cuda").uniform_(generator=gen)
    score[:, list(empty)] = -1.0
    ex = score.topk(k, 1).indices.int()
    w = torch.softmax(torch.empty(T, k, device="cuda").normal_(generator=gen), 1)
    g = {m: torch.full(s, float("nan"), device="cuda") for m, s in
         (("dx", (T, H)), ("dWg", (H, E)), ("dgb", (E,)), ("dW1", (E, H, I)), ("db1", (E, I)), ("dW2", (E, I, H)), ("db2", (E, H)))}
    ws = torch.full((moe.moe_backward_workspace_bytes(cfg),), 0xff, dtype=torch.uint8, device="cuda")
    moe.moe_backward(cfg, ws, x, Wg, W1, None, W2, None, ex, w, dout, *g.values())
    ref = {m: torch.zeros(v.shape, dtype=torch.float64, device="cuda") for m, v in g.items()}
    X, D, G, p = x.double(), dout.double(), Wg.double(), torch.zeros(T, k, dtype=torch.float64, device="cuda")
    rows = []
    for e in range(E):
        t, j = (ex == e).nonzero(as_tuple=True)            # token order, which is slot order
        t, j = t[:C], j[:C]
        rows.append(len(t))
        a, dh, we = X[t] @ W1[e].double(), D[t] @ W2[e].double().t(), w[t, j].double()[:, None]
        h, d = (a.clamp(min=0), (a > 0).double()) if act == "relu" else (a, 1.0)
        p[t, j] = we[:, 0] * (h * dh).sum(1)
        da = we * dh * d
        ref["dW2"][e], ref["dW1"][e] = (we * h).t() @ D[t], X[t].t() @ da
        ref["db1"][e], ref["db2"][e] = da.sum(0), (we * D[t]).sum(0)
        ref["dx"].index_add_(0, t, da @ W1[e].double().t())
    dl = p - w.double() * p.sum(1, keepdim=True)
    dL = torch.zeros(T, E, dtype=torch.float64, device="cuda").scatter_(1, ex.long(), dl)
    ref["dx"] += dL @ G.t()
    ref["dWg"], ref["dgb"] = X.t() @ dL, dL.sum(0)
    return cfg, g, ref, rows


def check(g, ref, rows, bounds):
    for m, bound in bounds.items():
        err = float((g[m].double() - ref[m]).norm() / ref[m].norm())
        assert err < bound, (m, err, bound)
    for e, r in enumerate(rows):                           # every expert by itself: a mistake in one does not hide behind the others
        for m in ("dW1", "dW2"):
            if r == 0:
                assert float(g[m][e].abs().max()) == 0.0, (m, e)
            else:
                err = float((g[m][e].double() - ref[m][e]).norm() / ref[m][e].norm())
                assert err < 2 * bounds[m], (m, e, err)


@pytest.mark.parametrize("T,H,I,E,k,C,dtype,empty,on", [
    # [slot][m] activations: one tile and 8 columns each way, full experts and an empty one; C_pad = 256 is the shortest K
    (16384, 264, 264, 128, 2, 250, "f16", (3,), ("128", "128", "stream")),
    (3500, 1032, 1000, 32, 2, 200, "bf16", (0, 31), ("128", "128", "stream")),
    # an odd number of experts, five and ten K-tiles of which the last ones are empty
    (1000, 2056, 1992, 9, 2, 253, "bf16", (), ("128", "128", "stream")),
    (2600, 2056, 1992, 9, 2, 600, "f16", (5,), ("128", "128", "stream")),
    # [n][k] weights: the shortest K and a ragged N for dh, then for dxe; few rows
    (4800, 256, 392, 64, 2, 200, "bf16", (7,), ("stream", "128", "wgrad")),
    (4800, 392, 256, 64, 2, 200, "f16", (63,), ("128", "stream", "wgrad")),
    (600, 320, 264, 130, 2, 12, "f16", (), ("stream", "128", "wgrad")),
    # 256-row tiles and 128-row ones, several K-tile pairs, both gradients
    (9000, 448, 512, 40, 2, 500, "bf16", (39,), ("stream", "stream", "wgrad")),
])
def test_streaming_forms(T, H, I, E, k, C, dtype, empty, on):
    print("case", T, H, I, E, k, C, dtype, flush=True)
    cfg, g, ref, rows = run(T, H, I, E, k, C, "identity", dtype, empty)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert tuple(moe.moe_gemm16_kernel(cfg, p, cus) for p in ("dh", "dxe", "dw")) == on
    u = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype]
    check(g, ref, rows, {"dW1": u, "dW2": u, "db1": u, "db2": 2.0 ** -20, "dx": u, "dWg": 2 * u})


# bodies of dW2 and dW1 (as moe_f32_gemm_body numbers them); after ReLU sums of more than 1024 padded slots are made in spans
@pytest.mark.parametrize("T,H,I,E,k,C,act,bodies", [
    (900, 64, 256, 2, 1, 1500, "relu", (64, 64)),          # the live slots end in the first span,
    (2450, 64, 256, 2, 1, 1500, "relu", (64, 64)),         # or in the second
    (1500, 1032, 2056, 8, 1, 1300, "relu", (128, 128)),
    (700, 2056, 2048, 24, 1, 1100, "relu", (256, 256)),
    (500, 64, 4104, 64, 1, 120, "identity", (64, 1)),      # the 64 x 256 body
    (1000, 520, 264, 8, 2, 600, "identity", (64, 64)),
    (1000, 520, 2056, 8, 4, 900, "identity", (128, 128)),
    (300, 2056, 2048, 24, 2, 256, "identity", (256, 256)),
])
def test_fp32_sums_end_with_the_live_slots(T, H, I, E, k, C, act, bodies):
    print("case", T, H, I, E, k, C, act, flush=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    cfg, g, ref, rows = run(T, H, I, E, k, C, act, "f32", (E - 1,) if E > 2 else ())
    assert (moe.moe_f32_gemm_body(E, I, H, C, False, cus), moe.moe_f32_gemm_body(E, H, I, C, False, cus)) == bodies
    u = 2.0 ** -24
    w = math.sqrt((max(rows) + H) / 8 + 2) * u
    check(g, ref, rows, {"dW1": w, "dW2": w, "db1": w, "dx": math.sqrt((H + I) / 8 + 2) * u})


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("T,H,I,E,C", [(3300, 1024, 2048, 17, 400), (2600, 2048, 1024, 17, 300), (9000, 448, 512, 40, 500)])
def test_gradients_do_not_depend_on_an_experts_number(T, H, I, E, C, dtype):
    # the same experts under other numbers (another division of a layer among GPUs): every sum is made in the same order, bit for bit
    print("case", T, H, I, E, C, dtype, flush=True)
    k, shift, td = 2, 3, moe.TORCH_DTYPE[dtype]
    cfg = moe.make_config(T, H, I, E, k, 1.0, "relu", dtype, capacity_override=C)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert {moe.moe_gemm16_kernel(cfg, p, cus) for p in ("dh", "dxe")} == {"stream"}
    gen = torch.Generator(device="cuda").manual_seed(T)
    n = lambda scale, *s: (torch.empty(s, device="cuda").normal_(generator=gen) * scale).to(td)
    x, Wg, W1, W2, dout = n(1, T, H), n(H ** -0.5, H, E), n(H ** -0.5, E, H, I), n(I ** -0.5, E, I, H), n(1, T, H)
    ex = torch.empty(T, E, device="cuda").uniform_(generator=gen).topk(k, 1).indices.int()
    w = torch.softmax(torch.empty(T, k, device="cuda").normal_(generator=gen), 1)

    def gradients(Wg, W1, W2, ex):
        g = [torch.full(s, float("nan"), device="cuda") for s in ((T, H), (H, E), (E,), (E, H, I), (E, I), (E, I, H), (E, H))]
        ws = torch.empty(moe.moe_backward_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
        moe.moe_backward(cfg, ws, x, Wg, W1, None, W2, None, ex, w, dout, *g)
        return g

    want = gradients(Wg, W1, W2, ex)
    got = gradients(Wg.roll(shift, 1), W1.roll(shift, 0), W2.roll(shift, 0), (ex + shift) % E)
    for name, a, b, axis in zip(("dx", "dWg", "dgb", "dW1", "db1", "dW2", "db2"), want, got, (None, 1, 0, 0, 0, 0, 0)):
        assert torch.equal(a if axis is None else a.roll(shift, axis), b), name
