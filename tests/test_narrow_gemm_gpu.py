"""16-bit expert FFNs in the 128 x 128 tiles that launches of few tasks and narrow layers take: edges of the tile, of its 32-deep K-tiles and of
the ring of five, against float64; and the same experts in a layer with enough tasks for the weight-streaming kernel, whose sums are made in
the same order, bit for bit."""
import pytest
import torch

from paper_2506_04667_amd import binding as moe

pytestmark = pytest.mark.gpu

ACTS = {"relu": torch.relu, "gelu_tanh": lambda v: torch.nn.functional.gelu(v, approximate="tanh"), "gelu_erf": torch.nn.functional.gelu,
        "identity": lambda v: v}


def _layer(E, rows, H, I, act, dtype, bias, seed):
    td = moe.TORCH_DTYPE[dtype]
    g = torch.Generator().manual_seed(seed)
    n = lambda scale, *s: (torch.randn(*s, generator=g) * scale).to(td)
    C = max(rows)
    t = {"xe": n(1, E, C, H), "W1": n(H ** -0.5, E, H, I), "W2": n(I ** -0.5, E, I, H),
         "b1": n(0.5, E, I) if bias else None, "b2": n(0.5, E, H) if bias else None}
    return t, C


def kernels(cfg):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return moe.moe_gemm16_kernel(cfg, "ffn1", cus), moe.moe_gemm16_kernel(cfg, "ffn2", cus)


def _ffn(t, rows, C, H, I, act, dtype, on):
    E = len(rows)
    cfg = moe.make_config(max(1, sum(rows)), H, I, E, 1, 1.0, act, dtype, capacity_override=C)
    assert kernels(cfg) == on
    b = moe.Buffers(cfg).alloc_staged()
    b.xe.zero_()
    b.xe[:, :C] = t["xe"].cuda()
    b.y.zero_()
    b.expert_demand.copy_(torch.tensor(rows, dtype=torch.int32))
    d = lambda k: None if t[k] is None else t[k].cuda()
    moe.moe_expert_ffn(cfg, b.workspace, b.xe, b.expert_demand, d("W1"), d("b1"), d("W2"), d("b2"), b.y)
    return b.y.cpu()


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("rows,H,I,act,bias", [
    ([1, 0, 5], 8, 16, "identity", True),                        # one chunk of k and of columns; an expert without rows
    ([15, 16, 17, 33, 48, 49, 64, 65, 0], 32, 128, "relu", False),          # row tiles and wavefronts with and without a live row
    ([127, 128, 129, 200], 40, 136, "gelu_tanh", True),          # tile remainders; K one chunk beyond a K-tile, a column tile 8 wide
    ([257, 384, 385], 120, 64, "gelu_erf", False),               # both unit lists; four K-tiles, the last one short
    ([300, 20], 160, 192, "gelu_erf", True),                     # as many K-tiles as the ring has, and one more
    ([90] * 11, 248, 328, "relu", True),                         # more units than XCDs, not a multiple of 8
    ([3] * 48, 1032, 264, "gelu_tanh", False),                   # few rows: a weight stream
])
def test_against_float64(rows, H, I, act, bias, dtype):
    check_against_float64(rows, H, I, act, bias, dtype, ("128", "128"))


def check_against_float64(rows, H, I, act, bias, dtype, on):
    print("case", rows, H, I, act, bias, dtype, flush=True)
    t, C = _layer(len(rows), rows, H, I, act, dtype, bias, H + I)
    y = _ffn(t, rows, C, H, I, act, dtype, on).double().cuda()
    f = {k: None if v is None else v.double().cuda() for k, v in t.items()}
    # h and y are each rounded once to storage: relative to each value 2^-8 (bf16) or 2^-11 (f16) at most
    tol = 2 * 2.0 ** (-8 if dtype == "bf16" else -11)
    for e, r in enumerate(rows):
        h = f["xe"][e, :r] @ f["W1"][e] + (f["b1"][e] if bias else 0)
        want = ACTS[act](h) @ f["W2"][e] + (f["b2"][e] if bias else 0)
        if r:
            assert float((y[e, :r] - want).norm() / want.norm()) < tol, e
        assert bool((y[e, r:] == 0).all()), e                    # rows beyond the live ones are not written


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("H,I", [(448, 512), (456, 520), (488, 408)])
def test_same_sums_as_the_streaming_kernel(H, I, dtype):
    # 4 experts are at most 40 tiles of 128 x 128, below one per CU; 76 are 608 and more, too many
    few = [200, 130, 1, 97]
    many = few + [140] * 72
    t, C = _layer(len(many), many, H, I, "gelu_erf", dtype, True, 5)
    wide = _ffn(t, many, C, H, I, "gelu_erf", dtype, ("stream", "stream"))
    narrow = _ffn({k: v[:4] for k, v in t.items()}, few, C, H, I, "gelu_erf", dtype, ("128", "128"))
    assert torch.equal(narrow, wide[:4])


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("H,I", [(448, 448), (1024, 1024)])     # rows of weights spread over the L2's channels, and rows that begin at the same one
def test_same_data_gradients_as_the_streaming_kernel(H, I, dtype):
    # tokens choose among the first 4 experts of 76; ReLU (the gradients of the weights do not enter)
    T, k, C = 300, 2, 200
    td = moe.TORCH_DTYPE[dtype]
    g = torch.Generator().manual_seed(9)
    n = lambda scale, *s: (torch.randn(*s, generator=g) * scale).to(td)
    x, Wg, W1, W2, dout = n(1, T, H), n(H ** -0.5, H, 76), n(H ** -0.5, 76, H, I), n(I ** -0.5, 76, I, H), n(1, T, H)
    ex = torch.rand(T, 4, generator=g).argsort(1)[:, :k].int().contiguous().cuda()
    w = torch.softmax(torch.randn(T, k, generator=g), 1).cuda()
    out = []
    for E in (4, 76):
        cfg = moe.make_config(T, H, I, E, k, 1.0, "relu", dtype, capacity_override=C)
        cus = torch.cuda.get_device_properties(0).multi_processor_count
        assert {moe.moe_gemm16_kernel(cfg, p, cus) for p in ("ffn1", "dh", "dxe")} == {"128" if E == 4 else "stream"}
        dx, dWg, dgb, dW1, db1, dW2, db2 = (torch.empty(s, device="cuda") for s in
                                            ((T, H), (H, E), (E,), (E, H, I), (E, I), (E, I, H), (E, H)))
        ws = torch.empty(moe.moe_backward_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
        c = lambda v: v.contiguous().cuda()
        moe.moe_backward(cfg, ws, c(x), c(Wg[:, :E]), c(W1[:E]), None, c(W2[:E]), None, ex, w, c(dout), dx, dWg, dgb, dW1, db1, dW2, db2)
        out.append(dx.cpu())
    assert torch.equal(out[0], out[1])
