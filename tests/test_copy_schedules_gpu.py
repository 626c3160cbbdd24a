"""Where the order of copies and products inside a tile can go wrong, against float64: 128-row tiles of the weight-streaming kernel at every edge
of their 16-row MFMA tiles (those beyond the live rows are left out), 256-row tiles of the fewest K-tiles over several tasks per workgroup
(copies cross from task to task), layers whose tasks go in blocks of row and column tiles, data gradients of weights whose rows are a multiple
of 2 KB long, and fp32 256 x 256 tiles of one to seven K-tiles."""
import math

import pytest
import torch

from paper_2506_04667_amd import binding as moe

from test_backward_streaming_gpu import check, run
from test_narrow_gemm_gpu import check_against_float64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("H,I,act,bias", [(320, 512, "gelu_tanh", True), (264, 264, "relu", False)])
def test_small_tiles(H, I, act, bias, dtype):
    # every multiple of 16 live rows, one less and one more; workgroups with several tasks of different heights one after the other
    rows = [r for m in range(0, 129, 16) for r in (m - 1, m, m + 1) if 0 <= r <= 128] * 6
    check_against_float64(rows, H, I, act, bias, dtype, ("stream", "stream"))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("H,I", [(256, 256), (320, 448), (192, 264)])   # eight K-tiles, ten and fourteen, and six
def test_large_tiles_of_few_k_tiles(H, I, dtype):
    rows = [129, 256, 300, 143, 145, 512, 255, 0, 1, 384] * 50
    check_against_float64(rows, H, I, "identity", False, dtype, ("stream", "stream" if H >= 256 else "128"))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("rows,H,I,on", [
    ([1024, 700, 256, 0, 1000, 300, 513, 897] * 3, 320, 3208, ("stream", "stream")),    # four row tiles to an expert: blocks of four by eight, 13 column tiles
    ([600, 512, 300, 257, 0, 129] * 4, 264, 4360, ("stream", "128")),                   # three: blocks of two by sixteen, 18 column tiles
])
def test_wide_layers(rows, H, I, on, dtype):
    check_against_float64(rows, H, I, "gelu_tanh", True, dtype, on)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("T,C,E", [(3300, 400, 17), (1500, 120, 19)])   # 256-row tiles and 128-row ones
def test_data_gradients_of_long_rows(T, C, E, dtype):
    print("case", T, C, E, dtype, flush=True)
    cfg, g, ref, rows = run(T, 1024, 2048, E, 2, C, "identity", dtype, (E - 1,))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    # few row tiles go to the 128 x 128 tiles where each has a CU of its own
    assert [moe.moe_gemm16_kernel(cfg, p, cus) for p in ("dh", "dxe")] == ["stream", "128" if C == 120 else "stream"]
    u = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype]
    check(g, ref, rows, {"dW1": u, "dW2": u, "db1": u, "db2": 2.0 ** -20, "dx": u, "dWg": 2 * u})


@pytest.mark.parametrize("H", [8, 32, 40, 64, 96, 104, 128, 200])
def test_fp32_large_tiles_of_few_k_tiles(H):
    E, I, rows = 32, 2048, [256, 1, 200, 0, 129, 64, 255, 31] * 4
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert moe.moe_f32_gemm_body(E, 256, I, H, True, cus) == 256
    gen = torch.Generator(device="cuda").manual_seed(H)
    n = lambda scale, *s: torch.empty(s, device="cuda").normal_(generator=gen) * scale
    W1, W2 = n(H ** -0.5, E, H, I), n(I ** -0.5, E, I, H)
    cfg = moe.make_config(sum(rows), H, I, E, 1, 1.0, "identity", "f32", capacity_override=256)
    b = moe.Buffers(cfg).alloc_staged()
    b.xe.normal_(generator=gen)
    b.expert_demand.copy_(torch.tensor(rows, dtype=torch.int32))
    moe.moe_expert_ffn(cfg, b.workspace, b.xe, b.expert_demand, W1, None, W2, None, b.y)
    for e, r in enumerate(rows):
        if r:
            want = b.xe[e, :r].double() @ W1[e].double() @ W2[e].double()
            # two roundings for every 32 / 6 products, counted with partial sums as large as the whole
            assert float((b.y[e, :r].double() - want).norm() / want.norm()) < math.sqrt((H + I) / 8 + 2) * 2.0 ** -24, e
