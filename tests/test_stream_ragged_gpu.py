"""16-bit expert FFNs whose contractions end inside a K-tile (K a multiple of 8, not of 64): every remainder of the streaming kernel's pair of
K-tiles, both tile heights, and an infinity right behind the last k; in layers of few tasks, which the 128 x 128 tiles take (against the oracle
at the layer's bar), and of more tasks than CUs, which the streaming kernel takes from K = 136 on (against float64)."""
import pytest
import torch

from paper_2506_04667_amd import binding as moe
from paper_2506_04667_amd.inputs import WORKLOADS, scaled

from test_narrow_gemm_gpu import check_against_float64, kernels
from test_parity_gpu import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rem", [8, 16, 24, 32, 40, 48, 56])
@pytest.mark.parametrize("dtype,T,act", [("bf16", 700, "gelu_erf"), ("f16", 90, "gelu_tanh")])
def test_every_remainder(oracle, dtype, T, act, rem):
    # 256-row tiles with a remainder (T = 700 over 4 experts), 128-row tiles; K = H = 256 + rem and K = I = 320 + rem (six K-tiles at 128 + 8)
    w = scaled(WORKLOADS["paper_bf16_e128"], name="ragged", seed=81, T=T, H=256 + rem, I=320 + rem, E=4, k=2, capacity_factor=2.0, with_bias=rem % 16 == 8,
               act=act, dtype=dtype)
    assert kernels(moe.config_of(w)) == ("128", "128")
    _run(oracle, w)


@pytest.mark.parametrize("rem", [8, 16, 24, 32, 40, 48, 56])
@pytest.mark.parametrize("dtype,most,act", [("bf16", 300, "gelu_erf"), ("f16", 90, "gelu_tanh")])
def test_every_remainder_in_the_streaming_kernel(dtype, most, act, rem):
    # 256-row tiles with 128-row ones and without, an expert without rows; 128-row tiles only.  K = H = 128 + rem is six K-tiles; rows
    # of y of fewer than 256 columns are left to the other kernel
    rows = [min(r, most) for r in [300, 1, 129, 0, 128, 257, 64, 200, 256, 33, 15] * 12]
    check_against_float64(rows, 256 + rem, 320 + rem, act, rem % 16 == 8, dtype, ("stream", "stream"))
    check_against_float64(rows, 128 + rem, 264, act, rem % 16 == 8, dtype, ("stream", "128"))


@pytest.mark.parametrize("case", [
    dict(T=600, H=136, I=1000, E=3, k=1, capacity_factor=3.0, act="relu"),         # shortest K; I * 2 bytes no multiple of a line
    dict(T=3000, H=1032, I=264, E=40, k=2, capacity_factor=0.7, act="identity"),   # many units, drops, second column tile 8 wide
    dict(T=20, H=4440, I=2648, E=32, k=2, capacity_factor=1.0, act="gelu_erf"),    # a weight stream
])
def test_ragged_shapes(oracle, case):
    w = scaled(WORKLOADS["paper_bf16_e128"], name="ragged", seed=82, **case)
    cpu, dev, b, host, rep = _run(oracle, w)
    from parity import gpu_forward
    b2, _ = gpu_forward(w, dev, staged=True)
    assert torch.equal(b.out, b2.out)


@pytest.mark.parametrize("E,on", [(2, "128"), (90, "stream")])
@pytest.mark.parametrize("rem", [8, 40])
def test_infinity_behind_the_last_k_stays_out(rem, E, on):
    # expert 1's first row, right behind expert 0's rows of W1, and the columns right behind a row's last k in xe (the next row) are infinite
    H, I, rows = 256 + rem, 264, 130
    cfg = moe.make_config(E * rows, H, I, E, 1, 1.0, "identity", "bf16")
    assert kernels(cfg) == (on, on)
    b = moe.Buffers(cfg).alloc_staged()
    b.xe.fill_(1.0)
    b.xe[:, 1::2] = float("inf")
    W1 = torch.full((E, H, I), 2.0 ** -10, dtype=torch.bfloat16, device="cuda")
    W1[1, 0] = float("inf")
    W2 = torch.full((E, I, H), 2.0 ** -4, dtype=torch.bfloat16, device="cuda")
    b.expert_demand.fill_(rows)
    moe.moe_expert_ffn(cfg, b.workspace, b.xe, b.expert_demand, W1, None, W2, None, b.y)
    y = b.y[0, :rows].float().cpu()
    want = float(torch.tensor(float(torch.tensor(H * 2.0 ** -10).bfloat16()) * 2.0 ** -4 * I).bfloat16())
    assert bool((y[0::2] == want).all()) and bool(torch.isinf(y[1::2]).all())
