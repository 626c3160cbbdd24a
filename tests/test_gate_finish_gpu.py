"""The gate with its sums in slices, whose last launch takes 16 tokens to a workgroup and adds its picks per expert to the chunk of 64 that they
belong to: edges of both, with the routing that follows, against the oracle; twice, since the second call finds the first one's counts."""
import pytest
import torch

from paper_2506_04667_amd.inputs import WORKLOADS, scaled

from parity import gpu_forward
from test_parity_gpu import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 15, 16, 17, 63, 64, 65, 80, 129, 200])
@pytest.mark.parametrize("dtype,H,E,k", [("bf16", 2048, 128, 2), ("f16", 1536, 12, 4), ("f32", 1024, 64, 8), ("bf16", 1600, 256, 3)])
def test_token_counts(oracle, T, dtype, H, E, k):
    w = scaled(WORKLOADS["paper_bf16_e128"], name="finish", seed=90 + T, T=T, H=H, I=64, E=E, k=k, capacity_factor=1.25, dtype=dtype)
    cpu, dev, b, host, rep = _run(oracle, w)
    b2, host2 = gpu_forward(w, dev)
    assert all((host[n] == host2[n]).all() for n in ("topk_expert", "slot", "expert_demand")) and torch.equal(b.out, b2.out)
