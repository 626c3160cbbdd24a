"""The slot assignment's forms (counting the earlier pairs again, adding up per-chunk counts, the scan in a launch of its own) at the
sizes where one takes over from the other, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from paper_2506_04667_amd import binding as moe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("policy", ["token_major", "choice_major"])
@pytest.mark.parametrize("T,E,k,C", [
    (4096, 12, 2, 0), (4097, 12, 2, 0),              # 8192 pairs: counted again; 8194: per-chunk counts
    (129, 40, 40, 17),                               # 40 steps of 64 pairs per chunk, 16 wavefronts at a time
    (65, 1024, 8, 3), (65, 1025, 8, 3),              # most experts of one launch; scan launch
    (65536, 8, 1, 0), (65537, 8, 1, 9000),           # most chunks of one launch; scan launch
    (3000, 6, 3, 1200), (200, 2500, 5, 1),           # experts not a multiple of 4; room for three wavefronts' counts
])
def test_slots_where_the_form_changes(oracle, T, E, k, C, policy):
    cfg = moe.make_config(T, 8, 8, E, k, 1.0, "relu", "f32", capacity_override=C, drop_policy=policy)
    b = moe.Buffers(cfg).alloc_staged()
    rng = np.random.default_rng(T + E + k)
    te = np.argpartition(rng.standard_normal((T, E)) - 0.02 * np.arange(E), -k, axis=1)[:, -k:].astype(np.int32)
    tw = rng.random((T, k), dtype=np.float32)
    b.topk_expert.copy_(torch.from_numpy(te))
    b.topk_weight.copy_(torch.from_numpy(tw))
    for t in (b.slot, b.expert_demand, b.slot_token):
        t.fill_(77)
    b.slot_weight.fill_(77.0)
    moe.moe_dispatch(cfg, b.workspace, None, b.topk_expert, b.topk_weight, b.slot, b.expert_demand, b.slot_token, b.slot_weight, None)
    slot, demand, st, sw = oracle.slots(te, tw, E, b.C, choice_major=(policy == "choice_major"))
    for got, want in ((b.slot, slot), (b.expert_demand, demand), (b.slot_token, st), (b.slot_weight, sw)):
        np.testing.assert_array_equal(got.cpu().numpy(), want)
