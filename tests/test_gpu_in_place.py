"""dK and dV written over K and V (dk = k, dv = v, and swapped): dQ still reads
K and V, so a backward that would run both work lists in one launch takes two,
with the same splits.  The gradients are those of separate buffers bit for bit,
for every shape of the one-launch backward, with one query head a KV head (the
workgroups write dK and dV themselves) and with grouped heads; so the kernels of
the separate launches are also compared with the one-launch kernel's."""
import pytest

from tests.helpers import bits_from_dev, lib_desc, make_shard, to_dev
from workloads import shard_inputs

pytestmark = pytest.mark.gpu

# name: (head dim, segments, heads, query heads a KV head, causal, plan of the backward)
CASES = {
    "4_2_d128": (128, [700, 97], 4, 1, True, (4, 0, 2, 0)),
    "4_2_d64": (64, [700, 97], 4, 1, True, (4, 0, 2, 0)),
    "4_2_gqa": (128, [700, 97], 4, 2, True, (4, 0, 2, 0)),
    "2_1_d128": (128, [700, 500], 8, 1, False, (2, 0, 1, 0)),
    "2_1_d64": (64, [1000, 900], 10, 1, True, (2, 0, 1, 0)),
    "1_1_d128": (128, [1, 130, 257] * 12, 6, 1, True, (1, 0, 1, 0)),
    "1_1_d64": (64, [1, 130, 257] * 12, 6, 1, True, (1, 0, 1, 0)),
    "two_a_cu": (64, [33, 1, 130, 257] * 15, 9, 1, True, (1, 1, 1, 1)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_gradients_over_keys_and_values(name):
    import numpy as np
    import torch
    import paper_2505_22296_amd as sp
    D, lens, H, g, causal, shape = CASES[name]
    T = sum(lens)
    sh = make_shard(name, T, T, D, H, 0, H, H, g, H // g, 0, lens, causal=causal, seed_base=820)
    print(f"{name}: T={T} D={D} H={H} g={g}", flush=True)
    d = lib_desc(sh)
    plan = sp.sp_attn_plan(d, sp.SP_OP_BWD)
    assert plan["one_launch"] and tuple(plan.values())[:4] == shape, plan
    q, k, v, do = (to_dev(x) for x in shard_inputs(sh))
    o, lse = sp.sp_attn_fwd(d, q, k, v)
    ref = [bits_from_dev(t) for t in sp.sp_attn_bwd(d, q, k, v, o, lse, do)]
    for swap in (False, True):
        K, V = k.clone(), v.clone()
        dk, dv = (V, K) if swap else (K, V)
        got = sp.sp_attn_bwd(d, q, K, V, o, lse, do, dk=dk, dv=dv)
        torch.cuda.synchronize()
        for what, a, r in zip(("dQ", "dK", "dV"), got, ref):
            assert np.array_equal(bits_from_dev(a), r), f"{what}, swapped: {swap}"
