"""Launches of few work items, whose items are split over several workgroups
(1, 2 or 4 for row items, 1 or 2 for key items): row and key counts at the
edges of the split tiles, one key, empty segments, dummy slots, the ring merge
and the dQ accumulator, against the fp64 oracle at the parity bars.  The
number of items (segments x heads) and their length decide the split: a
handful of items are split finest, about a hundred in two, several hundred
short ones not at all, where head dimension 64 runs two workgroups a CU if the
load decides.  Every case asserts the launch shapes that it is there for."""
import numpy as np
import pytest

import oracle
from tests.helpers import (LSE_MAX_ABS, assert_close, bits_from_dev, from_dev, lib_desc, make_shard,
                           oracle_kw, scaled_max_abs, to_dev)
from workloads import randn_bf16_bits, shard_inputs

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 193, 255, 256, 257, 0, 97]
CASES = {
    # name: (segment lengths, real heads, dummy slots, padding rows,
    #        forward (split, two a CU), backward (dQ split, dK/dV split, two a
    #        CU, one launch)); two a CU at head dimension 64 only
    "one_row": ([1], 1, 0, 0, (4, 0), (4, 2, 0, 1)),
    "finest": ([193], 2, 1, 3, (4, 0), (4, 2, 0, 1)),
    "finest_long": ([700], 2, 0, 0, (4, 0), (4, 2, 0, 1)),
    "finest_edges": ([257, 65, 1, 0, 130], 2, 0, 5, (4, 0), (4, 2, 0, 1)),
    "two": (EDGES + [250, 160, 200, 129, 140], 4, 1, 2, (2, 0), (1, 1, 0, 1)),
    "two_full": ([256] * 25, 4, 0, 0, (2, 0), None),
    "two_bwd": (EDGES + [512, 450], 4, 1, 2, (4, 0), (2, 1, 0, 1)),
    "none": (EDGES * 3, 7, 0, 0, (1, 0), (1, 1, 0, 1)),
    "two_a_cu": ([33, 1, 65, 40] * 18, 11, 1, 3, (1, 1), (1, 1, 1, 1)),
    "none_300": ([257, 30, 129, 128] * 15, 4, 1, 3, (1, 0), (1, 1, 0, 1)),
    "two_a_cu_split": ([769, 801, 770, 771, 783] * 5, 3, 1, 3, (2, 1), (1, 1, 0, 1)),
    # past 2048 items in both lists: two launches
    "apart": ([33, 1, 65, 40, 0, 7] * 38, 6, 1, 3, (1, 1), (1, 1, 1, 0)),
}


def _shapes(sp, d, D, fwd, bwd):
    """The planned shapes are the case's (two a CU for D = 64 only)."""
    two = int(D == 64)
    f, b = sp.sp_attn_plan(d, sp.SP_OP_FWD), sp.sp_attn_plan(d, sp.SP_OP_BWD)
    assert (f["row_split"], f["row_two"]) == (fwd[0], fwd[1] & two), f
    if bwd:
        assert (b["row_split"], b["key_split"], b["row_two"], b["key_two"], b["one_launch"]) == (
            bwd[0], bwd[1], bwd[2] & two, bwd[2] & two, bwd[3]), b


@pytest.fixture(scope="module")
def sp():
    import torch
    assert torch.cuda.is_available()
    import paper_2505_22296_amd as m
    m.load()
    return m


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("name", list(CASES))
def test_split_items(sp, name, D, causal):
    import torch
    lens, real, dummies, pad, fwd, bwd = CASES[name]
    if name == "two_a_cu_split" and D == 128:
        pytest.skip("a shape of head dimension 64")
    H, T = real + dummies, sum(lens) + pad
    # with a dummy slot: the last of two ranks
    off, nr, npad = (H, H + real, 2 * H) if dummies else (0, real, real)
    sh = make_shard(name, T, T, D, H, off, nr, npad, nr, 1, 0, lens, causal=causal, seed_base=640)
    q, k, v, do = shard_inputs(sh)
    Q, K, V, dO = (to_dev(x) for x in (q, k, v, do))
    d = lib_desc(sh)
    _shapes(sp, d, D, fwd, bwd)
    o, lse = sp.sp_attn_fwd(d, Q, K, V)
    dq, dk, dv = sp.sp_attn_bwd(d, Q, K, V, o, lse, dO)
    acc = torch.ones((T, H, D), dtype=torch.float32, device="cuda")
    sp.sp_attn_bwd(d, Q, K, V, o, lse, dO, dq_acc=acc)
    torch.cuda.synchronize()
    f = [oracle.bf16_bits_to_f64(x) for x in (q, k, v, do)]
    kw = oracle_kw(sh)
    RO, RL = oracle.attn_forward(*f[:3], **kw)
    RdQ, RdK, RdV = oracle.attn_backward(*f, **kw)
    for what, g, r in (("O", from_dev(o)[:, :real], RO[:, :real]),
                       ("dQ", from_dev(dq)[:, :real], RdQ[:, :real]),
                       ("dQ acc", from_dev(acc)[:, :real] - 1.0, RdQ[:, :real]),
                       ("dK", from_dev(dk), RdK), ("dV", from_dev(dv), RdV)):
        assert_close(g, r, f"{name} {what}", max_abs=scaled_max_abs(r))
    fin = np.isfinite(RL[:real])
    GL = lse.cpu().numpy()[:real]
    assert np.array_equal(np.isfinite(GL), fin)
    if fin.any():
        assert np.abs(GL[fin] - RL[:real][fin]).max() <= LSE_MAX_ABS
    assert np.all(bits_from_dev(o)[:, real:] == 0) and np.all(bits_from_dev(dq)[:, real:] == 0)
    assert bool((acc[:, real:] == 1.0).all())


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T,H,n1,fwd", [(1, 1, 161, (4, 0)), (97, 2, 161, (4, 0)), (300, 3, 161, (4, 0)),
                                        (257, 60, 161, (2, 0)), (200, 300, 161, (1, 1)),
                                        (33, 800, 161, (1, 1)), (769, 80, 769, (2, 1))])
def test_split_ring_merge(sp, T, H, n1, fwd, D):
    """Two ring steps over two KV chunks (the second shorter than one stage of
    keys) against the oracle over all keys; the first chunk's keys are hidden
    from the first rows."""
    import torch
    n2 = 31
    if n1 > 161 and D == 128:
        pytest.skip("a shape of head dimension 64")
    heads = dict(H_loc=H, head_offset=0, num_real=H, num_padded=H, gqa=H, Hkv_loc=1, kv_off=0)
    q = randn_bf16_bits((T, H, D), 900)
    k, v = (randn_bf16_bits((n1 + n2, 1, D), s) for s in (901, 902))
    Q = to_dev(q)
    # (n1 = 161: the rows before 161 do not see the second chunk)
    pos_q = 40 + np.arange(T) if n1 == 161 else n1 - 9 + np.arange(T)
    o_acc = torch.full((T, H, D), 7.0, device="cuda")
    lse = torch.full((H, T), 7.0, device="cuda")
    out = torch.empty((T, H, D), dtype=torch.bfloat16, device="cuda")
    for a, b in ((0, n1), (n1, n1 + n2)):
        sh = make_shard("ring", T, b - a, D, *heads.values(), [T], [b - a], pos_q=pos_q,
                        pos_k=a + np.arange(b - a))
        if a == 0:
            plan = sp.sp_attn_plan(lib_desc(sh), sp.SP_OP_RING_STEP)
            assert (plan["row_split"], plan["row_two"]) == (fwd[0], fwd[1] & int(D == 64)), plan
        sp.sp_ring_step(lib_desc(sh), Q, to_dev(k[a:b]), to_dev(v[a:b]), o_acc, lse, init=a == 0,
                        o_out=out if a else None)
    torch.cuda.synchronize()
    sh = make_shard("whole", T, n1 + n2, D, *heads.values(), [T], [n1 + n2], pos_q=pos_q,
                    pos_k=np.arange(n1 + n2))
    RO, RL = oracle.attn_forward(*(oracle.bf16_bits_to_f64(x) for x in (q, k, v)), **oracle_kw(sh))
    assert_close(from_dev(o_acc), RO, "O acc")
    assert_close(from_dev(out), RO, "O out")
    assert np.abs(lse.cpu().numpy() - RL).max() <= LSE_MAX_ABS


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("seg_q,seg_k,H,splits", [([95], [16000], 17, (4, 1)),
                                                  ([4000] + [1] * 510, [95] + [0] * 510, 4, (1, 2))])
def test_one_long_side(sp, seg_q, seg_k, H, splits, D):
    """Few rows against many keys and the reverse (beside rows without keys):
    past 2048 items in both lists together the few long items are split in a
    launch of their own."""
    import torch
    rows, keys = sum(seg_q), sum(seg_k)
    sh = make_shard("side", rows, keys, D, H, 0, H, H, H, 1, 0, seg_q, seg_k, causal=False, seed_base=990)
    d = lib_desc(sh)
    plan = sp.sp_attn_plan(d, sp.SP_OP_BWD)
    assert (plan["row_split"], plan["key_split"], plan["one_launch"]) == (*splits, 0), plan
    q, k, v, do = shard_inputs(sh)
    Q, K, V, dO = (to_dev(x) for x in (q, k, v, do))
    o, lse = sp.sp_attn_fwd(d, Q, K, V)
    grads = sp.sp_attn_bwd(d, Q, K, V, o, lse, dO)
    torch.cuda.synchronize()
    f = [oracle.bf16_bits_to_f64(x) for x in (q, k, v, do)]
    kw = oracle_kw(sh)
    RO, RL = oracle.attn_forward(*f[:3], **kw)
    for what, g, r in zip(("O", "dQ", "dK", "dV"), (o, *grads), (RO, *oracle.attn_backward(*f, **kw))):
        assert_close(from_dev(g), r, what, max_abs=scaled_max_abs(r))
    fin = np.isfinite(RL)
    GL = lse.cpu().numpy()
    assert np.array_equal(np.isfinite(GL), fin) and np.abs(GL[fin] - RL[fin]).max() <= LSE_MAX_ABS
