"""The launch shapes that the host chooses (sp_attn_plan, no GPU): its
arguments, and the range of shapes over small, large and one-sided problems."""
import ctypes

import pytest

import paper_2505_22296_amd as sp
from tests.helpers import lib_desc, make_shard


def _plan(D, H, seg_q, seg_k=None, op=sp.SP_OP_BWD, causal=True):
    T_k = sum(seg_q if seg_k is None else seg_k)
    sh = make_shard("plan", sum(seg_q), T_k, D, H, 0, H, H, 1, H, 0, seg_q, seg_k, causal=causal)
    return tuple(sp.sp_attn_plan(lib_desc(sh), op).values())


def test_arguments():
    sh = make_shard("plan", 300, 300, 64, 2, 0, 2, 2, 1, 2, 0, [300])
    d, out = lib_desc(sh), (ctypes.c_int32 * 6)()
    f = sp.load().sp_attn_plan
    assert f(d.ref, 7, out) == sp.SP_ERR_INVALID_ARG
    assert f(d.ref, sp.SP_OP_FWD, None) == sp.SP_ERR_INVALID_ARG
    d.c.head_dim = 96
    assert f(d.ref, sp.SP_OP_FWD, out) == sp.SP_ERR_UNSUPPORTED


@pytest.mark.parametrize("D", [64, 128])
def test_shapes_over_the_range(D):
    # few items: split finest, one backward launch; many: whole items, two launches
    assert _plan(D, 1, [1]) == (4, 0, 2, 0, 1, 0)
    assert _plan(D, 4, [4096], op=sp.SP_OP_FWD) == _plan(D, 4, [4096], op=sp.SP_OP_RING_STEP) == (4, 0, 0, 0, 0, 0)
    two = int(D == 64)
    assert _plan(D, 28, [16384], op=sp.SP_OP_FWD)[:2] == (1, two)
    assert _plan(D, 28, [16384]) == (1, two, 1, two, 0, 0)
    # one side long: the other side's few items are split in launches of their own
    assert _plan(D, 7, [95], [38517], causal=False)[:5] == (4, 0, 1, two, 0)
    assert _plan(D, 17, [38517], [95], causal=False)[2:5] == (2, 0, 0)
    # nothing to do
    assert _plan(D, 1, [0])[4] == 0


def test_two_workgroups_a_cu_by_costs():
    """Head dimension 64, unsplit lists: two workgroups a CU where the load
    decides, one where the longest item would share its CU, whatever the
    number of items."""
    f = lambda *a, **k: _plan(64, *a, op=sp.SP_OP_FWD, **k)[:2]  # noqa: E731
    assert f(16, [32768]) == f(12, [16384]) == f(3, [65536]) == f(8, [1024] * 24) == (1, 1)
    assert f(8, [16384]) == (1, 0)
    # 768 items as 12 heads of 16384 rows have, but the longest among short ones
    assert f(8, [16384] + [256] * 32) == (1, 0)
    assert f(8, [512] * 40, causal=False) == (1, 1)
    assert f(4, [32768] + [256] * 500) == (1, 0)  # more items than are scheduled in the model
    # backward, two launches: dQ's 768 items like the forward's, dK/dV's 1536 are shorter
    assert _plan(64, 8, [16384] + [256] * 32) == (1, 0, 1, 1, 0, 0)
    assert _plan(64, 12, [16384]) == (1, 1, 1, 1, 0, 0)
    # head dimension 128 has no such kernels
    assert _plan(128, 16, [32768], op=sp.SP_OP_FWD)[1] == 0
