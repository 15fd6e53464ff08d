"""The wrapper's workspace handling (host only): a caller's workspace that
fits is used as it is, one that is too small is replaced by a new one, and the
library's refusal of one that is large enough (misaligned) stands."""
import pytest
import torch

import paper_2505_22296_amd as sp
from paper_2505_22296_amd import _lib
from tests.helpers import lib_desc, make_shard


@pytest.mark.parametrize("size,aligned,calls", [(None, True, 1), (0, True, 2), (-1, True, 2), (0x40, True, 1),
                                                (0x40, False, 1)])
def test_workspace_of_the_caller(size, aligned, calls):
    """`size`: bytes past what is needed (None: no workspace; 0: an empty one)."""
    sh = make_shard("ws", 300, 300, 64, 2, 0, 2, 2, 1, 2, 0, [300])
    d = lib_desc(sh)
    need = sp.sp_attn_workspace_size(d, sp.SP_OP_BWD)
    ws = None if size is None else torch.empty(need + size if size else 0, dtype=torch.uint8)
    seen = []

    def call(ptr, n):  # the library's rule
        seen.append((ptr, n))
        return sp.SP_OK if ptr and n >= need and aligned else sp.SP_ERR_WORKSPACE

    def go():
        _lib._with_workspace(d, sp.SP_OP_BWD, "cpu", ws, call, "here")
    if aligned:
        go()
        assert seen[-1][1] >= need
    else:
        with pytest.raises(sp.SpError) as e:
            go()
        assert e.value.status == sp.SP_ERR_WORKSPACE
    assert len(seen) == calls
    if ws is not None:
        assert seen[0] == (ws.data_ptr(), ws.numel())


def test_other_refusals_are_not_retried():
    sh = make_shard("ws", 300, 300, 64, 2, 0, 2, 2, 1, 2, 0, [300])
    seen = []
    with pytest.raises(sp.SpError) as e:
        _lib._with_workspace(lib_desc(sh), sp.SP_OP_FWD, "cpu", torch.empty(16, dtype=torch.uint8),
                             lambda p, n: seen.append(n) or sp.SP_ERR_UNSUPPORTED, "here")
    assert e.value.status == sp.SP_ERR_UNSUPPORTED and len(seen) == 1
