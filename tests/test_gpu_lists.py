"""Work lists at the length where they move from the kernel arguments to the
workspace: 511, 512 and 513 items in the forward, 511 to 513 in both lists of a
backward together.  Every segment is one row, so the results have closed forms:
O = v, LSE = scale q.k, dV = dO, dQ = dK = 0 up to the rounding of dO.v (formed
twice, in bf16 products with float32 sums: D terms of about 1 each time)."""
import numpy as np
import pytest

from tests.helpers import bits_from_dev, from_dev, lib_desc, make_shard, to_dev
from workloads import shard_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rows,keys", [(511, 511), (512, 512), (513, 513), (255, 256), (256, 256), (256, 257)])
def test_lists_around_the_argument_limit(rows, keys, D):
    import torch
    import paper_2505_22296_amd as sp
    n = max(rows, keys)
    seg_q, seg_k = [1] * rows + [0] * (n - rows), [1] * keys + [0] * (n - keys)
    sh = make_shard("lists", rows, keys, D, 1, 0, 1, 1, 1, 1, 0, seg_q, seg_k, seed_base=960)
    d = lib_desc(sh)
    assert len(sp.sp_attn_schedule(d, sp.SP_OP_FWD)) == rows and len(sp.sp_attn_schedule(d, sp.SP_OP_BWD)) == keys
    q, k, v, do = (to_dev(x) for x in shard_inputs(sh))
    o, lse = sp.sp_attn_fwd(d, q, k, v)
    dq, dk, dv = sp.sp_attn_bwd(d, q, k, v, o, lse, do)
    torch.cuda.synchronize()
    assert np.array_equal(bits_from_dev(o), bits_from_dev(v[:rows]))
    ref = (q.double() * k[:rows].double()).sum(-1).T * sh.scale
    assert float((lse.double() - ref).abs().max()) <= 1e-5
    # P = exp(s - LSE) is 1 within a few float32 ulps of |s| <= 10 (2^-20), the
    # bf16 output rounds it back to 1
    assert np.array_equal(bits_from_dev(dv[:rows]), bits_from_dev(do))
    assert not bits_from_dev(dv[rows:]).any() and not bits_from_dev(dk[rows:]).any()
    # dP and D: two float32 sums of D products, each within D 2^-24 of sum |dO v|
    bound = 2.0 * D * 2.0 ** -24 * D * 4 * sh.scale * 6
    assert np.abs(from_dev(dq)).max() <= bound and np.abs(from_dev(dk)).max() <= bound
