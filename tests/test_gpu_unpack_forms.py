"""The unpack's forms, bit for bit against an index copy, with guard rows around
the output: heads that four divides and that it does not, one or four chunks a
thread (up to 2^21 16-byte chunks and past them), planes that end inside a
workgroup's tile, and head rows whose length is no power of two."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MANY = (1 << 21) // 8  # rows x heads at D = 64 whose chunks are 2^21


@pytest.mark.parametrize("T,heads,D", [
    (1, 1, 8), (33, 2, 64), (129, 2, 8), (MANY // 2 + 1, 2, 64), (127, 3, 64), (128, 3, 64), (129, 3, 64), (1000, 4, 128), (257, 5, 24), (511, 6, 128),
    (77, 13, 40), (50, 63, 128), (50, 65, 64),  # (maps of at most and of more than 64 entries)
    (MANY // 7, 7, 64), (MANY // 7 + 1, 7, 64), (MANY // 3 + 77, 3, 64), (MANY // 4 + 1, 4, 64)])
def test_unpack_forms(T, heads, D):
    import torch
    import paper_2505_22296_amd as sp
    n = 2
    H = -(-heads // n)
    print(f"T={T} heads={heads} D={D}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T + heads)
    src = torch.randint(-32768, 32767, (n, T, H, D), generator=gen, device="cuda", dtype=torch.int32).to(torch.int16)
    slots = np.random.default_rng(heads).permutation(n * H)
    hm = np.full(n * H, -1, np.int32)
    hm[slots[:heads]] = np.arange(heads)
    buf = torch.full((T + 2, heads, D), 77, dtype=torch.int16, device="cuda")
    sp.sp_ulysses_unpack(src.view(torch.bfloat16), hm, heads, dst=buf[1:T + 1].view(torch.bfloat16))
    torch.cuda.synchronize()
    assert bool((buf[0] == 77).all()) and bool((buf[T + 1] == 77).all())
    for s in range(n * H):
        if hm[s] >= 0:
            assert torch.equal(buf[1:T + 1, int(hm[s])], src[s // H, :, s % H])
