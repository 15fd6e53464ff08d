"""The logits' gradient: vocabularies one 16-byte chunk below, at and above the
lengths where a thread takes a second and a third load (2048, 4096), where the
workgroup walks on (8192) and where the row is split over workgroups of 8192
logits (12288), one chunk in all, and few long rows, against the float64 formula, with guard rows around
the output.  bf16 results: half an ulp of the value (2^-9 of it), plus the
float32 exponent's error (about 2e-6 of the value at these logits)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,V", [(1, 8), (5, 2048), (5, 2056), (5, 4096), (5, 4104), (5, 8184),
                                 (5, 8192), (5, 8200), (5, 12288), (5, 12296), (3, 16384), (3, 16392), (2, 152064),
                                 (1200, 2048)])
def test_gradient_of_split_rows(T, V):
    import torch
    import paper_2505_22296_amd as sp
    print(f"T={T} V={V}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T + V)
    x = (torch.randn((T, V), generator=gen, device="cuda") * 2).to(torch.bfloat16)
    lab = torch.randint(0, V, (T,), generator=gen, device="cuda", dtype=torch.int32)
    lab[0] = V - 1  # the last logit of a row
    if T > 2:
        lab[1], lab[2] = -100, 0  # a row that is not scored; the first logit
    cu = np.array([0, (T + 1) // 2, T], np.int32)
    g = torch.tensor([0.75, -1.25], device="cuda")
    _, lse, _ = sp.sp_token_logprob(x, lab, cu)
    buf = torch.full((T + 2, V), 3.0, dtype=torch.bfloat16, device="cuda")
    sp.sp_token_logprob_bwd(x, lab, lse, cu, g, dlogits=buf[1:T + 1])
    torch.cuda.synchronize()
    assert bool((buf[0] == 3.0).all()) and bool((buf[T + 1] == 3.0).all())
    d = x.double()
    ref = -torch.softmax(d, 1)
    ok = (lab >= 0)
    ref[torch.arange(T, device="cuda")[ok], lab[ok].long()] += 1.0
    ref *= (torch.where(torch.arange(T, device="cuda") < int(cu[1]), g[0], g[1]).double() * ok)[:, None]
    got = buf[1:T + 1].double()
    bound = ref.abs() * 2.0 ** -8 + 4e-6 * 1.25 * torch.softmax(d, 1)
    assert bool(((got - ref).abs() <= bound).all())
    if T > 2:
        assert bool((buf[2] == 0).all())


@pytest.mark.parametrize("T", [65535, 65536, 2 * 65535 + 1, (1 << 24) + 5])
def test_gradient_of_many_rows(T):
    """Rows past one grid dimension (65535 workgroups), and more workgroups of
    256 threads than one dimension holds (2^32 threads); the gradient is
    written over the logits."""
    import torch
    import paper_2505_22296_amd as sp
    V = 8
    print(f"T={T} V={V}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    buf = torch.full((T + 2, V), 3.0, dtype=torch.bfloat16, device="cuda")
    x = buf[1:T + 1]
    x.copy_(torch.randn((T, V), generator=gen, device="cuda"))
    lab = torch.randint(0, V, (T,), generator=gen, device="cuda", dtype=torch.int32)
    lse = torch.logsumexp(x.float(), 1)
    ref = (-0.5 * torch.exp(x.double() - lse.double()[:, None]))
    p = ref.abs()
    ref.scatter_add_(1, lab[:, None].long(), torch.full((T, 1), 0.5, dtype=torch.float64, device="cuda"))
    sp.sp_token_logprob_bwd(x, lab, lse, np.array([0, T], np.int32), torch.tensor([0.5], device="cuda"), dlogits=x)
    torch.cuda.synchronize()
    assert bool((buf[0] == 3.0).all()) and bool((buf[T + 1] == 3.0).all())
    assert bool(((x.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 4e-6 * p).all())
