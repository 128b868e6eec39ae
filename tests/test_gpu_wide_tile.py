"""The linear's 320 x 256 tile at shapes where the launcher takes it: rows and columns that end inside a tile, whole and ragged last
k-steps, more than one round of the chip.  Against float64: one bf16 rounding (2^-9), taken twice, and the fp32 sum's 2 sqrt(k) 2^-24 of the
terms' size, taken four times."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epi,N,n,k", [(0, 24893, 312, 256), (0, 16817, 592, 264), (0, 32003, 3072, 1152), (1, 16775, 784, 264), (1, 22105, 592, 768)])
def test_linear(epi, N, n, k):
    import paper_2506_13497_amd as m
    assert m.ddit_linear_form(epi, N, n, k, 256) == (320, 256) and m.ddit_linear_front_tokens(epi, N, n, k, 256) == 0
    g = torch.Generator(device="cuda").manual_seed(N)
    rnd = lambda *s: torch.randn(s, device="cuda", generator=g)
    u, W, bias = rnd(N, k + 8).bfloat16()[:, :k], rnd(n, k).bfloat16(), rnd(n).bfloat16()
    ref = u.double() @ W.double().t() + bias.double()
    fp32 = 8 * k ** 0.5 * 2.0 ** -24 * k ** 0.5
    out = torch.full((N, n + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    m.ddit_linear_fwd(epi, u, k + 8, W, bias, N, n, k, out, n + 8)
    torch.cuda.synchronize()
    want = ref if epi == 0 else torch.nn.functional.gelu(ref, approximate="tanh")
    assert torch.isnan(out[:, n:].float()).all()
    assert ((out[:, :n].double() - want).abs() <= 2.0 ** -8 * want.abs() + fp32 + 1e-5).all()
