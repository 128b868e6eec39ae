"""The modulated LayerNorm at the borders of its forms: rows per wavefront (8192 rows; one for wide rows), chunks per lane
(512, 1280, 2048 features), streaming loads (24 M elements), samples that end inside a workgroup; against float64 PyTorch.
One bf16 rounding (2^-9 of the value) and fp32 arithmetic of a few terms."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,D,tps", [(8191, 1152, 8191), (8193, 1152, 2731), (8193, 512, 8193), (8195, 520, 1639), (9001, 1280, 9001),
                                     (9001, 1288, 9001), (8194, 2048, 4097), (8195, 2056, 8195), (8195, 4096, 1639), (20000, 1280, 20000),
                                     (3, 2048, 1), (100001, 256, 100001)])
def test_forms(N, D, tps):
    import paper_2506_13497_amd as m
    g = torch.Generator(device="cuda").manual_seed(N + D)
    draw = lambda *s: torch.randn(*s, device="cuda", generator=g)
    x, tab, c6 = draw(N, D) * 1.5 + 0.3, draw(6, D) * 0.5, draw((N + tps - 1) // tps, 6 * D) * 0.5
    for which in (0, 1):
        out = torch.full((N, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        m.ddit_modulated_layernorm_fwd(x, tab, c6, which, tps, 1e-6, out)
        torch.cuda.synchronize()
        mod = (tab.double() + c6.double().view(-1, 6, D))[torch.arange(N, device="cuda") // tps]
        xd = x.double()
        xn = (xd - xd.mean(1, keepdim=True)) * torch.rsqrt(xd.var(1, unbiased=False, keepdim=True) + 1e-6)
        ref = xn * (1.0 + mod[:, 3 * which + 1]) + mod[:, 3 * which]
        assert ((out.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all(), (N, D, tps, which)
        del mod, xd, xn, ref
