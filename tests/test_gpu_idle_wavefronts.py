"""Attention where the last query tile of a unit leaves wavefronts without queries: they pass the barriers of the others and write
nothing.  Many units, so that no unit's keys are shared out; one, two and more key tiles, whole and ragged, in the streaming forms of
64 and 128 queries and in the resident one.  Against float64 on the same bf16 operands: the bars of the attention tests (2e-2 elementwise,
5e-3 of the norm; log-sum-exp 2e-2)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,dh", [(4, 72), (4, 64)])
@pytest.mark.parametrize("T,S", [(60, 1), (60, 31), (60, 33), (52, 65), (52, 96), (52, 129), (64, 144), (64, 161), (52, 321), (40, 385), (26, 527)])
def test_spatial(T, S, H, dh):
    import paper_2506_13497_amd as m
    g = torch.Generator(device="cuda").manual_seed(S)
    q, k, v = (torch.randn((T, S, H, dh), device="cuda", generator=g).bfloat16() for _ in range(3))
    q *= 2
    A = H * dh
    o = torch.full((T, S, H, dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((T, S, H), float("nan"), device="cuda")
    m.ddit_attn_fwd(m.DDIT_ATTN_SPATIAL, m.make_shape(1, T, 1, S, A, H, dh, 64, 8, 1), q, k, v, A, A, None, o, A, lse)
    torch.cuda.synchronize()
    h = lambda t: t.double().permute(0, 2, 1, 3).contiguous()
    s = torch.matmul(h(q), h(k).transpose(2, 3).contiguous()) * dh ** -0.5
    want = torch.matmul(torch.softmax(s, -1), h(v)).permute(0, 2, 1, 3)
    d = (o.double() - want).abs()
    assert (d <= 2e-2 * (1 + want.abs())).all() and d.norm() <= 5e-3 * want.norm()
    assert (lse.double() - torch.logsumexp(s, -1).permute(0, 2, 1)).abs().max() <= 2e-2


@pytest.mark.parametrize("L,Ly", [(2337, 300), (4650, 65), (2305, 64)])
def test_cross(L, Ly):
    import paper_2506_13497_amd as m
    H, dh = 16, 72
    A = H * dh
    g = torch.Generator(device="cuda").manual_seed(L)
    q, k, v = (torch.randn((1, n, H, dh), device="cuda", generator=g).bfloat16() for n in (L, Ly, Ly))
    o = torch.full((1, L, H, dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    m.ddit_attn_fwd(m.DDIT_ATTN_CROSS, m.make_shape(1, 1, 1, L, A, H, dh, 64, Ly, 1), q, k, v, A, A, [Ly - 1], o, A)
    torch.cuda.synchronize()
    h = lambda t, n: t.double()[:, :n].permute(0, 2, 1, 3).contiguous()
    s = torch.matmul(h(q, L), h(k, Ly - 1).transpose(2, 3).contiguous()) * dh ** -0.5
    want = torch.matmul(torch.softmax(s, -1), h(v, Ly - 1)).permute(0, 2, 1, 3)
    d = (o.double() - want).abs()
    assert (d <= 2e-2 * (1 + want.abs())).all() and d.norm() <= 5e-3 * want.norm()
