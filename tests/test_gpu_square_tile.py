"""The linear's 192 x 192 tile at shapes where the launcher takes it: rows and columns that end inside a tile and inside a wavefront's
part of it, contractions shorter than its ring, ragged last k-steps; residual updates also where samples meet inside a tile, at a
wavefront's edge (4704 = 49 x 96) or not, and with the tiles whose wavefronts fetch rows of the stream ahead.  Against float64: one bf16
rounding (2^-9), taken twice, and the fp32 sum's 2 sqrt(k) 2^-24 of the terms' size, taken four times."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def operands(N, n, k):
    g = torch.Generator(device="cuda").manual_seed(N + k)
    rnd = lambda *s: torch.randn(s, device="cuda", generator=g)
    u, W, bias = rnd(N, k + 8).bfloat16()[:, :k], rnd(n, k).bfloat16(), rnd(n).bfloat16()
    return rnd, u, W, bias, u.double() @ W.double().t() + bias.double(), 8 * k ** 0.5 * 2.0 ** -24 * k ** 0.5


@pytest.mark.parametrize("epi,N,n,k", [(0, 7200, 1152, 264), (0, 8064, 1144, 1152), (0, 13111, 568, 264), (0, 2400, 3456, 776),
                                            (1, 7187, 1152, 8), (1, 9300, 776, 72), (1, 8064, 1152, 192)])
def test_bf16(epi, N, n, k):
    import paper_2506_13497_amd as m
    assert m.ddit_linear_form(epi, N, n, k, 256) == (192, 192)
    rnd, u, W, bias, ref, fp32 = operands(N, n, k)
    out = torch.full((N, n + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    m.ddit_linear_fwd(epi, u, k + 8, W, bias, N, n, k, out, n + 8)
    torch.cuda.synchronize()
    want = ref if epi == 0 else torch.nn.functional.gelu(ref, approximate="tanh")
    assert torch.isnan(out[:, n:].float()).all()
    assert ((out[:, :n].double() - want).abs() <= 2.0 ** -8 * want.abs() + fp32 + 1e-5).all()


# tile None: the launcher's; else 192 x 384, 256 x 256 and 192 x 256 forced
@pytest.mark.parametrize("tile,copy,N,n,k", [(None, False, 7187, 1152, 8), (None, False, 8064, 1144, 4608), (None, False, 9301, 776, 776), (None, True, 7600, 1152, 1152),
                                             (None, True, 9301, 776, 264), (None, True, 13110, 568, 72), (0, False, 5001, 392, 264), (0, True, 4800, 1152, 72),
                                             (1, False, 5001, 392, 72), (1, True, 4800, 1152, 264), (3, False, 5001, 1152, 264), (3, True, 5001, 392, 72)])
def test_residual(tile, copy, N, n, k):
    import paper_2506_13497_amd as m
    assert tile is not None or m.ddit_linear_form(18 if copy else 2, N, n, k, 256) == (192, 192)
    assert tile is not None or m.ddit_linear_front_tokens(18 if copy else 2, N, n, k, 256) == 0
    rnd, u, W, bias, ref, fp32 = operands(N, n, k)
    out = torch.full((N, n + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    for tps in (N, 4704, 1701):   # one sample; meeting at a wavefront's edge; anywhere
        tab, c6 = rnd(6, n), rnd((N + tps - 1) // tps, 6 * n)
        x0 = rnd(N, n)
        x = x0.clone()
        where = (out, n + 8) if copy else (None, 0)
        args = (2, u, k + 8, W, bias, N, n, k, *where)
        call = m.ddit_linear_fwd if tile is None else lambda *a, **kw: m.ddit_linear_fwd_tile(tile, *a, **kw)
        call(*args, resid=x, ada_table=tab, c6=c6, gate_row=2, tokens_per_sample=tps)
        torch.cuda.synchronize()
        gate = tab[2].double() + c6.double()[torch.arange(N, device="cuda") // tps, 2 * n:3 * n]
        want = x0.double() + gate * ref
        assert ((x.double() - want).abs() <= (fp32 + 2.0 ** -20 * ref.abs()) * (1 + gate.abs()) + 2.0 ** -22 * want.abs()).all(), tps
        if copy:
            assert torch.equal(out[:, :n], x.bfloat16()) and torch.isnan(out[:, n:].float()).all()
