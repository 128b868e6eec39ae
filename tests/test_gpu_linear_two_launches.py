"""A linear with a long contraction in two launches: token counts that leave one row, a few rows and the most that is
split behind the full rounds of the largest tile (16320 tokens a round at 1152 out-features), and the first one that is
not.  Against fp32 PyTorch on the same bf16 operands, with samples that change inside either launch and at their border,
strided operands, and nothing written beyond the tokens: fp32 sums over k = 3072 in another order (1e-5 of the operands'
norms, measured 2e-7), plus half a bf16 unit where the output is bf16."""
import pytest
import torch

pytestmark = pytest.mark.gpu
K, M = 3072, 1152


@pytest.mark.parametrize("N", [16321, 16400, 26111, 26113, 32703])
@pytest.mark.parametrize("epilogue,copy,samples", [(0, False, 1), (2, False, 7), (2, True, 2)])
def test_linear_in_two_launches(N, epilogue, copy, samples):
    import paper_2506_13497_amd as m
    gen = torch.Generator(device="cuda").manual_seed(N)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda")
    N = N // samples * samples
    u, W, b = rnd(N, K + 8).bfloat16(), (rnd(M, K) / K ** 0.5).bfloat16(), rnd(M).bfloat16()
    tab, c6, x = rnd(6, M), rnd(samples, 6 * M), rnd(N + 3, M)
    lin = torch.addmm(b.float(), u[:, :K].float(), W.float().t())
    out = torch.full((N + 3, M + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    if epilogue == 2:
        gate = (tab[2] + c6[:, 2 * M:3 * M]).repeat_interleave(N // samples, 0)
        ref = x[:N] + gate * lin
        tail = x[N:].clone()
        m.ddit_linear_fwd(2, u, K + 8, W, b, N, M, K, out if copy else None, M + 8, resid=x, ada_table=tab, c6=c6, gate_row=2,
                          tokens_per_sample=N // samples)
        torch.cuda.synchronize()
        assert ((x[:N] - ref).abs() <= 1e-4 * (1 + ref.abs())).all()
        assert torch.equal(x[N:], tail)
    else:
        ref = lin
        m.ddit_linear_fwd(0, u, K + 8, W, b, N, M, K, out, M + 8)
        torch.cuda.synchronize()
    if copy or epilogue == 0:
        assert ((out[:N, :M].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all()
        assert torch.isnan(out[N:]).all() and torch.isnan(out[:, M:]).all()
