"""A linear with a long contraction in two launches (16320 tokens are a round of the largest tile at 1152 out-features): one
row behind the full rounds, a few rows, the most that is split behind two full rounds (three fifths of one; with the bf16 copy
what the launcher's model says) and the first count that is not.  Every case says how many tokens the first launch
has to have.  Against fp32 PyTorch on the same bf16 operands, for every epilogue, with samples that end before, at and behind
the border and inside a tile of the second launch, strided operands, and nothing written beyond the tokens: fp32 sums over
k = 3072 in another order (1e-5 of the operands' norms, measured 2e-7), plus half a bf16 unit where the output is bf16; GELU
(slope at most 1.13) adds its own fp32 error."""
import pytest
import torch

pytestmark = pytest.mark.gpu
K, M = 3072, 1152
GELU, RESIDUAL, COPY = 1, 2, 18
CASES = [   # epilogue, tokens, of them in the first launch, tokens per sample
    (0, 16321, 16320, 16321), (GELU, 32641, 32640, 32641), (RESIDUAL, 32641, 32640, 32640), (COPY, 32641, 32640, 200),
    (COPY, 16400, 16320, 16354), (RESIDUAL, 16400, 16320, 77), (COPY, 17000, 16320, 16352), (RESIDUAL, 17000, 16320, 400),
    (0, 42432, 32640, 42432), (GELU, 42432, 32640, 42432), (RESIDUAL, 42432, 32640, 16320), (COPY, 39808, 32640, 32700),
    (0, 42433, 0, 42433), (GELU, 42433, 0, 42433), (RESIDUAL, 42433, 0, 9000), (COPY, 39809, 0, 400),
]


@pytest.mark.parametrize("epilogue,N,front,per_sample", CASES)
def test_linear_in_two_launches(epilogue, N, front, per_sample):
    import paper_2506_13497_amd as m
    assert torch.cuda.get_device_properties(0).multi_processor_count != 256 or m.ddit_linear_front_tokens(epilogue, N, M, K) == front
    assert m.ddit_linear_front_tokens(epilogue, N, M, K, 256) == front
    gen = torch.Generator(device="cuda").manual_seed(N)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda")
    samples = -(-N // per_sample)
    u, W, b = rnd(N, K + 8).bfloat16(), (rnd(M, K) / K ** 0.5).bfloat16(), rnd(M).bfloat16()
    tab, c6, x = rnd(6, M), rnd(samples, 6 * M), rnd(N + 3, M)
    lin = torch.addmm(b.float(), u[:, :K].float(), W.float().t())
    out = torch.full((N + 3, M + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    if epilogue in (RESIDUAL, COPY):
        gate = (tab[2] + c6[:, 2 * M:3 * M]).repeat_interleave(per_sample, 0)[:N]
        ref = x[:N] + gate * lin
        tail = x[N:].clone()
        m.ddit_linear_fwd(2, u, K + 8, W, b, N, M, K, out if epilogue == COPY else None, M + 8, resid=x, ada_table=tab, c6=c6,
                          gate_row=2, tokens_per_sample=per_sample)
        torch.cuda.synchronize()
        assert ((x[:N] - ref).abs() <= 1e-4 * (1 + ref.abs())).all()
        assert torch.equal(x[N:], tail)
    else:
        ref = torch.nn.functional.gelu(lin, approximate="tanh") if epilogue == GELU else lin
        m.ddit_linear_fwd(epilogue, u, K + 8, W, b, N, M, K, out, M + 8)
        torch.cuda.synchronize()
    if epilogue != RESIDUAL:
        assert ((out[:N, :M].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all()
        assert torch.isnan(out[N:]).all() and torch.isnan(out[:, M:]).all()


@pytest.mark.parametrize("epilogue,N,form", [(RESIDUAL, 16401, (32, 32)), (RESIDUAL, 17100, (64, 64)), (COPY, 16700, (64, 32)), (GELU, 32700, (32, 32)),
                                             (0, 32990, (64, 32))])
def test_the_rest_takes_the_form_of_so_few_tokens(epilogue, N, form):
    """The second launch is the one that a linear of its tokens takes, which ddit_linear_form says: the same bits."""
    import paper_2506_13497_amd as m
    k = 4608
    front = m.ddit_linear_front_tokens(epilogue, N, M, k, 256)
    assert front in (16320, 32640) and m.ddit_linear_form(epilogue, N - front, M, k, 256) == form
    gen = torch.Generator(device="cuda").manual_seed(N)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda")
    u, W, b, x0 = rnd(N, k).bfloat16(), (rnd(M, k) / k ** 0.5).bfloat16(), rnd(M).bfloat16(), rnd(N, M)
    got = []
    for first in (0, front):
        x, out = x0[first:].clone(), torch.full((N - first, M), float("nan"), dtype=torch.bfloat16, device="cuda")
        m.ddit_linear_fwd(epilogue & 3, u[first:], k, W, b, N - first, M, k, None if epilogue == RESIDUAL else out, M,
                          resid=x if epilogue & 2 else None, tokens_per_sample=N)
        got.append((x[front - first:], out[front - first:]))
    torch.cuda.synchronize()
    for a, b in zip(*got):
        assert torch.equal(a, b) or (torch.isnan(a).all() and torch.isnan(b).all())
