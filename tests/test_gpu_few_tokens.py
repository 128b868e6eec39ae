"""The linear's forms for few tokens (32 x 32, 64 x 32 and 64 x 64 tiles, the k-steps dealt out to the wavefronts): rows and columns that end
inside a tile, contractions with fewer k-steps than wavefronts, with ragged last ones, with as many as all rings hold and one more,
strided operands, samples that change inside a tile; and fc2's parts through a step.  Every case says which form has to take it.  Against float64: bf16 results one rounding (2^-9),
fp32 results 2 sqrt(k) 2^-24 of the terms' size, taken four times."""
import numpy as np
import pytest
import torch

import ddit_synth as syn
from helpers import assert_parity, dev_to_f64, dict_dev, dict_f64, to_dev, to_f64
from oracle import stdit_oracle as ora

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n,k,form", [(1, 8, 8, 1), (31, 40, 56, 1), (32, 1152, 64, 1), (33, 264, 72, 1), (64, 1152, 1152, 1), (65, 392, 1160, 1),
                                        (100, 288, 1144, 1), (224, 1152, 1216, 1), (17, 1152, 4608, 1), (256, 256, 256, 1), (300, 24, 384, 1),
                                        (40, 520, 392, 1), (441, 1144, 1152, 2), (449, 1152, 1160, 0), (448, 1152, 1096, 2), (300, 1144, 4096, 2), (257, 1152, 776, 2),
                                        (760, 1144, 4600, 3), (515, 1152, 3080, 3), (896, 1152, 3008, 3), (897, 1152, 3008, 0), (833, 1096, 2952, 3)])
def test_linear(N, n, k, form):
    """Form 0: one more k-step or token than the forms for few tokens take."""
    import paper_2506_13497_amd as m
    assert m.ddit_linear_few_form(N, n, k, 1, 256) == form
    g = torch.Generator(device="cuda").manual_seed(N + k)
    rnd = lambda *s: torch.randn(s, device="cuda", generator=g)
    wide, W, bias = rnd(N, k + 16).bfloat16(), rnd(n, k).bfloat16(), rnd(n).bfloat16()
    u = wide[:, 8:8 + k]
    tps = max(1, N // 3)
    tab, c6 = rnd(6, n), rnd((N + tps - 1) // tps, 6 * n)
    ref = u.double() @ W.double().t() + bias.double()
    fp32 = 8 * k ** 0.5 * 2.0 ** -24 * k ** 0.5
    for epi, want in ((0, ref), (1, torch.nn.functional.gelu(ref, approximate="tanh"))):
        out = torch.full((N, n + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
        m.ddit_linear_fwd(epi, u, k + 16, W, bias, N, n, k, out, n + 8)
        torch.cuda.synchronize()
        assert torch.isnan(out[:, n:].float()).all()
        assert ((out[:, :n].double() - want).abs() <= 2.0 ** -8 * want.abs() + fp32 + 1e-5).all(), (N, n, k, epi)
    gate = tab[2].double() + c6.double()[torch.arange(N, device="cuda") // tps, 2 * n:3 * n]
    for copy in (False, True):
        x0 = rnd(N, n)
        x, out = x0.clone(), torch.full((N, n), float("nan"), dtype=torch.bfloat16, device="cuda")
        m.ddit_linear_fwd(2, u, k + 16, W, bias, N, n, k, out if copy else None, n if copy else 0, resid=x, ada_table=tab, c6=c6,
                          gate_row=2, tokens_per_sample=tps)
        torch.cuda.synchronize()
        want = x0.double() + gate * ref
        assert ((x.double() - want).abs() <= (fp32 + 2.0 ** -20 * ref.abs()) * (1 + gate.abs()) + 2.0 ** -22 * want.abs()).all(), (N, n, k, copy)
        assert not copy or torch.equal(out, x.bfloat16())


@pytest.mark.parametrize("B,T,Hp,Wp,M,parts,form", [(1, 1, 1, 3, 4608, 3, 1), (2, 2, 2, 8, 4608, 3, 1), (1, 5, 3, 5, 4608, 3, 2), (1, 5, 5, 8, 4608, 3, 0),
                                                    (1, 3, 10, 10, 6080, 2, 3)])
def test_parts_of_fc2(B, T, Hp, Wp, M, parts, form):
    """Two blocks of few tokens, where fc2 comes in parts, in each of the forms and in none; parts of 48 and 47 k-steps in the last."""
    import paper_2506_13497_amd as m
    D, H, dh, Ly = 1152, 16, 72, 20
    sh = syn.Shape(B, T, Hp, Wp, D, H, dh, M, Ly, 2)
    assert m.ddit_linear_partial_choice(sh.N, D, M)[0] == parts and m.ddit_linear_few_form(sh.N, D, M, parts, 256) == form
    sw = syn.make_step_weights(sh, 54)
    blocks = [syn.make_block_weights(sh, 54, i, table_std=0.1) for i in range(2)]
    act, temb = syn.make_activations(sh, 54), syn.make_temb(sh, 54)
    shape = m.make_shape(B, T, Hp, Wp, D, H, dh, M, Ly, 2)
    ws = m.alloc_workspace(shape)
    ws.fill_(0xFF)
    dsw, dblocks = {k: to_dev(v) for k, v in sw.items()}, [dict_dev(b) for b in blocks]
    x_out = torch.full((B, T, sh.S, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    m.ddit_denoise_step(shape, m.step_struct(dsw, dblocks), to_dev(act["x"]), to_dev(act["y"]), None, None, to_dev(temb), x_out, ws)
    torch.cuda.synchronize()
    ref = ora.denoise_step(to_f64(act["x"]), to_f64(act["y"]), None, None, dict_f64(sw), [dict_f64(b) for b in blocks],
                           H, dh, temb=temb.astype(np.float64))
    assert_parity(dev_to_f64(x_out), ref, "step of %d tokens" % sh.N)


@pytest.mark.parametrize("N,n,k", [(64, 1152, 1152), (300, 1152, 4096), (600, 1152, 4096), (17, 1152, 4608), (224, 512, 2048)])
def test_sums_are_as_exact_as_the_listed_tiles(N, n, k):
    """fp32 results against float64: dealing the k-steps out makes shorter chains, so the error is no larger than with the listed tile of
    64 x 64 (two chains); and a second call gives the same bits."""
    import paper_2506_13497_amd as m
    assert m.ddit_linear_few_form(N, n, k, 1, 256) > 0
    g = torch.Generator(device="cuda").manual_seed(N + k)
    rnd = lambda *s: torch.randn(s, device="cuda", generator=g)
    u, W, bias = rnd(N, k).bfloat16(), rnd(n, k).bfloat16(), rnd(n).bfloat16()
    ref = u.double() @ W.double().t() + bias.double()
    err, got = [], []
    for tile in (-1, -1, m.ddit_linear_tile_count() - 1):
        x = torch.zeros(N, n, device="cuda")
        m.ddit_linear_fwd_tile(tile, 2, u, k, W, bias, N, n, k, None, 0, resid=x)
        torch.cuda.synchronize()
        got.append(x)
        err.append((x.double() - ref).norm().item())
    assert torch.equal(got[0], got[1]) and err[0] <= err[2]
