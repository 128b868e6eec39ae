"""The linear's form for few tokens (32 x 32 tiles, the k-steps dealt to six wavefronts): rows and columns that end inside a tile,
contractions with fewer k-steps than wavefronts, with ragged last ones, with as many as all rings hold and one more, strided
operands, samples that change inside a tile; and fc2's parts through a step.  Against float64: bf16 results one rounding (2^-9),
fp32 results 2 sqrt(k) 2^-24 of the terms' size, taken four times."""
import numpy as np
import pytest
import torch

import ddit_synth as syn
from helpers import assert_parity, dev_to_f64, dict_dev, dict_f64, to_dev, to_f64
from oracle import stdit_oracle as ora

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n,k", [(1, 8, 8), (31, 40, 56), (32, 1152, 64), (33, 264, 72), (64, 1152, 1152), (65, 392, 1160), (100, 288, 1144),
                                   (224, 1152, 1216), (17, 1152, 4608), (256, 256, 256), (300, 24, 384), (40, 520, 392)])
def test_linear(N, n, k):
    import paper_2506_13497_amd as m
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


@pytest.mark.parametrize("B,T,Hp,Wp,parts", [(1, 1, 1, 3, 3), (2, 2, 2, 8, 3), (1, 5, 3, 5, 3)])
def test_parts_of_fc2(B, T, Hp, Wp, parts):
    """Two blocks of few tokens, where fc2 comes in parts in this form (the last shape is just too large for it)."""
    import paper_2506_13497_amd as m
    D, H, dh, M, Ly = 1152, 16, 72, 4608, 20
    sh = syn.Shape(B, T, Hp, Wp, D, H, dh, M, Ly, 2)
    assert m.ddit_linear_partial_choice(sh.N, D, M)[0] == parts
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
