"""fc2 in partial sums that the next LayerNorm, or the final cast, adds to the stream: a step of two blocks
against the CPU oracle at token counts where it comes in three and in two parts, with rows that end inside a
tile and samples that change inside a workgroup's rows, the gates of the update per sample, and a k whose
last part is ragged."""
import numpy as np
import pytest
import torch

import ddit_synth as syn
from helpers import assert_parity, dev_to_f64, dict_dev, dict_f64, to_dev, to_f64
from oracle import stdit_oracle as ora

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,Hp,Wp,D,H,dh,M", [
    (1, 2, 3, 5, 1152, 16, 72, 4608),
    (2, 3, 5, 11, 1152, 16, 72, 4616),    # 330 rows, 165 a sample
    (3, 3, 7, 9, 1152, 4, 72, 4608),      # 567 rows; attention narrower than the stream
    (2, 1, 23, 25, 1152, 16, 72, 4608),   # 1150 rows
    (1, 1, 45, 46, 1152, 16, 72, 4608),   # 2070 rows
    (1, 1, 5, 7, 1344, 21, 64, 5376),      # LayerNorm with more than five chunks a lane
])
def test_step_with_partial_sums(B, T, Hp, Wp, D, H, dh, M):
    import paper_2506_13497_amd as m
    sh = syn.Shape(B, T, Hp, Wp, D, H, dh, M, 20, 2)
    sw = syn.make_step_weights(sh, 51)
    blocks = [syn.make_block_weights(sh, 51, i, table_std=0.1) for i in range(2)]
    act = syn.make_activations(sh, 51)
    temb = syn.make_temb(sh, 51)
    shape = m.make_shape(B, T, Hp, Wp, D, H, dh, M, 20, 2, 0)
    ws = m.alloc_workspace(shape)
    ws.fill_(0xFF)
    dsw, dblocks = {k: to_dev(v) for k, v in sw.items()}, [dict_dev(b) for b in blocks]
    x_out = torch.full((B, T, sh.S, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    m.ddit_denoise_step(shape, m.step_struct(dsw, dblocks), to_dev(act["x"]), to_dev(act["y"]), None, None, to_dev(temb), x_out, ws)
    torch.cuda.synchronize()
    ref = ora.denoise_step(to_f64(act["x"]), to_f64(act["y"]), None, None, dict_f64(sw), [dict_f64(b) for b in blocks],
                           H, dh, temb=temb.astype(np.float64))
    assert_parity(dev_to_f64(x_out), ref, "step with fc2 in partial sums")


@pytest.mark.parametrize("B,T,Hp,Wp,D,H,dh,M,parts", [
    (2, 2, 5, 10, 1152, 16, 72, 4608, 3),
    (1, 4, 16, 31, 1152, 16, 72, 4608, 2),
    (1, 2, 4, 5, 256, 4, 64, 1024, 0),
])
def test_taps_show_what_an_untapped_step_runs(B, T, Hp, Wp, D, H, dh, M, parts):
    """Keeping taps changes neither how fc2 is split nor a bit of the result, and the last tap is the result."""
    import paper_2506_13497_amd as m
    sh = syn.Shape(B, T, Hp, Wp, D, H, dh, M, 20, 2)
    assert m.ddit_linear_partial_choice(sh.N, D, M)[0] == parts
    dsw = {k: to_dev(v) for k, v in syn.make_step_weights(sh, 52).items()}
    dblocks = [dict_dev(syn.make_block_weights(sh, 52, i, table_std=0.1)) for i in range(2)]
    act = syn.make_activations(sh, 52)
    x_in, y, temb = to_dev(act["x"]), to_dev(act["y"]), to_dev(syn.make_temb(sh, 52))
    out = []
    for flags in (0, m.DDIT_FLAG_TAPS):
        shape = m.make_shape(B, T, Hp, Wp, D, H, dh, M, 20, 2, flags)
        ws = m.alloc_workspace(shape)
        ws.fill_(0xFF)
        x_out = torch.empty((B, T, sh.S, D), dtype=torch.bfloat16, device="cuda")
        m.ddit_denoise_step(shape, m.step_struct(dsw, dblocks), x_in, y, None, None, temb, x_out, ws)
        torch.cuda.synchronize()
        out.append(x_out.reshape(sh.N, D))
    assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16))
    last = m.read_tap(shape, ws, 1, "x_out").reshape(sh.N, D)
    assert torch.equal(last.to(torch.bfloat16).view(torch.int16), out[1].view(torch.int16))


def test_workspace_query_touches_no_device():
    """The query in a process of its own opens no GPU: a parent that forks its workers may ask first."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = ("import os, paper_2506_13497_amd as m\n"
            "fds = lambda: sum('kfd' in os.readlink('/proc/self/fd/' + f) for f in os.listdir('/proc/self/fd') if os.path.exists('/proc/self/fd/' + f))\n"
            "before = fds()\n"
            "m.ddit_workspace_bytes(m.make_shape(1, 16, 9, 16, 1152, 16, 72, 4608, 300, 28))\n"
            "print('opened', fds() - before)\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "opened 0" in r.stdout, r.stdout + r.stderr


@pytest.mark.parametrize("n_blocks", [1, 28])
def test_static_scratch_takes_the_parts_that_fit(n_blocks):
    """One rank's share at 2500 tokens: with one block's text the two parts of fc2 fit the built-in scratch, with 28
    blocks' they do not and fc2 adds in one launch; both match the oracle, as the caller-owned workspace does."""
    import paper_2506_13497_amd as m
    B, T, Hp, Wp, D, H, dh, M, Ly = 1, 4, 25, 25, 1152, 4, 72, 4608, 300
    sh = syn.Shape(B, T, Hp, Wp, D, H, dh, M, Ly, n_blocks)
    shape = m.make_shape(B, T, Hp, Wp, D, H, dh, M, Ly, n_blocks)
    assert (m.ddit_workspace_bytes(shape) > 64 << 20) == (n_blocks == 28)
    w = syn.make_block_weights(sh, 57, 0, table_std=0.1)
    act, c6 = syn.make_activations(sh, 57), syn.make_c6(sh, 57, 0.5)
    dw = dict_dev(w)
    bw = m.block_struct(dw)
    x, y, dc6 = to_dev(act["x"]), to_dev(act["y"]), to_dev(c6)
    ref = ora.block_fwd(to_f64(act["x"]), to_f64(act["y"]), None, to_f64(c6), dict_f64(w), H, dh)
    ws = m.alloc_workspace(shape)
    ws.fill_(0xFF)
    for call in (lambda o: m.ddit_stdit_block_fwd(shape, bw, x, y, None, dc6, o, ws),
                 lambda o: m.ddit_stdit_block_fwd_static(shape, bw, x, y, None, dc6, o)):
        out = torch.empty((B, T, sh.S, D), dtype=torch.bfloat16, device="cuda")
        call(out)
        torch.cuda.synchronize()
        assert_parity(dev_to_f64(out), ref, "block, %d blocks' text" % n_blocks)


@pytest.mark.parametrize("tile", range(4, 10))   # the tiles compiled for partial sums
@pytest.mark.parametrize("N,n,k", [(70, 392, 4608), (1, 8, 520), (1300, 1152, 4608), (2600, 1152, 1160)])
def test_every_partial_sum_tile(tile, N, n, k):
    """One ragged tile; one row; a tile grid that fills the CUs and more than one round of it; a k whose last part is
    ragged: every part against float64 over its own k, the bias in the first.  fp32 sums of at most 4608 products:
    2 sqrt(k) 2^-24 of the terms' size, taken four times."""
    import paper_2506_13497_amd as m
    info = m.ddit_linear_tile_info(tile)
    g = torch.Generator(device="cuda").manual_seed(tile + N)
    u = torch.randn(N, k, device="cuda", generator=g).bfloat16()
    W, bias = torch.randn(n, k, device="cuda", generator=g).bfloat16(), torch.randn(n, device="cuda", generator=g).bfloat16()
    for parts in (2, 3):
        per = -(-(-(-k // 64)) // parts) * 64
        out = torch.full((parts, N, n), float("nan"), device="cuda")
        m.ddit_linear_partial_fwd(tile, parts, u, k, W, bias, N, n, k, out)
        torch.cuda.synchronize()
        for p in range(parts):
            ref = u[:, p * per:(p + 1) * per].double() @ W[:, p * per:(p + 1) * per].double().t()
            if p == 0:
                ref += bias.double()
            assert (out[p].double() - ref).abs().max() <= 8 * k ** 0.5 * 2.0 ** -24 * k ** 0.5, (info, parts, p)


@pytest.mark.parametrize("B,T,Hp,Wp,H,parts", [(2, 2, 5, 10, 16, 3), (1, 5, 10, 23, 4, 3), (1, 5, 20, 23, 4, 2), (1, 4, 10, 10, 4, 2)])
def test_parts_beside_the_treated_attention(B, T, Hp, Wp, H, parts):
    """The split is taken (the count is asserted), the regions behind the parts move for it (a third part; attention
    narrower than the stream), and with them the angles of the rotary embedding."""
    import paper_2506_13497_amd as m
    D, dh, M, Ly = 1152, 72, 4608, 20
    sh = syn.Shape(B, T, Hp, Wp, D, H, dh, M, Ly, 2)
    assert m.ddit_linear_partial_choice(sh.N, D, M)[0] == parts
    sw = syn.make_step_weights(sh, 53)
    blocks = [syn.make_block_weights(sh, 53, i, qk_norm=True, table_std=0.1) for i in range(2)]
    act, temb = syn.make_activations(sh, 53), syn.make_temb(sh, 53)
    shape = m.make_shape(B, T, Hp, Wp, D, H, dh, M, Ly, 2, m.DDIT_FLAG_QK_NORM | m.DDIT_FLAG_ROPE_TEMPORAL)
    ws = m.alloc_workspace(shape)
    ws.fill_(0xFF)
    dsw, dblocks = {k: to_dev(v) for k, v in sw.items()}, [dict_dev(b) for b in blocks]
    x_out = torch.full((B, T, sh.S, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    m.ddit_denoise_step(shape, m.step_struct(dsw, dblocks), to_dev(act["x"]), to_dev(act["y"]), None, None, to_dev(temb), x_out, ws)
    torch.cuda.synchronize()
    ref = ora.denoise_step(to_f64(act["x"]), to_f64(act["y"]), None, None, dict_f64(sw), [dict_f64(b) for b in blocks],
                           H, dh, temb=temb.astype(np.float64), rope_temporal=True)
    assert_parity(dev_to_f64(x_out), ref, "step with fc2 in %d parts and treated q, k" % parts)
