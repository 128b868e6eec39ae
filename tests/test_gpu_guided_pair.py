"""Guided sampling with both text caches: the two evaluations of a step run side by side where the workspace of one holds
them.  Against the oracle's loop, at shapes where fc2 comes in parts beside h, where h lies where q|k|v and o were, with two
samples of different text lengths, with the q/k treatment, and where there is no room and they run one by one; and against
the same steps taken call by call: the same operands, fp32 sums in another order and bf16 roundings of intermediates that
may fall the other way (2^-9 each; measured 1.2e-3 of a latent's change, of which the bar is four times).  Another order is
no larger error: the two errors against the oracle are norms over a latent's 1700 values and more of as many roundings
each, which differ by their scatter, a few hundredths; the bar is a fifth."""
import numpy as np
import pytest
import torch

import ddit_synth as syn
from helpers import assert_parity, dev_to_f64, rel_fro, to_dev
from oracle import latent_io_oracle as lio
from test_gpu_io import Setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,Hp,Wp,D,H,dh,M,Ly,blocks,options,together", [
    (1, 2, 6, 9, 1152, 16, 72, 4608, 300, 3, False, True),    # fc2 in three parts
    (2, 3, 5, 7, 1152, 16, 72, 256, 120, 3, False, True),     # h in the place of q|k|v and o
    (2, 3, 5, 7, 256, 4, 64, 1024, 120, 3, True, True),       # attention narrower than h, q and k treated
    (1, 35, 2, 3, 256, 4, 64, 512, 120, 3, True, True),       # temporal attention on the streaming kernel
    (1, 2, 10, 10, 1152, 16, 72, 4608, 300, 2, False, True),  # another order: fc2 in two parts instead of three
    (1, 4, 10, 15, 1152, 16, 72, 4608, 300, 2, True, True),   # another order: q|k|v and fc1 on a tile that sums k in one piece
    (1, 2, 20, 41, 1152, 4, 72, 4608, 16, 1, False, False),   # no room: one by one
])
def test_guided_steps_with_caches(B, T, Hp, Wp, D, H, dh, M, Ly, blocks, options, together):
    import paper_2506_13497_amd as lib
    st = Setup(lib, syn.Shape(B, T, Hp, Wp, D, H, dh, M, Ly, blocks), 4, 64, options=options)
    sh, n, guidance = st.sh, 4, 2.5
    valid = [Ly - 7 * b for b in range(1, B + 1)]
    y, y_u = st.caption_dev(lib, st.c_text), st.caption_dev(lib, st.c_unc)
    kv = torch.empty(lib.ddit_cross_kv_bytes(st.shape) // 2, dtype=torch.bfloat16, device="cuda")
    kv_u = torch.empty_like(kv)
    lib.ddit_cross_kv_precompute(st.shape, st.step, y, kv)
    lib.ddit_cross_kv_precompute(st.shape, st.step, y_u, kv_u)
    z, z1 = to_dev(st.z), to_dev(st.z)
    scratch = torch.full((2,) + tuple(z.shape), float("nan"), dtype=torch.float32, device="cuda")
    st.ws.fill_(0xFF)
    lib.ddit_sample(st.shape, st.step, st.io, z, y, valid, y_u, guidance, n, 1, 3, scratch, st.ws, kv, kv_u)
    torch.cuda.synchronize()
    # one by one, the workspace's own text cache (behind x, xh, q|k|v and o; parts of fc2 may reach 4 N D into it) stays as it was
    at = sum(-(-n // 256) * 256 for n in (4 * sh.N * D, 2 * sh.N * D, 6 * sh.N * sh.A, 2 * sh.N * sh.A))
    assert bool((st.ws[at + 4 * sh.N * D:at + kv.numel() * 2] != 0xFF).any()) == together
    mc, mu = st.oracle_model(st.c_text, np.array(valid)), st.oracle_model(st.c_unc, None)
    ref = lio.sample(st.z.astype(np.float64), lambda zz, t: lio.guide(mc(zz, t), mu(zz, t), guidance), n, 1, 3)
    assert_parity(dev_to_f64(z), ref, "latent after two guided steps")
    for i in (1, 2):
        t, tn = [1000.0 * (1 - i / n)] * B, [1000.0 * (1 - (i + 1) / n)] * B
        lib.ddit_eps_theta(st.shape, st.step, st.io, z1, y, valid, t, scratch[0], st.ws, cross_kv=kv)
        lib.ddit_eps_theta(st.shape, st.step, st.io, z1, y_u, None, t, scratch[1], st.ws, cross_kv=kv_u)
        lib.ddit_solver_step(z1, scratch[0], scratch[1], guidance, t, tn, z1.numel() // B)
    torch.cuda.synchronize()
    assert rel_fro(dev_to_f64(z) - st.z, dev_to_f64(z1) - st.z) < 5e-3
    error, error_one = (rel_fro(dev_to_f64(v) - st.z, ref - st.z) for v in (z, z1))
    print("error of the change: side by side %.3e, one by one %.3e" % (error, error_one))
    assert error < 1.2 * error_one


def test_guided_step_of_many_tokens():
    """25000 tokens an evaluation side by side (the text cache of 90 narrow blocks leaves the room), against call by call."""
    import paper_2506_13497_amd as lib
    st = Setup(lib, syn.Shape(1, 5, 50, 100, 72, 1, 72, 72, 300, 90), 4, 64)
    y, y_u = st.caption_dev(lib, st.c_text), st.caption_dev(lib, st.c_unc)
    kv = torch.empty(lib.ddit_cross_kv_bytes(st.shape) // 2, dtype=torch.bfloat16, device="cuda")
    kv_u = torch.empty_like(kv)
    lib.ddit_cross_kv_precompute(st.shape, st.step, y, kv)
    lib.ddit_cross_kv_precompute(st.shape, st.step, y_u, kv_u)
    z, z1 = to_dev(st.z), to_dev(st.z)
    scratch = torch.full((2,) + tuple(z.shape), float("nan"), dtype=torch.float32, device="cuda")
    st.ws.fill_(0xFF)
    lib.ddit_sample(st.shape, st.step, st.io, z, y, [200], y_u, 2.5, 4, 1, 2, scratch, st.ws, kv, kv_u)
    torch.cuda.synchronize()
    at = 14 * st.sh.N * 72 + 1024   # one by one, the workspace's own text cache (behind x, xh, q|k|v and o) stays as it was
    assert bool((st.ws[at:at + kv.numel()] != 0xFF).any())
    for ys, cache, valid, out in ((y, kv, [200], scratch[0]), (y_u, kv_u, None, scratch[1])):
        lib.ddit_eps_theta(st.shape, st.step, st.io, z1, ys, valid, [750.0], out, st.ws, cross_kv=cache)
    lib.ddit_solver_step(z1, scratch[0], scratch[1], 2.5, [750.0], [500.0], z1.numel())
    torch.cuda.synchronize()
    assert torch.isfinite(z).all() and rel_fro(dev_to_f64(z) - st.z, dev_to_f64(z1) - st.z) < 5e-3


@pytest.mark.parametrize("which", ["y", "y_uncond"])
def test_misaligned_text_is_refused_with_caches(which):
    """The text itself is not read when the caches are given, but a misaligned pointer is refused as without guidance."""
    import paper_2506_13497_amd as lib
    st = Setup(lib, syn.Shape(1, 2, 3, 4, 256, 4, 64, 1024, 16, 1), 4, 64)
    y = torch.zeros(16 * 256 + 1, dtype=torch.bfloat16, device="cuda")
    kv = torch.zeros(lib.ddit_cross_kv_bytes(st.shape) // 2, dtype=torch.bfloat16, device="cuda")
    z = to_dev(st.z)
    scratch = torch.empty((2,) + tuple(z.shape), dtype=torch.float32, device="cuda")
    with pytest.raises(lib.DditError) as e:
        lib.ddit_sample(st.shape, st.step, st.io, z, y[which == "y":], None, y[which == "y_uncond":], 2.5, 4, 1, 2, scratch,
                        st.ws, kv, kv)
    assert "aligned" in str(e.value)
