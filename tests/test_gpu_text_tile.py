"""Text k|v projections of all layers at the token counts where the launcher takes a tile of 320 rows: one row of tiles, full and
ragged, and a ragged second; and the first counts behind one row and two, which other tiles take.  Enough layers to fill the chip with it.  Against fp32 PyTorch on the
same bf16 operands: one bf16 rounding (2^-9 of the value) and fp32 sums over k = 256."""
import pytest
import torch

import ddit_synth as syn
from helpers import dict_dev, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Ly", [289, 300, 320, 321, 620, 641])
def test_text_projection(Ly):
    import paper_2506_13497_amd as m
    D, H, dh, blocks = 256, 4, 64, 64
    sh = syn.Shape(1, 1, 1, 2, D, H, dh, 64, Ly, blocks)
    shape = m.make_shape(1, 1, 1, 2, D, H, dh, 64, Ly, blocks)
    assert m.ddit_cross_kv_form(shape, 256) == {321: (192, 256), 641: (256, 256)}.get(Ly, (320, 256))
    dsw = {k: to_dev(v) for k, v in syn.make_step_weights(sh, 62).items()}
    dblocks = [dict_dev(syn.make_block_weights(sh, 62, 0, table_std=0.1)) for _ in range(blocks)]
    g = torch.Generator(device="cuda").manual_seed(Ly)
    for b in dblocks:
        for layer in b.values():
            layer["w_ckv"].normal_(0, 0.05, generator=g)
            layer["b_ckv"].normal_(0, 0.5, generator=g)
    y = torch.randn(Ly, D, device="cuda", generator=g).bfloat16()
    kv = torch.full((m.ddit_cross_kv_bytes(shape) // 2,), float("nan"), dtype=torch.bfloat16, device="cuda")
    m.ddit_cross_kv_precompute(shape, m.step_struct(dsw, dblocks), y, kv)
    torch.cuda.synchronize()
    got = kv.view(2 * blocks, Ly, 2 * H * dh).float()
    for l in range(2 * blocks):
        w = dblocks[l // 2]["spatial" if l % 2 == 0 else "temporal"]
        ref = torch.nn.functional.linear(y.float(), w["w_ckv"].float(), w["b_ckv"].float())
        assert ((got[l] - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all(), (Ly, l)
