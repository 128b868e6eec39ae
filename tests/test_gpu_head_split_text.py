"""Text k|v projections of all layers in one launch for a rank of a head split: 2, 6, 10 and 14 heads of 72 have
2 * A out-features that only a tile of 288 columns divides; text lengths at the edges of its 192 rows.  Against fp32
PyTorch on the same bf16 operands: one bf16 rounding (2^-9 of the value) and fp32 sums over k = 1152."""
import pytest
import torch

import ddit_synth as syn
from helpers import dict_dev, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [2, 6, 10, 14])
@pytest.mark.parametrize("Ly", [1, 192, 193, 300])
def test_text_projection_of_a_head_split(H, Ly):
    import paper_2506_13497_amd as m
    D, dh, blocks = 1152, 72, 2
    sh = syn.Shape(1, 1, 1, 2, D, H, dh, 64, Ly, blocks)
    dsw = {k: to_dev(v) for k, v in syn.make_step_weights(sh, 61).items()}
    dblocks = [dict_dev(syn.make_block_weights(sh, 61, i, table_std=0.1)) for i in range(blocks)]
    shape = m.make_shape(1, 1, 1, 2, D, H, dh, 64, Ly, blocks)
    y = to_dev(syn.make_activations(sh, 61)["y"])
    kv = torch.full((m.ddit_cross_kv_bytes(shape) // 2,), float("nan"), dtype=torch.bfloat16, device="cuda")
    m.ddit_cross_kv_precompute(shape, m.step_struct(dsw, dblocks), y, kv)
    torch.cuda.synchronize()
    got = kv.view(2 * blocks, Ly, 2 * H * dh).float()
    for l in range(2 * blocks):
        w = dblocks[l // 2]["spatial" if l % 2 == 0 else "temporal"]
        ref = torch.nn.functional.linear(y.float().view(Ly, D), w["w_ckv"].float(), w["b_ckv"].float())
        assert ((got[l] - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all(), (H, Ly, l)
