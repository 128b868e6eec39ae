"""Attention and LayerNorm launches whose further workgroups fetch the weights of the launches after them: blocks at the
token counts where that begins and ends (3200), with weights smaller than what one workgroup reads and weights for many
rows of workgroups beside a launch of few, spatial, short and long temporal layers, with and without the q/k treatment,
against the oracle.  What is fetched is not used, so the result has the parity bar of every block."""
import pytest
import torch

import ddit_synth as syn
from helpers import assert_parity, dev_to_f64, dict_dev, dict_f64, to_dev, to_f64
from oracle import stdit_oracle as ora

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("options", [False, True])
@pytest.mark.parametrize("B,T,Hp,Wp,D,H,dh,M", [
    (1, 1, 1, 1, 64, 1, 64, 8),         # one workgroup, and a fetch of 128 pieces and less
    (2, 3, 3, 5, 72, 1, 72, 40),        # weights that no number of workgroups divides
    (1, 2, 2, 3, 1152, 16, 72, 4608),   # many rows of workgroups for the weights of a launch of three
    (1, 34, 2, 4, 128, 2, 64, 256),     # temporal attention on the streaming kernel
    (1, 2, 40, 40, 72, 1, 72, 72),      # 3200 tokens
    (1, 3, 11, 97, 72, 1, 72, 72),      # 3201
])
def test_block_with_weights_fetched_ahead(B, T, Hp, Wp, D, H, dh, M, options):
    import paper_2506_13497_amd as m
    sh = syn.Shape(B, T, Hp, Wp, D, H, dh, M, 6, 1)
    act, c6 = syn.make_activations(sh, 71), syn.make_c6(sh, 71, 0.5)
    wb = syn.make_block_weights(sh, 71, 0, table_std=0.02, qk_norm=options)
    shape = m.make_shape(B, T, Hp, Wp, D, H, dh, M, 6, 1, m.DDIT_FLAG_QK_NORM | m.DDIT_FLAG_ROPE_TEMPORAL if options else 0)
    ws = m.alloc_workspace(shape)
    ws.fill_(0xFF)
    x_out = torch.full((B, T, sh.S, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    dwb = dict_dev(wb)
    m.ddit_stdit_block_fwd(shape, m.block_struct(dwb), to_dev(act["x"]), to_dev(act["y"]), None, to_dev(c6), x_out, ws)
    torch.cuda.synchronize()
    ref = ora.block_fwd(to_f64(act["x"]), to_f64(act["y"]), None, c6.astype("float64"), dict_f64(wb), H, dh, rope_temporal=options)
    assert_parity(dev_to_f64(x_out), ref, "block of %d tokens" % sh.N)


def test_weights_beyond_a_grids_rows():
    """fc1 and fc2 of 3.3 GB each beside launches of one workgroup: more rows of workgroups would be due than a grid may have.
    With weights of zero the MLP adds nothing, whatever its width."""
    import paper_2506_13497_amd as m
    D, widths = 4096, (8, 400000)
    sh = syn.Shape(1, 1, 1, 1, D, 1, 64, widths[0], 6, 1)
    act, c6, wb = syn.make_activations(sh, 71), to_dev(syn.make_c6(sh, 71, 0.5)), syn.make_block_weights(sh, 71, 0, table_std=0.02)
    dwb, x, y = dict_dev(wb), to_dev(act["x"]), to_dev(act["y"])
    zeros, out = torch.zeros(widths[1] * D, dtype=torch.bfloat16, device="cuda"), []
    for M in widths:
        for layer in dwb.values():
            layer.update(w_fc1=zeros, w_fc2=zeros, b_fc1=zeros, b_fc2=zeros)
        shape = m.make_shape(1, 1, 1, 1, D, 1, 64, M, 6, 1, 0)
        out.append(torch.full((1, 1, 1, D), float("nan"), dtype=torch.bfloat16, device="cuda"))
        m.ddit_stdit_block_fwd(shape, m.block_struct(dwb), x, y, None, c6, out[-1], m.alloc_workspace(shape))
        torch.cuda.synchronize()
    assert not torch.isnan(out[0]).any() and torch.equal(out[0], out[1])
