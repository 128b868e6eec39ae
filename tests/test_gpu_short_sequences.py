"""Self-attention at the sequence lengths where the streaming kernel changes its queries per workgroup (64 up to 64
queries, else 128): the edges of a wavefront, of the key tile and of both forms, against the oracle."""
import pytest
import torch

import ddit_synth as syn
from helpers import assert_parity, dev_to_f64, to_dev, to_f64
from oracle import stdit_oracle as ora

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,dh", [(5, 72), (4, 64)])   # 5 heads x 3 groups: units that do not divide the XCDs
@pytest.mark.parametrize("n", [1, 32, 33, 63, 64, 65, 128])
@pytest.mark.parametrize("kind", ["spatial", "temporal"])
def test_lengths_at_the_borders(kind, n, H, dh):
    import paper_2506_13497_amd as m
    T, S = (3, n) if kind == "spatial" else (n, 3)
    A = H * dh
    sh = syn.Shape(1, T, 1, S, A, H, dh, 64, 8, 1)
    d = syn.make_attn_inputs(kind, sh, 93, q_scale=2.0)
    o_ref, _ = (ora.spatial_attention if kind == "spatial" else ora.temporal_attention)(*(to_f64(d[k]) for k in "qkv"))
    o = torch.full((1, T, S, H, dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    m.ddit_attn_fwd(m.DDIT_ATTN_SPATIAL if kind == "spatial" else m.DDIT_ATTN_TEMPORAL,
                    m.make_shape(1, T, 1, S, A, H, dh, 64, 8, 1), *(to_dev(d[k]) for k in "qkv"), A, A, None, o, A)
    torch.cuda.synchronize()
    assert_parity(dev_to_f64(o), o_ref, "%s attention, %d long" % (kind, n))
