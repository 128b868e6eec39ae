"""Temporal attention with several locations in one matrix tile: frame counts around the packing's limit, location
counts that leave a pack partly empty, partial head groups, two samples; and an infinity or NaN of one location
stays there."""
import numpy as np
import pytest
import torch

import ddit_synth as syn
from helpers import assert_parity, dev_to_f64, to_dev, to_f64
from oracle import stdit_oracle as ora

pytestmark = pytest.mark.gpu


def _shape(m, sh):
    return m.make_shape(sh.B, sh.T, sh.Hp, sh.Wp, sh.D, sh.H, sh.dh, sh.M, sh.Ly, sh.n_blocks)


@pytest.mark.parametrize("B,T,Hp,Wp,H,dh", [
    (1, 1, 7, 5, 3, 72), (2, 1, 1, 3, 4, 64), (2, 2, 3, 7, 5, 72), (1, 3, 1, 1, 2, 64), (2, 4, 5, 5, 16, 72),
    (1, 7, 3, 3, 4, 72), (2, 8, 3, 3, 3, 64), (2, 10, 2, 5, 4, 72), (2, 11, 2, 3, 4, 72), (1, 31, 1, 3, 5, 72),
])
def test_packed_locations(B, T, Hp, Wp, H, dh):
    import paper_2506_13497_amd as m
    sh = syn.Shape(B, T, Hp, Wp, H * dh, H, dh, 64, 8, 1)
    d = syn.make_attn_inputs("temporal", sh, 80)
    o_ref, lse_ref = ora.temporal_attention(*(to_f64(d[n]) for n in "qkv"))
    A = sh.A
    o = torch.full((B, T, sh.S, H, dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full(lse_ref.shape, float("nan"), dtype=torch.float32, device="cuda")
    m.ddit_attn_fwd(m.DDIT_ATTN_TEMPORAL, _shape(m, sh), *(to_dev(d[n]) for n in "qkv"), A, A, None, o, A, lse)
    torch.cuda.synchronize()
    assert_parity(dev_to_f64(o).reshape(o_ref.shape), o_ref, "packed temporal attention")
    assert np.max(np.abs(dev_to_f64(lse) - lse_ref)) < 2e-2


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("operand", [0, 1, 2])
def test_packed_locations_keep_apart(value, operand):
    import paper_2506_13497_amd as m
    sh = syn.Shape(1, 4, 3, 5, 144, 2, 72, 64, 8, 1)
    d = syn.make_attn_inputs("temporal", sh, 81)
    clean = [to_dev(d[n]).reshape(sh.T, sh.S, sh.A) for n in "qkv"]
    dirty = [t.clone() for t in clean]
    dirty[operand][1, 2, 5] = value
    out = []
    for q, k, v in (clean, dirty):
        o = torch.empty((sh.T, sh.S, sh.A), dtype=torch.bfloat16, device="cuda")
        m.ddit_attn_fwd(m.DDIT_ATTN_TEMPORAL, _shape(m, sh), q, k, v, sh.A, sh.A, None, o, sh.A)
        out.append(o)
    torch.cuda.synchronize()
    others = [s for s in range(sh.S) if s != 2]
    assert torch.equal(out[0][:, others], out[1][:, others])
    assert torch.equal(out[0][:, 2, 72:], out[1][:, 2, 72:])           # the location's other head
    assert not torch.isfinite(out[1][:, 2, :72]).all()
