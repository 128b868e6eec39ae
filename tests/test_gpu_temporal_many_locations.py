"""Temporal attention of short clips with enough locations that several share a workgroup: packs of two, a power of two
below what the tile holds, and as many as it holds; last packs partly empty, partial head groups, two samples; treated
q and k; and an infinity or NaN of one location stays there."""
import numpy as np
import pytest
import torch

import ddit_synth as syn
from helpers import assert_parity, dev_to_f64, to_dev, to_f64
from oracle import stdit_oracle as ora

pytestmark = pytest.mark.gpu

SHAPES = [
    (1, 4, 531, 3, 72),    # two of the eight that fit
    (2, 4, 523, 4, 64),    # four, two samples
    (1, 2, 2081, 2, 72),   # eight of sixteen
    (1, 2, 4099, 2, 64),   # all sixteen
    (1, 10, 259, 12, 72),  # three frames' worth, three head groups
    (1, 3, 2563, 1, 72),   # ten
    (1, 7, 1031, 5, 72),   # four, two head groups
    (1, 11, 531, 3, 72),   # too long to share
]


def _inputs(B, T, S, H, dh, seed):
    sh = syn.Shape(B, T, 1, S, H * dh, H, dh, 64, 8, 1)
    return sh, syn.make_attn_inputs("temporal", sh, seed)


@pytest.mark.parametrize("B,T,S,H,dh", SHAPES)
def test_packs(B, T, S, H, dh):
    import paper_2506_13497_amd as m
    sh, d = _inputs(B, T, S, H, dh, 83)
    o_ref, lse_ref = ora.temporal_attention(*(to_f64(d[n]) for n in "qkv"))
    A = sh.A
    o = torch.full((B, T, S, H, dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full(lse_ref.shape, float("nan"), dtype=torch.float32, device="cuda")
    m.ddit_attn_fwd(m.DDIT_ATTN_TEMPORAL, m.make_shape(B, T, 1, S, A, H, dh, 64, 8, 1), *(to_dev(d[n]) for n in "qkv"), A, A, None, o, A, lse)
    torch.cuda.synchronize()
    assert_parity(dev_to_f64(o).reshape(o_ref.shape), o_ref, "packed temporal attention")
    assert np.max(np.abs(dev_to_f64(lse) - lse_ref)) < 2e-2


@pytest.mark.parametrize("norm,rope", [(True, False), (False, True), (True, True)], ids=["norm", "rope", "norm+rope"])
@pytest.mark.parametrize("B,T,S,H,dh", SHAPES + [(1, 30, 37, 5, 72), (1, 32, 37, 4, 64)])
def test_treated_packs(B, T, S, H, dh, norm, rope):
    """The treatment inside the attention kernel against the pass of its own that rounds q and k to bf16 as it does."""
    import paper_2506_13497_amd as m
    sh, d = _inputs(B, T, S, H, dh, 84)
    A, shape = sh.A, m.make_shape(B, T, 1, S, H * dh, H, dh, 64, 8, 1)
    gen = torch.Generator(device="cuda").manual_seed(7)
    g = [(1.0 + 0.2 * torch.randn(dh, device="cuda", generator=gen)).bfloat16() if norm else None for _ in range(2)]
    out = []
    for fuse in (True, False):
        qkv = torch.cat([to_dev(d[n]).reshape(B * T * S, A) for n in "qkv"], 1).contiguous()
        tab = torch.empty(T * dh, device="cuda") if rope else None
        o = torch.full((B * T * S, A), float("nan"), dtype=torch.bfloat16, device="cuda")
        m.ddit_self_attn_fwd(m.DDIT_ATTN_TEMPORAL, shape, qkv[:, :A], qkv[:, A:2 * A], qkv[:, 2 * A:], 3 * A, 3 * A, *g, tab, fuse, o, A)
        torch.cuda.synchronize()
        out.append(dev_to_f64(o))
    assert_parity(out[0], out[1], "treated temporal attention")


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("operand", [0, 1, 2])
def test_locations_of_a_pack_keep_apart(value, operand):
    import paper_2506_13497_amd as m
    T, S, H, dh = 4, 1051, 2, 72
    A, shape = H * dh, m.make_shape(1, T, 1, S, H * dh, H, dh, 64, 8, 1)
    d = syn.make_attn_inputs("temporal", syn.Shape(1, T, 1, S, A, H, dh, 64, 8, 1), 85)
    clean = [to_dev(d[n]).reshape(T, S, A) for n in "qkv"]
    dirty = [t.clone() for t in clean]
    dirty[operand][1, 6, 5] = value
    out = []
    for q, k, v in (clean, dirty):
        o = torch.empty((T, S, A), dtype=torch.bfloat16, device="cuda")
        m.ddit_attn_fwd(m.DDIT_ATTN_TEMPORAL, shape, q, k, v, A, A, None, o, A)
        out.append(o)
    torch.cuda.synchronize()
    others = [s for s in range(S) if s != 6]
    assert torch.equal(out[0][:, others], out[1][:, others])
    assert torch.equal(out[0][:, 6, dh:], out[1][:, 6, dh:])           # the location's other head
