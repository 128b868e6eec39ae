"""Attention whose wavefronts share a unit's keys (few queries for the chip): every set of key tiles keeps its own
softmax reference, and the sets meet at the end.  Key counts at the edges of a tile and of the forms, samples whose text
leaves some sets without a tile, a dominant key in a late tile; the kernel against the oracle, log-sum-exp included."""
import numpy as np
import pytest
import torch

import ddit_synth as syn
from helpers import assert_parity, dev_to_f64, to_dev, to_f64
from oracle import stdit_oracle as ora

pytestmark = pytest.mark.gpu


def run(kind, sh, d, valid=None):
    import paper_2506_13497_amd as m
    o = torch.full(tuple(d["q"].shape), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((sh.B, sh.L, sh.H), float("nan"), device="cuda")
    m.ddit_attn_fwd(kind, m.make_shape(sh.B, sh.T, sh.Hp, sh.Wp, sh.D, sh.H, sh.dh, sh.M, sh.Ly, sh.n_blocks),
                    *(to_dev(d[k]) if isinstance(d[k], np.ndarray) else d[k] for k in "qkv"), sh.A, sh.A, valid, o, sh.A, lse)
    torch.cuda.synchronize()
    return dev_to_f64(o), dev_to_f64(lse)


@pytest.mark.parametrize("H,dh", [(5, 72), (4, 64)])
@pytest.mark.parametrize("Ly,valid,L", [(300, [300, 1, 64], 65), (320, [65, 320, 129], 64), (321, [321, 2, 200], 129),
                                        (700, [700, 640, 63], 33), (128, [128, 65, 66], 1)])
def test_cross(Ly, valid, L, H, dh):
    import paper_2506_13497_amd as m
    sh = syn.Shape(3, 1, 1, L, H * dh, H, dh, 64, Ly, 1)
    d = syn.make_attn_inputs("cross", sh, 71, q_scale=3.0, Lq=L)
    o_ref, lse_ref = ora.cross_attention(*(to_f64(d[k]) for k in "qkv"), np.array(valid))
    o, lse = run(m.DDIT_ATTN_CROSS, sh, d, valid)
    assert_parity(o, o_ref.reshape(o.shape), "cross %d %s" % (Ly, valid))
    assert np.abs(lse - lse_ref.reshape(lse.shape)).max() <= 2e-2


@pytest.mark.parametrize("H,dh", [(4, 72), (4, 64)])
@pytest.mark.parametrize("S", [65, 192, 193, 320, 321, 450, 1031])
def test_spatial(S, H, dh):
    import paper_2506_13497_amd as m
    sh = syn.Shape(1, 2, 1, S, H * dh, H, dh, 64, 8, 1)
    d = syn.make_attn_inputs("spatial", sh, 72, q_scale=2.0)
    o_ref, lse_ref = ora.spatial_attention(*(to_f64(d[k]) for k in "qkv"))
    o, lse = run(m.DDIT_ATTN_SPATIAL, sh, d)
    assert_parity(o, o_ref, "spatial %d" % S)
    assert np.abs(lse - lse_ref.reshape(lse.shape)).max() <= 2e-2


@pytest.mark.parametrize("Ly", [300, 700])
@pytest.mark.parametrize("at", [3, 70, 257, 290])
def test_a_dominant_key_in_one_set(Ly, at):
    """One key far above all others: only its set has weight, whatever reference the other sets took."""
    import paper_2506_13497_amd as m
    H, dh, L = 4, 72, 96
    sh = syn.Shape(1, 1, 1, L, H * dh, H, dh, 64, Ly, 1)
    rng = np.random.default_rng(at)
    q = np.abs(rng.standard_normal((1, L, H, dh))) + 0.5
    k = -4.0 * np.abs(rng.standard_normal((1, Ly, H, dh)))
    k[:, at] = 4.0
    q, k, v = (torch.from_numpy(a).to(torch.bfloat16) for a in (q, k, rng.standard_normal((1, Ly, H, dh))))
    o, lse = run(m.DDIT_ATTN_CROSS, sh, {"q": q.cuda(), "k": k.cuda(), "v": v.cuda()})
    o_ref, lse_ref = ora.cross_attention(*(t.double().numpy() for t in (q, k, v)), np.array([Ly]))
    assert_parity(o, o_ref, "dominant key %d" % at)
    assert np.abs(lse / lse_ref.reshape(lse.shape) - 1).max() <= 1e-2


@pytest.mark.parametrize("Ly", [300, 700])
def test_scores_of_minus_infinity_in_one_set(Ly):
    """Keys whose scores are -inf have no weight, also where they fill a set's first tile or all of its tiles."""
    import paper_2506_13497_amd as m
    H, dh, L = 4, 72, 40
    sh = syn.Shape(1, 1, 1, L, H * dh, H, dh, 64, Ly, 1)
    rng = np.random.default_rng(5)
    q, k, v = (torch.from_numpy(rng.standard_normal(s)).to(torch.bfloat16) for s in ((1, L, H, dh), (1, Ly, H, dh), (1, Ly, H, dh)))
    q[..., 0], k[..., 0] = 1.0, 0.0
    cut = k.clone()
    cut[:, 64:256, :, 0] = float("-inf")
    keep = [j for j in range(Ly) if not 64 <= j < 256]
    o, _ = run(m.DDIT_ATTN_CROSS, sh, {"q": q.cuda(), "k": cut.cuda(), "v": v.cuda()})
    o_ref, _ = ora.cross_attention(*(t.double().numpy() for t in (q, k[:, keep], v[:, keep])), np.array([len(keep)]))
    assert_parity(o, o_ref, "-inf in one set")
