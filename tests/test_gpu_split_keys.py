"""Attention whose wavefronts share a unit's keys (few queries for the chip): the sets of key tiles begin with one softmax reference,
move it on their own, and meet at the end.  Key counts at the edges of a tile and of the forms, samples whose text
leaves some sets without a tile, a dominant key in a late tile; the kernel against the oracle, log-sum-exp included.  Every case says
how many sets have to share the keys: four with all keys fetched at once, two tile by tile, or one just beside those rules."""
import numpy as np
import pytest
import torch

import ddit_synth as syn
from helpers import assert_parity, dev_to_f64, to_dev, to_f64
from oracle import stdit_oracle as ora

pytestmark = pytest.mark.gpu


def sets_of(keys, queries):
    return 4 if (192 if 64 < queries <= 128 else 128) < keys <= 320 else 2 if keys > 704 else 1


def run(kind, sh, d, sets, valid=None):
    import paper_2506_13497_amd as m
    o = torch.full(tuple(d["q"].shape), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((sh.B, sh.L, sh.H), float("nan"), device="cuda")
    shape = m.make_shape(sh.B, sh.T, sh.Hp, sh.Wp, sh.D, sh.H, sh.dh, sh.M, sh.Ly, sh.n_blocks)
    assert m.ddit_attn_form(kind, shape, 256)[1:] == {4: (4, True), 2: (2, False), 1: (1, False)}[sets]
    m.ddit_attn_fwd(kind, shape,
                    *(to_dev(d[k]) if isinstance(d[k], np.ndarray) else d[k] for k in "qkv"), sh.A, sh.A, valid, o, sh.A, lse)
    torch.cuda.synchronize()
    return dev_to_f64(o), dev_to_f64(lse)


@pytest.mark.parametrize("H,dh", [(5, 72), (4, 64)])
@pytest.mark.parametrize("Ly,valid,L", [(300, [300, 1, 64], 65), (320, [65, 320, 129], 64), (321, [321, 2, 200], 129),
                                        (700, [700, 640, 63], 33), (128, [128, 65, 66], 1), (192, [192, 65, 129], 1), (129, [129, 128, 64], 200), (193, [193, 192, 1], 128), (300, [60, 64, 1], 65), (705, [705, 64, 65], 33),
                                        (720, [720, 128, 129], 33), (1031, [1031, 1, 700], 130), (768, [768, 767, 705], 96)])
def test_cross(Ly, valid, L, H, dh):
    import paper_2506_13497_amd as m
    sh = syn.Shape(3, 1, 1, L, H * dh, H, dh, 64, Ly, 1)
    d = syn.make_attn_inputs("cross", sh, 71, q_scale=3.0, Lq=L)
    o_ref, lse_ref = ora.cross_attention(*(to_f64(d[k]) for k in "qkv"), np.array(valid))
    o, lse = run(m.DDIT_ATTN_CROSS, sh, d, sets_of(Ly, L), valid)
    assert_parity(o, o_ref.reshape(o.shape), "cross %d %s" % (Ly, valid))
    assert np.abs(lse - lse_ref.reshape(lse.shape)).max() <= 2e-2


@pytest.mark.parametrize("H,dh", [(4, 72), (4, 64)])
@pytest.mark.parametrize("S", [65, 129, 192, 193, 320, 321, 450, 704, 705, 832, 1031])
def test_spatial(S, H, dh):
    import paper_2506_13497_amd as m
    sh = syn.Shape(1, 2, 1, S, H * dh, H, dh, 64, 8, 1)
    d = syn.make_attn_inputs("spatial", sh, 72, q_scale=2.0)
    o_ref, lse_ref = ora.spatial_attention(*(to_f64(d[k]) for k in "qkv"))
    o, lse = run(m.DDIT_ATTN_SPATIAL, sh, d, sets_of(S, S))
    assert_parity(o, o_ref, "spatial %d" % S)
    assert np.abs(lse - lse_ref.reshape(lse.shape)).max() <= 2e-2


@pytest.mark.parametrize("Ly,at", [(Ly, at) for Ly in (300, 700, 720, 1031) for at in (3, 70, 257, 290)] + [(720, 650), (720, 719), (1031, 1030)])
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
    o, lse = run(m.DDIT_ATTN_CROSS, sh, {"q": q.cuda(), "k": k.cuda(), "v": v.cuda()}, sets_of(Ly, L))
    o_ref, lse_ref = ora.cross_attention(*(t.double().numpy() for t in (q, k, v)), np.array([Ly]))
    assert_parity(o, o_ref, "dominant key %d" % at)
    assert np.abs(lse / lse_ref.reshape(lse.shape) - 1).max() <= 1e-2


@pytest.mark.parametrize("Ly,at", [(300, range(64, 256)), (700, range(64, 256)), (720, range(64, 256)), (1031, range(64, 128)),
                                   (1031, [j for j in range(1031) if j // 64 % 2 == 1])])
def test_scores_of_minus_infinity_in_one_set(Ly, at):
    """Keys whose scores are -inf have no weight, also where they fill a set's first tile or all of its tiles."""
    import paper_2506_13497_amd as m
    H, dh, L = 4, 72, 40
    sh = syn.Shape(1, 1, 1, L, H * dh, H, dh, 64, Ly, 1)
    rng = np.random.default_rng(5)
    q, k, v = (torch.from_numpy(rng.standard_normal(s)).to(torch.bfloat16) for s in ((1, L, H, dh), (1, Ly, H, dh), (1, Ly, H, dh)))
    q[..., 0], k[..., 0] = 1.0, 0.0
    cut = k.clone()
    cut[:, list(at), :, 0] = float("-inf")
    keep = [j for j in range(Ly) if j not in set(at)]
    o, _ = run(m.DDIT_ATTN_CROSS, sh, {"q": q.cuda(), "k": cut.cuda(), "v": v.cuda()}, sets_of(Ly, L))
    o_ref, _ = ora.cross_attention(*(t.double().numpy() for t in (q, k[:, keep], v[:, keep])), np.array([len(keep)]))
    assert_parity(o, o_ref, "-inf in one set")


def attend(q, k, v, keep=None):
    """The kernel's output and log-sum-exp of one sample of cross-attention, and the oracle's over the keys kept."""
    import paper_2506_13497_amd as m
    L, Ly, H, dh = q.shape[1], k.shape[1], q.shape[2], q.shape[3]
    o, lse = run(m.DDIT_ATTN_CROSS, syn.Shape(1, 1, 1, L, H * dh, H, dh, 64, Ly, 1), {"q": q.cuda(), "k": k.cuda(), "v": v.cuda()}, sets_of(Ly, L))
    keep = list(range(Ly)) if keep is None else keep
    o_ref, lse_ref = ora.cross_attention(*(t.double().numpy() for t in (q, k[:, keep], v[:, keep])), np.array([len(keep)]))
    return o, lse, o_ref, lse_ref.reshape(lse.shape)


def operands_with_a_bias(Ly, H, dh, seed):
    """q, k, v ~ N(0,1); the first two columns of q are ones and those of k zero, so that they add to a key's scores."""
    rng = np.random.default_rng(seed)
    q, k, v = (torch.from_numpy(rng.standard_normal(s)).to(torch.bfloat16) for s in ((1, 96, H, dh), (1, Ly, H, dh), (1, Ly, H, dh)))
    q[..., :2], k[..., :2] = 1.0, 0.0
    return q, k, v


@pytest.mark.parametrize("H,dh", [(4, 72), (4, 64)])
@pytest.mark.parametrize("level", [-1e6, -1e9, -3.3e38])
@pytest.mark.parametrize("Ly,tiles", [(300, (0,)), (300, (1,)), (300, (2,)), (300, (3,)), (300, (4,)), (300, (1, 2, 3)), (200, (1,)),
                                      (720, (0,)), (720, (1,)), (720, (2,)), (720, (3,)), (720, (1, 3, 5, 7, 9, 11)), (720, (11,)), (705, (1,))])
def test_whole_tiles_far_below(Ly, tiles, level, H, dh):
    """Key tiles whose scores lie far below the others' have no weight, whichever set has them and whether or not their level is a
    bf16 number (it is off the nearest one by 1.5e-3 of it)."""
    q, k, v = operands_with_a_bias(Ly, H, dh, 7)
    for t in tiles:
        k[:, 64 * t:64 * t + 64, :, 0], k[:, 64 * t:64 * t + 64, :, 1] = level, -1.5e-3 * level
    o, lse, o_ref, lse_ref = attend(q, k, v)
    assert_parity(o, o_ref, "%s at %g" % (tiles, level))
    assert np.abs(lse - lse_ref).max() <= 2e-2


@pytest.mark.parametrize("Ly,cut", [(300, (1,)), (300, (0, 1, 2)), (300, (0, 1, 2, 3)), (720, (0,)), (720, (1,)), (720, (1, 3, 5, 7, 9, 11))])
def test_first_tiles_of_minus_infinity_and_the_rest_far_below_zero(Ly, cut):
    """A set whose first tile holds -inf alone begins with the others' reference, not with zero.  (Where all sets' first tiles do, the
    reference is zero and the rest is near it.)"""
    q, k, v = operands_with_a_bias(Ly, 4, 72, 8)
    k[..., 0] = 0.0 if cut == (0, 1, 2, 3) else -1200.0
    for t in cut:
        k[:, 64 * t:64 * t + 64, :, 0] = float("-inf")
    o, lse, o_ref, lse_ref = attend(q, k, v, [j for j in range(Ly) if j // 64 not in cut])
    assert_parity(o, o_ref, "-inf in %s" % (cut,))
    assert np.abs(lse - lse_ref).max() <= 2e-2


@pytest.mark.parametrize("high,lower", [(2, 3), (3, 2), (10, 11), (6, 3)])
def test_a_later_tile_far_below_another_sets(high, lower):
    """Two tiles far above the first ones, in different sets: the lower one's sums overflow for its reference's rounding and have no
    weight.  (At 3e5 a score's fp32 sum is rounded to 1/32, a weight by a few thousandths.)"""
    q, k, v = operands_with_a_bias(720, 4, 72, 9)
    k[:, 64 * high:64 * high + 64, :, 0] = 299008.0
    k[:, 64 * lower:64 * lower + 64, :, 0], k[:, 64 * lower:64 * lower + 64, :, 1] = 266240.0, 1000.0
    o, _, o_ref, _ = attend(q, k, v)
    assert_parity(o, o_ref, "tile %d above tile %d" % (high, lower))
