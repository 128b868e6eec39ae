"""The linear's k loop where it can go wrong: fewer k-steps than the operand ring is deep, exactly as many, one
more, whole and partial last steps; tiles that begin while the ring still holds the tile before; rows and
columns that end inside a tile.  Every compiled tile, through the C ABI, against the oracle."""
import math

import numpy as np
import pytest
import torch

import ddit_synth as syn
from helpers import assert_parity, dev_to_f64, to_dev, to_f64
from oracle import stdit_oracle as ora

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2506_13497_amd as m
    assert torch.cuda.is_available()
    return m


@pytest.mark.parametrize("k", [56, 64, 72, 128, 136, 192, 320, 384, 456, 512, 520, 584])
@pytest.mark.parametrize("N,n", [(67, 136), (4500, 392)])   # one ragged tile; more than one round of the small tiles
def test_linear_k_steps(lib, N, n, k):
    u, W = syn.normal_bits((61, N, k), (N, k), 1.0), syn.normal_bits((62, n, k), (n, k), 1.0 / math.sqrt(k))
    b = syn.normal_bits((63, n), (n,), 0.5)
    resid = np.random.default_rng(k).standard_normal((N, n)).astype(np.float32)
    du, dW, db, tab = to_dev(u), to_dev(W), to_dev(b), torch.zeros(6, n, device="cuda")
    tab[2] = 0.75
    c6 = torch.zeros(1, 6 * n, device="cuda")
    lin = ora.linear(to_f64(u), to_f64(W), to_f64(b))
    for tile in range(lib.ddit_linear_tile_count()):
        out = torch.full((N, n), float("nan"), dtype=torch.bfloat16, device="cuda")
        lib.ddit_linear_fwd_tile(tile, 0, du, k, dW, db, N, n, k, out, n)
        x = to_dev(resid)
        lib.ddit_linear_fwd_tile(tile, 2, du, k, dW, db, N, n, k, None, 0, resid=x, ada_table=tab, c6=c6, gate_row=2,
                                 tokens_per_sample=N)
        torch.cuda.synchronize()
        assert_parity(dev_to_f64(out), lin, "tile %d" % tile)
        assert_parity(dev_to_f64(x), resid + 0.75 * lin, "tile %d, residual" % tile)
