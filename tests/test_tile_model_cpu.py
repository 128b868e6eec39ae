"""The rules that choose a linear's output tile and fc2's split, against the times they rest on (host only)."""
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def m():
    import paper_2506_13497_amd as mod
    return mod


def test_picks_against_the_recorded_sweep(m):
    """Every tile timed on linears of six layers at 31 token counts: what the launcher picks costs little more than the best
    tile there, on average and at worst."""
    import bench
    rows, tiles = bench.read_tile_sweep(os.path.join(ROOT, "profiles", "gemm_tile_sweep.txt"))
    info = [m.ddit_linear_tile_info(t) for t in range(m.ddit_linear_tile_count())]
    assert tiles == [(t["rows"], t["cols"]) for t in info] and len(rows) > 800
    ratio = [us[m.ddit_linear_tile_choice(epi, N, n, k, 256)[0]] / min(us) for epi, n, k, N, us in rows]
    assert sum(ratio) / len(ratio) <= 1.009 and max(ratio) <= 1.27


# microseconds of a layer (hidden 1152, MLP 4608, 16 heads) with fc2 in one launch and in two and three parts
SPLIT_TIMES = {200: (102.0, 97.0, 95.5), 400: (106.5, 103.5, 103.6), 800: (117.0, 119.5, 120.8), 1152: (144.3, 142.4, 138.2),
               1500: (149.8, 150.8, 150.6), 1800: (180.6, 175.5, 177.0), 2048: (187.9, 181.3), 2304: (199.8, 192.5),
               2500: (202.7, 198.2), 2720: (212.6, 213.4), 2900: (215.7, 215.6), 3200: (222.5, 221.8), 3500: (233.5, 233.4)}


@pytest.mark.parametrize("N", sorted(SPLIT_TIMES))
def test_split_of_fc2_against_measured_layers(m, N):
    """The split taken is within a microsecond or two of the best one, and none is taken where none was measured to pay."""
    us = SPLIT_TIMES[N]
    parts = m.ddit_linear_partial_choice(N, 1152, 4608)[0]
    assert us[max(parts - 1, 0)] <= min(us) + 2.0
    assert parts == 0 or us[parts - 1] < us[0]


# microseconds of linears (epilogue, tokens, out-features, in-features) whose largest tile leaves a small part of a round: in two launches and
# in one of the tile that ddit_linear_form says
TWO_OR_ONE_TIMES = {(0, 24618, 768, 3072): (115.0, 107.8), (1, 54077, 768, 4096): (289.1, 267.0), (0, 19653, 1024, 3072): (114.2, 97.0),
                    (1, 51098, 1024, 4096): (375.3, 361.9), (0, 12371, 1344, 3072): (100.2, 88.1), (1, 26273, 1536, 4096): (262.1, 248.1),
                    (0, 10054, 2048, 3072): (118.6, 96.7), (1, 25280, 2048, 4096): (366.0, 340.0), (0, 6413, 3072, 4096): (136.2, 124.8),
                    (0, 55401, 3072, 3072): (848.6, 901.2), (1, 49774, 3072, 3072): (781.9, 825.2), (0, 50105, 3072, 4096): (969.3, 1009.0)}


@pytest.mark.parametrize("linear", sorted(TWO_OR_ONE_TIMES))
def test_two_launches_or_one_of_the_wide_tile(m, linear):
    epi, N, n, k = linear
    two, one = TWO_OR_ONE_TIMES[linear]
    assert m.ddit_linear_form(epi, N, n, k, 256) == (320, 256)
    assert (m.ddit_linear_front_tokens(epi, N, n, k, 256) == 0) == (one < two)


# microseconds of short contractions of many tokens (epilogue, tokens, out-features, in-features) with the best listed tile and with 320 x 256
SHORT_TIMES = {(0, 101426, 256, 256): (26.4, 29.8), (0, 72024, 256, 256): (20.8, 18.5), (0, 35058, 768, 256): (23.3, 27.4), (0, 61654, 768, 256): (38.6, 44.3),
               (0, 48295, 768, 256): (32.2, 29.6), (0, 74891, 768, 256): (43.3, 46.2), (1, 103073, 1024, 256): (91.9, 93.9), (1, 56225, 1024, 256): (51.6, 48.2),
               (0, 102646, 1024, 384): (102.9, 110.0), (0, 37559, 1024, 384): (41.0, 37.2), (1, 96119, 1536, 384): (143.9, 151.2), (1, 90202, 1536, 384): (142.8, 133.1),
               (0, 95692, 1536, 512): (161.4, 169.0), (0, 77392, 1536, 512): (143.0, 130.7), (1, 63057, 2048, 512): (152.9, 158.4), (1, 50247, 2048, 512): (132.0, 117.1),
               (0, 87984, 768, 768): (105.3, 110.3), (0, 51933, 2304, 768): (177.8, 164.1)}


@pytest.mark.parametrize("linear", sorted(SHORT_TIMES))
def test_short_contractions_take_the_wide_tile_where_it_is_faster(m, linear):
    listed, wide = SHORT_TIMES[linear]
    assert (m.ddit_linear_form(*linear, 256) == (320, 256)) == (wide < listed)


def test_text_projections_of_short_contractions(m):
    """56 layers of 512 features, k = 256: 600 text tokens 18.3 us with the best listed tile, 16.6 with 320 x 256; 1600 35.2 and 41.8; 2000 42.7 and 49.3."""
    form = lambda Ly, B: m.ddit_cross_kv_form(m.make_shape(B, 1, 1, 2, 256, 4, 64, 64, Ly, 28), 256)
    assert form(300, 2) == (320, 256) and form(200, 8) != (320, 256) and form(500, 4) != (320, 256)


@pytest.mark.parametrize("table,forms,mean,worst", [("gemm_forms_sweep.txt", {(320, 256): 10}, 0.94, 1.06), ("gemm_forms_sweep.txt", {(192, 192): 11}, 0.92, 1.06),
                                                    ("gemm_few_tokens_sweep.txt", {1: 12, 2: 13, 3: 14}, 0.79, 1.04)])
def test_forms_beside_the_list_against_their_recorded_sweeps(m, table, forms, mean, worst):
    """Where the launcher takes a form beside the list, the form's recorded time over that of the best listed tile."""
    import bench
    rows, tiles = bench.read_tile_sweep(os.path.join(ROOT, "profiles", table))
    count = m.ddit_linear_tile_count()
    ratio = []
    for epi, n, k, N, us in rows:
        few = m.ddit_linear_few_form(N, n, k, 1, 256)
        column = forms.get(few or m.ddit_linear_form(epi, N, n, k, 256))
        if column is not None:
            ratio.append(us[column] / min(us[:count]))
    assert len(ratio) >= 15 and sum(ratio) / len(ratio) <= mean and max(ratio) <= worst


# kernel times of attention of few units (kind, heads, frames, queries of a unit, keys), microseconds, the keys shared by four sets of wavefronts or not
SPLIT_KEYS_TIMES = {("cross", 4, 1, 36, 100): (6.64, 6.04), ("cross", 4, 1, 36, 170): (7.48, 8.10), ("cross", 4, 1, 72, 170): (8.20, 7.28), ("cross", 4, 1, 160, 230): (8.60, 9.48),
                    ("cross", 4, 1, 512, 300): (9.10, 10.26), ("cross", 16, 1, 36, 300): (9.08, 11.60), ("cross", 16, 1, 72, 100): (7.82, 7.40), ("cross", 16, 1, 72, 170): (8.60, 8.26),
                    ("cross", 16, 1, 72, 230): (8.98, 9.34), ("cross", 16, 1, 640, 100): (8.16, 7.84), ("cross", 16, 1, 640, 300): (10.12, 10.58), ("spatial", 4, 2, 144, 144): (8.08, 8.48),
                    ("spatial", 16, 2, 80, 80): (7.82, 7.32), ("spatial", 16, 5, 128, 128): (8.04, 7.66), ("spatial", 16, 1, 300, 300): (9.72, 10.28), ("spatial", 4, 1, 128, 128): (7.36, 6.38)}


@pytest.mark.parametrize("case", sorted(SPLIT_KEYS_TIMES))
def test_keys_are_shared_where_that_was_faster(m, case):
    kind, H, T, L, keys = case
    split, whole = SPLIT_KEYS_TIMES[case]
    shape = m.make_shape(1, T, 1, L, H * 72, H, 72, 64, keys, 1)
    form = m.ddit_attn_form(m.DDIT_ATTN_CROSS if kind == "cross" else m.DDIT_ATTN_SPATIAL, shape, 256)
    assert (form[1] == 4) == (split < whole)


# kernel times of one frame after the other (heads, frames, tokens of a frame), 64 keys a tile through a ring or all keys fetched at once
RESIDENT_TIMES = {(16, 16, 144): (12.68, 12.18), (16, 16, 160): (12.80, 12.50), (16, 16, 192): (12.92, 13.30), (16, 16, 256): (15.20, 16.92), (16, 15, 240): (15.22, 16.12),
                  (16, 13, 160): (11.84, 11.20), (16, 13, 224): (14.00, 14.36), (16, 11, 200): (13.22, 12.66), (16, 11, 256): (13.40, 13.92), (16, 9, 256): (13.14, 12.60),
                  (4, 51, 130): (11.20, 10.22), (4, 51, 250): (14.24, 15.04), (4, 40, 224): (13.04, 12.74), (4, 64, 224): (15.04, 15.86)}


@pytest.mark.parametrize("case", sorted(RESIDENT_TIMES))
def test_keys_are_fetched_at_once_where_that_was_faster(m, case):
    H, T, S = case
    ring, resident = RESIDENT_TIMES[case]
    assert m.ddit_attn_form(m.DDIT_ATTN_SPATIAL, m.make_shape(1, T, 1, S, H * 72, H, 72, 64, 8, 1), 256)[2] == (resident < ring)
