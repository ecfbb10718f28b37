"""The launch plan where an estimate that was off made steps slower than they had been.  Times: the kernels of one step on the GPU, the
plan asked for / the one that was taken."""
import pytest

import paper_2605_12471_amd as kv
from paper_2605_12471_amd import binding


def _plan(dtype, hq, hkv, d, n, prev):
    cfg = binding.make_config(1, hq, hkv, d, max(n, 256), 131072, dtype)
    rc, plan = kv.kvfold_plan_for(cfg, 256, n, prev + n)
    assert rc == 0
    return plan


@pytest.mark.parametrize("hq,hkv,n,prev,units", [
    (28, 4, 3559, 95, 2),     # 98 / 125 us
    (28, 4, 3559, 0, 2),      # 95 / 120
    (28, 4, 3273, 153, 2),    # 89 / 117
    (28, 4, 2752, 536, 2),    # 93 / 110
    (28, 4, 3249, 0, 1),      # 78 / 115 (not taken, but the other way round: here two units are the ones not evenly dealt)
])
def test_unsplit_steps_whose_workgroups_are_not_evenly_dealt(hq, hkv, n, prev, units):
    plan = _plan(kv.KVFOLD_BF16, hq, hkv, 128, n, prev)
    assert plan.n_splits == 1 and plan.units_per_wave == units


@pytest.mark.parametrize("d,n,prev", [
    (128, 2500, 0),     # 78 / 85 us
    (128, 2500, 95),    # 81 / 88
    (64, 2867, 0),      # 54 / 73
    (64, 3013, 0),      # 57 / 78
])
def test_neither_form_evenly_dealt(d, n, prev):
    """One unit per wavefront: the XCD with the heavy workgroups has the power that the others leave."""
    plan = _plan(kv.KVFOLD_BF16, 28, 4, d, n, prev)
    assert plan.n_splits == 1 and plan.units_per_wave == 1


@pytest.mark.parametrize("hq,hkv,d,n,prev,splits", [
    (32, 8, 128, 286, 319, 1),    # 13.05 / 15.4 us with two pieces
    (32, 32, 128, 264, 409, 1),   # 15.4 / 18.0
    (32, 32, 128, 260, 597, 1),   # 16.7 / 19.9
    (32, 8, 128, 284, 699, 1),    # 16.7 / 18.7
    (28, 4, 128, 374, 497, 1),    # 15.6 / 17.7
    (64, 8, 128, 147, 718, 1),    # 16.4 / 17.8
    (8, 1, 64, 1202, 1710, 3),    # 22.4 / 27.5
    (16, 2, 64, 821, 5170, 4),    # 38.2 / 39.6
    (28, 4, 64, 565, 6793, 4),    # 45 / 49
    (32, 2, 128, 2182, 631, 1),   # 97 / 102.5
    (4, 1, 64, 3845, 1320, 4),    # 37 / 40.3
])
def test_pieces_that_meet_are_not_free(hq, hkv, d, n, prev, splits):
    """Two pieces need no merge kernel, but the later one waits for memory at its end."""
    assert _plan(kv.KVFOLD_BF16, hq, hkv, d, n, prev).n_splits == splits


@pytest.mark.parametrize("hq,hkv,d,n,prev", [
    (32, 8, 64, 596, 1222),     # 20.0 us / 26.7 whole
    (28, 4, 64, 2485, 8164),    # 195 / 240 with seven
    (32, 8, 64, 950, 3361),     # 43 / 54.6 whole
    (28, 4, 128, 670, 461),     # 19.5 / 24.5 whole
    (28, 4, 128, 632, 797),     # 21.6 / 29.3 whole
])
def test_two_pieces_that_meet(hq, hkv, d, n, prev):
    assert _plan(kv.KVFOLD_BF16, hq, hkv, d, n, prev).n_splits == 2


@pytest.mark.parametrize("hq,hkv,n,prev", [
    (8, 2, 295, 1252),     # 41 / 53 us with 13 pieces
    (4, 1, 897, 146),      # 38 / 49 with 9
    (8, 2, 506, 1131),     # 44 / 62 with 9 (dealt evenly, 255 of 288 workgroups with work)
    (8, 2, 1023, 305),     # 53 / 78 with 11
])
def test_fp32_pieces_fit_one_round(hq, hkv, n, prev):
    """... without the empty ones of early tokens making room for others."""
    assert _plan(kv.KVFOLD_F32, hq, hkv, 128, n, prev).n_workgroups <= 256


@pytest.mark.parametrize("hq,hkv,d,n,prev,waves", [
    (8, 2, 128, 64, 60000, 4),      # 124 / 149 us
    (8, 2, 128, 64, 25645, 4),      # 71 / 81
    (4, 1, 128, 127, 33421, 4),     # 90 / 109
    (32, 32, 64, 573, 858, 4),      # 66 / 78
    (28, 4, 128, 512, 16384, 8),    # 635 / 643 with 4 pieces instead of 9
])
def test_fp32_wavefronts_per_workgroup(hq, hkv, d, n, prev, waves):
    plan = _plan(kv.KVFOLD_F32, hq, hkv, d, n, prev)
    units = -(-n * (hq // hkv) // 32)
    assert plan.n_workgroups == plan.n_splits * hkv * -(-units // waves)


@pytest.mark.parametrize("hq,hkv,d,n,prev", [
    (32, 32, 128, 12, 1091),     # 13.1 / 16.4 us, unsplit
    (32, 32, 64, 21, 1196),      # 9.1 / 10.7
    (32, 32, 64, 1, 1111),       # 8.3 / 9.3
])
def test_few_rows_are_split_where_the_merge_is_worth_it(hq, hkv, d, n, prev):
    assert _plan(kv.KVFOLD_BF16, hq, hkv, d, n, prev).n_splits > 1


@pytest.mark.parametrize("n,prev", [
    (37, 32768),     # 41.4 / 44.1 us, 27 pieces
    (40, 16384),     # 27.3 / 30.3
])
def test_five_units_a_head_have_their_cus_to_themselves(n, prev):
    """Two workgroups a head of whose eight wavefronts three have no rows."""
    plan = _plan(kv.KVFOLD_BF16, 32, 8, 128, n, prev)
    assert plan.units_per_wave == 1 and plan.n_workgroups == 256


@pytest.mark.parametrize("hq,hkv,d,n,prev,units", [
    (14, 2, 128, 4282, 65, 2),      # 83 / 111 us
    (14, 2, 64, 4201, 0, 2),        # 57 / 68
    (8, 1, 128, 7507, 0, 2),        # 142 / 198
    (8, 2, 128, 7255, 196, 2),      # 127 / 162
    (16, 4, 128, 2909, 2237, 2),    # 103 / 112
    (28, 4, 128, 2038, 0, 1),       # (448 workgroups, dealt in turn)
])
def test_heavy_and_light_workgroups_share_cus_only_if_dealt_in_turn(hq, hkv, d, n, prev, units):
    plan = _plan(kv.KVFOLD_BF16, hq, hkv, d, n, prev)
    assert plan.units_per_wave == units and plan.pair_order == (1 if units == 1 else 0)


@pytest.mark.parametrize("n,prev", [(4045, 189), (4045, 300)])
def test_64_wide_two_unit_grids_do_not_count_on_empty_workgroups_beyond_a_round(n, prev):
    """31 to 36 us; 45 with seven pieces of two units a wavefront, 448 workgroups of which 256 have work."""
    plan = _plan(kv.KVFOLD_BF16, 4, 1, 64, n, prev)
    assert not (plan.units_per_wave == 2 and plan.n_workgroups > 256 * 5 // 4)


@pytest.mark.parametrize("hq,hkv,d,n,prev", [
    (16, 2, 64, 15, 66000),      # 20.7 / 25.5 us with one unit a workgroup
    (16, 2, 64, 15, 114000),     # 27.1 / 39.1
    (32, 8, 64, 221, 6855),      # 29.2 / 31.8 (with the rotary embedding)
])
def test_units_share_a_workgroup_where_each_reading_its_keys_alone_is_slower(hq, hkv, d, n, prev):
    plan = _plan(kv.KVFOLD_BF16, hq, hkv, d, n, prev)
    units = -(-n * (hq // hkv) // 32)
    assert plan.n_workgroups < hkv * units * plan.n_splits


@pytest.mark.parametrize("hq,hkv,d,n,prev,dealt", [
    (8, 2, 128, 128, 4187, True),      # 30.9 us with a unit's keys dealt to the wavefronts / 39.9 without
    (8, 2, 128, 128, 20000, False),    # 92.7 / 78.0
    (32, 8, 64, 37, 30000, False),     # 89.2 / 83.7
    (4, 1, 64, 128, 0, True),          # 7.5 / 12.0
    (28, 4, 128, 28, 0, True),         # 28 keys: a single block has nothing to deal
])
def test_fp32_keys_are_dealt_to_wavefronts_where_units_are_few(hq, hkv, d, n, prev, dealt):
    plan = _plan(kv.KVFOLD_F32, hq, hkv, d, n, prev)
    units = -(-n * (hq // hkv) // 32)
    assert (plan.n_workgroups == hkv * units * plan.n_splits) == (dealt and n + prev > 32)


@pytest.mark.parametrize("hq,hkv,d,n,prev,units", [
    (32, 8, 128, 37, 32768, 1),     # one unit a wavefront as fast, and what these steps have always taken
    (16, 16, 128, 213, 25614, 1),   # 60.9 / 69.9 us
    (32, 8, 128, 52, 32711, 1),     # 44.8 / 50.4
    (28, 4, 128, 20, 104146, 2),    # 54.1 / 73.6: the two workgroups of a piece do not share an L2
])
def test_two_units_a_wavefront_where_a_piece_would_be_read_twice(hq, hkv, d, n, prev, units):
    assert _plan(kv.KVFOLD_BF16, hq, hkv, d, n, prev).units_per_wave == units


@pytest.mark.parametrize("hq,hkv,d,n,prev,dealt", [
    (28, 4, 128, 10, 65536, False),    # 113.6 us / 124.5 with a unit's keys dealt to the wavefronts
    (16, 16, 64, 124, 15584, False),   # 71.7 / 77.5
    (12, 4, 64, 39, 55847, False),     # 63.1 / 68.0
    (8, 2, 128, 22, 62438, True),      # 105.2 without / 63.4: few units in all
    (32, 8, 128, 11, 26579, True),     # 87.1 / 77.0: two units a head
])
def test_fp32_keys_of_three_and_four_units_a_head_on_long_caches(hq, hkv, d, n, prev, dealt):
    plan = _plan(kv.KVFOLD_F32, hq, hkv, d, n, prev)
    units = -(-n * (hq // hkv) // 32)
    assert (plan.n_workgroups == hkv * units * plan.n_splits) == dealt
