"""Which form an attention call takes (tr_block_attn_plan, tr_attn_workgroup: host only, nothing is launched): parts of the keys,
packed heads, shape of the workgroups."""
import pytest

from gpu_util import RING, RING_BF16, STEP_BF16, STEP_F32, attn_per_unit as per_unit, attn_plan as plan, attn_shape as shape


@pytest.fixture(scope="module")
def tr():
    from paper_2412_20501_amd.build import ensure_built
    ensure_built()
    import paper_2412_20501_amd as m
    return m


def test_calls_that_are_not_cut_are_packed_only_for_fewer_rounds(tr):
    assert plan(tr, 8, 32, 16, 100, 2048, 128) == (1, 0)      # 256 plain workgroups are one round: 40 us, 48 in two parts
    assert plan(tr, 16, 16, 2, 53, 1618, 128) == (1, 0)
    assert plan(tr, 4, 24, 8, 87, 1823, 128) == (1, 0)
    assert plan(tr, 2, 64, 8, 538, 1070, 64) == (1, 0)        # 384 plain, 272 packed: two rounds either way
    assert plan(tr, 32, 32, 8, 1, 4096, 128) == (1, 1)        # 1024 plain, 256 packed
    assert plan(tr, 64, 32, 8, 1, 2048, 128) == (1, 1)


def test_few_rows_on_many_keys_are_cut(tr):
    assert plan(tr, 4, 32, 8, 1, 8192, 128) == (4, 1)
    assert plan(tr, 1, 32, 8, 500, 12500, 128, 12000) == (4, 0)
    assert plan(tr, 1, 8, 1, 1, 256, 128) == (1, 0)
    assert plan(tr, 1, 32, 32, 4096, 4096, 128) == (1, 0)


def test_workgroups_of_fewer_rows_make_a_cut_needless(tr):
    """us, cut and uncut: 29.5 and 19.2, 29.7 and 20.5, 31.4 and 24.4; still cut: 17.1 and 40.6, 47.7 and 137."""
    assert plan(tr, 4, 3, 1, 935, 1385, 128) == (1, 0)
    assert plan(tr, 1, 12, 4, 1611, 1611, 128, 0) == (1, 0)
    assert plan(tr, 1, 16, 16, 1594, 2428, 64, 834) == (1, 0)
    assert plan(tr, 1, 3, 3, 234, 4714, 128, 4480)[0] > 1
    assert plan(tr, 1, 3, 3, 1307, 27907, 64, 26600)[0] > 1


def test_short_calls_of_few_heads_are_cut(tr):
    """us, cut and in one piece whose reference is renewed where the parts would begin."""
    assert plan(tr, 1, 3, 3, 1251, 1251, 64)[0] > 1                             # 12.4 and 14.3
    assert plan(tr, 1, 12, 12, 286, 1282, 64)[0] > 1                            # 12.3 and 14.7
    assert plan(tr, 1, 4, 1, 1694, 1906, 64, 212)[0] > 1                        # 14.7 and 17.2
    assert plan(tr, 1, 2, 2, 1053, 1053, 128)[0] > 1                            # 15.0 and 17.0
    assert plan(tr, 1, 1, 1, 6762, 1812, 128, -4950)[0] > 1                     # 17.6 and 21.8


def test_long_calls_of_few_rows_are_cut_at_head_dim_128(tr):
    """us, cut and in one piece."""
    assert plan(tr, 2, 32, 32, 165, 8866, 128, 8701)[0] > 1                     # 73 and 90
    assert plan(tr, 2, 32, 32, 147, 7438, 128)[0] > 1                           # 62 and 81
    assert plan(tr, 4, 4, 2, 889, 8060, 128)[0] > 1                             # 67 and 80
    assert plan(tr, 2, 12, 3, 419, 4343, 128, 3924)[0] > 1                      # 37 and 42


def test_a_packed_grid_stays_within_the_dispatch_limit(tr):
    """2^32 threads in one dimension: the plain form's second grid dimension holds what a packed launch would not."""
    assert plan(tr, 2_700_000, 2, 1, 257, 8, 64) == (1, 1)
    assert plan(tr, 2_800_000, 2, 1, 257, 8, 64) == (1, 0)


def test_workgroups_of_a_causal_cut_are_counted_as_they_are(tr):
    """A row tile has as many workgroups as parts that its rows see, one at least and never more than there are parts; us in 256 rows and in
    the shape chosen: 31.6 and 27.7, 27.0 and 23.8, 23.9 and 20.7, 20.0 and 17.3."""
    for case in ((1, 32, 32, 120, 6905, 128, 6785), (2, 32, 32, 122, 2508, 128, 2386), (1, 32, 4, 26, 26034, 64, 26008), (1, 12, 3, 206, 2534, 128, 2328)):
        assert plan(tr, *case)[0] > 1 and shape(tr, STEP_F32, *case) == (64, 2)
    # 255 workgroups of 128 rows, but 58 of them on the first XCD's 32 compute units: 41.8 in (128, 2)
    assert plan(tr, 1, 3, 3, 3929, 3929, 128, 0) == (5, 0) and shape(tr, STEP_F32, 1, 3, 3, 3929, 3929, 128, 0) == (128, 1)
    assert plan(tr, 1, 3, 3, 2646, 2646, 128, 0)[0] > 1 and shape(tr, STEP_F32, 1, 3, 3, 2646, 2646, 128, 0) == (128, 1)     # 33.3 -> 25.7


def test_shapes_of_a_workgroup(tr):
    assert shape(tr, RING, 1, 32, 32, 32768, 32768, 128, 0, 8) == (256, 1)      # a full chip
    assert shape(tr, RING, 2, 24, 24, 16384, 16384, 64, None, 4) == (128, 1)
    assert shape(tr, RING, 1, 1, 1, 8192, 8192, 128) == (64, 2)                 # an idle one
    assert shape(tr, RING_BF16, 1, 16, 4, 6008, 6008, 128, 0, 4) == (128, 1)
    assert shape(tr, RING, 1, 1, 1, 34 * 288, 34 * 288, 128, 0, 34)[1] == 1     # more references than key groups keep
    for H in (1, 2, 4, 8, 16):
        for n in (2, 3, 33):                                                    # segments of one sub-tile: key groups would both start in the first
            assert shape(tr, RING, 1, H, H, 33 * n, 33 * n, 64, None, n)[1] == 1
    assert shape(tr, STEP_BF16, 4, 32, 8, 1, 8192, 128) == (64, 2)


def test_workgroups_that_share_a_compute_unit(tr):
    for D, small in ((64, 3), (128, 2)):
        assert shape(tr, RING, 4, 96, 96, 1024, 1024, D, 0) == (128, 1) and per_unit(tr, RING, 4, 96, 96, 1024, 1024, D, 0) == small
        assert per_unit(tr, RING, 1, 1, 1, 8192, 8192, D) == 1                     # 64 rows, two key groups, a unit each
        assert per_unit(tr, RING, 1, 32, 32, 32768, 32768, 128, 0, 8) == 1         # 256 rows
    assert shape(tr, STEP_F32, 2, 12, 12, 1777, 1777, 64, 0) == (64, 2) and per_unit(tr, STEP_F32, 2, 12, 12, 1777, 1777, 64, 0) == 3


def test_where_three_workgroups_of_64_rows_share_a_unit(tr):
    """us, the best other shape and three of 64 rows a unit."""
    def three(*case):
        return shape(tr, *case) == (64, 2) and per_unit(tr, *case) == 3
    for form in (RING, STEP_F32):
        assert three(form, 1, 8, 8, 4096, 4096, 64, 0)                          # 33.1 and 28.7
        assert three(form, 1, 4, 4, 8192, 8192, 64, 0)                          # 55.4 and 51.4, cut in three 89.3
        assert three(form, 1, 4, 4, 9000, 9000, 64, 0)                          # 68.6 and 58.4
        assert not three(form, 1, 24, 24, 1777, 1777, 64)
        assert not three(form, 4, 32, 32, 280, 280, 64, 0)                      # a few keys: 7.3 and 7.9
        assert three(form, 4, 32, 32, 238, 238, 64, 0)                          # two a unit: 7.3 and 6.9
    assert three(RING, 1, 2, 2, 17644, 17644, 64, 0, 4)                         # 119 and 108
    assert not three(STEP_F32, 8, 32, 32, 138, 5315, 64, 5177)                  # few row tiles a head, K and V from beyond the L2s: 82 and 142
    assert not three(STEP_BF16, 16, 24, 24, 106, 2905, 64, 2799)                # 53 and 78
    assert not three(STEP_F32, 8, 24, 24, 256, 2568, 64, 2312)                  # 45 and 59
    assert three(STEP_F32, 4, 24, 12, 321, 1322, 64, 1001)                      # 22.5 and 20.3
    assert plan(tr, 1, 16, 16, 2462, 27776, 64, 25314)[0] > 1                   # uncut 323, in three parts 287


def test_short_rings_of_an_odd_number_of_sub_tiles(tr):
    """One of two key groups has a step more then; us, one key group and two."""
    for H, S, n, D, groups in ((6, 288, 4, 128, 1), (2, 292, 4, 128, 2),        # 10.6 and 11.3, 11.7 and 11.5
                               (8, 412, 4, 128, 1), (4, 464, 4, 128, 2),        # 12.6 and 13.1, 13.9 and 13.7
                               (4, 156, 2, 64, 1), (4, 280, 4, 64, 1), (4, 408, 4, 64, 2)):   # 6.3 and 6.9, 8.4 and 8.8, 10.0 and 9.6
        assert shape(tr, RING, 1, H, H, S, S, D, None, n)[1] == groups
    assert shape(tr, RING, 1, 2, 2, 256, 256, 64, None, 4) == (64, 2)


def test_packed_rings_have_one_key_group(tr):
    """Rings whose heads share a row space, which fills the chip: no kernel with key groups is there for them."""
    for D in (64, 128):
        for off in (None, 0):
            for B, g, seg, n in ((300, 2, 40, 3), (64, 4, 32, 2), (32, 8, 33, 4), (200, 16, 65, 2), (64, 2, 150, 2), (300, 3, 100, 8)):
                assert shape(tr, RING, B, 2 * g, 2, seg * n, seg * n, D, off, n)[1] == 1


def test_invalid_arguments(tr):
    assert shape(tr, 5, 1, 2, 2, 8, 8, 64)[0] == -1 and shape(tr, STEP_F32, 1, 3, 2, 8, 8, 64)[0] == -1
    assert shape(tr, RING, 1, 2, 2, 8, 8, 64, None, 3)[0] == -1 and shape(tr, RING_BF16, 1, 2, 2, 8, 16, 64)[0] == -1
    assert tr.raw_lib().tr_attn_workgroup(None, None, 0, 0, 0, 0, 1, None) == -1
    assert tr.raw_lib().tr_attn_workgroups_per_unit(None, None, 0, 0, 0, 0, 1) == -1 and per_unit(tr, RING, 1, 2, 2, 8, 8, 64, None, 3) == -1
    assert plan(tr, 1, 3, 2, 8, 8, 64)[0] == -1 and plan(tr, 1, 2, 2, 8, 8, 96)[0] == -1
    assert tr.raw_lib().tr_block_attn_plan(None, None, 0, 0, 0, None) == -1
    q = tr.TrTensor(0x7F0000000000, tr.TR_BF16, 1, 2, 8, 64, 1024, 512, 64)
    assert tr.raw_lib().tr_block_attn_plan(q, q, 1, -1, 0, None) == -1 and "positions" in tr.raw_lib().tr_last_error().decode()
