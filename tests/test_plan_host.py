"""Which form an attention call takes (tr_block_attn_plan: host only, nothing is launched): parts of the keys, packed heads."""
import pytest

from gpu_util import attn_plan as plan


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
    """us, cut and uncut: 31.2 and 19.0, 30.5 and 20.4, 33.5 and 25.4; still cut: 17.1 and 40.6, 47.7 and 137."""
    assert plan(tr, 4, 3, 1, 935, 1385, 128) == (1, 0)
    assert plan(tr, 1, 12, 4, 1611, 1611, 128, 0) == (1, 0)
    assert plan(tr, 1, 16, 16, 1594, 2428, 64, 834) == (1, 0)
    assert plan(tr, 1, 3, 3, 234, 4714, 128, 4480)[0] > 1
    assert plan(tr, 1, 3, 3, 1307, 27907, 64, 26600)[0] > 1


def test_a_packed_grid_stays_within_the_dispatch_limit(tr):
    """2^32 threads in one dimension: the plain form's second grid dimension holds what a packed launch would not."""
    assert plan(tr, 2_700_000, 2, 1, 257, 8, 64) == (1, 1)
    assert plan(tr, 2_800_000, 2, 1, 257, 8, 64) == (1, 0)


def test_invalid_arguments(tr):
    assert plan(tr, 1, 3, 2, 8, 8, 64)[0] == -1 and plan(tr, 1, 2, 2, 8, 8, 96)[0] == -1
    assert tr.raw_lib().tr_block_attn_plan(None, None, 0, 0, 0, None) == -1
    q = tr.TrTensor(0x7F0000000000, tr.TR_BF16, 1, 2, 8, 64, 1024, 512, 64)
    assert tr.raw_lib().tr_block_attn_plan(q, q, 1, -1, 0, None) == -1 and "positions" in tr.raw_lib().tr_last_error().decode()
