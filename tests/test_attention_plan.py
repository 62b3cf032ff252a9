"""The work division of calls with few queries over caches larger than the L2s."""
import pytest

import paper_2603_06664_amd as P
from paper_2603_06664_amd import binding as B


@pytest.mark.parametrize("n_q,n_heads,n_keys", [(16, 40, 32760), (100, 40, 32760), (24, 40, 14040), (16, 12, 32760),
                                                (100, 12, 100000), (24, 12, 32760)])
def test_one_query_tile_fills_the_gpu_by_splits(n_q, n_heads, n_keys):
    """One query tile per head: only the splits bring work-groups, and HBM wants three quarters of the CUs or the
    16 splits that there are (measured: 4 to 6 splits of 40 heads and 16 of 12 are the fastest)."""
    plan = P.chunk_attention_choose_plan(n_q, n_heads, n_keys)
    assert plan[1] == 16 or 192 <= n_heads * plan[1] <= 256, plan


@pytest.mark.parametrize("n_q,n_heads,n_keys", [(262, 22, 27422), (257, 38, 17991), (269, 15, 67003), (545, 44, 15519),
                                                (293, 26, 102830), (351, 37, 44483), (268, 49, 36223), (384, 49, 27425)])
def test_few_query_tiles_over_caches_beyond_the_last_level(n_q, n_heads, n_keys):
    """K and V above 256 MB: 128-query work-groups read them twice as often and lose 6 to 20 % (measured)."""
    assert n_heads * n_keys * 512 > 256 << 20
    assert P.chunk_attention_choose_plan(n_q, n_heads, n_keys)[0] == 8


@pytest.mark.parametrize("n_q,n_heads,n_keys", [(9048, 29, 108576), (17160, 38, 102960), (4000, 40, 120000)])
def test_large_caches_take_any_number_of_splits(n_q, n_heads, n_keys):
    """More than 3 M heads x keys, taken by chunk_attention_static: no jump to 8 splits where fewer are as fast (9048
    queries: 10.93 ms in 8 splits and 1.1 GB of scratch, 10.90 in 6)."""
    assert n_heads * n_keys > 3000000
    splits = P.chunk_attention_choose_plan(n_q, n_heads, n_keys)[1]
    assert 1 <= splits < 8, splits


@pytest.mark.parametrize("n_q,n_heads,n_keys", [(50432, 4, 8192), (83200, 4, 30000)])
def test_nearly_empty_last_round_among_several(n_q, n_heads, n_keys):
    """3.08 and 5.08 rounds: splitting to fill the last of them loses (measured unsplit and in 2 splits: 674 and 723 us,
    3802 and 3953)."""
    assert P.chunk_attention_choose_plan(n_q, n_heads, n_keys)[1] == 1
