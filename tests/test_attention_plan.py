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
