"""Workspace of a score call with few voting columns a KV head: the columns' operands take 4 D bytes a column, not those
of a block of 32.  Host only."""
import pytest

import paper_2502_14317_amd as pc


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G,obs", [(1, 1), (1, 8), (4, 3), (1, 31)])
def test_columns_are_not_padded_to_a_block(D, G, obs):
    H, cols = 16, G * obs
    size = lambda c: pc.pc_chunk_query_scores_workspace_bytes(pc.make_shape(c, 40, 40, G * H, H, D, obs, 1.0e4))
    # beyond 350 key blocks (one a group here): a group's operands, its (max, sum) and logsumexp, block sum
    per_group = (size(2000) - size(1000)) / (1000 * H)
    assert per_group <= cols * (4 * D + 8) + 32 * 4 + 4 + 1
