"""Which kernel a call takes, and calls at the lines between them."""
import pytest
import torch

import paper_2606_19849_amd as vico
from synth import ChunkShape, make_chunk_inputs
from tests._route import BALANCED, TILE, chunk_route

# one and two whole row tiles of equal length per work-group: the balanced shares hold no part of a row tile
WHOLE_TILES = [ChunkShape(256, 256, 64, 0, 200, 300, 170, 40), ChunkShape(512, 512, 64, 3, 256, 300, 190, 9),
               ChunkShape(256, 32, 128, 0, 64, 0, 0, 256)]


@pytest.mark.parametrize("sh", WHOLE_TILES + [ChunkShape(32, 4, 128, 64, 16384, 16384, 16384, 2048),
                                              ChunkShape(16, 2, 128, 0, 512, 512, 512, 4096)])
def test_balanced_shares_of_whole_row_tiles_take_the_plain_schedule(sh):
    """The balanced schedule writes partial results for a merge.  A plan of one part has neither workspace nor merge."""
    for flags in (0, vico.VICO_ATTN_BIDIRECTIONAL):
        parts, wb = vico.vico_attn_plan(sh.chunk_len, sh.sink_len, sh.ring_slots, sh.hist_len, sh.window, sh.num_q_heads,
                                        sh.num_kv_heads, sh.head_dim, vico.VICO_SPLIT_BALANCED, flags)
        kernel, _, groups = chunk_route(sh, vico.VICO_SPLIT_BALANCED, flags)
        assert (kernel == BALANCED) == (parts > 1) == (wb > 0)
        if parts == 1:
            assert kernel == TILE and groups >= 256


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(WHOLE_TILES)))
def test_balanced_calls_of_whole_row_tiles(case):
    from tests._gpu import DeviceChunk, check_f32, oracle_and_bound
    inp = make_chunk_inputs(WHOLE_TILES[case], seed=1200 + case, family="F2")
    dc = DeviceChunk(inp)
    o, lse = dc.attention(torch.float32, num_splits=vico.VICO_SPLIT_BALANCED)
    assert dc.parts == 1
    ref, ref_lse, b = oracle_and_bound(inp)
    check_f32(o, ref, b, lse, ref_lse)
