"""Which kernel a call takes, and calls at the lines between them."""
import pytest
import torch

import paper_2606_19849_amd as vico
from synth import ChunkShape, QueryShape, make_chunk_inputs, make_query_inputs
from tests._route import BALANCED, GATHER, ROWS, TILE, chunk_route, gather_route

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
        kernel, _, groups = chunk_route(sh, vico.VICO_SPLIT_BALANCED, flags)[:3]
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


HEADS = {"7b": (28, 4, 128), "3b": (16, 2, 128), "small": (8, 2, 64), "mha": (32, 32, 128)}

# (segments, keys in them), hint given; per head set the query lengths at which one kernel was measured
# clearly faster than the other (sink of 64, the tail as long as the query)
FASTER = [
    (0, 0, False, {"7b": ([8, 64, 256, 384, 512], [1024, 2048]), "3b": ([8, 256, 768], [2048]),
                   "small": ([64, 1024, 2048], []), "mha": ([64, 256, 512], [1024, 2048])}),
    (8, 512, True, {"7b": ([8, 64, 256, 384, 512], [1024, 2048]), "3b": ([8, 256, 512], [1024, 2048]),
                    "small": ([64, 1024], []), "mha": ([64, 256, 512], [768, 1024, 2048])}),
    (8, 512, False, {"7b": ([8, 64, 256, 384, 512], [768, 1024, 2048]), "3b": ([8, 256, 512, 768], [1024, 2048]),
                     "small": ([64, 1024], []), "mha": ([64, 256, 384], [768, 1024, 2048])}),
    (32, 20480, True, {"7b": ([8, 16], [96, 128, 512, 2048]), "3b": ([8, 48], [192, 512, 2048]), "mha": ([8], [96, 512])}),
    (32, 20480, False, {"7b": ([8, 64, 256, 384], [768, 1024, 2048]), "3b": ([8, 256, 384], [1024, 2048]),
                        "small": ([64, 1024], [2048]), "mha": ([64, 384], [512, 768, 1024, 2048])}),
]


@pytest.mark.parametrize("segments,keys,known,by_heads", FASTER)
def test_gathered_calls_take_the_faster_kernel(segments, keys, known, by_heads):
    """Long queries, which the rows kernel walks in rounds, stay on the 256-row kernel; without a hint also
    where only the store's keys make it the faster one."""
    for name, (rows, gather) in by_heads.items():
        for q_len in rows + gather:
            got = gather_route(q_len, q_len, 64, 24000, segments, keys if known else 0, HEADS[name])[0]
            assert got == (ROWS if q_len in rows else GATHER), (name, q_len)


def test_forced_parts_count_as_rounds():
    for name, keys, parts in (("mha", 0, 64), ("mha", 256, 16), ("mha", 4096, 16), ("small", 4096, 64), ("small", 10000, 64)):
        assert gather_route(64, 300, 64, 24000, 8, keys, HEADS[name], parts)[0] == GATHER, (name, parts)
    assert gather_route(64, 300, 64, 24000, 8, 4096, HEADS["small"], 16)[0] == ROWS       # one round
    # 64 parts of a 32-token query: seven row tiles each would be 1792 work-groups
    assert gather_route(32, 32, 64, 24000, 32, 2000, HEADS["7b"], 64)[0] == GATHER
    assert gather_route(1, 64, 64, 24000, 32, 2000, HEADS["7b"], 64)[0] == ROWS


@pytest.mark.gpu
@pytest.mark.parametrize("q_len,kernel", [(384, ROWS), (500, ROWS), (1000, GATHER)])
def test_long_queries(q_len, kernel):
    from tests._gpu import check_f32
    from tests.test_gpu_retrieval import DeviceQuery
    qi = make_query_inputs(QueryShape(28, 4, 128, 16, 64, 6, 20, 60, q_len, q_len + 3, 4), seed=77, family="F2")
    d = DeviceQuery(qi)
    st, ln = qi.chunk_start[:4], qi.chunk_len[:4]
    assert gather_route(q_len, q_len + 3, 16, qi.store_len, 4, int(ln.sum()), (28, 4, 128))[0] == kernel
    o, lse, parts = d.attend(st, ln)
    ro, rl, b = d.reference(st, ln, parts=max(parts, 8))
    check_f32(o, ro, b, lse, rl)


@pytest.mark.parametrize("sh,splits,groups", [
    (ChunkShape(28, 4, 128, 64, 18432, 9 * 18432, 16384, 2048), 0, 32),       # 224 work-groups: beside, on idle CUs
    (ChunkShape(16, 2, 128, 64, 512, 4001, 307, 77), 0, 10),                  # all that the copy has work for
    (ChunkShape(32, 32, 128, 64, 640, 2000, 0, 512), 0, 256),                 # two full rounds: the copy runs after them
    (ChunkShape(32, 32, 128, 64, 640, 2000, 256, 256), 0, 256),
    (ChunkShape(32, 4, 128, 64, 4096, 9000, 1024, 2048), 1, 256),             # the tile kernel, one full round
    (ChunkShape(16, 2, 128, 64, 576, 2000, 320, 256), 0, 32),                 # a small copy after a full round
    (ChunkShape(16, 2, 128, 64, 575, 2000, 320, 256), 0, 0)])                 # no room beside the window
def test_append_groups_beside_the_attention(sh, splits, groups):
    assert chunk_route(sh, splits, vico.VICO_ATTN_APPEND)[3] == groups
    assert chunk_route(sh, splits)[3] == 0
