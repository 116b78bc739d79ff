"""The register-streamed rows kernel (small chunks, decode steps, short
queries) and the pipelined tile kernel at the sizes where they can go wrong:
edges of 16- and 32-row tiles, of 32-key blocks and 64-key tiles, ranges
shorter than the pipeline, blocks across segments.  Reference: the fp64 oracle
with the derived per-element bound; and the same call on the other kernel,
each within its bound."""
import numpy as np
import pytest
import torch

import paper_2606_19849_amd as vico
from synth import ChunkShape, QueryShape, make_chunk_inputs, make_query_inputs
from tests._gpu import DeviceChunk, check_bf16, check_f32, oracle_and_bound
from tests._route import GATHER, ROWS, TILE, chunk_route, gather_route
from tests.test_gpu_retrieval import DeviceQuery

pytestmark = pytest.mark.gpu


# heads, kv heads, d, sink, ring, history, window, chunk: packed rows g*C around 16 and 32, keys
# around multiples of 32, no history, one token, wrapped ring
ROWS_CHUNKS = [
    (4, 4, 64, 0, 64, 0, 0, 1),
    (4, 4, 128, 0, 64, 31, 31, 1),
    (8, 1, 128, 1, 40, 90, 30, 2),
    (7, 1, 128, 16, 80, 177, 64, 5),
    (8, 2, 64, 32, 128, 300, 128, 8),
    (16, 2, 128, 5, 200, 333, 187, 33),
    (6, 2, 128, 64, 96, 100, 96, 11),
    (3, 3, 64, 3, 500, 1203, 467, 65),
    (28, 4, 128, 64, 700, 2000, 612, 77),
]


@pytest.mark.parametrize("case", range(len(ROWS_CHUNKS)))
@pytest.mark.parametrize("flags", [0, vico.VICO_ATTN_BIDIRECTIONAL])
def test_small_chunks_on_both_kernels(case, flags):
    """The library's choice (the rows kernel here) and the tile kernel (a split
    count given by the caller) against the oracle, fp32 and bf16 results."""
    inp = make_chunk_inputs(ChunkShape(*ROWS_CHUNKS[case]), seed=700 + case, family="F2")
    dc = DeviceChunk(inp)
    for splits in (0, 1, 3):
        assert chunk_route(inp.shape, splits, flags)[0] == (TILE if splits else ROWS)
        o, lse = dc.attention(torch.float32, num_splits=splits, flags=flags)
        ref, ref_lse, b = oracle_and_bound(inp, parts=max(dc.parts, 8), bidirectional=bool(flags))
        check_f32(o, ref, b, lse, ref_lse)
        check_bf16(dc.attention(torch.bfloat16, num_splits=splits, flags=flags)[0], ref, b)


def _table(rng, n_seg, cap):
    """Segments of 0 to 70 keys in scattered order, some reaching outside the store."""
    st = rng.integers(-20, cap, n_seg)
    ln = rng.integers(-2, 71, n_seg)
    return st.astype(np.int64), ln.astype(np.int32)


@pytest.mark.parametrize("heads", [(8, 2, 128), (7, 1, 128), (4, 4, 64), (12, 2, 64)])
@pytest.mark.parametrize("q_len,tail", [(1, 1), (2, 31), (4, 4), (5, 40), (9, 9), (33, 64)])
@pytest.mark.parametrize("n_seg", [0, 1, 7, 64])
def test_gathered_rows(heads, q_len, tail, n_seg):
    """Tables of up to 64 entries take the rows kernel; the same table padded
    with empty entries to 65 takes the 256-row kernel."""
    Hq, Hkv, D = heads
    sh = QueryShape(Hq, Hkv, D, 19, 64, 12, 20, 90, q_len, tail, 6)
    qi = make_query_inputs(sh, seed=900 + q_len + n_seg, family="F2")
    d = DeviceQuery(qi)
    st, ln = _table(np.random.default_rng(31 * q_len + n_seg), n_seg, qi.store_len)
    lo = np.clip(st, 0, qi.store_len)
    hi = np.clip(st + ln, 0, qi.store_len)
    keep = hi > lo
    pad = 65 - n_seg
    wide = (np.concatenate([st, np.zeros(pad, np.int64)]), np.concatenate([ln, np.zeros(pad, np.int32)]))
    for splits in (0, 3):
        for table, kernel in (((st, ln), ROWS), (wide, GATHER)):
            hint = int(np.maximum(table[1], 0).sum())
            assert gather_route(q_len, tail, 19, qi.store_len, len(table[0]), hint, heads, splits)[0] == kernel
            o, lse, parts = d.attend(*table, num_splits=splits)
            ro, rl, b = d.reference(lo[keep], (hi - lo)[keep], parts=max(parts, 8))
            check_f32(o, ro, b, lse, rl)


@pytest.mark.parametrize("heads,q_len", [((7, 1, 128), 33), ((16, 2, 128), 20), ((12, 2, 64), 6)])
@pytest.mark.parametrize("n_seg", [1, 9, 64])
@pytest.mark.parametrize("splits", [1, 2])
def test_gathered_rows_through_lds(heads, q_len, n_seg, splits):
    """Five or more row tiles over key ranges of several blocks a wave (K staged
    through LDS), blocks inside a segment and across segments.  Few parts and a
    hint of 1200 keys take that route whatever the table holds."""
    Hq, Hkv, D = heads
    qi = make_query_inputs(QueryShape(Hq, Hkv, D, 40, 64, 12, 20, 90, q_len, q_len + 3, 6), seed=950 + n_seg, family="F2")
    d = DeviceQuery(qi)
    rng = np.random.default_rng(n_seg)
    st = rng.integers(-20, qi.store_len - 64, n_seg).astype(np.int64)
    ln = rng.integers(30, 1 + 1800 // n_seg if n_seg < 10 else 71, n_seg).astype(np.int32)
    lo, hi = np.clip(st, 0, qi.store_len), np.clip(st + ln, 0, qi.store_len)
    keep = hi > lo
    kernel, *_, staged = gather_route(q_len, q_len + 3, 40, qi.store_len, n_seg, 1200, heads, splits)
    assert kernel == ROWS and staged
    o, lse, parts = d.attend(st, ln, num_splits=splits, hint=1200)
    ro, rl, b = d.reference(lo[keep], (hi - lo)[keep], parts=max(parts, 8))
    check_f32(o, ro, b, lse, rl)


# key ranges of one to six 64-key tiles per split (the pipeline runs three tiles ahead), row counts
# around a wave's 32 rows and a work-group's 256, ring end and chunk end inside a tile
TILE_CHUNKS = [
    (2, 2, 128, 0, 64, 0, 0, 64, 1),
    (2, 2, 64, 0, 64, 64, 64, 65, 1),
    (4, 2, 128, 16, 300, 777, 250, 33, 5),
    (2, 1, 128, 64, 200, 456, 192, 257, 16),
    (8, 2, 128, 70, 1000, 4321, 1000, 300, 12),
    (8, 2, 64, 1, 513, 1500, 512, 255, 7),
    (4, 1, 128, 64, 640, 1280, 640, 256, 3),
]


@pytest.mark.parametrize("case", range(len(TILE_CHUNKS)))
@pytest.mark.parametrize("flags", [0, vico.VICO_ATTN_BIDIRECTIONAL])
def test_tile_kernel_short_ranges(case, flags):
    """Split counts that leave each work-group one to a few key tiles.  The
    workspace is filled with NaN patterns first: every partial that the merge
    reads has been written."""
    *shape, splits = TILE_CHUNKS[case]
    inp = make_chunk_inputs(ChunkShape(*shape), seed=800 + case, family="F2")
    sh = inp.shape
    dc = DeviceChunk(inp)
    parts, wb = vico.vico_attn_plan(sh.chunk_len, sh.sink_len, sh.ring_slots, sh.hist_len, sh.window, sh.num_q_heads,
                                    sh.num_kv_heads, sh.head_dim, splits, flags)
    ws = torch.full((max(wb, 16),), 255, dtype=torch.uint8, device="cuda")
    out = torch.empty((sh.chunk_len, sh.num_q_heads, sh.head_dim), dtype=torch.float32, device="cuda")
    lse = torch.empty((sh.num_q_heads, sh.chunk_len), dtype=torch.float32, device="cuda")
    vico.vico_chunk_prefill_attn(dc.q, dc.kc, dc.vc, dc.sk, dc.sv, dc.rk, dc.rv, sh.hist_len, sh.window, out, lse=lse,
                                 workspace=ws, num_splits=splits, flags=flags)
    torch.cuda.synchronize()
    ref, ref_lse, b = oracle_and_bound(inp, parts=parts, bidirectional=bool(flags))
    check_f32(out.cpu().numpy().astype(np.float64), ref, b, lse.cpu().numpy().astype(np.float64), ref_lse)


@pytest.mark.parametrize("shape", [
    # ring with room for window and chunk (the copy rides on the attention launch), exactly and with a wrap
    (8, 2, 128, 16, 400, 777, 300, 77), (8, 2, 128, 0, 377, 5000, 300, 77), (8, 1, 64, 3, 2000, 3999, 1500, 300),
    # one slot short of it (the copy is a launch of its own)
    (8, 2, 128, 16, 376, 777, 300, 77),
    # 256 work-groups, and twice 256: a wide copy behind the full rounds
    (32, 32, 128, 3, 400, 900, 100, 256), (32, 32, 64, 0, 700, 1500, 10, 512)])
@pytest.mark.parametrize("splits", [0, 1, 2])
def test_append_beside_the_attention(shape, splits):
    """One call with the append equals the attention and then vico_kv_append, bit for bit, ring included."""
    inp = make_chunk_inputs(ChunkShape(*shape), seed=611, family="F2")
    a, b = DeviceChunk(inp), DeviceChunk(inp)
    o, lse = a.attention(num_splits=splits)
    vico.vico_kv_append(a.kc, a.vc, a.rk, a.rv, inp.shape.hist_len)
    oa, la = b.attention(num_splits=splits, flags=vico.VICO_ATTN_APPEND)
    torch.cuda.synchronize()
    assert np.array_equal(o, oa) and np.array_equal(lse, la)
    assert torch.equal(a.rk, b.rk) and torch.equal(a.rv, b.rv)
    ref, ref_lse, bound = oracle_and_bound(inp, parts=max(a.parts, 8))
    check_f32(oa, ref, bound, la, ref_lse)


@pytest.mark.parametrize("shape", [(4, 2, 128, 5, 200, 300, 150, 256), (8, 2, 64, 0, 300, 500, 260, 300),
                                   (7, 1, 128, 64, 128, 100, 90, 77), (8, 2, 128, 64, 4096, 4596, 4000, 600)])
@pytest.mark.parametrize("splits", [0, 1, 3, vico.VICO_SPLIT_BALANCED])
@pytest.mark.parametrize("poison", [float("nan"), float("inf")])
def test_later_tokens_stay_out_of_earlier_rows(shape, splits, poison):
    """NaN or infinity in the last chunk token's K and V reaches no row of a
    wave whose own key tiles end before it: a wave holds 32 rows (at most 32
    tokens, from a multiple of 32), and tiles have 64 keys.  The rest of the
    result keeps its bits."""
    dc = DeviceChunk(make_chunk_inputs(ChunkShape(*shape), seed=431, family="F2"))
    sh = dc.inp.shape
    clean, clean_lse = dc.attention(num_splits=splits)
    dc.kc[-1] = poison
    dc.vc[-1] = poison
    o, lse = dc.attention(num_splits=splits)
    first = sh.sink_len + sh.visible_window
    last_of_wave = np.minimum(np.arange(sh.chunk_len) // 32 * 32 + 31, sh.chunk_len - 1)
    apart = (first + last_of_wave) // 64 < (first + sh.chunk_len - 1) // 64
    assert apart.any()
    assert np.array_equal(o[apart], clean[apart]) and np.array_equal(lse[:, apart], clean_lse[:, apart])


@pytest.mark.parametrize("poison", [float("nan"), float("inf")])
@pytest.mark.parametrize("splits", [0, 1, 3, 16, vico.VICO_SPLIT_BALANCED])
@pytest.mark.parametrize("shape", [(4, 2, 128, 5, 1200, 2000, 1150, 40), (8, 2, 128, 64, 4096, 4596, 4000, 600),
                                   (8, 2, 64, 0, 4096, 4500, 4000, 64)])
def test_nan_logits_stay_in_a_split_result(shape, splits, poison):
    """A NaN or infinite logit makes its row NaN, however the keys are split: the part that holds it is not
    taken for an empty one.  The key is the oldest of the window, which every row sees."""
    dc = DeviceChunk(make_chunk_inputs(ChunkShape(*shape), seed=432, family="F2"))
    sh = dc.inp.shape
    dc.rk[(sh.hist_len - sh.visible_window) % sh.ring_slots] = poison
    o, lse = dc.attention(num_splits=splits)
    assert np.isnan(o).all()


@pytest.mark.parametrize("splits", [0, 1, 5, 24])
@pytest.mark.parametrize("pad", [0, 60])
@pytest.mark.parametrize("q_len", [1, 20])
def test_nan_logits_stay_in_a_split_gathered_result(splits, pad, q_len):
    """The same for the gathered call, on the rows kernel and (65 table entries) on the 256-row kernel."""
    qi = make_query_inputs(QueryShape(8, 2, 128, 19, 64, 12, 100, 300, q_len, q_len, 5), seed=433, family="F2")
    d = DeviceQuery(qi)
    st = np.concatenate([qi.chunk_start[:5], np.zeros(pad, np.int64)])
    ln = np.concatenate([qi.chunk_len[:5], np.zeros(pad, np.int32)])
    d.gk[int(st[2])] = float("nan")
    o, lse, parts = d.attend(st, ln, num_splits=splits)
    assert np.isnan(o).all()
