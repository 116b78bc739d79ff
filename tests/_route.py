"""Which kernel a call runs: the library's own routing, asked without launching anything."""
from __future__ import annotations

import ctypes

import paper_2606_19849_amd as vico

TILE, BALANCED, ROWS, GATHER = "tile", "balanced", "rows", "gather"
_NAMES = (TILE, BALANCED, ROWS, GATHER)
_lib = vico.load_library()
_lib.vico_attn_route.argtypes = [ctypes.c_int32] * 3 + [ctypes.c_int64] * 2 + [ctypes.c_int32] * 5 + [ctypes.c_void_p]
_lib.vico_gather_route.argtypes = [ctypes.c_int32] * 5 + [ctypes.c_int64] + [ctypes.c_int32] * 4 + [ctypes.c_void_p]


def _route(call, *args):
    out = (ctypes.c_int32 * 5)()
    assert call(*args, out) == 0
    return _NAMES[out[0]], *out[1:]


def chunk_route(sh, splits=0, flags=0):
    """(kernel, key-range parts, work-groups, append work-groups, K through LDS) of vico_chunk_prefill_attn on a ChunkShape."""
    return _route(_lib.vico_attn_route, sh.chunk_len, sh.sink_len, sh.ring_slots, sh.hist_len, sh.window,
                  sh.num_q_heads, sh.num_kv_heads, sh.head_dim, splits, flags)


def gather_route(q_len, tail, sink, slots, segments, hint, heads, splits=0):
    """(kernel, key-range parts, work-groups, 0, K through LDS) of vico_gather_attn; heads: (query, key/value, size)."""
    return _route(_lib.vico_gather_route, q_len, tail, sink, slots, segments, hint, *heads, splits)
