"""The C++ calls of the binding against its ctypes path: what the first takes
gives the same results, what it does not take is accepted or rejected by the
second in its own words."""
import warnings

import numpy as np
import pytest
import torch

import paper_2606_19849_amd as vico
import paper_2606_19849_amd._binding as binding
from synth import CONFIGS, make_chunk_inputs


class _Never:
    """Stands in for the C++ calls and takes none."""

    def __getattr__(self, name):
        return lambda *a: None


def test_host_tensors_go_to_the_general_path():
    calls = binding._fast()
    bf = lambda *s: torch.zeros(*s, dtype=torch.bfloat16)   # noqa: E731
    assert calls.prefill(bf(4, 2, 64), bf(4, 1, 64), bf(4, 1, 64), None, None, bf(8, 1, 64), bf(8, 1, 64), 8, 8,
                         bf(4, 2, 64), None, None, 0, 0.0, None, 0) is None
    assert calls.token_mean(bf(3, 64), torch.zeros(64), None) is None
    assert calls.token_mean() is None and calls.gather(1, 2, 3) is None
    with pytest.raises(ValueError, match="expected a contiguous"):
        vico.vico_token_mean(bf(3, 64), torch.zeros(64))
    with pytest.raises(ValueError, match="expected a contiguous"):
        vico.vico_kv_append(bf(4, 1, 64), bf(4, 1, 64), bf(8, 1, 64), bf(8, 1, 64), 0)


def test_without_the_cpp_calls_the_ctypes_path_runs(monkeypatch, tmp_path):
    """A tree with libvico alone still works: a warning once, then the general path in its own words."""
    monkeypatch.setattr(binding, "_calls", None)
    monkeypatch.setattr(binding, "CALL_PATH", str(tmp_path / "_vico_call.so"))
    x, out = torch.zeros(3, 64, dtype=torch.bfloat16), torch.zeros(64)
    with pytest.warns(RuntimeWarning, match="build it"), pytest.raises(ValueError, match="expected a contiguous"):
        vico.vico_token_mean(x, out)
    with warnings.catch_warnings(), pytest.raises(ValueError, match="expected a contiguous"):
        warnings.simplefilter("error")
        vico.vico_token_mean(x, out)
    # as vico_kv_append, up to the library: an empty chunk is accepted there
    seen = []
    monkeypatch.setattr(binding, "_dev_bf16", lambda *a: None)
    monkeypatch.setattr(binding, "_stream", lambda s: seen.append(s) or None)
    empty = torch.zeros(0, 1, 64, dtype=torch.bfloat16)
    vico.vico_kv_append(empty, empty, torch.zeros(8, 1, 64), torch.zeros(8, 1, 64), 0)
    assert seen == [None]


@pytest.mark.gpu
@pytest.mark.parametrize("stream", ["current", "object", "handle"])
def test_both_paths_give_the_same(stream, monkeypatch):
    from tests._gpu import DeviceChunk
    dc = DeviceChunk(make_chunk_inputs(CONFIGS["tiny"], seed=5, family="F2"))
    sh = dc.inp.shape
    s = torch.cuda.current_stream() if stream == "current" else torch.cuda.Stream()
    arg = {"current": None, "object": s, "handle": s.cuda_stream}[stream]
    x = torch.randn(9, 128, device="cuda").to(torch.bfloat16)
    feats = torch.randn(20, 128, device="cuda")
    starts = torch.arange(0, 200, 10, device="cuda")
    lens = torch.full((20,), 10, dtype=torch.int32, device="cuda")
    frames = torch.randn(2, 4, 6, 64, device="cuda").to(torch.bfloat16)
    torch.cuda.synchronize()

    def everything():
        new = lambda shape, dt: torch.zeros(shape, dtype=dt, device="cuda")   # noqa: E731
        out, lse = new((sh.chunk_len, sh.num_q_heads, sh.head_dim), torch.float32), new((sh.num_q_heads, sh.chunk_len), torch.float32)
        rk, rv = dc.rk.clone(), dc.rv.clone()
        qf, sc = new(128, torch.float32), new(20, torch.float32)
        oc, osc, cnt = new(5, torch.int32), new(5, torch.float32), new(1, torch.int32)
        ss, sl = new(5, torch.int64), new(5, torch.int32)
        go, go2 = new((1, sh.num_q_heads, sh.head_dim), torch.bfloat16), new((1, sh.num_q_heads, sh.head_dim), torch.bfloat16)
        keep, idx, n = new((2, 6), torch.uint8), new(48, torch.int32), new(1, torch.int32)
        tok = new((48, 64), torch.bfloat16)
        torch.cuda.synchronize()
        vico.vico_chunk_prefill_attn(dc.q, dc.kc, dc.vc, dc.sk, dc.sv, rk, rv, sh.hist_len, sh.window, out, lse=lse,
                                     stream=arg)
        vico.vico_kv_append(dc.kc, dc.vc, rk, rv, sh.hist_len, stream=arg)
        vico.vico_token_mean(x, qf, stream=arg)
        vico.vico_chunk_scores(qf, feats, sc, stream=arg)
        vico.vico_topk_chunks(sc, 5, oc, osc, cnt, chunk_start=starts, chunk_len=lens, seg_start=ss, seg_len=sl,
                              stream=arg)
        for f, o in ((vico.vico_gather_attn, go), (vico.vico_gather_attn_noalloc, go2)):
            f(dc.q[:1], dc.kc, dc.vc, dc.sk, dc.sv, rk, rv, ss, sl, o, keys_hint=50, stream=arg)
        vico.vico_temporal_drop(frames, 0.1, keep, idx, n, out_tokens=tok, stream=arg)
        torch.cuda.synchronize()
        return out, lse, rk, rv, qf, sc, oc, osc, cnt, ss, sl, go, go2, keep, idx, n, tok

    fast = everything()
    monkeypatch.setattr(binding, "_calls", _Never())
    for a, b in zip(fast, everything()):
        assert torch.equal(a, b)


@pytest.mark.gpu
def test_rejections_are_the_general_ones():
    """Wrong types, shapes and numbers raise what the ctypes path raises; an
    error status of the library raises VicoError on either path."""
    bf = lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device="cuda")   # noqa: E731
    k = bf(4, 1, 64)
    with pytest.raises(ValueError):
        vico.vico_kv_append(k.float(), k, bf(8, 1, 64), bf(8, 1, 64), 0)
    with pytest.raises(ValueError):
        vico.vico_kv_append(k, bf(4, 64, 1).transpose(1, 2)[:, :, ::2], bf(8, 1, 64), bf(8, 1, 64), 0)
    with pytest.raises(vico.VicoError) as e:
        vico.vico_kv_append(k, k.clone(), bf(2, 1, 64), bf(2, 1, 64), 0)
    assert e.value.status == -3
    with pytest.raises(ValueError, match="out"):
        vico.vico_chunk_prefill_attn(k, k, k, None, None, None, None, 0, 0, bf(3, 1, 64))
    ring = bf(8, 1, 64), bf(8, 1, 64)
    vico.vico_kv_append(k + 1, k + 2, *ring, np.int64(6))      # an index type of numpy: the general path
    torch.cuda.synchronize()
    assert float(ring[0][6:].sum()) == 128 and float(ring[1][:2].sum()) == 256


@pytest.mark.gpu
def test_lazily_cloned_outputs_get_memory_of_their_own():
    """A copy-on-write clone as an output leaves the tensor that it was cloned from alone, and inputs may be clones."""
    bf = lambda *s: torch.randn(*s, device="cuda").to(torch.bfloat16)   # noqa: E731
    new = lambda dt, *s: torch.zeros(*s, dtype=dt, device="cuda")   # noqa: E731
    i32, i64, f32 = torch.int32, torch.int64, torch.float32
    k, v, q, frames, feats = bf(4, 1, 64), bf(4, 1, 64), bf(4, 2, 64), bf(2, 4, 6, 64), torch.randn(9, 64, device="cuda")
    seg = torch.arange(2, device="cuda"), torch.ones(2, dtype=i32, device="cuda")
    lens = torch.ones(9, dtype=i32, device="cuda")
    ring = lambda: [new(torch.bfloat16, 8, 1, 64), new(torch.bfloat16, 8, 1, 64)]   # noqa: E731
    attn = lambda: [new(f32, 4, 2, 64), new(f32, 2, 4)]   # noqa: E731
    calls = [
        (ring(), lambda o: vico.vico_kv_append(k, v, *o, 6)),
        (attn() + ring(), lambda o: vico.vico_chunk_prefill_attn(q, k, v, None, None, o[2], o[3], 6, 4, o[0], lse=o[1],
                                                                 flags=vico.VICO_ATTN_APPEND)),
        (attn(), lambda o: vico.vico_gather_attn(q, k, v, None, None, k, v, *seg, o[0], lse=o[1])),
        (attn(), lambda o: vico.vico_gather_attn_noalloc(q, k, v, None, None, k, v, *seg, o[0], lse=o[1])),
        ([new(f32, 64)], lambda o: vico.vico_token_mean(k.view(4, 64), *o)),
        ([new(f32, 9)], lambda o: vico.vico_chunk_scores(feats[0], feats, *o)),
        ([new(i32, 3), new(f32, 3), new(i32, 1), new(i64, 3), new(i32, 3)],
         lambda o: vico.vico_topk_chunks(feats[:, 0].contiguous(), 3, *o[:3], chunk_start=torch.arange(9, device="cuda"),
                                         chunk_len=lens, seg_start=o[3], seg_len=o[4])),
        ([new(torch.uint8, 2, 6), new(i32, 48), new(i32, 1), new(f32, 2, 6), new(torch.bfloat16, 48, 64)],
         lambda o: vico.vico_temporal_drop(frames, 0.1, *o[:3], sim=o[3], out_tokens=o[4])),
    ]
    for base, call in calls:
        want = [t.clone() for t in base]
        call(want)
        before = [t.clone() for t in base]
        clones = [torch._lazy_clone(t) for t in base]
        call(clones)
        torch.cuda.synchronize()
        for t, b, c, w in zip(base, before, clones, want):
            assert torch.equal(t, b) and torch.equal(c, w)
    lazy = torch._lazy_clone(k)
    out = [attn(), attn()]
    for x, o in zip((k, lazy), out):
        vico.vico_chunk_prefill_attn(q, x, v, None, None, None, None, 0, 0, o[0], lse=o[1])
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
