// The binding's calls in C++: checks of plain arguments, their pointers, and
// the call of libvico.
//
// A Python wrapper that looks at up to ten tensors attribute by attribute and
// hands 26 arguments to ctypes takes 10-14 us, as long as the kernels of the
// small calls run; here the same takes under 2.  Every function returns the
// library's status, or None for anything out of the ordinary (a tensor
// subclass, a wrong type or shape, a number that is not an int): the Python
// wrapper then takes its general path, which accepts or rejects the call in
// its own words.

#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>

#include "vico.h"

namespace {

// Arguments in order; `ok` turns false at the first one that is not plain.
struct Args {
  PyObject* const* a;
  Py_ssize_t n, i = 0;
  bool ok = true;

  PyObject* next() {
    if (i < n) return a[i++];
    ok = false;
    return Py_None;
  }
  // a contiguous device tensor of the given type and dimensions, or None where allowed
  const at::Tensor* tensor(at::ScalarType type, int dims, bool optional = false) {
    PyObject* o = next();
    if (o == Py_None) {
      if (!optional) ok = false;
      return nullptr;
    }
    if (!THPVariable_CheckExact(o)) return no();
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != type || t.dim() != dims || !t.is_contiguous()) return no();
    return &t;
  }
  // the output of an attention call: bf16 or fp32
  const at::Tensor* output() {
    PyObject* o = next();
    if (!THPVariable_CheckExact(o)) return no();
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.dim() != 3 || !t.is_contiguous()) return no();
    if (t.scalar_type() != at::kBFloat16 && t.scalar_type() != at::kFloat) return no();
    return &t;
  }
  // a workspace: any tensor's memory, by its size in bytes
  const at::Tensor* memory(bool device_only) {
    PyObject* o = next();
    if (o == Py_None) return nullptr;
    if (!THPVariable_CheckExact(o)) return no();
    const at::Tensor& t = THPVariable_Unpack(o);
    if (t.layout() != at::kStrided || (device_only && (!t.is_cuda() || !t.is_contiguous()))) return no();
    return &t;
  }
  const at::Tensor* no() {
    ok = false;
    return nullptr;
  }
  int64_t integer() {
    PyObject* o = next();
    if (!PyLong_CheckExact(o)) {
      ok = false;
      return 0;
    }
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    return v;
  }
  int32_t int32() {
    const int64_t v = integer();
    if (v != (int32_t)v) ok = false;
    return (int32_t)v;
  }
  float real() {
    PyObject* o = next();
    if (!PyFloat_CheckExact(o)) {
      ok = false;
      return 0.f;
    }
    return (float)PyFloat_AS_DOUBLE(o);
  }
  // None: the current stream of the current device; else a stream handle
  void* stream() {
    PyObject* o = next();
    if (o == Py_None) return ok ? (void*)c10::hip::getCurrentHIPStream().stream() : nullptr;
    return (void*)(uintptr_t)integer();
  }
};

// Address of a tensor that the library reads, and of one that it writes: the
// second gives a copy-on-write tensor memory of its own first.
void* ptr(const at::Tensor* t) { return t && t->numel() > 0 ? const_cast<void*>(t->const_data_ptr()) : nullptr; }
void* wptr(const at::Tensor* t) { return t && t->numel() > 0 ? t->mutable_data_ptr() : nullptr; }
int32_t size(const at::Tensor* t, int d) { return t ? (int32_t)t->size(d) : 0; }
int64_t bytes(const at::Tensor* t) { return t ? t->numel() * (int64_t)t->element_size() : 0; }
bool shape3(const at::Tensor* t, int64_t a, int64_t b, int64_t c) {
  return t->size(0) == a && t->size(1) == b && t->size(2) == c;
}
bool fits(const at::Tensor* t) { return !t || t->numel() < (int64_t(1) << 40); }

struct WithoutGil {
  PyThreadState* state = PyEval_SaveThread();
  ~WithoutGil() { PyEval_RestoreThread(state); }
};

template <class F>
PyObject* called(const Args& in, F&& call) {
  if (!in.ok || in.i != in.n) Py_RETURN_NONE;
  int st;
  {
    WithoutGil free;
    st = call();
  }
  return PyLong_FromLong(st);
}

// A tensor without memory throws when its address is asked for, before the
// library is called: also a case for the general path.
template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  try {
    return F(args, n);
  } catch (...) {
    Py_RETURN_NONE;
  }
}

// q, k_chunk, v_chunk, sink_k, sink_v, ring_k, ring_v, hist_len, window, out, lse, workspace, num_splits,
// softmax_scale, stream, flags
PyObject* prefill(PyObject* const* args, Py_ssize_t n) {
  Args in{args, n};
  const at::Tensor *q = in.tensor(at::kBFloat16, 3), *kc = in.tensor(at::kBFloat16, 3), *vc = in.tensor(at::kBFloat16, 3);
  const at::Tensor *sk = in.tensor(at::kBFloat16, 3, true), *sv = in.tensor(at::kBFloat16, 3, true);
  const at::Tensor *rk = in.tensor(at::kBFloat16, 3, true), *rv = in.tensor(at::kBFloat16, 3, true);
  const int64_t hist = in.integer(), window = in.integer();
  const at::Tensor* out = in.output();
  const at::Tensor* lse = in.tensor(at::kFloat, 2, true);
  const at::Tensor* ws = in.memory(false);
  const int32_t splits = in.int32();
  const float scale = in.real();
  void* stream = in.stream();
  const int32_t flags = in.int32();
  if (!in.ok || !shape3(out, q->size(0), q->size(1), q->size(2))) Py_RETURN_NONE;
  if (lse && (lse->size(0) != q->size(1) || lse->size(1) != q->size(0))) Py_RETURN_NONE;
  if (!fits(q) || !fits(kc) || !fits(sk) || !fits(rk)) Py_RETURN_NONE;
  const bool append = flags & VICO_ATTN_APPEND;
  void *const o = wptr(out), *const l = wptr(lse), *const w = wptr(ws);
  void *const ring_k = append ? wptr(rk) : ptr(rk), *const ring_v = append ? wptr(rv) : ptr(rv);
  return called(in, [&] {
    return vico_chunk_prefill_attn_ex(ptr(q), ptr(kc), ptr(vc), size(q, 0), ptr(sk), ptr(sv), size(sk, 0), ring_k, ring_v,
                                      size(rk, 0), hist, window, size(q, 1), size(kc, 1), size(q, 2), scale, o,
                                      out->scalar_type() == at::kFloat ? VICO_DTYPE_F32 : VICO_DTYPE_BF16, (float*)l,
                                      splits, flags, w, bytes(ws), stream);
  });
}

// q, tail_k, tail_v, sink_k, sink_v, store_k, store_v, seg_start, seg_len, out, lse, keys_hint, num_splits,
// softmax_scale, stream; then the workspace unless `noalloc`
PyObject* gather_call(PyObject* const* args, Py_ssize_t n, bool noalloc) {
  Args in{args, n};
  const at::Tensor *q = in.tensor(at::kBFloat16, 3), *tk = in.tensor(at::kBFloat16, 3), *tv = in.tensor(at::kBFloat16, 3);
  const at::Tensor *sk = in.tensor(at::kBFloat16, 3, true), *sv = in.tensor(at::kBFloat16, 3, true);
  const at::Tensor *gk = in.tensor(at::kBFloat16, 3, true), *gv = in.tensor(at::kBFloat16, 3, true);
  const at::Tensor* ss = in.tensor(at::kLong, 1, true);
  const at::Tensor* sl = in.tensor(at::kInt, 1, true);
  const at::Tensor* out = in.output();
  const at::Tensor* lse = in.tensor(at::kFloat, 2, true);
  const int64_t hint = in.integer();
  const int32_t splits = in.int32();
  const float scale = in.real();
  void* stream = in.stream();
  const at::Tensor* ws = noalloc ? nullptr : in.memory(false);
  if (!in.ok || !shape3(out, q->size(0), q->size(1), q->size(2)) || !ss != !sl) Py_RETURN_NONE;
  if (lse && (lse->size(0) != q->size(1) || lse->size(1) != q->size(0))) Py_RETURN_NONE;
  if (!fits(q) || !fits(tk) || !fits(sk) || !fits(gk) || !fits(ss)) Py_RETURN_NONE;
  const int32_t dt = out->scalar_type() == at::kFloat ? VICO_DTYPE_F32 : VICO_DTYPE_BF16;
  void *const o = wptr(out), *const l = wptr(lse), *const w = wptr(ws);
  return called(in, [&] {
    if (noalloc)
      return vico_gather_attn_noalloc(ptr(q), size(q, 0), ptr(tk), ptr(tv), size(tk, 0), ptr(sk), ptr(sv), size(sk, 0),
                                      ptr(gk), ptr(gv), size(gk, 0), (const int64_t*)ptr(ss), (const int32_t*)ptr(sl),
                                      size(ss, 0), hint, size(q, 1), size(tk, 1), size(q, 2), scale, o, dt, (float*)l, splits,
                                      stream);
    return vico_gather_attn(ptr(q), size(q, 0), ptr(tk), ptr(tv), size(tk, 0), ptr(sk), ptr(sv), size(sk, 0), ptr(gk),
                            ptr(gv), size(gk, 0), (const int64_t*)ptr(ss), (const int32_t*)ptr(sl), size(ss, 0), hint,
                            size(q, 1), size(tk, 1), size(q, 2), scale, o, dt, (float*)l, splits, w, bytes(ws), stream);
  });
}
PyObject* gather(PyObject* const* args, Py_ssize_t n) { return gather_call(args, n, false); }
PyObject* gather_noalloc(PyObject* const* args, Py_ssize_t n) { return gather_call(args, n, true); }

// k_chunk, v_chunk, ring_k, ring_v, hist_len, stream
PyObject* kv_append(PyObject* const* args, Py_ssize_t n) {
  Args in{args, n};
  const at::Tensor *kc = in.tensor(at::kBFloat16, 3), *vc = in.tensor(at::kBFloat16, 3);
  const at::Tensor *rk = in.tensor(at::kBFloat16, 3), *rv = in.tensor(at::kBFloat16, 3);
  const int64_t hist = in.integer();
  void* stream = in.stream();
  if (!in.ok || !fits(kc) || !fits(rk)) Py_RETURN_NONE;
  void *const ring_k = wptr(rk), *const ring_v = wptr(rv);
  return called(in, [&] {
    return vico_kv_append(ptr(kc), ptr(vc), size(kc, 0), ring_k, ring_v, size(rk, 0), hist, size(kc, 1), size(kc, 2),
                          stream);
  });
}

// x, out, stream
PyObject* token_mean(PyObject* const* args, Py_ssize_t n) {
  Args in{args, n};
  const at::Tensor *x = in.tensor(at::kBFloat16, 2), *out = in.tensor(at::kFloat, 1);
  void* stream = in.stream();
  if (!in.ok || out->size(0) != x->size(1) || !fits(x)) Py_RETURN_NONE;
  void* const o = wptr(out);
  return called(in, [&] { return vico_token_mean(ptr(x), size(x, 0), size(x, 1), (float*)o, stream); });
}

// query_feat, chunk_feat, scores, stream
PyObject* chunk_scores(PyObject* const* args, Py_ssize_t n) {
  Args in{args, n};
  const at::Tensor *qf = in.tensor(at::kFloat, 1), *cf = in.tensor(at::kFloat, 2), *sc = in.tensor(at::kFloat, 1);
  void* stream = in.stream();
  if (!in.ok || qf->size(0) != cf->size(1) || sc->size(0) != cf->size(0) || !fits(cf)) Py_RETURN_NONE;
  void* const o = wptr(sc);
  return called(in, [&] {
    return vico_chunk_scores((const float*)ptr(qf), (const float*)ptr(cf), size(cf, 0), size(cf, 1), (float*)o, stream);
  });
}

// scores, top_k, out_chunks, out_scores, out_count, min_score, chunk_start, chunk_len, seg_start, seg_len, stream
PyObject* topk_chunks(PyObject* const* args, Py_ssize_t n) {
  Args in{args, n};
  const at::Tensor* sc = in.tensor(at::kFloat, 1);
  const int32_t k = in.int32();
  const at::Tensor *oc = in.tensor(at::kInt, 1), *os = in.tensor(at::kFloat, 1), *cnt = in.tensor(at::kInt, 1);
  const float lowest = in.real();
  const at::Tensor *cs = in.tensor(at::kLong, 1, true), *cl = in.tensor(at::kInt, 1, true);
  const at::Tensor *ss = in.tensor(at::kLong, 1, true), *sl = in.tensor(at::kInt, 1, true);
  void* stream = in.stream();
  if (!in.ok || !fits(sc)) Py_RETURN_NONE;
  if (!cs != !cl || !cs != !ss || !cs != !sl) Py_RETURN_NONE;       // all four or none
  if (oc->size(0) < k || os->size(0) < k) Py_RETURN_NONE;
  if (cs && (cs->size(0) < sc->size(0) || cl->size(0) < sc->size(0) || ss->size(0) < k || sl->size(0) < k))
    Py_RETURN_NONE;
  void *const c = wptr(oc), *const v = wptr(os), *const b = wptr(ss), *const e = wptr(sl), *const m = wptr(cnt);
  return called(in, [&] {
    return vico_topk_chunks((const float*)ptr(sc), size(sc, 0), k, lowest, (const int64_t*)ptr(cs),
                            (const int32_t*)ptr(cl), (int32_t*)c, (float*)v, (int64_t*)b, (int32_t*)e, (int32_t*)m,
                            stream);
  });
}

// frames, tau, keep, out_index, out_count, sim, out_tokens, prev_frame, workspace, stream
PyObject* temporal_drop(PyObject* const* args, Py_ssize_t n) {
  Args in{args, n};
  const at::Tensor* f = in.tensor(at::kBFloat16, 4);
  const float tau = in.real();
  const at::Tensor *keep = in.tensor(at::kByte, 2), *idx = in.tensor(at::kInt, 1), *cnt = in.tensor(at::kInt, 1);
  const at::Tensor *sim = in.tensor(at::kFloat, 2, true), *tok = in.tensor(at::kBFloat16, 2, true);
  const at::Tensor* prev = in.tensor(at::kBFloat16, 2, true);
  const at::Tensor* ws = in.memory(true);
  void* stream = in.stream();
  if (!in.ok || !fits(f)) Py_RETURN_NONE;
  const int64_t B = f->size(0), C = f->size(1), n_f = f->size(2), dm = f->size(3), rows = B * C * n_f;
  if (keep->size(0) != B || keep->size(1) != n_f || idx->size(0) < rows) Py_RETURN_NONE;
  if (sim && (sim->size(0) != B || sim->size(1) != n_f)) Py_RETURN_NONE;
  if (tok && (tok->size(0) < rows || tok->size(1) != dm)) Py_RETURN_NONE;
  void *const k = wptr(keep), *const s = wptr(sim), *const o = wptr(tok), *const i = wptr(idx), *const m = wptr(cnt);
  void* const w = wptr(ws);
  return called(in, [&] {
    return vico_temporal_drop(ptr(f), (int32_t)B, (int32_t)C, (int32_t)n_f, (int32_t)dm, tau, ptr(prev), (uint8_t*)k,
                              (float*)s, o, (int32_t*)i, (int32_t*)m, w, bytes(ws), stream);
  });
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))entry<name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(prefill),      FAST(gather),      FAST(gather_noalloc), FAST(kv_append), FAST(token_mean),
                         FAST(chunk_scores), FAST(topk_chunks), FAST(temporal_drop),  {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_vico_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__vico_call(void) { return PyModule_Create(&module); }
