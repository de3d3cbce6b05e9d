// The hot calls of the Python binding (kvq.py) as C functions of an extension module: argument reading only.
//
// What a call costs a program that launches one small kernel after another is the interpreter's time in front of the launch:
// tensor attributes read one by one (0.1 us each), arguments converted by ctypes (0.1 us each).  Here they are read from the
// tensors' own structures.  Every function takes the arguments of the kvq.py function of its name, makes that function's checks, and
// returns the library's status; for anything but the plain case (tensor subclasses and wrappers, function modes, other types of
// number, a check that does not hold, the first call in a process) it returns None without having done anything, and kvq.py goes on
// as if it were not there, so that what is refused, and how, is said in one place.
// Host time per call through kvq.py, without and with it: a 2048-token append of one sequence 5.6 and 3.9 us (4.0 of them the
// library and the launch, by ctypes with everything at hand), a fused step 6.7 and 4.1; back to back that append takes 5.7 and 4.5 us.
#include <Python.h>
#include <string.h>
#include <unistd.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "kvq.h"

// torch's current stream (a build that runs without a device names another source)
#ifndef KVQ_CURRENT_STREAM
#define KVQ_CURRENT_STREAM() c10::hip::getCurrentHIPStream().stream()
#endif

namespace {

// The library's entry points, as kvq.py has loaded them (bind), and the process that torch's device runtime was started in
// (0: not yet; a forked child is another process, and what it may not do is torch's to say).
decltype(&kvq_quantize_append) g_append = nullptr;
decltype(&kvq_decode_attention) g_attention = nullptr;
decltype(&kvq_decode_attention_varlen) g_attention_varlen = nullptr;
decltype(&kvq_decode_step) g_step = nullptr;
decltype(&kvq_decode_step_varlen) g_step_varlen = nullptr;
pid_t g_pid = 0;

PyObject* g_layout_attr = nullptr;                 // "_c", "_struct": where kvq.py's objects keep their C structs
PyObject* g_cache_attr = nullptr;
PyObject* g_c = nullptr;                           // "c": the method that builds them
PyObject* g_layout_class = nullptr;                // kvq.py's Layout and Cache (bind)
PyObject* g_cache_class = nullptr;

// Copies the C struct of `obj` to `to`; false where there is none.  An object of kvq.py's own class keeps its struct under `attr`; where
// nothing is kept yet, and for any other class, which may build it in its own way, it is what obj.c() returns.  A copy, made with
// the interpreter's lock held: `obj` may drop its struct (a new page table does) while the library, which runs without the lock,
// still reads it.
template <typename T> bool copy_struct(PyObject* obj, PyObject* own, PyObject* attr, T* to) {
  PyObject* s = (PyObject*)Py_TYPE(obj) == own ? PyObject_GetAttr(obj, attr) : nullptr;
  if (!s || s == Py_None) {
    PyErr_Clear();
    Py_XDECREF(s);
    s = PyObject_CallMethodNoArgs(obj, g_c);
    if (!s) return false;
  }
  Py_buffer view;
  bool copied = false;
  if (PyObject_GetBuffer(s, &view, PyBUF_SIMPLE) == 0) {
    copied = view.len == (Py_ssize_t)sizeof(T);
    if (copied) memcpy(to, view.buf, sizeof(T));
    PyBuffer_Release(&view);
  } else {
    PyErr_Clear();
  }
  Py_DECREF(s);
  return copied;
}

// Reads the arguments of one call; `ok` turns false at the first that is not plain.
struct Reader {
  bool ok = true;
  kvq_layout layout;
  kvq_cache cache;
  void* stream = nullptr;

  Reader(bool right_form, PyObject* l, PyObject* c) {
    if (!need(right_form && g_pid != 0 && getpid() == g_pid && !at::impl::torch_function_mode_enabled())) return;
    if (need(copy_struct(l, g_layout_class, g_layout_attr, &layout) && copy_struct(c, g_cache_class, g_cache_attr, &cache))) stream = KVQ_CURRENT_STREAM();
  }
  bool need(bool holds) { ok = ok && holds; return ok; }
  const at::Tensor* tensor(PyObject* o) { return need(THPVariable_CheckExact(o)) ? &THPVariable_Unpack(o) : nullptr; }
  int32_t int32(PyObject* o) {
    if (!need(PyLong_CheckExact(o))) return 0;
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    return need(!overflow && v >= INT32_MIN && v <= INT32_MAX) ? (int32_t)v : 0;
  }
  float real(PyObject* o) { return need(PyFloat_CheckExact(o)) ? (float)PyFloat_AS_DOUBLE(o) : 0.0f; }
  kvq_dtype dtype(const at::Tensor& t) {
    const auto st = t.scalar_type();
    need(st == at::kHalf || st == at::kBFloat16 || st == at::kFloat);
    return st == at::kHalf ? KVQ_F16 : st == at::kBFloat16 ? KVQ_BF16 : KVQ_F32;
  }
};
// Key and value rows: alike in everything, the last axis contiguous.
struct Rows {
  const void *k = nullptr, *v = nullptr;
  kvq_dtype type = KVQ_F16;
  int64_t sb = 0, sh = 0, st = 0, n = 0;
  // tokens: [B, H, n, D]; otherwise one token each, [B, H, D] or [B, H, 1, D]
  Rows(Reader& r, PyObject* ko, PyObject* vo, bool tokens) {
    const at::Tensor *kt = r.tensor(ko), *vt = r.tensor(vo);
    if (!r.ok) return;
    const int64_t dims = kt->dim();
    if (!r.need((dims == 4 || (dims == 3 && !tokens)) && kt->sizes() == vt->sizes() && kt->scalar_type() == vt->scalar_type() &&
                kt->strides() == vt->strides() && kt->stride(dims - 1) == 1 && (tokens || dims == 3 || kt->size(2) == 1)))
      return;
    k = kt->data_ptr(); v = vt->data_ptr();
    type = r.dtype(*kt);
    sb = kt->stride(0); sh = kt->stride(1);
    if (tokens) { st = kt->stride(2); n = kt->size(2); r.need(n <= INT32_MAX); }
  }
};
struct Attention {
  const void* q = nullptr;
  void *out = nullptr, *ws = nullptr;
  kvq_dtype q_type = KVQ_F16, out_type = KVQ_F16;
  int32_t heads = 0;
  float scale = 0.0f;
  size_t ws_bytes = 0;
  Attention(Reader& r, PyObject* qo, PyObject* so, PyObject* oo, PyObject* wo) {
    const at::Tensor *qt = r.tensor(qo), *ot = r.tensor(oo), *wt = wo == Py_None ? nullptr : r.tensor(wo);
    scale = r.real(so);
    if (!r.ok || !r.need(qt->dim() == 3 && qt->is_contiguous() && ot->is_contiguous() && ot->sizes() == qt->sizes())) return;
    if (!r.need(qt->size(1) <= INT32_MAX)) return;
    q = qt->data_ptr(); out = ot->data_ptr();
    q_type = r.dtype(*qt); out_type = r.dtype(*ot);
    heads = (int32_t)qt->size(1);
    if (wt) { ws = wt->data_ptr(); ws_bytes = wt->nbytes(); }
  }
};
const int32_t* lengths(Reader& r, PyObject* o) {
  const at::Tensor* t = r.tensor(o);
  if (!r.ok || !r.need(t->scalar_type() == at::kInt && t->is_contiguous() && t->numel() == r.layout.batch)) return nullptr;
  return static_cast<const int32_t*>(t->data_ptr());
}

// What `body` returns (the library's status, or a negative number for a case that is not plain) as Python has it.
template <typename F> PyObject* plain(F body) {
  long status;
  try {
    status = (long)body();
  } catch (...) {                                  // (whatever a tensor without plain storage or strides raises)
    status = -1;
  }
  if (status < 0) {                                // (an object's own c() may have raised: kvq.py meets that again, an interrupt goes on)
    if (PyErr_Occurred() && !PyErr_ExceptionMatches(PyExc_Exception)) return nullptr;
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  return PyLong_FromLong(status);
}
// The library's call itself, other threads running.
template <typename F> int released(F call) {
  PyThreadState* state = PyEval_SaveThread();
  const kvq_status st = call();
  PyEval_RestoreThread(state);
  return (int)st;
}

// (layout, cache, k_new, v_new, pos)
PyObject* quantize_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return plain([&]() -> int {
    if (n != 5) return -1;
    Reader r(g_append != nullptr, a[0], a[1]);
    if (!r.ok) return -1;
    const Rows w(r, a[2], a[3], true);
    const int32_t pos = r.int32(a[4]);
    if (!r.ok) return -1;
    return released([&] { return g_append(&r.layout, &r.cache, w.k, w.v, w.type, w.sb, w.sh, w.st, pos, (int32_t)w.n, r.stream); });
  });
}

// (layout, cache, q, seq_len, softmax_scale, out, workspace)
PyObject* decode_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return plain([&]() -> int {
    if (n != 7) return -1;
    Reader r(g_attention != nullptr, a[0], a[1]);
    if (!r.ok) return -1;
    const Attention t(r, a[2], a[4], a[5], a[6]);
    const int32_t len = r.int32(a[3]);
    if (!r.ok) return -1;
    return released([&] {
      return g_attention(&r.layout, &r.cache, t.q, t.q_type, t.heads, len, t.scale, t.out, t.out_type, t.ws, t.ws_bytes, r.stream);
    });
  });
}

// (layout, cache, q, seq_lens, max_seq_len, softmax_scale, out, workspace)
PyObject* decode_attention_varlen(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return plain([&]() -> int {
    if (n != 8) return -1;
    Reader r(g_attention_varlen != nullptr, a[0], a[1]);
    if (!r.ok) return -1;
    const Attention t(r, a[2], a[5], a[6], a[7]);
    const int32_t* lens = lengths(r, a[3]);
    const int32_t bound = r.int32(a[4]);
    if (!r.ok) return -1;
    return released([&] {
      return g_attention_varlen(&r.layout, &r.cache, t.q, t.q_type, t.heads, lens, bound, t.scale, t.out, t.out_type, t.ws, t.ws_bytes,
                                r.stream);
    });
  });
}

// (layout, cache, k_new, v_new, pos, q, softmax_scale, out, workspace)
PyObject* decode_step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return plain([&]() -> int {
    if (n != 9) return -1;
    Reader r(g_step != nullptr, a[0], a[1]);
    if (!r.ok) return -1;
    const Rows w(r, a[2], a[3], false);
    const Attention t(r, a[5], a[6], a[7], a[8]);
    const int32_t pos = r.int32(a[4]);
    if (!r.ok) return -1;
    return released([&] {
      return g_step(&r.layout, &r.cache, w.k, w.v, w.type, w.sb, w.sh, pos, t.q, t.q_type, t.heads, t.scale, t.out, t.out_type, t.ws,
                    t.ws_bytes, r.stream);
    });
  });
}

// (layout, cache, k_new, v_new, pos, max_pos, q, softmax_scale, out, workspace)
PyObject* decode_step_varlen(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return plain([&]() -> int {
    if (n != 10) return -1;
    Reader r(g_step_varlen != nullptr, a[0], a[1]);
    if (!r.ok) return -1;
    const Rows w(r, a[2], a[3], false);
    const Attention t(r, a[6], a[7], a[8], a[9]);
    const int32_t* pos = lengths(r, a[4]);
    const int32_t bound = r.int32(a[5]);
    if (!r.ok) return -1;
    return released([&] {
      return g_step_varlen(&r.layout, &r.cache, w.k, w.v, w.type, w.sb, w.sh, pos, bound, t.q, t.q_type, t.heads, t.scale, t.out,
                           t.out_type, t.ws, t.ws_bytes, r.stream);
    });
  });
}

// (five addresses, in the order of the pointers above: the entry points of the library that kvq.py has loaded; then its classes
// Layout and Cache)
PyObject* bind(PyObject*, PyObject* args) {
  unsigned long long p[5];
  PyObject *layout, *cache;
  if (!PyArg_ParseTuple(args, "KKKKKOO", &p[0], &p[1], &p[2], &p[3], &p[4], &layout, &cache)) return nullptr;
  g_append = reinterpret_cast<decltype(g_append)>(p[0]);
  g_attention = reinterpret_cast<decltype(g_attention)>(p[1]);
  g_attention_varlen = reinterpret_cast<decltype(g_attention_varlen)>(p[2]);
  g_step = reinterpret_cast<decltype(g_step)>(p[3]);
  g_step_varlen = reinterpret_cast<decltype(g_step_varlen)>(p[4]);
  Py_INCREF(layout); Py_XSETREF(g_layout_class, layout);
  Py_INCREF(cache); Py_XSETREF(g_cache_class, cache);
  Py_RETURN_NONE;
}
// torch's device runtime is up in this process (kvq.py says so after a call that went its own way).
PyObject* ready(PyObject*, PyObject*) {
  g_pid = getpid();
  Py_RETURN_NONE;
}

#define KVQ_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {KVQ_FAST(quantize_append), KVQ_FAST(decode_attention), KVQ_FAST(decode_attention_varlen),
                         KVQ_FAST(decode_step), KVQ_FAST(decode_step_varlen), {"bind", bind, METH_VARARGS, nullptr},
                         {"ready", ready, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_kvq_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__kvq_binding(void) {
  g_layout_attr = PyUnicode_InternFromString("_c");
  g_cache_attr = PyUnicode_InternFromString("_struct");
  g_c = PyUnicode_InternFromString("c");
  if (!g_layout_attr || !g_cache_attr || !g_c) return nullptr;
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "torch_version", KVQ_TORCH_VERSION) != 0) Py_CLEAR(m);   // (whose structures it reads)
  return m;
}
