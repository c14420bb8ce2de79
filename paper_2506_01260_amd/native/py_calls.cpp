// The binding's calls in native code: each function takes the arguments of the
// Python function of the same name, turns the tensors into the C ABI's plain
// pointers, sizes and strides, allocates the output where none is given, and
// calls the library (whose entry points are handed over by bind(), so this
// module works with whichever build of the library the package loaded).
//
// It takes the ordinary call only.  Anything else (a tensor subclass, another
// device, dtype, shape or stride, a tracing or function mode, an object of
// another type) returns None before anything is launched, and the Python
// function goes on with the call and its errors.  A status other than SN_OK is
// raised by the package's own check.
//
// Why: the Python form of a call took 12.5 us, 3.5 of them the launch, and a
// small launch runs for less than that; this form takes about 5.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "sn.h"

namespace {

#define SN_CALLS(X)                                                                            \
  X(sn_compress) X(sn_decompress) X(sn_grad_compress) X(sn_compress_projected)                \
  X(sn_project_weights) X(sn_project_weights_workspace_bytes) X(sn_project_weights_multi)     \
  X(sn_project_weights_multi_workspace_bytes) X(sn_grassmann_accumulate)                      \
  X(sn_grassmann_workspace_bytes) X(sn_embed_lowrank_forward) X(sn_embed_lowrank_backward)    \
  X(sn_embed_lowrank_workspace_bytes) X(sn_adamw_step) X(sn_adamw_workspace_bytes)

struct Calls {
#define X(f) decltype(&::f) f = nullptr;
  SN_CALLS(X)
#undef X
} g_lib;
PyObject *g_check = nullptr;  // the package's status check

// names of the attributes read, interned once
PyObject *s_packed, *s_d, *s_k, *s_dt, *s_buf, *s_basis, *s_vocab, *s_n_pos, *s_cuda_stream;

struct Mat {
  void *p = nullptr;
  int64_t rows = 0, cols = 0, ld = 0;
  at::ScalarType type = at::ScalarType::Undefined;
};

// The tensor of an argument if it is a plain device tensor, else nullptr.
const at::Tensor *plain(PyObject *o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage()) return nullptr;
  constexpr c10::DispatchKeySet wrapped(
      {c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
       c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize});
  if (t.key_set().has_any(wrapped)) return nullptr;
  return &t;
}

bool mat(PyObject *o, Mat &m) {
  const at::Tensor *t = plain(o);
  if (!t || t->dim() != 2) return false;
  m.rows = t->size(0);
  m.cols = t->size(1);
  if (m.cols > 1 && t->stride(1) != 1) return false;
  m.ld = m.rows > 1 ? t->stride(0) : m.cols;
  if (m.ld < m.cols) return false;
  m.type = t->scalar_type();
  m.p = t->data_ptr();
  return true;
}

// A matrix of the given type and width (absent: None).
bool table(PyObject *o, at::ScalarType type, int64_t cols, Mat &m) {
  if (o == Py_None) return true;
  return mat(o, m) && m.type == type && m.cols == cols;
}

// n contiguous int32 ids; not looked at where `used` is false, as in Python.
bool ids(PyObject *o, bool used, int64_t n, const int32_t *&p) {
  p = nullptr;
  if (!used || o == Py_None) return true;
  const at::Tensor *t = plain(o);
  if (!t || t->scalar_type() != at::kInt || t->dim() != 1 || t->size(0) != n ||
      (n > 1 && t->stride(0) != 1))
    return false;
  p = static_cast<const int32_t *>(t->data_ptr());
  return true;
}

bool flag(PyObject *o, int32_t *&p) {
  p = nullptr;
  if (o == Py_None) return true;
  const at::Tensor *t = plain(o);
  if (!t) return false;
  p = static_cast<int32_t *>(t->data_ptr());
  return true;
}

bool int_of(PyObject *o, int64_t &v) {
  if (!PyLong_CheckExact(o)) return false;
  v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}

bool int_attr(PyObject *o, PyObject *name, int64_t &v) {
  PyObject *a = PyObject_GetAttr(o, name);
  if (!a) {
    PyErr_Clear();
    return false;
  }
  const bool ok = int_of(a, v);
  Py_DECREF(a);
  return ok;
}

// A tensor attribute's data pointer (and size in bytes).
bool buffer_attr(PyObject *o, PyObject *name, void *&p, int64_t &bytes) {
  PyObject *a = PyObject_GetAttr(o, name);
  if (!a) {
    PyErr_Clear();
    return false;
  }
  const at::Tensor *t = plain(a);
  if (t) {
    p = t->data_ptr();
    bytes = static_cast<int64_t>(t->nbytes());
  }
  Py_DECREF(a);  // the object keeps its tensor
  return t != nullptr;
}

struct Basis {
  void *p = nullptr;
  int64_t d = 0, k = 0, dt = 0;
  at::ScalarType type = at::ScalarType::Undefined;
};
bool basis(PyObject *o, Basis &b) {
  int64_t bytes;
  if (!buffer_attr(o, s_packed, b.p, bytes) || !int_attr(o, s_d, b.d) || !int_attr(o, s_k, b.k) ||
      !int_attr(o, s_dt, b.dt))
    return false;
  b.type = b.dt == SN_F32 ? at::kFloat : at::kBFloat16;
  return b.dt == SN_F32 || b.dt == SN_BF16;
}

bool stream(PyObject *o, sn_stream &s) {
  if (o == Py_None) {
    s = c10::hip::getCurrentHIPStream().stream();
    return true;
  }
  PyObject *a = PyObject_GetAttr(o, s_cuda_stream);
  if (!a) {
    PyErr_Clear();
    return false;
  }
  const bool ok = PyLong_CheckExact(a);
  if (ok) s = PyLong_AsVoidPtr(a);
  Py_DECREF(a);
  if (ok && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return ok;
}

// The output argument, or a new tensor like the Python functions make (`t`
// keeps it until it is returned).
bool output(PyObject *o, PyObject *like, at::ScalarType type, int64_t rows, int64_t cols, Mat &m,
            at::Tensor &t) {
  if (o != Py_None) return mat(o, m) && m.type == type && m.rows == rows && m.cols == cols;
  t = at::empty({rows, cols}, THPVariable_Unpack(like).options().dtype(type).requires_grad(false));
  m.p = t.data_ptr();
  m.rows = rows;
  m.cols = m.ld = cols;
  m.type = type;
  return true;
}

bool workspace(PyObject *o, PyObject *like, size_t need, void *&p, size_t &bytes, at::Tensor &t) {
  if (o != Py_None) {
    const at::Tensor *w = plain(o);
    if (!w || static_cast<size_t>(w->numel()) < need) return false;
    p = w->data_ptr();
    bytes = static_cast<size_t>(w->numel());
    return true;
  }
  bytes = need > 1 ? need : 1;
  t = at::empty({static_cast<int64_t>(bytes)},
                THPVariable_Unpack(like).options().dtype(at::kByte).requires_grad(false));
  p = t.data_ptr();
  return true;
}

// A mode that sees or replaces calls on tensors.
bool modes() {
  return at::impl::torch_function_mode_enabled() ||
         c10::impl::TorchDispatchModeTLS::any_modes_set();
}

PyObject *given(PyObject *o) {
  Py_INCREF(o);
  return o;
}

PyObject *finish(int32_t status, PyObject *out, at::Tensor &made) {
  if (status != SN_OK) {
    PyObject *r = PyObject_CallFunction(g_check, "i", status);
    Py_XDECREF(r);
    if (!r) return nullptr;
  }
  return made.defined() ? THPVariable_Wrap(std::move(made)) : given(out);
}

// The library call without the interpreter lock, as ctypes makes it.
template <typename F>
int32_t launch(F &&f) {
  int32_t st;
  Py_BEGIN_ALLOW_THREADS st = f();
  Py_END_ALLOW_THREADS return st;
}

// Runs a call; an exception (a tensor without data, an allocation that fails)
// leaves it to the Python form, which meets the same one and reports it.
template <typename F>
PyObject *guarded(Py_ssize_t have, Py_ssize_t want, F &&f) {
  if (have != want) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    if (!modes()) {
      bool taken = true;
      PyObject *r = f(taken);
      if (taken) return r;
    }
  } catch (const std::exception &) {
  }
  Py_RETURN_NONE;
}

#define SN_FAST(name) PyObject *name(PyObject *, PyObject *const *a, Py_ssize_t n)
#define SN_LEAVE return taken = false, nullptr

// (basis, X or C, tok, E, P, pos, seq_len, out, err_flag, stream)
PyObject *codec(PyObject *const *a, Py_ssize_t n, bool compress) {
  return guarded(n, 10, [&](bool &taken) -> PyObject * {
    Basis b;
    Mat in, E, P, out;
    const int32_t *tok, *pos;
    int32_t *err;
    int64_t seq = 0;
    sn_stream s;
    at::Tensor made;
    if (!basis(a[0], b) || !mat(a[1], in) || in.type != b.type ||
        in.cols != (compress ? b.d : b.k) || !table(a[3], b.type, b.d, E) ||
        !table(a[4], b.type, b.d, P) || !ids(a[2], a[3] != Py_None, in.rows, tok) ||
        !ids(a[5], a[4] != Py_None, in.rows, pos) || (a[6] != Py_None && !int_of(a[6], seq)) ||
        !flag(a[8], err) || !stream(a[9], s) ||
        !output(a[7], a[1], b.type, in.rows, compress ? b.k : b.d, out, made))
      SN_LEAVE;
    const int32_t dt = static_cast<int32_t>(b.dt);
    const int32_t st = launch([&] {
      return (compress ? g_lib.sn_compress : g_lib.sn_decompress)(
          b.p, b.d, b.k, dt, in.p, in.rows, in.ld, tok, E.p, E.rows, E.ld, pos, P.p, P.rows, P.ld,
          seq, out.p, out.ld, err, s);
    });
    return finish(st, a[7], made);
  });
}
SN_FAST(compress) { return codec(a, n, true); }
SN_FAST(decompress) { return codec(a, n, false); }

// (basis, G, out, stream)
SN_FAST(grad_compress) {
  return guarded(n, 4, [&](bool &taken) -> PyObject * {
    Basis b;
    Mat g, out;
    sn_stream s;
    at::Tensor made;
    if (!basis(a[0], b) || !mat(a[1], g) || g.type != b.type || g.cols != b.d || !stream(a[3], s) ||
        !output(a[2], a[1], b.type, g.rows, b.k, out, made))
      SN_LEAVE;
    const int32_t st = launch([&] {
      return g_lib.sn_grad_compress(b.p, b.d, b.k, static_cast<int32_t>(b.dt), g.p, g.rows, g.ld,
                                    out.p, out.ld, s);
    });
    return finish(st, a[2], made);
  });
}

// (basis, X, proj, tok, pos, seq_len, out, err_flag, stream)
SN_FAST(compress_projected) {
  return guarded(n, 9, [&](bool &taken) -> PyObject * {
    Basis b;
    Mat x, out;
    const int32_t *tok, *pos;
    int32_t *err;
    int64_t seq = 0, vocab = 0, n_pos = 0, bytes = 0;
    void *proj = nullptr;
    sn_stream s;
    at::Tensor made;
    PyObject *pb = PyObject_GetAttr(a[2], s_basis);
    if (!pb) {
      PyErr_Clear();
      SN_LEAVE;
    }
    const bool same = pb == a[0];
    Py_DECREF(pb);
    if (!same || !basis(a[0], b) || !mat(a[1], x) || x.type != b.type || x.cols != b.d ||
        !buffer_attr(a[2], s_buf, proj, bytes) || !int_attr(a[2], s_vocab, vocab) ||
        !int_attr(a[2], s_n_pos, n_pos) || !ids(a[3], vocab != 0, x.rows, tok) ||
        !ids(a[4], n_pos != 0, x.rows, pos) || (a[5] != Py_None && !int_of(a[5], seq)) ||
        !flag(a[7], err) || !stream(a[8], s) ||
        !output(a[6], a[1], b.type, x.rows, b.k, out, made))
      SN_LEAVE;
    const int32_t st = launch([&] {
      return g_lib.sn_compress_projected(b.p, b.d, b.k, static_cast<int32_t>(b.dt), x.p, x.rows,
                                         x.ld, tok, pos, seq, bytes ? proj : nullptr, vocab, n_pos,
                                         out.p, out.ld, err, s);
    });
    return finish(st, a[6], made);
  });
}

// (basis, W, workspace, stream)
SN_FAST(project_weights) {
  return guarded(n, 4, [&](bool &taken) -> PyObject * {
    Basis b;
    Mat w;
    sn_stream s;
    void *ws;
    size_t bytes;
    at::Tensor made, none;
    if (!basis(a[0], b) || !mat(a[1], w) || w.type != b.type || w.rows != b.d || !stream(a[3], s))
      SN_LEAVE;
    const int32_t dt = static_cast<int32_t>(b.dt);
    const size_t need = g_lib.sn_project_weights_workspace_bytes(b.d, b.k, dt, w.cols);
    if (!workspace(a[2], a[1], need, ws, bytes, made)) SN_LEAVE;
    const int32_t st = launch([&] {
      return g_lib.sn_project_weights(b.p, b.d, b.k, dt, w.p, w.cols, w.ld, ws, bytes, s);
    });
    return finish(st, a[1], none);
  });
}

// (basis, Ws, workspace, stream)
SN_FAST(project_weights_multi) {
  return guarded(n, 4, [&](bool &taken) -> PyObject * {
    Basis b;
    sn_stream s;
    void *p[SN_PROJECT_MAX_MATRICES], *ws;
    int64_t m[SN_PROJECT_MAX_MATRICES], ld[SN_PROJECT_MAX_MATRICES];
    size_t bytes;
    at::Tensor made, none;
    if (!basis(a[0], b) || !PyList_CheckExact(a[1]) || !stream(a[3], s)) SN_LEAVE;
    const Py_ssize_t count = PyList_GET_SIZE(a[1]);
    if (count < 1 || count > SN_PROJECT_MAX_MATRICES) SN_LEAVE;
    for (Py_ssize_t i = 0; i < count; ++i) {
      Mat w;
      if (!mat(PyList_GET_ITEM(a[1], i), w) || w.type != b.type || w.rows != b.d) SN_LEAVE;
      p[i] = w.p;
      m[i] = w.cols;
      ld[i] = w.ld;
    }
    const int32_t dt = static_cast<int32_t>(b.dt), c = static_cast<int32_t>(count);
    const size_t need = g_lib.sn_project_weights_multi_workspace_bytes(b.d, b.k, dt, c, m);
    if (!workspace(a[2], PyList_GET_ITEM(a[1], 0), need, ws, bytes, made)) SN_LEAVE;
    const int32_t st = launch([&] {
      return g_lib.sn_project_weights_multi(b.p, b.d, b.k, dt, c, p, m, ld, ws, bytes, s);
    });
    return finish(st, a[1], none);
  });
}

// (basis, G, state, with_su, want_cg, out, workspace, stream)
SN_FAST(grassmann_accumulate) {
  return guarded(n, 8, [&](bool &taken) -> PyObject * {
    Basis b;
    Mat g, out;
    sn_stream s;
    void *state, *ws;
    int64_t d, k, sb;
    size_t bytes;
    at::Tensor made, wmade;
    const int su = PyObject_IsTrue(a[3]), cg = PyObject_IsTrue(a[4]);
    if (su < 0 || cg < 0) {
      PyErr_Clear();
      SN_LEAVE;
    }
    if (!basis(a[0], b) || !mat(a[1], g) || g.type != b.type || g.cols != b.d ||
        !buffer_attr(a[2], s_buf, state, sb) || !int_attr(a[2], s_d, d) ||
        !int_attr(a[2], s_k, k) || d != b.d || k != b.k || !stream(a[7], s))
      SN_LEAVE;
    const int32_t dt = static_cast<int32_t>(b.dt);
    const size_t need = g_lib.sn_grassmann_workspace_bytes(b.d, b.k, dt, g.rows);
    const bool wire = a[5] != Py_None || cg;
    if ((wire && !output(a[5], a[1], b.type, g.rows, b.k, out, made)) ||
        !workspace(a[6], a[1], need, ws, bytes, wmade))
      SN_LEAVE;
    const int32_t st = launch([&] {
      return g_lib.sn_grassmann_accumulate(b.p, b.d, b.k, dt, g.p, g.rows, g.ld,
                                           wire ? out.p : nullptr, wire ? out.ld : 0, su, state,
                                           ws, bytes, s);
    });
    return finish(st, a[5], made);
  });
}

// (basis, CS, tok, E, P, pos, seq_len, out, err_flag, workspace, stream)
SN_FAST(embed_lowrank_forward) {
  return guarded(n, 11, [&](bool &taken) -> PyObject * {
    Basis b;
    Mat cs, E, P, out;
    const int32_t *tok, *pos;
    int32_t *err;
    int64_t seq = 0;
    sn_stream s;
    void *ws;
    size_t bytes;
    at::Tensor made, wmade;
    const at::Tensor *tt = plain(a[2]);
    if (!tt || tt->dim() != 1) SN_LEAVE;
    const int64_t N = tt->size(0);
    if (!basis(a[0], b) || !mat(a[1], cs) || cs.type != b.type || cs.cols != b.k ||
        !table(a[3], b.type, b.d, E) || (a[3] != Py_None && E.rows != cs.rows) ||
        !table(a[4], b.type, b.d, P) || !ids(a[2], true, N, tok) ||
        !ids(a[5], a[4] != Py_None, N, pos) || (a[6] != Py_None && !int_of(a[6], seq)) ||
        !flag(a[8], err) || !stream(a[10], s))
      SN_LEAVE;
    const int32_t dt = static_cast<int32_t>(b.dt);
    const size_t need = g_lib.sn_embed_lowrank_workspace_bytes(b.d, b.k, dt, N, cs.rows);
    if (!output(a[7], a[1], b.type, N, b.d, out, made) ||
        !workspace(a[9], a[1], need, ws, bytes, wmade))
      SN_LEAVE;
    const int32_t st = launch([&] {
      return g_lib.sn_embed_lowrank_forward(b.p, b.d, b.k, dt, cs.p, cs.rows, cs.ld, tok, E.p, E.ld,
                                            pos, P.p, P.rows, P.ld, seq, out.p, N, out.ld, err, ws,
                                            bytes, s);
    });
    return finish(st, a[7], made);
  });
}

// (basis, dX0, tok, gCS, err_flag, workspace, stream)
SN_FAST(embed_lowrank_backward) {
  return guarded(n, 7, [&](bool &taken) -> PyObject * {
    Basis b;
    Mat g, gcs;
    const int32_t *tok;
    int32_t *err;
    sn_stream s;
    void *ws;
    size_t bytes;
    at::Tensor wmade, none;
    if (!basis(a[0], b) || !mat(a[1], g) || g.type != b.type || g.cols != b.d || !mat(a[3], gcs) ||
        gcs.type != at::kFloat || gcs.cols != b.k || a[2] == Py_None ||
        !ids(a[2], true, g.rows, tok) || !flag(a[4], err) || !stream(a[6], s))
      SN_LEAVE;
    const int32_t dt = static_cast<int32_t>(b.dt);
    const size_t need = g_lib.sn_embed_lowrank_workspace_bytes(b.d, b.k, dt, g.rows, gcs.rows);
    if (!workspace(a[5], a[1], need, ws, bytes, wmade)) SN_LEAVE;
    const int32_t st = launch([&] {
      return g_lib.sn_embed_lowrank_backward(b.p, b.d, b.k, dt, g.p, g.rows, g.ld, tok, gcs.rows,
                                             static_cast<float *>(gcs.p), gcs.ld, err, ws, bytes,
                                             s);
    });
    return finish(st, a[3], none);
  });
}

// (W, G, M, V, t, lr, beta1, beta2, eps, weight_decay, subspace, workspace, stream)
SN_FAST(adamw_step) {
  return guarded(n, 13, [&](bool &taken) -> PyObject * {
    Mat w, g, m, v;
    int64_t t;
    double f[5];
    sn_stream s;
    void *ws = nullptr;
    size_t bytes = 0;
    at::Tensor wmade, none;
    for (int i = 0; i < 5; ++i) {
      if (!PyFloat_CheckExact(a[5 + i])) SN_LEAVE;
      f[i] = PyFloat_AS_DOUBLE(a[5 + i]);
    }
    const int sub = PyObject_IsTrue(a[10]);
    if (sub < 0) {
      PyErr_Clear();
      SN_LEAVE;
    }
    if (!mat(a[0], w) || (w.type != at::kFloat && w.type != at::kBFloat16) || !mat(a[1], g) ||
        !mat(a[2], m) || !mat(a[3], v) || g.type != w.type || m.type != at::kFloat ||
        v.type != at::kFloat || g.rows != w.rows || g.cols != w.cols || m.rows != w.rows ||
        m.cols != w.cols || v.rows != w.rows || v.cols != w.cols || m.ld != v.ld ||
        !int_of(a[4], t) || !stream(a[12], s))
      SN_LEAVE;
    const size_t need = sub ? g_lib.sn_adamw_workspace_bytes(w.rows, w.cols) : 0;
    if (need && !workspace(a[11], a[0], need, ws, bytes, wmade)) SN_LEAVE;
    const int32_t st = launch([&] {
      return g_lib.sn_adamw_step(w.p, w.ld, g.p, g.ld, w.type == at::kFloat ? SN_F32 : SN_BF16,
                                 static_cast<float *>(m.p), static_cast<float *>(v.p), m.ld, w.rows,
                                 w.cols, t, f[0], f[1], f[2], f[3], f[4], sub, ws, need, s);
    });
    return finish(st, a[0], none);
  });
}

// bind(addresses: dict of entry point -> address, check: status check)
SN_FAST(bind) {
  if (n != 2 || !PyDict_Check(a[0])) {
    PyErr_SetString(PyExc_TypeError, "bind(addresses, check)");
    return nullptr;
  }
#define X(f)                                                                  \
  {                                                                           \
    PyObject *v = PyDict_GetItemString(a[0], #f);                             \
    if (!v) return PyErr_Format(PyExc_KeyError, "%s", #f);                    \
    g_lib.f = reinterpret_cast<decltype(&::f)>(PyLong_AsVoidPtr(v));          \
    if (PyErr_Occurred()) return nullptr;                                     \
  }
  SN_CALLS(X)
#undef X
  Py_XDECREF(g_check);
  g_check = given(a[1]);
  Py_RETURN_NONE;
}

#define SN_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {SN_METHOD(bind),
                           SN_METHOD(compress),
                           SN_METHOD(decompress),
                           SN_METHOD(grad_compress),
                           SN_METHOD(compress_projected),
                           SN_METHOD(project_weights),
                           SN_METHOD(project_weights_multi),
                           SN_METHOD(grassmann_accumulate),
                           SN_METHOD(embed_lowrank_forward),
                           SN_METHOD(embed_lowrank_backward),
                           SN_METHOD(adamw_step),
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, g_methods,
                        nullptr,               nullptr,  nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
  const struct {
    PyObject **to;
    const char *name;
  } names[] = {{&s_packed, "packed"}, {&s_d, "d"},         {&s_k, "k"},
               {&s_dt, "dt"},         {&s_buf, "buf"},     {&s_basis, "basis"},
               {&s_vocab, "vocab"},   {&s_n_pos, "n_pos"}, {&s_cuda_stream, "cuda_stream"}};
  for (const auto &e : names)
    if (!(*e.to = PyUnicode_InternFromString(e.name))) return nullptr;
  return PyModule_Create(&g_module);
}
