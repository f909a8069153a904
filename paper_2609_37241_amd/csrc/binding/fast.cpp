// The op calls of the Python binding, marshalled in native code.
//
// A short kernel's call from Python is host work: for a float32 RMSNorm of
// 1024 x 128 the interpreter's shape checks, stride and pointer queries and
// argument conversion took 4.5 of the call's 7.0 us. A Handle (one per
// SpecCache) takes the same tensors in one C call: it makes the binding's
// checks on the unpacked tensors, allocates the outputs that were not given
// and issues the entry call.
//
// Only the plain case is taken here: exact torch.Tensor / Parameter operands
// on the cache's device, float32 or bfloat16, of the expected shapes and
// strides, no torch function or dispatch mode, default stream or a stream
// object. For anything else -- wrong arguments included -- a method returns
// None before it has done anything, and the Python method of the same name
// makes its checks and raises its errors. A MISS is handled by the owner's
// _on_miss, as in the Python methods.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/TensorSubclassLikeUtils.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "tri.h"

namespace {

PyObject *g_error = nullptr;        // TriError
PyObject *g_rope_ext = nullptr;     // the ctypes structures
PyObject *g_chain_args = nullptr;

struct Handle {
  PyObject_HEAD
  tri_cache *cache;                 // null once the cache is closed
  int dev;
};

// Releases the GIL for its lifetime, as a ctypes call does.
struct NoGil {
  PyThreadState *s = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(s); }
};

// A plain tensor on GPU `dev`, or null.
const at::Tensor *plain(PyObject *o, int dev) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided ||
      t.device().index() != dev || at::isTensorSubclassLike(t) || t._is_zerotensor())
    return nullptr;
  return &t;
}

int dtype_of(const at::Tensor &t) {
  switch (t.scalar_type()) {
    case at::kFloat: return TRI_F32;
    case at::kBFloat16: return TRI_BF16;
    default: return -1;
  }
}

bool same(const at::Tensor &t, const at::Tensor &like) {
  return t.scalar_type() == like.scalar_type() && t.sizes() == like.sizes();
}

bool weight(const at::Tensor &t, int64_t n, const at::Tensor &like) {
  return t.dim() == 1 && t.size(0) == n && t.scalar_type() == like.scalar_type() &&
         (n <= 1 || t.stride(0) == 1);
}

// Row stride of a [T, W] tensor with unit inner stride, or -1; a single row
// reports at least W.
int64_t rows(const at::Tensor &t) {
  const int64_t T = t.size(0), W = t.size(1), s = t.stride(0);
  if (W > 1 && t.stride(1) != 1) return -1;
  return T > 1 || s >= W ? s : W;
}

// Token stride of a [T, nh, hd] tensor with packed heads, or -1.
int64_t tokens(const at::Tensor &t) {
  const int64_t T = t.size(0), nh = t.size(1), hd = t.size(2), s = t.stride(0);
  if ((hd > 1 && t.stride(2) != 1) || (nh > 1 && t.stride(1) != hd)) return -1;
  return T > 1 || s >= nh * hd ? s : nh * hd;
}

bool number(PyObject *o, float *v) {
  if (!PyFloat_Check(o) && !PyLong_Check(o)) return false;
  const double d = PyFloat_AsDouble(o);
  if (d == -1.0 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  *v = float(d);
  return true;
}

bool stream_of(const Handle *h, PyObject *o, void **s) {
  if (o == Py_None) {
    *s = c10::hip::getCurrentHIPStream(c10::DeviceIndex(h->dev)).stream();
    return true;
  }
  PyObject *p = PyObject_GetAttrString(o, "cuda_stream");
  if (p) {
    *s = PyLong_AsVoidPtr(p);
    Py_DECREF(p);
  }
  if (!PyErr_Occurred()) return true;
  PyErr_Clear();
  return false;
}

bool modes() {
  return at::impl::torch_function_mode_enabled() ||
         c10::impl::TorchDispatchModeTLS::any_modes_set();
}

// The bytes of a ctypes structure of class `type` (which the caller keeps
// alive), or null.
void *structure(PyObject *o, PyObject *type, size_t size) {
  if (reinterpret_cast<PyObject *>(Py_TYPE(o)) != type) return nullptr;
  Py_buffer b;
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
    PyErr_Clear();
    return nullptr;
  }
  void *p = size_t(b.len) >= size ? b.buf : nullptr;
  PyBuffer_Release(&b);
  return p;
}

// `call` until it no longer misses, at most `misses` times handled by the
// owner's _on_miss; raises TriError for any other status. True on OK.
template <class F>
bool issue(PyObject *owner, const char *what, F &&call, int64_t misses = 1) {
  int st;
  {
    NoGil g;
    st = call();
  }
  for (int64_t i = 0; st == TRI_MISS && i < misses; ++i) {
    PyObject *r = PyObject_CallMethod(owner, "_on_miss", nullptr);
    if (!r) return false;
    Py_DECREF(r);
    NoGil g;
    st = call();
  }
  if (st == TRI_OK) return true;
  if (PyObject *e = PyObject_CallFunction(g_error, "is", st, what)) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  }
  return false;
}

// An output: the tensor given (checked against `like`), or a new one.
struct Out {
  at::Tensor t;
  PyObject *given = nullptr;
  bool take(PyObject *o, const at::Tensor &like, int dev) {
    if (o == Py_None) {
      NoGil g;
      t = at::empty_like(like);
      return true;
    }
    const at::Tensor *p = plain(o, dev);
    if (!p || !same(*p, like)) return false;
    t = *p;
    given = o;
    return true;
  }
  PyObject *result() {
    if (!given) return THPVariable_Wrap(std::move(t));
    Py_INCREF(given);
    return given;
  }
};

PyObject *pair(PyObject *a, PyObject *b) {
  if (!a || !b) {
    Py_XDECREF(a);
    Py_XDECREF(b);
    return nullptr;
  }
  PyObject *r = PyTuple_Pack(2, a, b);
  Py_DECREF(a);
  Py_DECREF(b);
  return r;
}

// A method: `n` positional arguments after the owner; not the plain case or
// a C++ exception (nothing has been launched then): None.
typedef PyObject *(*Body)(Handle *h, PyObject *owner, PyObject *const *a);
template <Body B, int N>
PyObject *method(PyObject *self, PyObject *const *args, Py_ssize_t n) {
  Handle *h = reinterpret_cast<Handle *>(self);
  if (n != N + 1 || !h->cache || modes()) Py_RETURN_NONE;
  try {
    return B(h, args[0], args + 1);
  } catch (...) {
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
  }
}

// rmsnorm(owner, x, w, eps, out, stream)
PyObject *rmsnorm(Handle *h, PyObject *owner, PyObject *const *a) {
  const at::Tensor *x = plain(a[0], h->dev), *w = plain(a[1], h->dev);
  float eps;
  void *s;
  if (!x || !w || x->dim() != 2 || dtype_of(*x) < 0 || !weight(*w, x->size(1), *x) ||
      !number(a[2], &eps) || !stream_of(h, a[4], &s))
    Py_RETURN_NONE;
  const int64_t T = x->size(0), H = x->size(1), xs = rows(*x);
  Out y;
  if (xs < 0 || !y.take(a[3], *x, h->dev)) Py_RETURN_NONE;
  const int64_t ys = rows(y.t);
  if (ys < 0) Py_RETURN_NONE;
  const tri_dtype dt = tri_dtype(dtype_of(*x));
  const void *xp = x->data_ptr(), *wp = w->data_ptr();
  void *yp = y.t.data_ptr();
  if (!issue(owner, "tri_rmsnorm",
             [&] { return tri_rmsnorm(h->cache, dt, xp, xs, wp, yp, ys, T, H, eps, s); }))
    return nullptr;
  return y.result();
}

// residual_rmsnorm(owner, x, residual, w, eps, out, residual_out, stream)
PyObject *residual_rmsnorm(Handle *h, PyObject *owner, PyObject *const *a) {
  const at::Tensor *x = plain(a[0], h->dev), *r = plain(a[1], h->dev), *w = plain(a[2], h->dev);
  float eps;
  void *s;
  if (!x || !r || !w || x->dim() != 2 || dtype_of(*x) < 0 || !same(*r, *x) ||
      !weight(*w, x->size(1), *x) || !number(a[3], &eps) || !stream_of(h, a[6], &s))
    Py_RETURN_NONE;
  const int64_t T = x->size(0), H = x->size(1), xs = rows(*x), rs = rows(*r);
  Out y, o;
  if (xs < 0 || rs < 0 || !y.take(a[4], *x, h->dev) || !o.take(a[5], *r, h->dev)) Py_RETURN_NONE;
  const int64_t ys = rows(y.t), os = rows(o.t);
  if (ys < 0 || os < 0) Py_RETURN_NONE;
  const tri_dtype dt = tri_dtype(dtype_of(*x));
  const void *xp = x->data_ptr(), *rp = r->data_ptr(), *wp = w->data_ptr();
  void *yp = y.t.data_ptr(), *op = o.t.data_ptr();
  if (!issue(owner, "tri_residual_rmsnorm", [&] {
        return tri_residual_rmsnorm(h->cache, dt, xp, xs, rp, rs, wp, yp, ys, op, os, T, H, eps, s);
      }))
    return nullptr;
  return pair(y.result(), o.result());
}

// Two inputs and an output of one shape [T, W] (swiglu, add), or one input
// (silu): (owner, a, [b,] out, stream).
template <int OP>
PyObject *flat(Handle *h, PyObject *owner, PyObject *const *a) {
  constexpr bool one = OP == TRI_OP_SILU;
  const at::Tensor *x = plain(a[0], h->dev);
  const at::Tensor *b = one ? x : plain(a[1], h->dev);
  PyObject *const *rest = a + (one ? 1 : 2);
  void *s;
  if (!x || !b || x->dim() != 2 || dtype_of(*x) < 0 || !same(*b, *x) || !stream_of(h, rest[1], &s))
    Py_RETURN_NONE;
  const int64_t T = x->size(0), W = x->size(1), xs = rows(*x), bs = rows(*b);
  Out y;
  if (xs < 0 || bs < 0 || !y.take(rest[0], *x, h->dev)) Py_RETURN_NONE;
  const int64_t ys = rows(y.t);
  if (ys < 0) Py_RETURN_NONE;
  const tri_dtype dt = tri_dtype(dtype_of(*x));
  const void *xp = x->data_ptr(), *bp = b->data_ptr();
  void *yp = y.t.data_ptr();
  const char *what = OP == TRI_OP_SWIGLU ? "tri_swiglu" : one ? "tri_silu" : "tri_add";
  if (!issue(owner, what, [&] {
        if constexpr (OP == TRI_OP_SWIGLU)
          return tri_swiglu(h->cache, dt, xp, xs, bp, bs, yp, ys, T, W, s);
        else if constexpr (one)
          return tri_silu(h->cache, dt, xp, xs, yp, ys, T, W, s);
        else
          return tri_add(h->cache, dt, xp, xs, bp, bs, yp, ys, T, W, s);
      }))
    return nullptr;
  return y.result();
}

// masked_fill(owner, x, mask, value, out, stream)
PyObject *masked_fill(Handle *h, PyObject *owner, PyObject *const *a) {
  const at::Tensor *x = plain(a[0], h->dev), *m = plain(a[1], h->dev);
  float value;
  void *s;
  if (!x || !m || x->dim() != 2 || dtype_of(*x) < 0 || m->sizes() != x->sizes() ||
      (m->scalar_type() != at::kByte && m->scalar_type() != at::kBool) || !number(a[2], &value) ||
      !stream_of(h, a[4], &s))
    Py_RETURN_NONE;
  const int64_t T = x->size(0), W = x->size(1), xs = rows(*x), ms = rows(*m);
  Out y;
  if (xs < 0 || ms < 0 || !y.take(a[3], *x, h->dev)) Py_RETURN_NONE;
  const int64_t ys = rows(y.t);
  if (ys < 0) Py_RETURN_NONE;
  const tri_dtype dt = tri_dtype(dtype_of(*x));
  const void *xp = x->data_ptr();
  const uint8_t *mp = static_cast<const uint8_t *>(m->data_ptr());
  void *yp = y.t.data_ptr();
  if (!issue(owner, "tri_masked_fill", [&] {
        return tri_masked_fill(h->cache, dt, xp, xs, mp, ms, value, yp, ys, T, W, s);
      }))
    return nullptr;
  return y.result();
}

// embedding(owner, table, ids, out, stream)
PyObject *embedding(Handle *h, PyObject *owner, PyObject *const *a) {
  const at::Tensor *t = plain(a[0], h->dev), *ids = plain(a[1], h->dev);
  void *s;
  if (!t || !ids || t->dim() != 2 || dtype_of(*t) < 0 || ids->dim() != 1 ||
      (ids->scalar_type() != at::kInt && ids->scalar_type() != at::kLong) ||
      !stream_of(h, a[3], &s))
    Py_RETURN_NONE;
  const int64_t n = t->size(0), H = t->size(1), T = ids->size(0), ts = rows(*t);
  if (ts < 0 || (T > 1 && ids->stride(0) != 1)) Py_RETURN_NONE;
  Out y;
  if (a[2] == Py_None) {
    NoGil g;
    y.t = at::empty({T, H}, t->options());
  } else {
    const at::Tensor *o = plain(a[2], h->dev);
    if (!o || o->dim() != 2 || o->size(0) != T || o->size(1) != H ||
        o->scalar_type() != t->scalar_type())
      Py_RETURN_NONE;
    y.t = *o;
    y.given = a[2];
  }
  const int64_t ys = rows(y.t);
  if (ys < 0) Py_RETURN_NONE;
  const tri_dtype dt = tri_dtype(dtype_of(*t));
  const void *tp = t->data_ptr(), *ip = ids->data_ptr();
  const int32_t wide = ids->scalar_type() == at::kLong;
  void *yp = y.t.data_ptr();
  if (!issue(owner, "tri_embedding", [&] {
        return tri_embedding(h->cache, dt, tp, ts, n, ip, wide, yp, ys, T, H, s);
      }))
    return nullptr;
  return y.result();
}

// The rotation: (owner, q, k, pos, base, ext, q_w, k_w, eps, stream, kind),
// kind 0: tri_rope_qk, 1: tri_qk_norm_rope, 2: tri_rope_qk_ext.
PyObject *rope(Handle *h, PyObject *owner, PyObject *const *a) {
  const at::Tensor *q = plain(a[0], h->dev), *pos = plain(a[2], h->dev);
  const at::Tensor *k = nullptr, *qw = nullptr, *kw = nullptr;
  float base, eps;
  void *s;
  if (!q || !pos || q->dim() != 3 || dtype_of(*q) < 0 || !number(a[3], &base) ||
      !number(a[7], &eps) || !stream_of(h, a[8], &s))
    Py_RETURN_NONE;
  const int64_t T = q->size(0), nq = q->size(1), hd = q->size(2), qs = tokens(*q);
  if (qs < 0 || nq > INT32_MAX || hd > INT32_MAX) Py_RETURN_NONE;
  const tri_rope_ext *ext = nullptr;
  if (a[4] != Py_None) {
    ext = static_cast<const tri_rope_ext *>(structure(a[4], g_rope_ext, sizeof(tri_rope_ext)));
    if (!ext) Py_RETURN_NONE;
    if (ext->cos_sin) {
      // the table's tensor travels with the struct: its width and device
      // must be what the kernels read through the bare address
      PyObject *to = PyObject_GetAttrString(a[4], "_cos_sin");
      if (!to) {
        PyErr_Clear();
        Py_RETURN_NONE;
      }
      const at::Tensor *t = plain(to, h->dev);
      const bool ok = t && t->dim() == 2 && t->size(1) == (ext->rotary_dim ? ext->rotary_dim : hd);
      Py_DECREF(to);
      if (!ok) Py_RETURN_NONE;
    }
  }
  int64_t nk = 0, ks = 0;
  void *kp = nullptr;
  if (a[1] != Py_None) {
    k = plain(a[1], h->dev);
    if (!k || k->dim() != 3 || k->size(0) != T || k->size(2) != hd ||
        k->scalar_type() != q->scalar_type() || k->size(1) > INT32_MAX)
      Py_RETURN_NONE;
    nk = k->size(1);
    if (nk) {
      ks = tokens(*k);
      if (ks < 0) Py_RETURN_NONE;
      kp = k->data_ptr();
    }
  }
  if (pos->dim() != 1 || pos->size(0) != T || (T > 1 && pos->stride(0) != 1) ||
      pos->scalar_type() != (ext && ext->pos_int64 ? at::kLong : at::kInt))
    Py_RETURN_NONE;
  if (a[5] != Py_None && (!(qw = plain(a[5], h->dev)) || !weight(*qw, hd, *q))) Py_RETURN_NONE;
  if (a[6] != Py_None && (!(kw = plain(a[6], h->dev)) || !weight(*kw, hd, *q))) Py_RETURN_NONE;
  const long kind = PyLong_AsLong(a[9]);
  if (kind == 1 && !qw) Py_RETURN_NONE;
  const tri_dtype dt = tri_dtype(dtype_of(*q));
  void *qp = q->data_ptr(), *pp = pos->data_ptr();
  const void *qwp = qw ? qw->data_ptr() : nullptr, *kwp = kw ? kw->data_ptr() : nullptr;
  const int32_t q_ = int32_t(nq), k_ = int32_t(nk), d_ = int32_t(hd);
  const char *what = kind == 0 ? "tri_rope_qk" : kind == 1 ? "tri_qk_norm_rope" : "tri_rope_qk_ext";
  if (!issue(owner, what, [&] {
        if (kind == 0)
          return tri_rope_qk(h->cache, dt, qp, qs, kp, ks, static_cast<const int32_t *>(pp), T, q_,
                             k_, d_, base, s);
        if (kind == 1)
          return tri_qk_norm_rope(h->cache, dt, qp, qs, kp, ks, static_cast<const int32_t *>(pp),
                                  T, q_, k_, d_, base, qwp, kwp, eps, s);
        return tri_rope_qk_ext(h->cache, dt, qp, qs, kp, ks, pp, T, q_, k_, d_, base, ext, qwp,
                               kwp, eps, s);
      }))
    return nullptr;
  return PyTuple_Pack(2, a[0], a[1]);
}

// decode_chain_args(owner, args, stream)
PyObject *chain(Handle *h, PyObject *owner, PyObject *const *a) {
  const void *p = structure(a[0], g_chain_args, sizeof(tri_chain_args));
  void *s;
  if (!p || !stream_of(h, a[1], &s)) Py_RETURN_NONE;
  if (!issue(owner, "tri_decode_chain", [&] {
        return tri_decode_chain(h->cache, static_cast<const tri_chain_args *>(p), s);
      }))
    return nullptr;
  Py_RETURN_TRUE;
}

// decode_chain_layers(owner, list of args, stream)
PyObject *layers(Handle *h, PyObject *owner, PyObject *const *a) {
  void *s;
  if (!PyList_CheckExact(a[0]) || !stream_of(h, a[1], &s)) Py_RETURN_NONE;
  const Py_ssize_t n = PyList_GET_SIZE(a[0]);
  std::vector<tri_chain_args> v;
  v.reserve(size_t(n) + 1);
  for (Py_ssize_t i = 0; i < n; ++i) {
    const void *p = structure(PyList_GET_ITEM(a[0], i), g_chain_args, sizeof(tri_chain_args));
    if (!p) Py_RETURN_NONE;
    v.push_back(*static_cast<const tri_chain_args *>(p));
  }
  if (n > TRI_MAX_LAYERS) Py_RETURN_NONE;
  if (!issue(owner, "tri_decode_chain_layers",
             [&] { return tri_decode_chain_layers(h->cache, v.data(), uint32_t(n), s); }, n))
    return nullptr;
  Py_RETURN_TRUE;
}

PyObject *close(PyObject *self, PyObject *) {
  reinterpret_cast<Handle *>(self)->cache = nullptr;
  Py_RETURN_NONE;
}

template <Body B, int N>
PyCFunction fn() {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&method<B, N>));
}

PyMethodDef g_methods[] = {
    {"rmsnorm", fn<rmsnorm, 5>(), METH_FASTCALL, nullptr},
    {"residual_rmsnorm", fn<residual_rmsnorm, 7>(), METH_FASTCALL, nullptr},
    {"swiglu", fn<flat<TRI_OP_SWIGLU>, 4>(), METH_FASTCALL, nullptr},
    {"silu", fn<flat<TRI_OP_SILU>, 3>(), METH_FASTCALL, nullptr},
    {"add", fn<flat<TRI_OP_ADD>, 4>(), METH_FASTCALL, nullptr},
    {"masked_fill", fn<masked_fill, 5>(), METH_FASTCALL, nullptr},
    {"embedding", fn<embedding, 4>(), METH_FASTCALL, nullptr},
    {"rope", fn<rope, 10>(), METH_FASTCALL, nullptr},
    {"chain", fn<chain, 2>(), METH_FASTCALL, nullptr},
    {"layers", fn<layers, 2>(), METH_FASTCALL, nullptr},
    {"close", close, METH_NOARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};

// Handle(cache address, device index)
PyObject *handle_new(PyTypeObject *type, PyObject *args, PyObject *) {
  unsigned long long p;
  int dev;
  if (!PyArg_ParseTuple(args, "Ki", &p, &dev)) return nullptr;
  Handle *h = reinterpret_cast<Handle *>(type->tp_alloc(type, 0));
  if (h) {
    h->cache = reinterpret_cast<tri_cache *>(p);
    h->dev = dev;
  }
  return reinterpret_cast<PyObject *>(h);
}

void handle_free(PyObject *self) {
  PyTypeObject *type = Py_TYPE(self);
  type->tp_free(self);
  Py_DECREF(type);
}

PyType_Slot g_slots[] = {{Py_tp_new, reinterpret_cast<void *>(&handle_new)},
                         {Py_tp_dealloc, reinterpret_cast<void *>(&handle_free)},
                         {Py_tp_methods, g_methods},
                         {0, nullptr}};
PyType_Spec g_spec = {"paper_2609_37241_amd._fast.Handle", int(sizeof(Handle)), 0,
                      Py_TPFLAGS_DEFAULT, g_slots};

// setup(TriError, RopeExt, ChainArgs)
PyObject *setup(PyObject *, PyObject *args) {
  PyObject *e, *r, *c;
  if (!PyArg_ParseTuple(args, "OOO", &e, &r, &c)) return nullptr;
  Py_INCREF(e);
  Py_INCREF(r);
  Py_INCREF(c);
  g_error = e;
  g_rope_ext = r;
  g_chain_args = c;
  Py_RETURN_NONE;
}

PyMethodDef g_functions[] = {{"setup", setup, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_fast", nullptr, -1, g_functions,
                        nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fast() {
  PyObject *m = PyModule_Create(&g_module);
  if (!m) return nullptr;
  PyObject *type = PyType_FromSpec(&g_spec);
  if (!type || PyModule_AddObject(m, "Handle", type) < 0) {
    Py_XDECREF(type);
    Py_DECREF(m);
    return nullptr;
  }
  // what the package compares with the torch it runs on
  if (PyModule_AddStringConstant(m, "torch_version", TRI_TORCH_VERSION) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
