// Argument marshalling of the Python binding: fills mt_tensor descriptors from
// torch tensors through their Python attributes and calls the C entry points.
// In native code because a call of the smallest layer is bound by it: with
// ctypes and descriptors built in Python a call took 11 us, more than its
// kernels. Nothing is kept between calls.
//
// init(handle, float32, bfloat16, describe, current_stream, stream_of): the
// library's dlopen handle, torch's two dtypes, binding.desc (called to raise
// its error for a tensor that is refused) and how a stream is found (none
// given / given). Every other function returns the entry point's status.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <dlfcn.h>

#include "../../include/minitensor_hip.h"

namespace {

PyObject *g_f32, *g_bf16, *g_describe, *g_current, *g_stream_of;
PyObject *s_is_cuda, *s_dtype, *s_shape, *s_stride, *s_data_ptr, *s_numel, *s_element_size;

struct Lib {
  decltype(&mt_linear_fwd) linear_fwd;
  decltype(&mt_linear_act_fwd) linear_act_fwd;
  decltype(&mt_linear_bwd) linear_bwd;
  decltype(&mt_matmul) matmul;
  decltype(&mt_reduce_broadcast_grad) reduce_broadcast_grad;
  decltype(&mt_act_bwd) act_bwd;
  decltype(&mt_mse_loss) mse_loss;
  decltype(&mt_sgd_step) sgd_step;
  decltype(&mt_adam_step) adam_step;
  decltype(&mt_rmsprop_step) rmsprop_step;
  decltype(&mt_conv2d_fwd) conv2d_fwd;
  decltype(&mt_conv2d_bwd) conv2d_bwd;
} L;

bool as_i64(PyObject* o, int64_t* v) {
  if (PyLong_Check(o)) {
    *v = PyLong_AsLongLong(o);
  } else {
    PyObject* i = PyNumber_Long(o);
    if (!i) return false;
    *v = PyLong_AsLongLong(i);
    Py_DECREF(i);
  }
  return *v != -1 || !PyErr_Occurred();
}

bool as_address(PyObject* o, void** p) {  // consumes o
  if (!o) return false;
  const unsigned long long v = PyLong_AsUnsignedLongLong(o);
  Py_DECREF(o);
  *p = (void*)(uintptr_t)v;
  return v != (unsigned long long)-1 || !PyErr_Occurred();
}

bool ints(PyObject* tuple, int64_t* out, Py_ssize_t* n) {  // consumes tuple
  if (!tuple) return false;
  bool ok = PyTuple_Check(tuple);
  if (!ok) PyErr_SetString(PyExc_TypeError, "expected a tuple of sizes");
  *n = ok ? PyTuple_GET_SIZE(tuple) : 0;
  for (Py_ssize_t i = 0; ok && i < *n && i < MT_MAX_DIMS; ++i) ok = as_i64(PyTuple_GET_ITEM(tuple, i), &out[i]);
  Py_DECREF(tuple);
  return ok;
}

bool refuse(PyObject* t) {
  PyObject* r = PyObject_CallOneArg(g_describe, t);  // raises what is wrong with it
  if (r) {
    Py_DECREF(r);
    PyErr_SetString(PyExc_RuntimeError, "tensor cannot be described");
  }
  return false;
}

bool describe(PyObject* t, mt_tensor* d) {
  PyObject* v = PyObject_GetAttr(t, s_is_cuda);
  if (!v) return false;
  Py_DECREF(v);
  if (v != Py_True) return refuse(t);
  if (!(v = PyObject_GetAttr(t, s_dtype))) return false;
  Py_DECREF(v);
  if (v == g_f32) d->dtype = MT_F32;
  else if (v == g_bf16) d->dtype = MT_BF16;
  else return refuse(t);
  Py_ssize_t n, m;
  if (!ints(PyObject_GetAttr(t, s_shape), d->shape, &n)) return false;
  if (n > MT_MAX_DIMS) return refuse(t);
  if (!ints(PyObject_CallMethodNoArgs(t, s_stride), d->stride, &m)) return false;
  if (m != n) return refuse(t);
  d->ndim = (int32_t)n;
  return as_address(PyObject_CallMethodNoArgs(t, s_data_ptr), &d->data);
}

// A call's arguments, converted in the order they are asked for; `ok` turns
// false with a Python error set, and later conversions do nothing.
struct Args {
  PyObject* const* a;
  bool ok = true;
  mt_tensor d[6];
  int used = 0;
  Args(PyObject* const* args, Py_ssize_t n, Py_ssize_t want) : a(args) {
    if (n != want) {
      PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
      ok = false;
    }
  }
  const mt_tensor* tensor(int i) {
    if (!ok || a[i] == Py_None) return nullptr;
    mt_tensor* t = &d[used++];
    ok = describe(a[i], t);
    return t;
  }
  int64_t i64(int i) {
    int64_t v = 0;
    if (ok) ok = as_i64(a[i], &v);
    return v;
  }
  float f32(int i) {
    if (!ok) return 0.f;
    const double v = PyFloat_AsDouble(a[i]);
    ok = v != -1.0 || !PyErr_Occurred();
    return (float)v;
  }
  struct Ws {
    void* p = nullptr;
    size_t n = 0;
  };
  Ws ws(int i) {
    Ws w;
    if (!ok || a[i] == Py_None) return w;
    PyObject* c = PyObject_GetAttr(a[i], s_is_cuda);
    ok = c != nullptr;
    if (c) Py_DECREF(c);
    if (ok && c != Py_True) {
      PyErr_SetString(PyExc_AssertionError, "the workspace is a device tensor");
      ok = false;
    }
    void *count = nullptr, *size = nullptr;
    ok = ok && as_address(PyObject_CallMethodNoArgs(a[i], s_data_ptr), &w.p) &&
         as_address(PyObject_CallMethodNoArgs(a[i], s_numel), &count) &&
         as_address(PyObject_CallMethodNoArgs(a[i], s_element_size), &size);
    w.n = (size_t)(uintptr_t)count * (size_t)(uintptr_t)size;
    return w;
  }
  void* stream(int i) {
    void* s = nullptr;
    if (ok)
      ok = as_address(a[i] == Py_None ? PyObject_CallNoArgs(g_current) : PyObject_CallOneArg(g_stream_of, a[i]), &s);
    return s;
  }
};

template <typename F>
PyObject* call(bool ok, F f) {
  if (!ok) return nullptr;
  mt_status s;
  Py_BEGIN_ALLOW_THREADS
  s = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong((long)s);
}

#define FN(name) PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n)

FN(linear_fwd) {  // x, w, b, y, stream
  Args g(a, n, 5);
  const mt_tensor *x = g.tensor(0), *w = g.tensor(1), *b = g.tensor(2), *y = g.tensor(3);
  void* st = g.stream(4);
  return call(g.ok, [&] { return L.linear_fwd(x, w, b, y, st); });
}
FN(linear_act_fwd) {  // x, w, b, act, z, y, stream
  Args g(a, n, 7);
  const mt_tensor *x = g.tensor(0), *w = g.tensor(1), *b = g.tensor(2);
  const int32_t act = (int32_t)g.i64(3);
  const mt_tensor *z = g.tensor(4), *y = g.tensor(5);
  void* st = g.stream(6);
  return call(g.ok, [&] { return L.linear_act_fwd(x, w, b, act, z, y, st); });
}
FN(linear_bwd) {  // x, w, dy, dx, dw, db, flags, ws, stream
  Args g(a, n, 9);
  const mt_tensor *x = g.tensor(0), *w = g.tensor(1), *dy = g.tensor(2), *dx = g.tensor(3), *dw = g.tensor(4),
                  *db = g.tensor(5);
  const uint32_t flags = (uint32_t)g.i64(6);
  const Args::Ws ws = g.ws(7);
  void* st = g.stream(8);
  return call(g.ok, [&] { return L.linear_bwd(x, w, dy, dx, dw, db, flags, ws.p, ws.n, st); });
}
FN(matmul) {  // a, b, c, flags, ws, stream
  Args g(a, n, 6);
  const mt_tensor *x = g.tensor(0), *y = g.tensor(1), *c = g.tensor(2);
  const uint32_t flags = (uint32_t)g.i64(3);
  const Args::Ws ws = g.ws(4);
  void* st = g.stream(5);
  return call(g.ok, [&] { return L.matmul(x, y, c, flags, ws.p, ws.n, st); });
}
FN(reduce_broadcast_grad) {  // grad_out, grad_in, flags, ws, stream
  Args g(a, n, 5);
  const mt_tensor *o = g.tensor(0), *i = g.tensor(1);
  const uint32_t flags = (uint32_t)g.i64(2);
  const Args::Ws ws = g.ws(3);
  void* st = g.stream(4);
  return call(g.ok, [&] { return L.reduce_broadcast_grad(o, i, flags, ws.p, ws.n, st); });
}
FN(act_bwd) {  // act, z, dy, dz, db, flags, ws, stream
  Args g(a, n, 8);
  const int32_t act = (int32_t)g.i64(0);
  const mt_tensor *z = g.tensor(1), *dy = g.tensor(2), *dz = g.tensor(3), *db = g.tensor(4);
  const uint32_t flags = (uint32_t)g.i64(5);
  const Args::Ws ws = g.ws(6);
  void* st = g.stream(7);
  return call(g.ok, [&] { return L.act_bwd(act, z, dy, dz, db, flags, ws.p, ws.n, st); });
}
FN(mse_loss) {  // pred, target, loss, dpred, ws, stream
  Args g(a, n, 6);
  const mt_tensor *p = g.tensor(0), *t = g.tensor(1), *l = g.tensor(2), *d = g.tensor(3);
  const Args::Ws ws = g.ws(4);
  void* st = g.stream(5);
  return call(g.ok, [&] { return L.mse_loss(p, t, l, d, ws.p, ws.n, st); });
}
FN(conv2d_fwd) {  // x, w, b, y, sh, sw, ph, pw, ws, stream
  Args g(a, n, 10);
  const mt_tensor *x = g.tensor(0), *w = g.tensor(1), *b = g.tensor(2), *y = g.tensor(3);
  int32_t v[4];
  for (int i = 0; i < 4; ++i) v[i] = (int32_t)g.i64(4 + i);
  const Args::Ws ws = g.ws(8);
  void* st = g.stream(9);
  return call(g.ok, [&] { return L.conv2d_fwd(x, w, b, y, v[0], v[1], v[2], v[3], ws.p, ws.n, st); });
}
FN(conv2d_bwd) {  // x, w, dy, dx, dw, db, sh, sw, ph, pw, flags, ws, stream
  Args g(a, n, 13);
  const mt_tensor *x = g.tensor(0), *w = g.tensor(1), *dy = g.tensor(2), *dx = g.tensor(3), *dw = g.tensor(4),
                  *db = g.tensor(5);
  int32_t v[4];
  for (int i = 0; i < 4; ++i) v[i] = (int32_t)g.i64(6 + i);
  const uint32_t flags = (uint32_t)g.i64(10);
  const Args::Ws ws = g.ws(11);
  void* st = g.stream(12);
  return call(g.ok, [&] { return L.conv2d_bwd(x, w, dy, dx, dw, db, v[0], v[1], v[2], v[3], flags, ws.p, ws.n, st); });
}

// Descriptors of up to four lists of n tensors each, one list after another.
// The lists' tensors are held until the call has returned: it runs without
// the interpreter's lock, while another thread may change a list, and an
// iterable may make its tensors as it is read. What has no length is refused.
struct Lists {
  PyObject* held[4] = {};
  mt_tensor* d = nullptr;
  Py_ssize_t n = 0;
  bool ok = true;
  Lists(PyObject* const* a, int lists) {
    for (int l = 0; ok && l < lists; ++l) ok = PyObject_Size(a[l]) >= 0 && (held[l] = PySequence_Tuple(a[l])) != nullptr;
    if (!ok) return;
    n = PyTuple_GET_SIZE(held[0]);
    for (int l = 1; l < lists; ++l) {
      if (PyTuple_GET_SIZE(held[l]) == n) continue;
      PyErr_SetString(PyExc_AssertionError, "the lists of tensors have different lengths");
      ok = false;
      return;
    }
    d = (mt_tensor*)PyMem_Malloc(sizeof(mt_tensor) * (size_t)(lists * (n > 0 ? n : 1)));
    if (!d) {
      PyErr_NoMemory();
      ok = false;
    }
    for (int l = 0; ok && l < lists; ++l)
      for (Py_ssize_t i = 0; ok && i < n; ++i) ok = describe(PyTuple_GET_ITEM(held[l], i), &d[l * n + i]);
  }
  ~Lists() {
    PyMem_Free(d);
    for (PyObject* h : held) Py_XDECREF(h);
  }
  const mt_tensor* operator[](int l) const { return d + l * n; }
};

FN(sgd_step) {  // params, grads, velocity, lr, momentum, weight_decay, stream
  Args g(a, n, 7);
  if (!g.ok) return nullptr;
  const Lists t(a, 3);
  if (!t.ok) return nullptr;
  const float lr = g.f32(3), mu = g.f32(4), wd = g.f32(5);
  void* st = g.stream(6);
  return call(g.ok, [&] { return L.sgd_step((int32_t)t.n, t[0], t[1], t[2], lr, mu, wd, st); });
}
FN(adam_step) {  // params, grads, exp_avg, exp_avg_sq, lr, beta1, beta2, eps, step, stream
  Args g(a, n, 10);
  if (!g.ok) return nullptr;
  const Lists t(a, 4);
  if (!t.ok) return nullptr;
  const float lr = g.f32(4), b1 = g.f32(5), b2 = g.f32(6), eps = g.f32(7);
  const int64_t step = g.i64(8);
  void* st = g.stream(9);
  return call(g.ok, [&] { return L.adam_step((int32_t)t.n, t[0], t[1], t[2], t[3], lr, b1, b2, eps, step, st); });
}
FN(rmsprop_step) {  // params, grads, sq_avg, lr, alpha, eps, stream
  Args g(a, n, 7);
  if (!g.ok) return nullptr;
  const Lists t(a, 3);
  if (!t.ok) return nullptr;
  const float lr = g.f32(3), alpha = g.f32(4), eps = g.f32(5);
  void* st = g.stream(6);
  return call(g.ok, [&] { return L.rmsprop_step((int32_t)t.n, t[0], t[1], t[2], lr, alpha, eps, st); });
}

FN(init) {
  if (n != 6) {
    PyErr_SetString(PyExc_TypeError, "init(handle, float32, bfloat16, describe, current_stream, stream_of)");
    return nullptr;
  }
  void* h = PyLong_AsVoidPtr(a[0]);
  if (!h) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null library handle");
    return nullptr;
  }
#define SYM(f)                                              \
  if (!(L.f = (decltype(L.f))dlsym(h, "mt_" #f))) {         \
    PyErr_SetString(PyExc_ImportError, "no symbol mt_" #f); \
    return nullptr;                                         \
  }
  SYM(linear_fwd) SYM(linear_act_fwd) SYM(linear_bwd) SYM(matmul) SYM(reduce_broadcast_grad) SYM(act_bwd)
  SYM(mse_loss) SYM(sgd_step) SYM(adam_step) SYM(rmsprop_step) SYM(conv2d_fwd) SYM(conv2d_bwd)
#undef SYM
  PyObject** to[] = {&g_f32, &g_bf16, &g_describe, &g_current, &g_stream_of};
  for (int i = 0; i < 5; ++i) {
    Py_INCREF(a[i + 1]);
    Py_XSETREF(*to[i], a[i + 1]);
  }
  Py_RETURN_NONE;
}

#define METHOD(f) {#f, (PyCFunction)(void (*)())f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(init), METHOD(linear_fwd), METHOD(linear_act_fwd), METHOD(linear_bwd), METHOD(matmul),
                         METHOD(reduce_broadcast_grad), METHOD(act_bwd), METHOD(mse_loss), METHOD(sgd_step),
                         METHOD(adam_step), METHOD(rmsprop_step), METHOD(conv2d_fwd), METHOD(conv2d_bwd),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "argument marshalling of the binding", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
  struct {
    PyObject** to;
    const char* name;
  } names[] = {{&s_is_cuda, "is_cuda"}, {&s_dtype, "dtype"},       {&s_shape, "shape"},
               {&s_stride, "stride"},   {&s_data_ptr, "data_ptr"}, {&s_numel, "numel"},
               {&s_element_size, "element_size"}};
  for (auto& e : names)
    if (!(*e.to = PyUnicode_InternFromString(e.name))) return nullptr;
  return PyModule_Create(&module);
}
