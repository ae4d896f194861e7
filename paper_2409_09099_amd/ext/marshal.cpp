// Native argument marshalling of the Python binding: the calls of binding.py that a training or inference loop makes for every layer,
// from Python objects to the C ABI of include/sste.h without Python code in between.
//
// Why: a call through ctypes costs 8...10 us of host time (a dozen attribute and method calls on each tensor, the stream lookup, the
// conversion of up to 19 arguments), more than the kernels of a small layer or of a decode batch run; through this module it costs
// 2...4 us, nearly all of it the kernel launches.
//
// Every function takes the arguments of the function of the same name in binding.py.  It handles the ordinary case (tensors on the GPU
// with the right element size and layout) and hands everything else, errors included, to that Python function, which stays the definition
// of the argument rules.  Addresses of the library's entry points and the Python functions arrive through bind().
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cstdint>

#include "../../include/sste.h"

namespace {

struct Entry {                     // one marshalled function: its Python definition (called when the fast path declines)
  PyObject* python = nullptr;
};
enum Fn { PROJECT_PACK, SGD_PROJECT_PACK, LINEAR_FWD, LINEAR_FWD_EX, LINEAR_FWD_ACT, LINEAR_DGRAD, LINEAR_DGRAD_ACT, LINEAR_WGRAD, CAST_FP8, N_FN };
Entry g_fn[N_FN];
PyObject* g_error = nullptr;       // SsteError
bool g_bound = false;

decltype(&sste_project_pack_gamma) p_project_pack_gamma;
decltype(&sste_sgd_project_pack) p_sgd_project_pack;
decltype(&sste_linear_fwd_ex) p_linear_fwd_ex;
decltype(&sste_linear_fwd_act) p_linear_fwd_act;
decltype(&sste_linear_dgrad_act) p_linear_dgrad_act;
decltype(&sste_linear_wgrad_at) p_linear_wgrad_at;
decltype(&sste_wgrad_workspace_bytes) p_wgrad_workspace_bytes;
decltype(&sste_cast_fp8) p_cast_fp8;
decltype(&sste_project_pack_batch) p_project_pack_batch;
decltype(&sste_sgd_project_pack_batch) p_sgd_project_pack_batch;
decltype(&sste_last_error) p_last_error;

// ---- arguments ------------------------------------------------------------------------------------------
// Positional and keyword arguments into slots; false if a keyword is unknown, given twice, or there are too many positions (the
// Python function then reports it).
template <int N>
bool collect(PyObject* (&names)[N], PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames, PyObject* (&out)[N]) {
  if (nargs > N) return false;
  for (int i = 0; i < N; i++) out[i] = i < nargs ? args[i] : nullptr;
  const Py_ssize_t nk = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
  for (Py_ssize_t k = 0; k < nk; k++) {
    PyObject* name = PyTuple_GET_ITEM(kwnames, k);
    int at = -1;
    for (int i = 0; i < N && at < 0; i++)
      if (names[i] == name) at = i;                                     // interned on both sides: pointers are equal
    for (int i = 0; i < N && at < 0; i++)
      if (PyUnicode_Compare(names[i], name) == 0) at = i;
    if (at < 0 || out[at]) return false;
    out[at] = args[nargs + k];
  }
  return true;
}
template <int N>
void intern(PyObject* (&names)[N], const char* const (&text)[N]) {
  for (int i = 0; i < N; i++) names[i] = PyUnicode_InternFromString(text[i]);
}

struct Args {
  bool ok = true;                  // stays true while everything read so far is of the ordinary kind
  static bool given(PyObject* o) { return o && o != Py_None; }

  double number(PyObject* o, double otherwise) {
    if (!o) return otherwise;
    if (PyFloat_Check(o)) return PyFloat_AS_DOUBLE(o);
    if (!PyLong_Check(o)) return ok = false, 0.0;
    const double v = PyLong_AsDouble(o);
    if (PyErr_Occurred()) PyErr_Clear(), ok = false;
    return v;
  }
  int64_t integer(PyObject* o, int64_t otherwise) {
    if (!o) return otherwise;
    if (!PyLong_Check(o)) return ok = false, 0;
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) PyErr_Clear(), ok = false;
    return v;
  }
  int small(PyObject* o, int otherwise) {
    const int64_t v = integer(o, otherwise);
    if (v < -0x7FFFFFFF || v > 0x7FFFFFFF) ok = false;
    return (int)v;
  }
  uint64_t word(PyObject* o) {                                          // 64 bits of any Python integer
    if (!o || !PyLong_Check(o)) return ok = false, 0;
    const uint64_t v = PyLong_AsUnsignedLongLongMask(o);
    if (PyErr_Occurred()) PyErr_Clear(), ok = false;
    return v;
  }
  const at::Tensor* tensor(PyObject* o) {
    if (!given(o)) return nullptr;
    if (!THPVariable_CheckExact(o)) return ok = false, nullptr;           // Tensor or Parameter; subclasses keep the Python route
    return &THPVariable_Unpack(o);
  }
  const at::Tensor* needed(PyObject* o) {
    const at::Tensor* t = tensor(o);
    if (!t) ok = false;
    return t;
  }
};

// a 2-D GPU tensor with unit inner stride: rows, columns, leading dimension
struct Matrix {
  void* p = nullptr;
  int64_t rows = 0, cols = 0, ld = 0;
};
Matrix matrix(Args& a, const at::Tensor* t, int itemsize) {
  Matrix m;
  if (!a.ok || !t) return m;
  if (t->dim() != 2 || !t->is_cuda() || (int)t->element_size() != itemsize || (t->size(1) > 1 && t->stride(1) != 1)) return a.ok = false, m;
  m.rows = t->size(0);
  m.cols = t->size(1);
  m.ld = m.rows >= 1 ? std::max(m.cols, t->stride(0)) : m.cols;
  m.p = t->numel() > 0 ? t->data_ptr() : nullptr;
  return m;
}
void* address(const at::Tensor* t) { return t && t->numel() > 0 ? t->data_ptr() : nullptr; }
int item(int dtype) { return dtype == SSTE_F8E4M3 || dtype == SSTE_F8E5M2 ? 1 : 2; }
void* stream_of(const at::Tensor& t) { return (void*)c10::hip::getCurrentHIPStream(t.device().index()).stream(); }
at::Tensor make(const at::Tensor& like, int64_t rows, int64_t cols, at::ScalarType type) {
  return at::empty({rows, cols}, at::TensorOptions().dtype(type).device(like.device()));
}
PyObject* keep(PyObject* o) {
  PyObject* r = o ? o : Py_None;
  Py_INCREF(r);
  return r;
}
// the caller's tensor if there is one, else the one made here
PyObject* result(PyObject* given, const at::Tensor& made) { return Args::given(given) ? keep(given) : THPVariable_Wrap(made); }

PyObject* fail(int status) {
  PyObject* e = PyObject_CallFunction(g_error, "is", status, p_last_error());
  if (e) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  }
  return nullptr;
}
PyObject* decline(Fn f, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  if (!g_fn[f].python) {
    PyErr_SetString(PyExc_RuntimeError, "bind() has not been called");
    return nullptr;
  }
  return PyObject_Vectorcall(g_fn[f].python, args, (size_t)nargs, kwnames);
}

#define CALL(status, expr)    \
  int status;                 \
  Py_BEGIN_ALLOW_THREADS;     \
  status = (expr);            \
  Py_END_ALLOW_THREADS

// ---- the calls ------------------------------------------------------------------------------------------
PyObject* n_pp[8];
PyObject* project_pack(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  PyObject* o[8];  // W beta val_dtype val_scale vals meta amax_out gamma
  Args a;
  if (!g_bound || !collect(n_pp, args, nargs, kwnames, o)) return decline(PROJECT_PACK, args, nargs, kwnames);
  const at::Tensor* W = a.needed(o[0]);
  const Matrix w = matrix(a, W, 2);
  if (!o[1]) a.ok = false;
  const double beta = a.number(o[1], 0), scale = a.number(o[3], 1.0), gamma = a.number(o[7], 0.0);
  const int dt = a.small(o[2], SSTE_BF16);
  const at::Tensor *vals = a.tensor(o[4]), *meta = a.tensor(o[5]), *amax = a.tensor(o[6]);
  if (!a.ok || !vals || !meta) return decline(PROJECT_PACK, args, nargs, kwnames);
  void* s = stream_of(*W);
  CALL(st, p_project_pack_gamma(w.p, w.rows, w.cols, w.ld, (float)beta, (float)gamma, dt, (float)scale, address(vals), address(meta), (float*)address(amax), s));
  if (st) return fail(st);
  return PyTuple_Pack(2, o[4], o[5]);
}

PyObject* n_sgd[8];
PyObject* sgd_project_pack(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  PyObject* o[8];  // W G alpha beta val_dtype val_scale vals meta
  Args a;
  if (!g_bound || !collect(n_sgd, args, nargs, kwnames, o)) return decline(SGD_PROJECT_PACK, args, nargs, kwnames);
  const at::Tensor *W = a.needed(o[0]), *G = a.needed(o[1]);
  const bool f32 = W && W->scalar_type() == at::kFloat;
  const Matrix w = matrix(a, W, f32 ? 4 : 2), g = matrix(a, G, 4);
  if (!o[2] || !o[3] || !a.ok || G->scalar_type() != at::kFloat || g.rows != w.rows || g.cols != w.cols) return decline(SGD_PROJECT_PACK, args, nargs, kwnames);
  const double alpha = a.number(o[2], 0), beta = a.number(o[3], 0), scale = a.number(o[5], 1.0);
  const int dt = a.small(o[4], SSTE_BF16);
  const at::Tensor *vals = a.tensor(o[6]), *meta = a.tensor(o[7]);
  if (!a.ok || !vals || !meta) return decline(SGD_PROJECT_PACK, args, nargs, kwnames);
  void* s = stream_of(*W);
  CALL(st, p_sgd_project_pack(w.p, f32 ? SSTE_F32 : SSTE_BF16, w.rows, w.cols, w.ld, (const float*)g.p, g.ld, (float)alpha, (float)beta, dt, (float)scale,
                              address(vals), address(meta), s));
  if (st) return fail(st);
  return PyTuple_Pack(2, o[6], o[7]);
}

PyObject* n_fwd[8];
PyObject* linear_fwd(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  PyObject* o[8];  // X vals meta O dtype x_scale w_scale Z
  Args a;
  if (!g_bound || !collect(n_fwd, args, nargs, kwnames, o)) return decline(LINEAR_FWD, args, nargs, kwnames);
  const at::Tensor *X = a.needed(o[0]), *vals = a.needed(o[1]), *meta = a.needed(o[2]), *Z = a.tensor(o[7]);
  if (!o[3]) a.ok = false;
  const int64_t O = a.integer(o[3], 0);
  const int dt = a.small(o[4], SSTE_BF16);
  const double xs = a.number(o[5], 1.0), ws = a.number(o[6], 1.0);
  const Matrix x = matrix(a, X, item(dt));
  if (!a.ok || O < 0) return decline(LINEAR_FWD, args, nargs, kwnames);
  at::Tensor made;
  if (!Z) made = make(*X, x.rows, O, at::kBFloat16);
  const Matrix z = matrix(a, Z ? Z : &made, 2);
  if (!a.ok) return decline(LINEAR_FWD, args, nargs, kwnames);
  void* s = stream_of(*X);
  CALL(st, p_linear_fwd_ex(x.p, x.rows, x.cols, x.ld, dt, (float)xs, address(vals), address(meta), O, (float)ws, z.p, z.ld, SSTE_BF16, 1.0f, nullptr, s));
  if (st) return fail(st);
  return result(o[7], made);
}

PyObject* n_fwd_ex[11];
PyObject* linear_fwd_ex(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  PyObject* o[11];  // X vals meta O dtype x_scale w_scale z_dtype z_scale Z amax_out
  Args a;
  if (!g_bound || !collect(n_fwd_ex, args, nargs, kwnames, o)) return decline(LINEAR_FWD_EX, args, nargs, kwnames);
  const at::Tensor *X = a.needed(o[0]), *vals = a.needed(o[1]), *meta = a.needed(o[2]), *Z = a.tensor(o[9]), *amax = a.tensor(o[10]);
  if (!o[3]) a.ok = false;
  const int64_t O = a.integer(o[3], 0);
  const int dt = a.small(o[4], SSTE_BF16), zdt = a.small(o[7], SSTE_BF16);
  const double xs = a.number(o[5], 1.0), ws = a.number(o[6], 1.0), zs = a.number(o[8], 1.0);
  const Matrix x = matrix(a, X, item(dt));
  if (!a.ok || !Z || (!amax && zdt == SSTE_F8E4M3)) return decline(LINEAR_FWD_EX, args, nargs, kwnames);
  const Matrix z = matrix(a, Z, item(zdt));
  if (!a.ok) return decline(LINEAR_FWD_EX, args, nargs, kwnames);
  void* s = stream_of(*X);
  CALL(st, p_linear_fwd_ex(x.p, x.rows, x.cols, x.ld, dt, (float)xs, address(vals), address(meta), O, (float)ws, z.p, z.ld, zdt, (float)zs, (float*)address(amax), s));
  if (st) return fail(st);
  return PyTuple_Pack(2, o[9], amax ? o[10] : Py_None);
}

PyObject* n_fwd_act[14];
PyObject* linear_fwd_act(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  PyObject* o[14];  // X vals meta O dtype x_scale w_scale act a_dtype a_scale H A amax_out store_pre
  Args a;
  if (!g_bound || !collect(n_fwd_act, args, nargs, kwnames, o)) return decline(LINEAR_FWD_ACT, args, nargs, kwnames);
  const at::Tensor *X = a.needed(o[0]), *vals = a.needed(o[1]), *meta = a.needed(o[2]), *H = a.tensor(o[10]), *A = a.tensor(o[11]), *amax = a.tensor(o[12]);
  if (!o[3]) a.ok = false;
  const int64_t O = a.integer(o[3], 0);
  const int dt = a.small(o[4], SSTE_BF16), act = a.small(o[7], SSTE_ACT_GELU_TANH), adt = a.small(o[8], SSTE_BF16);
  const double xs = a.number(o[5], 1.0), ws = a.number(o[6], 1.0), as = a.number(o[9], 1.0);
  const bool no_pre = o[13] == Py_False;
  if (o[13] && o[13] != Py_True && o[13] != Py_False) a.ok = false;
  const Matrix x = matrix(a, X, item(dt));
  if (!a.ok || !A || (!H && !no_pre) || (!amax && adt == SSTE_F8E4M3)) return decline(LINEAR_FWD_ACT, args, nargs, kwnames);
  const Matrix h = matrix(a, H, 2), am = matrix(a, A, item(adt));
  if (!a.ok) return decline(LINEAR_FWD_ACT, args, nargs, kwnames);
  void* s = stream_of(*X);
  CALL(st, p_linear_fwd_act(x.p, x.rows, x.cols, x.ld, dt, (float)xs, address(vals), address(meta), O, (float)ws, act, h.p, H ? h.ld : 0, am.p, am.ld, adt, (float)as,
                            (float*)address(amax), s));
  if (st) return fail(st);
  return PyTuple_Pack(3, H ? o[10] : Py_None, o[11], amax ? o[12] : Py_None);
}

// grad_X with and without the activation's derivative
PyObject* dgrad(Fn f, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames, PyObject* oy, PyObject* ov, PyObject* om, PyObject* oi, PyObject* oh, PyObject* odt,
                PyObject* os, PyObject* ow, PyObject* oact, PyObject* ox) {
  Args a;
  const at::Tensor *dY = a.needed(oy), *vals = a.needed(ov), *meta = a.needed(om), *H = f == LINEAR_DGRAD_ACT ? a.needed(oh) : nullptr, *dX = a.tensor(ox);
  if (!oi) a.ok = false;
  const int64_t I = a.integer(oi, 0);
  const int dt = a.small(odt, SSTE_BF16), act = f == LINEAR_DGRAD_ACT ? a.small(oact, SSTE_ACT_GELU_TANH) : SSTE_ACT_NONE;
  const double dys = a.number(os, 1.0), ws = a.number(ow, 1.0);
  const Matrix y = matrix(a, dY, item(dt));
  if (!a.ok || I < 0) return decline(f, args, nargs, kwnames);
  at::Tensor made;
  if (!dX) made = make(*dY, y.rows, I, at::kBFloat16);
  const Matrix x = matrix(a, dX ? dX : &made, 2), h = matrix(a, H, 2);
  if (!a.ok) return decline(f, args, nargs, kwnames);
  void* s = stream_of(*dY);
  CALL(st, p_linear_dgrad_act(y.p, y.rows, y.cols, y.ld, dt, (float)dys, address(vals), address(meta), I, (float)ws, act, h.p, h.ld, x.p, x.ld, s));
  if (st) return fail(st);
  return result(ox, made);
}
PyObject* n_dgrad[8];
PyObject* linear_dgrad(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  PyObject* o[8];  // dY vals meta I dtype dy_scale w_scale dX
  if (!g_bound || !collect(n_dgrad, args, nargs, kwnames, o)) return decline(LINEAR_DGRAD, args, nargs, kwnames);
  return dgrad(LINEAR_DGRAD, args, nargs, kwnames, o[0], o[1], o[2], o[3], nullptr, o[4], o[5], o[6], nullptr, o[7]);
}
PyObject* n_dgrad_act[10];
PyObject* linear_dgrad_act(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  PyObject* o[10];  // dY vals meta I H dtype dy_scale w_scale act dX
  if (!g_bound || !collect(n_dgrad_act, args, nargs, kwnames, o)) return decline(LINEAR_DGRAD_ACT, args, nargs, kwnames);
  return dgrad(LINEAR_DGRAD_ACT, args, nargs, kwnames, o[0], o[1], o[2], o[3], o[4], o[5], o[6], o[7], o[8], o[9]);
}

PyObject* n_wgrad[11];
PyObject* linear_wgrad(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  PyObject* o[11];  // dY X seed offset dtype dy_scale x_scale dW accumulate workspace first_token
  Args a;
  if (!g_bound || !collect(n_wgrad, args, nargs, kwnames, o)) return decline(LINEAR_WGRAD, args, nargs, kwnames);
  const at::Tensor *dY = a.needed(o[0]), *X = a.needed(o[1]), *dW = a.tensor(o[7]), *ws = a.tensor(o[9]);
  const uint64_t seed = a.word(o[2]), offset = a.word(o[3]);
  const int dt = a.small(o[4], SSTE_BF16);
  const double dys = a.number(o[5], 1.0), xs = a.number(o[6], 1.0);
  const int64_t first = a.integer(o[10], 0);
  const int acc = !o[8] || o[8] == Py_False ? 0 : 1;
  if (o[8] && o[8] != Py_True && o[8] != Py_False) a.ok = false;
  const Matrix y = matrix(a, dY, item(dt)), x = matrix(a, X, item(dt));
  if (!a.ok || y.rows != x.rows || (acc && !dW)) return decline(LINEAR_WGRAD, args, nargs, kwnames);
  at::Tensor made, scratch;
  if (!dW) made = make(*X, y.cols, x.cols, at::kFloat);
  const Matrix w = matrix(a, dW ? dW : &made, 4);
  if (!a.ok) return decline(LINEAR_WGRAD, args, nargs, kwnames);
  if (!ws) {
    const size_t need = p_wgrad_workspace_bytes(y.rows, y.cols, x.cols, dt);
    if (need > 0) {
      scratch = at::empty({(int64_t)need}, at::TensorOptions().dtype(at::kByte).device(X->device()));
      ws = &scratch;
    }
  }
  const size_t ws_bytes = ws ? (size_t)ws->numel() * ws->element_size() : 0;
  void* s = stream_of(*X);
  CALL(st, p_linear_wgrad_at(y.p, y.rows, y.cols, y.ld, dt, (float)dys, x.p, x.cols, x.ld, (float)xs, seed, offset, first, (float*)w.p, w.ld, acc, address(ws), ws_bytes, s));
  if (st) return fail(st);
  return result(o[7], made);
}

PyObject* n_cast[6];
PyObject* cast_fp8(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  PyObject* o[6];  // X scale out_dtype Q amax_out store
  Args a;
  if (!g_bound || !collect(n_cast, args, nargs, kwnames, o)) return decline(CAST_FP8, args, nargs, kwnames);
  const at::Tensor *X = a.needed(o[0]), *Q = a.tensor(o[3]), *amax = a.tensor(o[4]);
  if (!o[1] || (o[5] && o[5] != Py_True)) a.ok = false;
  const double scale = a.number(o[1], 1.0);
  const int dt = a.small(o[2], SSTE_F8E4M3);
  const Matrix x = matrix(a, X, 2);
  if (!a.ok || !Q || !amax) return decline(CAST_FP8, args, nargs, kwnames);
  const Matrix q = matrix(a, Q, 1);
  if (!a.ok) return decline(CAST_FP8, args, nargs, kwnames);
  void* s = stream_of(*X);
  CALL(st, p_cast_fp8(x.p, x.rows, x.cols, x.ld, dt, (float)scale, q.p, q.ld, (float*)address(amax), s));
  if (st) return fail(st);
  return PyTuple_Pack(2, o[3], o[4]);
}

// launches of the prepared multi-tensor tables: (table tensor, n_items, total_blocks, val_dtype) and (..., w_dtype, val_dtype, alpha)
PyObject* pack_batch_launch(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  Args a;
  if (nargs != 4 || !g_bound) return PyErr_SetString(PyExc_TypeError, "pack_batch_launch(table, n_items, total_blocks, val_dtype)"), nullptr;
  const at::Tensor* t = a.needed(args[0]);
  const int n = a.small(args[1], 0), dt = a.small(args[3], 0);
  const int64_t total = a.integer(args[2], 0);
  if (!a.ok) return PyErr_SetString(PyExc_TypeError, "pack_batch_launch: a tensor and three integers"), nullptr;
  void* s = stream_of(*t);
  CALL(st, p_project_pack_batch(address(t), n, total, dt, s));
  if (st) return fail(st);
  Py_RETURN_NONE;
}
PyObject* update_batch_launch(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  Args a;
  if (nargs != 6 || !g_bound) return PyErr_SetString(PyExc_TypeError, "update_batch_launch(table, n_items, total_blocks, w_dtype, val_dtype, alpha)"), nullptr;
  const at::Tensor* t = a.needed(args[0]);
  const int n = a.small(args[1], 0), wdt = a.small(args[3], 0), dt = a.small(args[4], 0);
  const int64_t total = a.integer(args[2], 0);
  const double alpha = a.number(args[5], 0);
  if (!a.ok) return PyErr_SetString(PyExc_TypeError, "update_batch_launch: a tensor, four integers and a number"), nullptr;
  void* s = stream_of(*t);
  CALL(st, p_sgd_project_pack_batch(address(t), n, total, wdt, dt, (float)alpha, s));
  if (st) return fail(st);
  Py_RETURN_NONE;
}

// bind(addresses: dict of entry point name -> address, python: dict of function name -> Python function, error class)
template <class F>
bool take(PyObject* d, const char* name, F& f) {
  PyObject* v = PyDict_GetItemString(d, name);
  if (!v) return PyErr_Format(PyExc_KeyError, "%s", name), false;
  f = (F)PyLong_AsVoidPtr(v);
  return !PyErr_Occurred();
}
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *addr, *fns, *err;
  if (!PyArg_ParseTuple(args, "O!O!O", &PyDict_Type, &addr, &PyDict_Type, &fns, &err)) return nullptr;
  const char* const names[N_FN] = {"project_pack", "sgd_project_pack", "linear_fwd", "linear_fwd_ex", "linear_fwd_act", "linear_dgrad", "linear_dgrad_act", "linear_wgrad", "cast_fp8"};
  for (int i = 0; i < N_FN; i++) {
    PyObject* f = PyDict_GetItemString(fns, names[i]);
    if (!f) return PyErr_Format(PyExc_KeyError, "%s", names[i]);
    Py_INCREF(f);
    Py_XSETREF(g_fn[i].python, f);
  }
  Py_INCREF(err);
  Py_XSETREF(g_error, err);
  if (PyDict_Size(addr) > 0) {
    if (!(take(addr, "sste_project_pack_gamma", p_project_pack_gamma) && take(addr, "sste_sgd_project_pack", p_sgd_project_pack) &&
          take(addr, "sste_linear_fwd_ex", p_linear_fwd_ex) && take(addr, "sste_linear_fwd_act", p_linear_fwd_act) &&
          take(addr, "sste_linear_dgrad_act", p_linear_dgrad_act) && take(addr, "sste_linear_wgrad_at", p_linear_wgrad_at) &&
          take(addr, "sste_wgrad_workspace_bytes", p_wgrad_workspace_bytes) && take(addr, "sste_cast_fp8", p_cast_fp8) &&
          take(addr, "sste_project_pack_batch", p_project_pack_batch) && take(addr, "sste_sgd_project_pack_batch", p_sgd_project_pack_batch) &&
          take(addr, "sste_last_error", p_last_error)))
      return nullptr;
    g_bound = true;
  }
  Py_RETURN_NONE;
}

// No C++ exception may leave an entry (a result that does not fit the memory, a tensor without storage): it becomes the Python error
// that the ctypes route raises.
using FastCall = PyObject* (*)(PyObject*, PyObject* const*, Py_ssize_t, PyObject*);
template <FastCall F>
PyObject* guarded(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  HANDLE_TH_ERRORS
  return F(self, args, nargs, kwnames);
  END_HANDLE_TH_ERRORS
}
using PlainCall = PyObject* (*)(PyObject*, PyObject* const*, Py_ssize_t);
template <PlainCall F>
PyObject* guarded(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  return F(self, args, nargs);
  END_HANDLE_TH_ERRORS
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))(FastCall)guarded<name>, METH_FASTCALL | METH_KEYWORDS, nullptr}
PyObject* document(PyObject*, PyObject* docs);
PyMethodDef methods[] = {
  FAST(project_pack), FAST(sgd_project_pack), FAST(linear_fwd), FAST(linear_fwd_ex), FAST(linear_fwd_act), FAST(linear_dgrad), FAST(linear_dgrad_act),
  FAST(linear_wgrad), FAST(cast_fp8),
  {"pack_batch_launch", (PyCFunction)(void (*)(void))(PlainCall)guarded<pack_batch_launch>, METH_FASTCALL, "Launches a prepared sste_project_pack_batch table."},
  {"update_batch_launch", (PyCFunction)(void (*)(void))(PlainCall)guarded<update_batch_launch>, METH_FASTCALL, "Launches a prepared sste_sgd_project_pack_batch table."},
  {"bind", bind, METH_VARARGS, "bind(addresses, functions, error)"},
  {"document", document, METH_O, "document(dict of function name -> signature and documentation)"},
  {nullptr, nullptr, 0, nullptr}};
// The functions' signatures and documentation, from the Python definitions.  The dict is kept: a method table holds plain pointers.
PyObject* document(PyObject*, PyObject* docs) {
  static PyObject* kept = nullptr;
  if (!PyDict_Check(docs)) return PyErr_SetString(PyExc_TypeError, "document: a dict"), nullptr;
  PyObject* d = PyDict_Copy(docs);
  if (!d) return nullptr;
  for (PyMethodDef* m = methods; m->ml_name; m++)
    if (PyObject* text = PyDict_GetItemString(d, m->ml_name)) {
      const char* p = PyUnicode_AsUTF8(text);
      if (!p) return Py_DECREF(d), nullptr;
      m->ml_doc = p;
    }
  Py_XSETREF(kept, d);
  Py_RETURN_NONE;
}
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "Native argument marshalling of the binding.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
  intern(n_pp, {"W", "beta", "val_dtype", "val_scale", "vals", "meta", "amax_out", "gamma"});
  intern(n_sgd, {"W", "G", "alpha", "beta", "val_dtype", "val_scale", "vals", "meta"});
  intern(n_fwd, {"X", "vals", "meta", "O", "dtype", "x_scale", "w_scale", "Z"});
  intern(n_fwd_ex, {"X", "vals", "meta", "O", "dtype", "x_scale", "w_scale", "z_dtype", "z_scale", "Z", "amax_out"});
  intern(n_fwd_act, {"X", "vals", "meta", "O", "dtype", "x_scale", "w_scale", "act", "a_dtype", "a_scale", "H", "A", "amax_out", "store_pre"});
  intern(n_dgrad, {"dY", "vals", "meta", "I", "dtype", "dy_scale", "w_scale", "dX"});
  intern(n_dgrad_act, {"dY", "vals", "meta", "I", "H", "dtype", "dy_scale", "w_scale", "act", "dX"});
  intern(n_wgrad, {"dY", "X", "seed", "offset", "dtype", "dy_scale", "x_scale", "dW", "accumulate", "workspace", "first_token"});
  intern(n_cast, {"X", "scale", "out_dtype", "Q", "amax_out", "store"});
  return PyModule_Create(&module);
}
