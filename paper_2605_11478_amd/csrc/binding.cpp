// The per-call part of the Python binding for encode, decode and attention:
// argument checks, output allocation and the library call, without the Python
// interpreter between them (14 us of checks around a 7 us kernel before, about
// 2 us here).  Every function returns None, having done nothing, for any
// argument that it does not recognise as valid; the Python code then goes
// through its own checks, which name what is wrong.  Once the library has been
// entered, its status is final: anything but FIBQ_OK raises FibqError.
//
// The library is reached through the entry points that bind() is given (the
// loaded library's own), so this module does not load it.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/python_arg_parser.h>

#include <ATen/ATen.h>

#include <cmath>
#include <cstdint>

#include "fibq.h"

namespace {

decltype(&fibq_encode) g_encode;
decltype(&fibq_decode) g_decode;
decltype(&fibq_attn_decode) g_attn;
decltype(&fibq_attn_workspace_bytes) g_ws;
decltype(&fibq_payload_bytes) g_payload;
PyObject* g_check;  // the package's _check(status, where): raises FibqError

using at::Tensor;

// A plain dense device tensor (no subclass, no wrapper without storage).
const Tensor* tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() ||
      t.is_conj() || t.is_neg())
    return nullptr;
  return &t;
}
bool int_arg(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  *v = PyLong_AsLongLongAndOverflow(o, &over);
  return over == 0 && *v >= -1 && *v < (1LL << 62);
}
bool shaped(const Tensor* t, at::ScalarType ty, std::initializer_list<int64_t> s) {
  if (!t || t->scalar_type() != ty || t->dim() != (int64_t)s.size() || !t->is_contiguous())
    return false;
  int64_t i = 0;
  for (int64_t v : s)
    if (t->size(i++) != v) return false;
  return true;
}
bool norm_type(const Tensor* t) {
  return t && (t->scalar_type() == at::kShort || t->scalar_type() == at::kUInt16);
}
int dtype_code(const Tensor& t) {
  switch (t.scalar_type()) {
    case at::kFloat: return FIBQ_F32;
    case at::kHalf: return FIBQ_F16;
    case at::kBFloat16: return FIBQ_BF16;
    default: return -1;
  }
}
const void* ptr(const Tensor& t) { return t.const_data_ptr(); }

// d, k, N of the call: R [d, d] and C [N, k] float32 on x's device
bool codec(const Tensor* R, const Tensor* C, int64_t d, int64_t k, int64_t N, at::Device dev,
           int64_t* P, double* rate) {
  if (d < 1 || d > 4096 || k < 1 || k > d || N < 2 || N > 65536) return false;
  if (!shaped(R, at::kFloat, {d, d}) || !shaped(C, at::kFloat, {N, k})) return false;
  if (R->device() != dev || C->device() != dev) return false;
  *P = g_payload((int)d, (int)k, (int)N);
  *rate = std::log2((double)N) / (double)k;
  return *P > 0;
}

// Raises FibqError for a status of the library.  (Not None: the Python code
// would enter the library a second time, and a HIP error is reported once.)
PyObject* raise_status(int rc, const char* where) {
  PyObject* r = PyObject_CallFunction(g_check, "is", rc, where);
  if (r) {  // (_check returned)
    Py_DECREF(r);
    PyErr_SetString(PyExc_RuntimeError, where);
  }
  return nullptr;
}

// Other Python threads run while this lives: an allocation may wait for the
// allocator, and a launch for a free place in the queue or, the first time,
// for the kernels to be loaded.  Raw pointers are taken before.
struct NoGil {
  PyThreadState* state = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(state); }
};

#define FIBQ_NONE return Py_NewRef_(Py_None)
PyObject* Py_NewRef_(PyObject* o) {
  Py_INCREF(o);
  return o;
}
PyObject* keep(PyObject* given, const Tensor& t) {
  return given != Py_None ? Py_NewRef_(given) : THPVariable_Wrap(t);
}

// encode(x, k, N, R, C, payload, norms, stream) -> (payload, norms)
PyObject* encode(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  if (!g_encode || n_args != 8) FIBQ_NONE;
  const Tensor* x = tensor(a[0]);
  int64_t k, N, st, P;
  double rate;
  if (!x || x->dim() != 2 || !int_arg(a[1], &k) || !int_arg(a[2], &N) || !int_arg(a[7], &st)) FIBQ_NONE;
  const int64_t n = x->size(0), d = x->size(1);
  const int dt = dtype_code(*x);
  if (dt < 0 || x->stride(1) != 1 || (n > 1 && x->stride(0) < d)) FIBQ_NONE;
  const Tensor *R = tensor(a[3]), *C = tensor(a[4]);
  if (!codec(R, C, d, k, N, x->device(), &P, &rate)) FIBQ_NONE;
  Tensor payload, norms;
  if (a[5] != Py_None) {
    const Tensor* t = tensor(a[5]);
    if (!shaped(t, at::kByte, {n, P}) || t->device() != x->device()) FIBQ_NONE;
    payload = *t;
  }
  if (a[6] != Py_None) {
    const Tensor* t = tensor(a[6]);
    if (!norm_type(t) || !shaped(t, t->scalar_type(), {n}) || t->device() != x->device()) FIBQ_NONE;
    norms = *t;
  }
  const auto opt = at::TensorOptions().device(x->device());
  const void* px = ptr(*x);
  const int64_t stride = x->stride(0);
  const float *pR = static_cast<const float*>(ptr(*R)), *pC = static_cast<const float*>(ptr(*C));
  int rc;
  {
    NoGil no_gil;
    if (!payload.defined()) payload = at::empty({n, P}, opt.dtype(at::kByte));
    if (!norms.defined()) norms = at::empty({n}, opt.dtype(at::kShort));
    rc = g_encode(px, dt, n, stride, (int)d, (int)k, rate, (int)N, pR, pC,
                  static_cast<uint8_t*>(payload.data_ptr()),
                  static_cast<uint16_t*>(norms.data_ptr()), reinterpret_cast<void*>(st));
  }
  if (rc != FIBQ_OK) return raise_status(rc, "fibq_encode");
  PyObject* r = PyTuple_New(2);
  if (!r) return nullptr;
  PyTuple_SET_ITEM(r, 0, keep(a[5], payload));
  PyTuple_SET_ITEM(r, 1, keep(a[6], norms));
  return r;
  END_HANDLE_TH_ERRORS
}

// decode(payload, norms, d, k, N, R, C, token_ids, out, stream) -> out
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  if (!g_decode || n_args != 10) FIBQ_NONE;
  const Tensor *p = tensor(a[0]), *h = tensor(a[1]);
  int64_t d, k, N, st, P;
  double rate;
  if (!p || !h || !int_arg(a[2], &d) || !int_arg(a[3], &k) || !int_arg(a[4], &N) ||
      !int_arg(a[9], &st) || p->dim() != 2)
    FIBQ_NONE;
  const at::Device dev = p->device();
  const Tensor *R = tensor(a[5]), *C = tensor(a[6]);
  if (!codec(R, C, d, k, N, dev, &P, &rate)) FIBQ_NONE;
  const int64_t cache = p->size(0);
  if (!shaped(p, at::kByte, {cache, P}) || !norm_type(h) || !shaped(h, h->scalar_type(), {cache}) ||
      h->device() != dev)
    FIBQ_NONE;
  const int64_t* ids = nullptr;
  int64_t n = cache;
  if (a[7] != Py_None) {
    const Tensor* t = tensor(a[7]);
    if (!t || t->dim() != 1 || !shaped(t, at::kLong, {t->size(0)}) || t->device() != dev) FIBQ_NONE;
    n = t->size(0);
    ids = static_cast<const int64_t*>(ptr(*t));
  }
  Tensor out;
  if (a[8] != Py_None) {
    const Tensor* t = tensor(a[8]);
    if (!shaped(t, at::kFloat, {n, d}) || t->device() != dev) FIBQ_NONE;
    out = *t;
  }
  const uint8_t* pp = static_cast<const uint8_t*>(ptr(*p));
  const uint16_t* ph = static_cast<const uint16_t*>(ptr(*h));
  const float *pR = static_cast<const float*>(ptr(*R)), *pC = static_cast<const float*>(ptr(*C));
  int rc;
  {
    NoGil no_gil;
    if (!out.defined()) out = at::empty({n, d}, at::TensorOptions().device(dev).dtype(at::kFloat));
    rc = g_decode(pp, ph, ids, n, cache, (int)d, (int)k, rate, (int)N, pR, pC,
                  static_cast<float*>(out.data_ptr()), reinterpret_cast<void*>(st));
  }
  if (rc != FIBQ_OK) return raise_status(rc, "fibq_decode");
  return keep(a[8], out);
  END_HANDLE_TH_ERRORS
}

// attn(q, k_payload, k_norms, v_payload, v_norms, T, k, N, R, C, scale,
//      workspace, out, stream) -> out
PyObject* attn(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  if (!g_attn || n_args != 14) FIBQ_NONE;
  const Tensor *q = tensor(a[0]), *kp = tensor(a[1]), *kn = tensor(a[2]), *vp = tensor(a[3]),
               *vn = tensor(a[4]);
  int64_t T, k, N, st, P;
  double rate;
  if (!q || !kp || q->dim() != 3 || kp->dim() != 3 || !q->is_contiguous() || !int_arg(a[5], &T) ||
      !int_arg(a[6], &k) || !int_arg(a[7], &N) || !PyFloat_CheckExact(a[10]) || !int_arg(a[13], &st))
    FIBQ_NONE;
  const int64_t ng = q->size(0), G = q->size(1), d = q->size(2), Ts = kp->size(1);
  const at::Device dev = q->device();
  const int dt = dtype_code(*q);
  const Tensor *R = tensor(a[8]), *C = tensor(a[9]);
  if (dt < 0 || G < 1 || G > 16 || T < 0 || T > Ts || !codec(R, C, d, k, N, dev, &P, &rate)) FIBQ_NONE;
  if (!shaped(kp, at::kByte, {ng, Ts, P}) || !shaped(vp, at::kByte, {ng, Ts, P}) ||
      !norm_type(kn) || !norm_type(vn) || !shaped(kn, kn->scalar_type(), {ng, Ts}) ||
      !shaped(vn, vn->scalar_type(), {ng, Ts}))
    FIBQ_NONE;
  if (kp->device() != dev || vp->device() != dev || kn->device() != dev || vn->device() != dev)
    FIBQ_NONE;
  Tensor out, ws;
  const auto opt = at::TensorOptions().device(dev);
  const int64_t need = (int64_t)g_ws(ng, (int)G, T, (int)d, (int)k, (int)N);
  if (a[11] != Py_None) {
    const Tensor* t = tensor(a[11]);
    if (!t || t->dim() != 1 || !shaped(t, at::kByte, {t->size(0)}) || t->size(0) < need ||
        t->device() != dev)
      FIBQ_NONE;
    ws = *t;
  }
  if (a[12] != Py_None) {
    const Tensor* t = tensor(a[12]);
    if (!shaped(t, at::kFloat, {ng, G, d}) || t->device() != dev) FIBQ_NONE;
    out = *t;
  }
  const void* pq = ptr(*q);
  const uint8_t *pkp = static_cast<const uint8_t*>(ptr(*kp)), *pvp = static_cast<const uint8_t*>(ptr(*vp));
  const uint16_t *pkn = static_cast<const uint16_t*>(ptr(*kn)), *pvn = static_cast<const uint16_t*>(ptr(*vn));
  const float *pR = static_cast<const float*>(ptr(*R)), *pC = static_cast<const float*>(ptr(*C));
  const float scale = (float)PyFloat_AS_DOUBLE(a[10]);
  int rc;
  {
    NoGil no_gil;
    if (!ws.defined()) ws = at::empty({need > 1 ? need : 1}, opt.dtype(at::kByte));
    if (!out.defined()) out = at::empty({ng, G, d}, opt.dtype(at::kFloat));
    rc = g_attn(pq, dt, pkp, pkn, pvp, pvn, ng, (int)G, T, Ts, (int)d, (int)k, rate, (int)N, pR, pC,
                scale, static_cast<float*>(out.data_ptr()), ws.data_ptr(), (size_t)ws.numel(),
                reinterpret_cast<void*>(st));
  }
  if (rc != FIBQ_OK) return raise_status(rc, "fibq_attn_decode");
  return keep(a[12], out);
  END_HANDLE_TH_ERRORS
}

// bind(encode, decode, attn_decode, attn_workspace_bytes, payload_bytes,
// check): addresses of the loaded library's entry points, and _check
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  if (n_args != 6) {
    PyErr_SetString(PyExc_TypeError, "bind takes five addresses and a callable");
    return nullptr;
  }
  void* p[5];
  for (int i = 0; i < 5; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred()) return nullptr;
  }
  g_encode = reinterpret_cast<decltype(g_encode)>(p[0]);
  g_decode = reinterpret_cast<decltype(g_decode)>(p[1]);
  g_attn = reinterpret_cast<decltype(g_attn)>(p[2]);
  g_ws = reinterpret_cast<decltype(g_ws)>(p[3]);
  g_payload = reinterpret_cast<decltype(g_payload)>(p[4]);
  Py_INCREF(a[5]);
  Py_XSETREF(g_check, a[5]);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void*)bind, METH_FASTCALL, nullptr},
    {"encode", (PyCFunction)(void*)encode, METH_FASTCALL, nullptr},
    {"decode", (PyCFunction)(void*)decode, METH_FASTCALL, nullptr},
    {"attn", (PyCFunction)(void*)attn, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr,
                      nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
