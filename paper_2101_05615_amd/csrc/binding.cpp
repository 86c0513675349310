// The calls that a program repeats, from Python straight into the C ABI: a CPython extension module.
//
// Marshalling a call of the GEMM in Python -- checks of shapes, types and strides, a parameter struct, a ctypes call with ten
// arguments -- took 4.1 us of its 7.8, beside 3.7 for the launch itself; through here the call takes 5.1, of which the stream (two
// calls into torch), the new output tensor and the marshalling are 1.4.  Anything out of the ordinary (a check that fails, an
// argument of another type, an error code) makes the function return None, and the caller in qgemm.py goes through its own
// checks, which name the error.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/autograd/python_variable.h>

#include <limits.h>

#include "qgemm.h"

namespace {

PyObject* g_stream_of = nullptr;  // device -> raw handle of its current stream
PyObject* g_device = nullptr;     // () -> current device
PyObject* g_name_fast = nullptr;  // "_fast"
PyObject* g_error = nullptr;      // exception for an error code: (code, name of the call)

// A C++ exception of the tensor library ends here: the slow path meets it again and reports it its own way
#define QG_OR_SLOW(...)     \
  try {                     \
    __VA_ARGS__             \
  } catch (...) {           \
    PyErr_Clear();          \
    Py_RETURN_NONE;         \
  }

bool slow() {  // an error of the CPython API: as above
  PyErr_Clear();
  return false;
}

struct reference {  // a new reference, given up on every way out that does not return it
  PyObject* o;
  ~reference() { Py_XDECREF(o); }
  PyObject* give() {
    PyObject* const r = o;
    o = nullptr;
    return r;
  }
};

bool stream(void** out) {
  PyObject* const dev = PyObject_CallNoArgs(g_device);
  if (!dev) return slow();
  PyObject* const s = PyObject_CallOneArg(g_stream_of, dev);
  Py_DECREF(dev);
  if (!s) return slow();
  *out = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  return !PyErr_Occurred() || slow();
}

bool integer(PyObject* o, int* out) {
  if (!PyIndex_Check(o)) return false;
  const long v = PyLong_AsLong(o);
  if (v == -1 && PyErr_Occurred()) return slow();
  *out = (int)v;
  return true;
}

// plain tensors only: what a subclass makes of its methods is for the slow path
const at::Tensor* tensor(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

struct packed {
  const qg_packed_b* handle;
  int K, N;
};
bool descriptor(PyObject* o, packed* out) {  // (address, K, N); None once it is closed
  PyObject* const t = PyObject_GetAttr(o, g_name_fast);
  if (!t) return slow();
  const bool ok = PyTuple_CheckExact(t) && PyTuple_GET_SIZE(t) == 3;
  if (ok) {
    out->handle = static_cast<const qg_packed_b*>(PyLong_AsVoidPtr(PyTuple_GET_ITEM(t, 0)));
    out->K = (int)PyLong_AsLong(PyTuple_GET_ITEM(t, 1));
    out->N = (int)PyLong_AsLong(PyTuple_GET_ITEM(t, 2));
  }
  Py_DECREF(t);
  if (PyErr_Occurred()) return slow();
  return ok && out->handle;
}

// bias and scales of an output pipeline
bool columns(PyObject* bias, PyObject* scales, const int32_t** b, const float** s, int* n_scales) {
  *b = nullptr;
  if (bias != Py_None) {
    const at::Tensor* const t = tensor(bias);
    if (!t || !t->is_cuda() || t->scalar_type() != at::kInt || !t->is_contiguous()) return false;
    *b = static_cast<const int32_t*>(t->data_ptr());
  }
  const at::Tensor* const t = tensor(scales);
  if (!t || !t->is_cuda() || t->scalar_type() != at::kFloat || !t->is_contiguous()) return false;
  *s = static_cast<const float*>(t->data_ptr());
  *n_scales = (int)t->numel();
  return true;
}

bool matrix(const at::Tensor* t, at::ScalarType type) {
  return t && t->is_cuda() && t->scalar_type() == type && t->dim() == 2 && t->stride(1) == 1;
}

// the caller's output, or a new one; both as a new reference
PyObject* output(PyObject* given, const at::Tensor& A, int64_t M, int N, at::ScalarType type, at::Tensor* out) {
  if (given == Py_None) {
    *out = at::empty({M, N}, A.options().dtype(type));
    return THPVariable_Wrap(*out);
  }
  const at::Tensor* const t = tensor(given);
  if (!matrix(t, type) || t->size(0) != M || t->size(1) != N) return nullptr;
  *out = *t;
  return Py_NewRef(given);
}

bool extents(const at::Tensor& A, const at::Tensor& C) {  // the C ABI's ints
  return A.size(0) <= INT_MAX && A.stride(0) <= INT_MAX && C.stride(0) <= INT_MAX && A.stride(0) >= INT_MIN && C.stride(0) >= INT_MIN;
}

// (A, a_zp, Bp, bias, scales, c_zp, relu, out or None, workspace or None, kernel id) -> out, or None: slow path
PyObject* gemm_u8s8_requant(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 10) Py_RETURN_NONE;
  QG_OR_SLOW(
    const at::Tensor* const A = tensor(a[0]);
    packed B;
    qg_requant_params p = {};
    int kernel = 0;
    void* s = nullptr;
    if (!matrix(A, at::kByte) || !descriptor(a[2], &B) || A->size(1) != B.K || !integer(a[1], &p.a_zp) || !integer(a[5], &p.c_zp) ||
        !integer(a[9], &kernel) || !columns(a[3], a[4], &p.bias, &p.scales, &p.n_scales))
      Py_RETURN_NONE;
    p.relu = PyObject_IsTrue(a[6]);
    if (p.relu < 0 || !stream(&s)) { PyErr_Clear(); Py_RETURN_NONE; }
    void* ws = nullptr;
    if (a[8] != Py_None) {
      const at::Tensor* const w = tensor(a[8]);
      if (!w) Py_RETURN_NONE;
      ws = w->data_ptr();
    }
    at::Tensor C;
    reference result{output(a[7], *A, A->size(0), B.N, at::kByte, &C)};
    if (!result.o) { PyErr_Clear(); Py_RETURN_NONE; }
    int rc = QG_EINVAL;
    if (extents(*A, C)) {
      const uint8_t* const ap = static_cast<const uint8_t*>(A->data_ptr());
      uint8_t* const cp = static_cast<uint8_t*>(C.data_ptr());
      const int M = (int)A->size(0); const int lda = (int)A->stride(0); const int ldc = (int)C.stride(0);
      Py_BEGIN_ALLOW_THREADS
      rc = qg_gemm_u8s8_requant_kernel(ap, M, lda, B.handle, &p, cp, ldc, ws, s, kernel);
      Py_END_ALLOW_THREADS
    }
    if (rc != QG_OK) Py_RETURN_NONE;
    return result.give();)
}

// (A, 1 / alpha, a_zp, Bp, bias, scales, c_zp or None: fp32 output, relu, out or None, workspace or None, kernel id)
PyObject* gemm_f32s8(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 11) Py_RETURN_NONE;
  QG_OR_SLOW(
    const at::Tensor* const A = tensor(a[0]);
    packed B;
    qg_requant_params p = {};
    qg_dequant_params d = {};
    int kernel = 0;
    void* s = nullptr;
    const bool f32 = a[6] == Py_None;
    if (!matrix(A, at::kFloat) || !descriptor(a[3], &B) || A->size(1) != B.K || !integer(a[2], &p.a_zp) ||
        (!f32 && !integer(a[6], &p.c_zp)) || !integer(a[10], &kernel) || !columns(a[4], a[5], &p.bias, &p.scales, &p.n_scales))
      Py_RETURN_NONE;
    const double inv = PyFloat_AsDouble(a[1]);
    if (inv == -1.0 && PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
    p.relu = PyObject_IsTrue(a[7]);
    if (p.relu < 0 || A->size(0) > INT_MAX || !stream(&s)) { PyErr_Clear(); Py_RETURN_NONE; }
    const int M = (int)A->size(0);
    at::Tensor own; const at::Tensor* w = &own;
    if (a[9] == Py_None)
      own = at::empty({(int64_t)qg_gemm_f32_workspace_bytes(M, B.handle)}, A->options().dtype(at::kByte));
    else if (!(w = tensor(a[9])))
      Py_RETURN_NONE;
    void* const ws = w->data_ptr();
    at::Tensor C;
    reference result{output(a[8], *A, M, B.N, f32 ? at::kFloat : at::kByte, &C)};
    if (!result.o) { PyErr_Clear(); Py_RETURN_NONE; }
    int rc = QG_EINVAL;
    if (extents(*A, C)) {
      const float* const ap = static_cast<const float*>(A->data_ptr());
      void* const cp = C.data_ptr();
      const int lda = (int)A->stride(0); const int ldc = (int)C.stride(0);
      d.a_zp = p.a_zp; d.bias = p.bias; d.scales = p.scales; d.n_scales = p.n_scales; d.relu = p.relu;
      Py_BEGIN_ALLOW_THREADS
      rc = f32 ? qg_gemm_f32s8_dequant_f32(ap, M, lda, (float)inv, B.handle, &d, static_cast<float*>(cp), ldc, ws, s, kernel)
               : qg_gemm_f32s8_requant(ap, M, lda, (float)inv, B.handle, &p, static_cast<uint8_t*>(cp), ldc, ws, s, kernel);
      Py_END_ALLOW_THREADS
    }
    if (rc != QG_OK) Py_RETURN_NONE;
    return result.give();)
}

// ---- a call whose arguments are marshalled once
enum call_kind { CALL_GEMM, CALL_CONV_GROUP, CALL_CONV_DENSE, CALL_KINDS };
const char* const call_names[CALL_KINDS] = {"qg_gemm_u8s8_requant", "qg_conv_groupwise_u8s8_requant", "qg_conv_dense_u8s8_requant"};
const int call_ints[CALL_KINDS] = {4, 6, 9};
struct call_args {
  int kind;
  const void* in;
  const qg_packed_b* weights;
  void* out;
  void* workspace;
  void* stream;
  qg_requant_params p;
  int i[9];
};
struct call_object {  // base class of the prepared calls in qgemm.py, whose attributes keep alive what the addresses belong to
  PyObject_HEAD
  call_args c;
};

PyObject* call_launch(PyObject* self, PyObject*) {
  const call_args c = reinterpret_cast<call_object*>(self)->c;  // (its own copy: another thread may change the stream)
  const uint8_t* const in = static_cast<const uint8_t*>(c.in);
  uint8_t* const out = static_cast<uint8_t*>(c.out);
  int rc;
  Py_BEGIN_ALLOW_THREADS
  switch (c.kind) {
    case CALL_GEMM: rc = qg_gemm_u8s8_requant_kernel(in, c.i[0], c.i[1], c.weights, &c.p, out, c.i[2], c.workspace, c.stream, c.i[3]); break;
    case CALL_CONV_GROUP:
      rc = qg_conv_groupwise_u8s8_requant(in, c.i[0], c.i[1], c.i[2], c.i[3], c.i[4], c.i[5], c.weights, &c.p, out, c.stream);
      break;
    default:
      rc = qg_conv_dense_u8s8_requant(in, c.i[0], c.i[1], c.i[2], c.i[3], c.i[4], c.i[5], c.i[6], c.i[7], c.weights, &c.p, out, c.stream, c.i[8]);
  }
  Py_END_ALLOW_THREADS
  if (rc == QG_OK) Py_RETURN_NONE;
  PyObject* const e = PyObject_CallFunction(g_error, "is", rc, call_names[c.kind]);
  if (e) {
    PyErr_SetObject((PyObject*)Py_TYPE(e), e);
    Py_DECREF(e);
  }
  return nullptr;
}

// (kind, input, weights, output, workspace: addresses, a_zp, bias, scales: addresses, n_scales, c_zp, relu, the call's other ints ...)
PyObject* call_set(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  if (n < 11) return PyErr_Format(PyExc_TypeError, "_set: too few arguments");
  call_args c = {};
  c.kind = (int)PyLong_AsLong(a[0]);
  if (PyErr_Occurred()) return nullptr;
  if (c.kind < 0 || c.kind >= CALL_KINDS || n != 11 + call_ints[c.kind]) return PyErr_Format(PyExc_TypeError, "_set: wrong kind or number of arguments");
  auto address = [](PyObject* o) { return o == Py_None ? nullptr : PyLong_AsVoidPtr(o); };
  c.in = address(a[1]);
  c.weights = static_cast<const qg_packed_b*>(address(a[2]));
  c.out = address(a[3]);
  c.workspace = address(a[4]);
  c.p.a_zp = (int)PyLong_AsLong(a[5]);
  c.p.bias = static_cast<const int32_t*>(address(a[6]));
  c.p.scales = static_cast<const float*>(address(a[7]));
  c.p.n_scales = (int)PyLong_AsLong(a[8]);
  c.p.c_zp = (int)PyLong_AsLong(a[9]);
  c.p.relu = (int)PyLong_AsLong(a[10]);
  for (int k = 0; k < call_ints[c.kind]; ++k) c.i[k] = (int)PyLong_AsLong(a[11 + k]);
  if (PyErr_Occurred()) return nullptr;
  reinterpret_cast<call_object*>(self)->c = c;
  Py_RETURN_NONE;
}

PyObject* call_set_stream(PyObject* self, PyObject* stream) {
  void* const s = PyLong_AsVoidPtr(stream);
  if (PyErr_Occurred()) return nullptr;
  reinterpret_cast<call_object*>(self)->c.stream = s;
  Py_RETURN_NONE;
}

#define QG_FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f))
PyMethodDef call_methods[] = {{"launch", call_launch, METH_NOARGS, "Issues the call on its stream."},
                              {"_set", QG_FAST(call_set), METH_FASTCALL, nullptr},
                              {"_set_stream", call_set_stream, METH_O, nullptr},
                              {nullptr, nullptr, 0, nullptr}};
PyTypeObject call_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// the functions and the exception that this module takes from Python
PyObject* init(PyObject*, PyObject* args) {
  PyObject *device, *stream_of, *error;
  if (!PyArg_ParseTuple(args, "OOO", &device, &stream_of, &error)) return nullptr;
  Py_XSETREF(g_device, Py_NewRef(device));
  Py_XSETREF(g_stream_of, Py_NewRef(stream_of));
  Py_XSETREF(g_error, Py_NewRef(error));
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"gemm_u8s8_requant", QG_FAST(gemm_u8s8_requant), METH_FASTCALL, nullptr},
    {"gemm_f32s8", QG_FAST(gemm_f32s8), METH_FASTCALL, nullptr},
    {"init", init, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
  call_type.tp_name = "_binding.Call";
  call_type.tp_basicsize = sizeof(call_object);
  call_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE;
  call_type.tp_methods = call_methods;
  call_type.tp_new = PyType_GenericNew;  // (zeroed: launch() of an object without arguments is refused by the call)
  if (PyType_Ready(&call_type) < 0) return nullptr;
  g_name_fast = PyUnicode_InternFromString("_fast");
  PyObject* const m = g_name_fast ? PyModule_Create(&module) : nullptr;
  if (m && PyModule_AddObjectRef(m, "Call", reinterpret_cast<PyObject*>(&call_type)) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
