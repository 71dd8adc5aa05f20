// CPython entry to the launch calls of the C ABI (no Python types beyond integers and floats, no HIP).
//
// A launch on small inputs is bound by the host: of 7.2 us for one tw_gemm issued from Python, 0.7 us were the
// ctypes call and the wrappers around it.  Here the arguments are read straight from the vector call
// (0.2 us).  Anything but plain integers (floats) in range returns None, and the caller takes the ctypes route,
// which converts or refuses as it always has.  The functions are bound by address, so that they are those
// of the library that the process has loaded.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <climits>
#include <cstdint>

namespace {

typedef int (*gemm_fn)(const void*, int, int, int, void*, void*, int, void*);
typedef int (*gemm_i8_fn)(const void*, int, int, void*, void*, int, int, float, void*);
typedef int (*conv_fn)(const void*, void*, void*, int, void*);
typedef int (*conv_i8_fn)(const void*, void*, void*, int, int, float, void*);
gemm_fn f_gemm = nullptr;
gemm_i8_fn f_gemm_i8 = nullptr;
conv_fn f_conv = nullptr;
conv_i8_fn f_conv_i8 = nullptr;

// Each sets `ok` to false when the object is not a plain number that the C type holds.
void* ptr(PyObject* o, bool& ok) {
  if (!PyLong_CheckExact(o)) { ok = false; return nullptr; }
  const unsigned long long v = PyLong_AsUnsignedLongLong(o);
  if (v == ~0ull && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
  return (void*)(uintptr_t)v;
}
int num(PyObject* o, bool& ok) {
  if (!PyLong_CheckExact(o)) { ok = false; return 0; }
  int over = 0;
  const long v = PyLong_AsLongAndOverflow(o, &over);
  if (over || v < INT_MIN || v > INT_MAX) { ok = false; return 0; }
  return (int)v;
}
float real(PyObject* o, bool& ok) {
  if (!PyFloat_CheckExact(o)) { ok = false; return 0.f; }
  return (float)PyFloat_AS_DOUBLE(o);
}
template <class F>
PyObject* run(F f) {
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  bool ok = n == 4;
  void* p[4] = {};
  for (int i = 0; ok && i < 4; ++i) p[i] = ptr(a[i], ok);
  if (!ok) { PyErr_SetString(PyExc_TypeError, "four function addresses expected"); return nullptr; }
  f_gemm = (gemm_fn)p[0]; f_gemm_i8 = (gemm_i8_fn)p[1]; f_conv = (conv_fn)p[2]; f_conv_i8 = (conv_i8_fn)p[3];
  Py_RETURN_NONE;
}
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {      // A, M, lda, layout, handle, C, ldc, stream
  bool ok = n == 8 && f_gemm;
  if (!ok) Py_RETURN_NONE;
  void* A = ptr(a[0], ok); const int M = num(a[1], ok), lda = num(a[2], ok), layout = num(a[3], ok);
  void* h = ptr(a[4], ok); void* C = ptr(a[5], ok); const int ldc = num(a[6], ok); void* s = ptr(a[7], ok);
  if (!ok) Py_RETURN_NONE;
  return run([&] { return f_gemm(A, M, lda, layout, h, C, ldc, s); });
}
PyObject* gemm_i8(PyObject*, PyObject* const* a, Py_ssize_t n) {   // A, M, lda, handle, C, ldc, c_dtype, scale, stream
  bool ok = n == 9 && f_gemm_i8;
  if (!ok) Py_RETURN_NONE;
  void* A = ptr(a[0], ok); const int M = num(a[1], ok), lda = num(a[2], ok);
  void* h = ptr(a[3], ok); void* C = ptr(a[4], ok); const int ldc = num(a[5], ok), dt = num(a[6], ok);
  const float scale = real(a[7], ok); void* s = ptr(a[8], ok);
  if (!ok) Py_RETURN_NONE;
  return run([&] { return f_gemm_i8(A, M, lda, h, C, ldc, dt, scale, s); });
}
PyObject* conv(PyObject*, PyObject* const* a, Py_ssize_t n) {      // X, binding, C, ldc, stream
  bool ok = n == 5 && f_conv;
  if (!ok) Py_RETURN_NONE;
  void* X = ptr(a[0], ok); void* b = ptr(a[1], ok); void* C = ptr(a[2], ok); const int ldc = num(a[3], ok);
  void* s = ptr(a[4], ok);
  if (!ok) Py_RETURN_NONE;
  return run([&] { return f_conv(X, b, C, ldc, s); });
}
PyObject* conv_i8(PyObject*, PyObject* const* a, Py_ssize_t n) {   // X, binding, C, ldc, c_dtype, scale, stream
  bool ok = n == 7 && f_conv_i8;
  if (!ok) Py_RETURN_NONE;
  void* X = ptr(a[0], ok); void* b = ptr(a[1], ok); void* C = ptr(a[2], ok);
  const int ldc = num(a[3], ok), dt = num(a[4], ok); const float scale = real(a[5], ok); void* s = ptr(a[6], ok);
  if (!ok) Py_RETURN_NONE;
  return run([&] { return f_conv_i8(X, b, C, ldc, dt, scale, s); });
}

PyMethodDef methods[] = {{"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
                         {"gemm", (PyCFunction)(void (*)(void))gemm, METH_FASTCALL, nullptr},
                         {"gemm_i8", (PyCFunction)(void (*)(void))gemm_i8, METH_FASTCALL, nullptr},
                         {"conv", (PyCFunction)(void (*)(void))conv, METH_FASTCALL, nullptr},
                         {"conv_i8", (PyCFunction)(void (*)(void))conv_i8, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_twcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__twcall() { return PyModule_Create(&module); }
