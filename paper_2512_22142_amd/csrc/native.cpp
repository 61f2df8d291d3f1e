// Argument checks of the calls a program makes once or twice per GEMM, as a
// CPython extension: a pass over small GEMMs is a few launches of a few
// microseconds each, and the same checks written in Python (one interpreter call
// per tensor property, one ctypes conversion per argument) take longer than the
// kernels.  Host time of the six calls of a 256 x 768 x 768 bf16 linear layer,
// forward and backward: 24 us through this file, 52 us through ctypes (a pass
// 27 / 53 us; the 512^3 fp32 GEMM 12.5 / 17 us).
//
// execute, reduce and reduce_residual check the tensors, take their addresses and
// call the C entry point of the same name; matrix, partials and stream serve the
// calls that go through ctypes.  Nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>

#include "cleave.h"

// The torch and Python this file is compiled for, read from the built file before it is loaded.
extern "C" __attribute__((used)) const char cleave_native_tag[] = CLEAVE_NATIVE_TAG;

namespace {

// The Python exception is set.
struct Raised {};

[[noreturn]] void raise(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw Raised{};
}

const at::Tensor& tensor(PyObject* o, const char* what) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "%s must be a torch tensor, not %s", what, Py_TYPE(o)->tp_name);
    throw Raised{};
  }
  return THPVariable_Unpack(o);
}

struct Matrix {
  void* ptr;
  int64_t ld, rows, cols;
  at::ScalarType type;
};

Matrix matrix(PyObject* o, const char* what) {
  const at::Tensor& t = tensor(o, what);
  if (t.dim() != 2 || t.stride(1) != 1 || !t.is_cuda()) {
    PyErr_Format(PyExc_ValueError, "%s must be a 2-D device tensor with unit column stride", what);
    throw Raised{};
  }
  return Matrix{t.data_ptr(), t.stride(0), t.size(0), t.size(1), t.scalar_type()};
}

// The partial blocks of a plan, `elems` elements.
float* partial_blocks(PyObject* o, int64_t elems) {
  const at::Tensor& t = tensor(o, "partials");
  if (t.scalar_type() != at::kFloat || !t.is_cuda() || !t.is_contiguous() || t.numel() < elems)
    raise(PyExc_ValueError, "partials must be a contiguous fp32 device tensor of partial_elems elements");
  return static_cast<float*>(t.data_ptr());
}

int dtype_code(at::ScalarType t) {
  if (t == at::kFloat) return CLEAVE_F32;
  if (t == at::kBFloat16) return CLEAVE_BF16;
  PyErr_Format(PyExc_TypeError, "unsupported dtype torch.%s", c10::toString(t));
  throw Raised{};
}

int64_t integer(PyObject* o) {   // as int(o)
  if (PyLong_Check(o)) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
  }
  PyObject* n = PyNumber_Long(o);
  if (!n) throw Raised{};
  const long long v = PyLong_AsLongLong(n);
  Py_DECREF(n);
  if (v == -1 && PyErr_Occurred()) throw Raised{};
  return v;
}

void* address(PyObject* o) {   // an int; None is null
  if (o == Py_None) return nullptr;
  void* p = PyLong_AsVoidPtr(o);
  if (!p && PyErr_Occurred()) throw Raised{};
  return p;
}

// None: torch's current stream; else an object with a `cuda_stream` (None there is
// the null stream), or an address in any form that int() takes.
void* stream_of(PyObject* o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  if (PyLong_Check(o)) return address(o);
  if (PyObject* s = PyObject_GetAttrString(o, "cuda_stream")) {
    void* p = s == Py_None ? nullptr : PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    if (!p && PyErr_Occurred()) throw Raised{};
    return p;
  }
  if (!PyErr_ExceptionMatches(PyExc_AttributeError)) throw Raised{};
  PyErr_Clear();
  PyObject* n = PyNumber_Long(o);
  if (!n) throw Raised{};
  void* p = PyLong_AsVoidPtr(n);
  Py_DECREF(n);
  if (!p && PyErr_Occurred()) throw Raised{};
  return p;
}

template <typename F>
PyObject* guarded(F&& body) {
  try {
    return body();
  } catch (const Raised&) {
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}

void expect_args(Py_ssize_t n, Py_ssize_t want) {
  if (n != want) raise(PyExc_TypeError, "wrong number of arguments");
}

// matrix(t, what) -> (address, leading dimension)
PyObject* py_matrix(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    expect_args(n, 2);
    const char* what = PyUnicode_AsUTF8(a[1]);
    if (!what) throw Raised{};
    const Matrix m = matrix(a[0], what);
    return Py_BuildValue("(NL)", PyLong_FromVoidPtr(m.ptr), static_cast<long long>(m.ld));
  });
}

// stream(s) -> address
PyObject* py_stream(PyObject*, PyObject* o) {
  return guarded([&]() -> PyObject* { return PyLong_FromVoidPtr(stream_of(o)); });
}

// execute(plan address, M, N, K, partial_elems, A, B, partials, transA, transB, ids address, n_ids, stream, noalloc)
PyObject* py_execute(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    expect_args(n, 14);
    const int64_t M = integer(a[1]), N = integer(a[2]), K = integer(a[3]);
    const Matrix A = matrix(a[5], "A"), B = matrix(a[6], "B");
    if (A.type != B.type) raise(PyExc_TypeError, "A and B must have the same dtype");
    float* p = partial_blocks(a[7], integer(a[4]));
    // stored shapes must hold the logical operands
    const int ta = static_cast<int>(integer(a[8])), tb = static_cast<int>(integer(a[9]));
    if (A.rows != (ta ? K : M) || A.cols != (ta ? M : K) || B.rows != (tb ? N : K) || B.cols != (tb ? K : N)) {
      PyErr_Format(PyExc_ValueError, "operand shapes (%lld, %lld), (%lld, %lld) do not match the plan",
                   static_cast<long long>(A.rows), static_cast<long long>(A.cols), static_cast<long long>(B.rows),
                   static_cast<long long>(B.cols));
      throw Raised{};
    }
    cleave_plan* plan = static_cast<cleave_plan*>(address(a[0]));
    const int64_t* ids = static_cast<const int64_t*>(address(a[10]));
    const int64_t n_ids = integer(a[11]);
    const int dt = dtype_code(A.type);
    void* stream = stream_of(a[12]);
    const int noalloc = PyObject_IsTrue(a[13]);
    if (noalloc < 0) throw Raised{};
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = (noalloc ? cleave_execute_noalloc : cleave_execute)(plan, ids, n_ids, A.ptr, A.ld, ta, B.ptr, B.ld, tb, dt, p,
                                                             stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
  });
}

// partials(t, elems) -> address
PyObject* py_partials(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    expect_args(n, 2);
    return PyLong_FromVoidPtr(partial_blocks(a[0], integer(a[1])));
  });
}

// reduce(plan address, M, N, partial_elems, partials, C, stream)
PyObject* py_reduce(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    expect_args(n, 7);
    const Matrix C = matrix(a[5], "C");
    if (C.rows != integer(a[1]) || C.cols != integer(a[2])) raise(PyExc_ValueError, "C must be M x N");
    cleave_plan* plan = static_cast<cleave_plan*>(address(a[0]));
    const float* p = partial_blocks(a[4], integer(a[3]));
    const int dt = dtype_code(C.type);
    void* stream = stream_of(a[6]);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = cleave_reduce(plan, p, C.ptr, C.ld, dt, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
  });
}

// reduce_residual(plan address, M, N, partial_elems, partials, R, C, stream)
PyObject* py_reduce_residual(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    expect_args(n, 8);
    const Matrix C = matrix(a[6], "C"), R = matrix(a[5], "R");
    const int64_t M = integer(a[1]), N = integer(a[2]);
    if (C.rows != M || C.cols != N || R.rows != M || R.cols != N || R.ld != C.ld || R.type != C.type)
      raise(PyExc_ValueError, "R and C must be M x N with the same dtype and leading dimension");
    cleave_plan* plan = static_cast<cleave_plan*>(address(a[0]));
    const float* p = partial_blocks(a[4], integer(a[3]));
    const int dt = dtype_code(C.type);
    void* stream = stream_of(a[7]);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = cleave_reduce_residual(plan, p, R.ptr, C.ptr, C.ld, dt, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
  });
}

template <typename F>
PyCFunction as_function(F* f) {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(f));
}

PyMethodDef kMethods[] = {
    {"matrix", as_function(py_matrix), METH_FASTCALL, nullptr},
    {"stream", py_stream, METH_O, nullptr},
    {"partials", as_function(py_partials), METH_FASTCALL, nullptr},
    {"execute", as_function(py_execute), METH_FASTCALL, nullptr},
    {"reduce", as_function(py_reduce), METH_FASTCALL, nullptr},
    {"reduce_residual", as_function(py_reduce_residual), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&kModule); }
