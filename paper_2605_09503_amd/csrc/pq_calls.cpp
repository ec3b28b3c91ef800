// The calls of the Python binding that a forward pass or a calibration hook makes once a layer, as a CPython module:
// their arguments go from the interpreter's objects to the C entry points without ctypes.  A call of these launches one or two
// kernels that may take 3 us, and the host has to keep up: issuing a launch takes 2.7 us by itself, a wrapper in Python, its
// tensors' methods and ctypes took 2 more.  NVFP4 256 x 512 x 512, quantizer and product, one pair after another: 10.4 us before, 6.8
// then, where the kernels alone took 6.5 (in a graph, 5.5 now); INT4 g128 77 x 1000 x 1152 from the stored layout 13.9 -> 10.2 (7.6 with
// one launch less).
//
// Marshalling only: pointers, sizes and strides of the tensors, the current stream, the result code.  pq.py holds the
// declarations that users read, the exception type and the helpers that allocate (handed over by bind()).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <new>

#include "../../include/permuquant.h"

namespace {

PyObject* g_raise = nullptr;        // raise(rc): raises the error of the last call
PyObject* g_operand = nullptr;      // operand(fmt, group, rows, K, like) -> tensor
PyObject* g_workspace = nullptr;    // workspace(op, fmt, group, M, N, K, n_batches, like) -> tensor or None

// thrown when a Python error is set
struct PyFailed {};

[[noreturn]] void fail(PyObject* type, const char* what) {
  PyErr_SetString(type, what);
  throw PyFailed{};
}

struct Ref {
  PyObject* p;
  explicit Ref(PyObject* o) : p(o) {
    if (!o) throw PyFailed{};
  }
  ~Ref() { Py_XDECREF(p); }
  Ref(const Ref&) = delete;
  Ref& operator=(const Ref&) = delete;
};

// integers and what stands for one (__index__: numpy's integers, a tensor of one)
int64_t as_int(PyObject* o) {
  if (!PyLong_Check(o)) {
    if (!PyIndex_Check(o)) fail(PyExc_TypeError, "an integer is required");
    Ref n(PyNumber_Index(o));
    return as_int(n.p);
  }
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw PyFailed{};
  return v;
}

// what int(o) gives
int64_t to_int(PyObject* o) {
  Ref n(PyNumber_Long(o));
  return as_int(n.p);
}

bool given(PyObject* o) { return o && o != Py_None; }

// a torch tensor itself; other objects, subclasses that override methods among them, are asked through their methods
const at::Tensor* tensor(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

void* pointer(PyObject* o) {
  if (!given(o)) return nullptr;
  if (const at::Tensor* t = tensor(o)) return t->data_ptr();
  Ref r(PyObject_CallMethod(o, "data_ptr", nullptr));
  void* p = PyLong_AsVoidPtr(r.p);
  if (!p && PyErr_Occurred()) throw PyFailed{};
  return p;
}
int64_t size(PyObject* o, int64_t dim) {
  if (const at::Tensor* t = tensor(o)) {
    if (dim >= t->dim()) fail(PyExc_IndexError, "tuple index out of range");
    return t->size(dim);
  }
  Ref shape(PyObject_GetAttrString(o, "shape"));
  Ref n(PySequence_GetItem(shape.p, dim));
  return as_int(n.p);
}
int64_t row_stride(PyObject* o) {
  if (const at::Tensor* t = tensor(o)) return t->stride(0);
  Ref r(PyObject_CallMethod(o, "stride", "i", 0));
  return as_int(r.p);
}
size_t numel(PyObject* o) {
  if (const at::Tensor* t = tensor(o)) return (size_t)t->numel();
  Ref r(PyObject_CallMethod(o, "numel", nullptr));
  return (size_t)as_int(r.p);
}
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

int64_t or_size(PyObject* o, PyObject* t, int64_t dim) { return given(o) ? as_int(o) : size(t, dim); }
int64_t or_stride(PyObject* o, PyObject* t) { return given(o) ? as_int(o) : row_stride(t); }

// Arguments by position or name into slots, nullptr where absent; the first `required` must be there.
struct Spec {
  const char* name;
  int n, required;
  const char* const* args;
};
void take(const Spec& s, PyObject* const* args, Py_ssize_t nargs, PyObject* names, PyObject** slot) {
  for (int i = 0; i < s.n; ++i) slot[i] = nullptr;
  if (nargs > s.n) {
    PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", s.name, s.n, nargs);
    throw PyFailed{};
  }
  for (Py_ssize_t i = 0; i < nargs; ++i) slot[i] = args[i];
  const Py_ssize_t n_names = names ? PyTuple_GET_SIZE(names) : 0;
  for (Py_ssize_t k = 0; k < n_names; ++k) {
    PyObject* name = PyTuple_GET_ITEM(names, k);
    int at = 0;
    while (at < s.n && PyUnicode_CompareWithASCIIString(name, s.args[at]) != 0) ++at;
    if (at == s.n) {
      PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", s.name, name);
      throw PyFailed{};
    }
    if (slot[at]) {
      PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", s.name, name);
      throw PyFailed{};
    }
    slot[at] = args[nargs + k];
  }
  for (int i = 0; i < s.required; ++i) {
    if (!slot[i]) {
      PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", s.name, s.args[i]);
      throw PyFailed{};
    }
  }
}

// the entry point without the interpreter's lock, as ctypes calls it
template <class F>
void call(F&& f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f();
  Py_END_ALLOW_THREADS
  if (rc != PQ_OK) {
    Ref unused(PyObject_CallFunction(g_raise, "i", rc));
    fail(PyExc_RuntimeError, "the library reported an error");       // not reached: raise() raises
  }
}

// runs a call's body; errors of the interpreter and C++ exceptions of torch become Python exceptions
template <class F>
PyObject* guarded(F&& f) {
  try {
    return f();
  } catch (const PyFailed&) {
    return nullptr;
  } catch (const c10::IndexError& e) {
    PyErr_SetString(PyExc_IndexError, e.what_without_backtrace());
  } catch (const c10::Error& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
  } catch (const std::bad_alloc&) {
    PyErr_NoMemory();
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}

PyObject* none() { Py_RETURN_NONE; }

// the operand buffer that was passed, or a new one: a new reference
PyObject* operand_of(PyObject* o, int64_t fmt, int64_t group, int64_t rows, int64_t K, PyObject* like) {
  if (given(o)) {
    Py_INCREF(o);
    return o;
  }
  return PyObject_CallFunction(g_operand, "LLLLO", (long long)fmt, (long long)group, (long long)rows, (long long)K, like);
}

#define PQ_CALL(fn) static PyObject* fn(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* names)
#define PQ_TAKE(fn, required, ...)                                                    \
  static const char* const arg_names[] = {__VA_ARGS__};                               \
  constexpr int n_args = sizeof(arg_names) / sizeof(arg_names[0]);                    \
  static const Spec spec = {#fn, n_args, required, arg_names};                        \
  PyObject* a[n_args];                                                                \
  take(spec, args, nargs, names, a)

PQ_CALL(quantize_act) {
  return guarded([&] {
    PQ_TAKE(pq_quantize_act, 7, "fmt", "group", "x", "perm", "tensor_scale", "codes", "scales", "M", "K", "ld");
    const int fmt = (int)as_int(a[0]), group = (int)as_int(a[1]);
    const int64_t M = or_size(a[7], a[2], 0), K = or_size(a[8], a[2], 1), ld = or_stride(a[9], a[2]);
    void *x = pointer(a[2]), *perm = pointer(a[3]), *ts = pointer(a[4]), *codes = pointer(a[5]), *scales = pointer(a[6]), *st = stream();
    call([&] {
      return pq_quantize_act((pq_format)fmt, group, x, M, K, ld, (const int32_t*)perm, (const float*)ts, (uint8_t*)codes, scales, st);
    });
    return none();
  });
}

PQ_CALL(quantize_act_packed) {
  return guarded([&] {
    PQ_TAKE(pq_quantize_act_packed, 4, "fmt", "group", "x", "tensor_scale", "operand", "codes", "scales", "K");
    const int fmt = (int)as_int(a[0]), group = (int)as_int(a[1]);
    const int64_t M = size(a[2], 0), K = or_size(a[7], a[2], 1);
    Ref out(operand_of(a[4], fmt, group, M, K, a[2]));
    void *x = pointer(a[2]), *ts = pointer(a[3]), *op = pointer(out.p), *codes = pointer(a[5]), *scales = pointer(a[6]), *st = stream();
    const int64_t ld = row_stride(a[2]);
    const size_t bytes = numel(out.p);
    call([&] {
      return pq_quantize_act_packed((pq_format)fmt, group, x, M, K, ld, (const float*)ts, op, bytes, (uint8_t*)codes, scales, st);
    });
    Py_INCREF(out.p);
    return out.p;
  });
}

PQ_CALL(norm_quantize_act_packed) {
  return guarded([&] {
    PQ_TAKE(pq_norm_quantize_act_packed, 6, "kind", "fmt", "group", "x", "eps", "tensor_scale", "perm", "gamma", "mod_scale",
            "mod_shift", "rows_per_mod", "operand", "y", "K");
    const int fmt = (int)as_int(a[1]), group = (int)as_int(a[2]);
    const int64_t M = size(a[3], 0), K = or_size(a[13], a[3], 1);
    Ref out(operand_of(a[11], fmt, group, M, K, a[3]));
    pq_norm_params p;
    p.kind = (decltype(p.kind))to_int(a[0]);
    p.perm = (decltype(p.perm))pointer(a[6]);
    p.gamma = pointer(a[7]);
    p.mod_scale = pointer(a[8]);
    p.mod_shift = pointer(a[9]);
    p.rows_per_mod = a[10] ? to_int(a[10]) : 0;
    p.eps = (float)PyFloat_AsDouble(a[4]);
    if (PyErr_Occurred()) throw PyFailed{};
    void *x = pointer(a[3]), *ts = pointer(a[5]), *op = pointer(out.p), *y = pointer(a[12]), *st = stream();
    const int64_t ld = row_stride(a[3]), ldy = given(a[12]) ? row_stride(a[12]) : 0;
    const size_t bytes = numel(out.p);
    call([&] {
      return pq_norm_quantize_act_packed(&p, (pq_format)fmt, group, x, M, K, ld, (const float*)ts, op, bytes, y, ldy, st);
    });
    Py_INCREF(out.p);
    return out.p;
  });
}

PQ_CALL(hadamard_quantize_act_packed) {
  return guarded([&] {
    PQ_TAKE(pq_hadamard_quantize_act_packed, 4, "fmt", "group", "x", "tensor_scale", "perm", "operand", "y", "K");
    const int fmt = (int)as_int(a[0]), group = (int)as_int(a[1]);
    const int64_t M = size(a[2], 0), K = or_size(a[7], a[2], 1);
    Ref out(operand_of(a[5], fmt, group, M, K, a[2]));
    void *x = pointer(a[2]), *ts = pointer(a[3]), *perm = pointer(a[4]), *op = pointer(out.p), *y = pointer(a[6]), *st = stream();
    const int64_t ld = row_stride(a[2]), ldy = given(a[6]) ? row_stride(a[6]) : 0;
    const size_t bytes = numel(out.p);
    call([&] {
      return pq_hadamard_quantize_act_packed((const int32_t*)perm, (pq_format)fmt, group, x, M, K, ld, (const float*)ts, op, bytes, y,
                                             ldy, st);
    });
    Py_INCREF(out.p);
    return out.p;
  });
}

template <class F>
PyObject* product_packed(PyObject* const* a, PyObject* y, PyObject* m, PyObject* n, PyObject* k, PyObject* ldy, F&& entry) {
  const int fmt = (int)as_int(a[0]), group = (int)as_int(a[1]);
  void *ao = pointer(a[2]), *ats = pointer(a[3]), *wo = pointer(a[4]), *wts = pointer(a[5]), *yp = pointer(y), *st = stream();
  const int64_t M = as_int(m), N = as_int(n), K = as_int(k), ld = or_stride(ldy, y);
  call([&] { return entry((pq_format)fmt, group, ao, (const float*)ats, wo, (const float*)wts, M, N, K, yp, ld, st); });
  return none();
}

PQ_CALL(qgemm_packed) {
  return guarded([&] {
    PQ_TAKE(pq_qgemm_packed, 10, "fmt", "group", "a_operand", "a_tensor_scale", "w_operand", "w_tensor_scale", "y", "M", "N", "K", "ldy");
    return product_packed(a, a[6], a[7], a[8], a[9], a[10], pq_qgemm_packed);
  });
}
PQ_CALL(qgemm_packed_f32) {
  return guarded([&] {
    PQ_TAKE(pq_qgemm_packed_f32, 10, "fmt", "group", "a_operand", "a_tensor_scale", "w_operand", "w_tensor_scale", "y", "M", "N", "K",
            "ldy");
    return product_packed(a, a[6], a[7], a[8], a[9], a[10],
                          [](pq_format fmt, int group, const void* ao, const float* ats, const void* wo, const float* wts, int64_t M,
                             int64_t N, int64_t K, void* y, int64_t ldy, void* st) {
                            return pq_qgemm_packed_f32(fmt, group, ao, ats, wo, wts, M, N, K, (float*)y, ldy, st);
                          });
  });
}
PQ_CALL(qgemm_packed_bias) {
  return guarded([&] {
    PQ_TAKE(pq_qgemm_packed_bias, 11, "fmt", "group", "a_operand", "a_tensor_scale", "w_operand", "w_tensor_scale", "bias", "y", "M",
            "N", "K", "ldy");
    void* bias = pointer(a[6]);
    return product_packed(a, a[7], a[8], a[9], a[10], a[11],
                          [&](pq_format fmt, int group, const void* ao, const float* ats, const void* wo, const float* wts, int64_t M,
                              int64_t N, int64_t K, void* y, int64_t ldy, void* st) {
                            return pq_qgemm_packed_bias(fmt, group, ao, ats, wo, wts, M, N, K, bias, y, ldy, st);
                          });
  });
}

// a workspace that was passed, or a new one (None where none is needed): a new reference
PyObject* workspace_of(PyObject* o, int op, int fmt, int group, int64_t M, int64_t N, int64_t K, int n_batches, PyObject* like) {
  if (given(o)) {
    Py_INCREF(o);
    return o;
  }
  return PyObject_CallFunction(g_workspace, "iiiLLLiO", op, fmt, group, (long long)M, (long long)N, (long long)K, n_batches, like);
}

PQ_CALL(qgemm) {
  return guarded([&] {
    PQ_TAKE(pq_qgemm, 9, "fmt", "group", "a_codes", "a_scales", "a_tensor_scale", "w_codes", "w_scales", "w_tensor_scale", "y",
            "workspace", "M", "N", "K", "ldy");
    const int fmt = (int)as_int(a[0]), group = (int)as_int(a[1]);
    const int64_t M = or_size(a[10], a[2], 0), K = given(a[12]) ? as_int(a[12]) : 2 * size(a[2], 1), N = or_size(a[11], a[5], 0);
    const int64_t ldy = or_stride(a[13], a[8]);
    Ref ws(workspace_of(a[9], PQ_OP_QGEMM, fmt, group, M, N, K, 0, a[2]));
    void *ac = pointer(a[2]), *as = pointer(a[3]), *ats = pointer(a[4]), *wc = pointer(a[5]), *wsc = pointer(a[6]),
         *wts = pointer(a[7]), *y = pointer(a[8]), *wp = pointer(ws.p), *st = stream();
    const size_t bytes = given(ws.p) ? numel(ws.p) : 0;
    call([&] {
      return pq_qgemm((pq_format)fmt, group, (const uint8_t*)ac, as, (const float*)ats, (const uint8_t*)wc, wsc, (const float*)wts, M, N,
                      K, y, ldy, wp, bytes, st);
    });
    return none();
  });
}

PQ_CALL(calib_moments) {
  return guarded([&] {
    PQ_TAKE(pq_calib_moments, 2, "x", "sumsq", "absmax", "workspace", "rows", "K", "ld");
    const int64_t rows = or_size(a[4], a[0], 0), K = or_size(a[5], a[0], 1), ld = or_stride(a[6], a[0]);
    Ref ws(workspace_of(a[3], PQ_OP_CALIB_MOMENTS, 0, 0, rows, 0, K, 1, a[0]));
    void *x = pointer(a[0]), *sumsq = pointer(a[1]), *absmax = pointer(a[2]), *wp = pointer(ws.p), *st = stream();
    const size_t bytes = given(ws.p) ? numel(ws.p) : 0;
    call([&] { return pq_calib_moments(x, rows, K, ld, (double*)sumsq, (float*)absmax, wp, bytes, st); });
    return none();
  });
}

PyObject* bind(PyObject*, PyObject* args) {
  PyObject *raise, *operand, *workspace;
  if (!PyArg_ParseTuple(args, "OOO", &raise, &operand, &workspace)) return nullptr;
  Py_INCREF(raise);
  Py_INCREF(operand);
  Py_INCREF(workspace);
  Py_XSETREF(g_raise, raise);
  Py_XSETREF(g_operand, operand);
  Py_XSETREF(g_workspace, workspace);
  Py_RETURN_NONE;
}

#define PQ_METHOD(fn, signature, text) \
  {"pq_" #fn, (PyCFunction)(void (*)(void))fn, METH_FASTCALL | METH_KEYWORDS, "pq_" #fn signature "\n--\n\n" text}
PyMethodDef methods[] = {
    PQ_METHOD(quantize_act, "(fmt, group, x, perm, tensor_scale, codes, scales, M=None, K=None, ld=None)",
              "Dynamic activation quantization into the stored layout."),
    PQ_METHOD(quantize_act_packed, "(fmt, group, x, tensor_scale, operand=None, codes=None, scales=None, K=None)",
              "Dynamic activation quantization straight into the GEMM's panel layout."),
    PQ_METHOD(norm_quantize_act_packed,
              "(kind, fmt, group, x, eps, tensor_scale, perm=None, gamma=None, mod_scale=None, mod_shift=None, rows_per_mod=0, "
              "operand=None, y=None, K=None)",
              "pq_norm_reorder feeding the activation quantizer directly: returns the GEMM operand."),
    PQ_METHOD(hadamard_quantize_act_packed, "(fmt, group, x, tensor_scale, perm=None, operand=None, y=None, K=None)",
              "The rotation feeding the activation quantizer directly: returns the GEMM operand."),
    PQ_METHOD(qgemm_packed, "(fmt, group, a_operand, a_tensor_scale, w_operand, w_tensor_scale, y, M, N, K, ldy=None)",
              "y[M, N] (bf16) = the product of two packed operands."),
    PQ_METHOD(qgemm_packed_f32, "(fmt, group, a_operand, a_tensor_scale, w_operand, w_tensor_scale, y, M, N, K, ldy=None)",
              "The packed product in fp32, before the rounding to bf16."),
    PQ_METHOD(qgemm_packed_bias, "(fmt, group, a_operand, a_tensor_scale, w_operand, w_tensor_scale, bias, y, M, N, K, ldy=None)",
              "The packed product plus the layer's bias (bf16 [N]), added before the rounding to bf16."),
    PQ_METHOD(qgemm,
              "(fmt, group, a_codes, a_scales, a_tensor_scale, w_codes, w_scales, w_tensor_scale, y, workspace=None, M=None, N=None, "
              "K=None, ldy=None)",
              "y[M, N] (bf16) = dequant(A) @ dequant(W)^T."),
    PQ_METHOD(calib_moments, "(x, sumsq, absmax=None, workspace=None, rows=None, K=None, ld=None)",
              "sumsq[K] (float64, in/out) += column sums of squares of bf16 x[rows, ld]."),
    {"bind", bind, METH_VARARGS, "bind(raise_, operand, workspace): the helpers of pq.py"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pq_calls", "Hot calls of the binding (see pq.py).", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pq_calls() { return PyModule_Create(&module); }
