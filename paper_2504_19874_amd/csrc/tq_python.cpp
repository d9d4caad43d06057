// The per-call half of the Python binding: reads what a call's tensors are, and calls the C ABI.
//
// A decoding step makes three calls whose kernels take 5 - 20 us each.  Marshalled in Python (attribute look-ups on a
// dozen tensors, a ctypes object per pointer, a stream object) such a call costs the host 10 - 15 us, more than the GPU
// needs for it; here the same work is a few hundred nanoseconds.
//
// Every function takes the tq_params struct as a buffer and returns the library's status, or None where an argument is
// not what the plain call has (a wrong type, dtype, device, layout or size, a workspace to be grown): nothing has been
// done then, and the caller takes its checked path, which raises the error or does the call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/turboquant.h"

namespace {

struct NotPlain {};

const tq_params* params(PyObject* o) {
  // the struct belongs to a Params object that the caller holds for the length of the call
  Py_buffer b;
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
    PyErr_Clear();
    throw NotPlain{};
  }
  const bool whole = (size_t)b.len == sizeof(tq_params);
  const tq_params* p = static_cast<const tq_params*>(b.buf);
  PyBuffer_Release(&b);
  if (!whole) throw NotPlain{};
  return p;
}

int64_t integer(PyObject* o) {
  if (!PyLong_CheckExact(o)) throw NotPlain{};
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow != 0) throw NotPlain{};
  return v;
}

int32_t integer32(PyObject* o) {
  const int64_t v = integer(o);
  if (v != (int32_t)v) throw NotPlain{};
  return (int32_t)v;
}

// (plain Tensor or Parameter objects only: a subclass may answer questions about itself in its own way)
const at::Tensor* tensor(PyObject* o) {
  if (o == Py_None) return nullptr;
  if (!THPVariable_CheckExact(o)) throw NotPlain{};
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda()) throw NotPlain{};
  return &t;
}

// a code array: contiguous, at least `numel` elements of `type`
template <class T>
T* array(PyObject* o, c10::ScalarType type, int64_t numel) {
  const at::Tensor* t = tensor(o);
  if (t == nullptr) return nullptr;
  if (t->scalar_type() != type || t->numel() < numel || !t->is_contiguous()) throw NotPlain{};
  return static_cast<T*>(t->data_ptr());
}

// a matrix with contiguous rows, which may be padded
struct Rows {
  void* ptr;
  int64_t rows, cols, stride;
  c10::ScalarType type;
};
Rows matrix(PyObject* o) {
  const at::Tensor* t = tensor(o);
  if (t == nullptr || t->dim() != 2 || (t->size(1) > 1 && t->stride(1) != 1)) throw NotPlain{};
  return Rows{t->data_ptr(), t->size(0), t->size(1), t->stride(0), t->scalar_type()};
}

struct Codes {
  uint32_t *idx, *qjl;
  float *gamma, *norm;
};
Codes codes(const tq_params* p, PyObject* const* o, int64_t rows) {
  const int64_t words = (int64_t)(p->d_hi / 32) * p->bits_mse_hi + (int64_t)((p->d - p->d_hi) / 32) * p->bits_mse;
  const int64_t scalars = p->d_hi != 0 ? 2 : 1;
  if (rows < 0) throw NotPlain{};
  Codes c;
  c.idx = array<uint32_t>(o[0], at::kInt, rows * words);
  c.qjl = array<uint32_t>(o[1], at::kInt, rows * (p->d / 32));
  c.gamma = array<float>(o[2], at::kFloat, rows * scalars);
  c.norm = array<float>(o[3], at::kFloat, rows * scalars);
  return c;
}

int32_t vector_type(const Rows& x) {
  if (x.type == at::kFloat) return TQ_F32;
  if (x.type == at::kBFloat16) return TQ_BF16;
  throw NotPlain{};
}

void* stream() { return static_cast<void*>(c10::hip::getCurrentHIPStream().stream()); }

template <class F>
PyObject* call(Py_ssize_t got, Py_ssize_t want, F f) {
  if (got != want) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    return PyLong_FromLong((long)f());
  } catch (const NotPlain&) {
    Py_RETURN_NONE;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// the library's calls run without the interpreter's lock
template <class F>
tq_status unlocked(F f) {
  tq_status st;
  Py_BEGIN_ALLOW_THREADS;
  st = f();
  Py_END_ALLOW_THREADS;
  return st;
}

// p, x, idx, norm
PyObject* quantize_mse(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 4, [&] {
    const tq_params* p = params(a[0]);
    const Rows x = matrix(a[1]);
    PyObject* const arrays[4] = {a[2], Py_None, Py_None, a[3]};
    const Codes c = codes(p, arrays, x.rows);
    const int32_t type = vector_type(x);
    void* const s = stream();
    return unlocked([&] { return tq_quantize_mse(p, x.ptr, type, x.rows, x.rows ? x.stride : p->d, c.idx, c.norm, s); });
  });
}

// p, x, idx, qjl, gamma, norm
PyObject* quantize_prod(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 6, [&] {
    const tq_params* p = params(a[0]);
    const Rows x = matrix(a[1]);
    const Codes c = codes(p, a + 2, x.rows);
    const int32_t type = vector_type(x);
    void* const s = stream();
    return unlocked(
        [&] { return tq_quantize_prod(p, x.ptr, type, x.rows, x.rows ? x.stride : p->d, c.idx, c.qjl, c.gamma, c.norm, s); });
  });
}

// p, x, idx, qjl, gamma, norm, first_row, row_step
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 8, [&] {
    const tq_params* p = params(a[0]);
    const Rows x = matrix(a[1]);
    const int64_t first = integer(a[6]), step = integer(a[7]);
    if (first < 0 || step < 1 || first > (int64_t(1) << 40) || step > (int64_t(1) << 40) || x.rows > (1 << 20)) throw NotPlain{};
    const Codes c = codes(p, a + 2, x.rows > 0 ? first + (x.rows - 1) * step + 1 : 0);
    const int32_t type = vector_type(x);
    void* const s = stream();
    return unlocked([&] {
      return tq_append(p, x.ptr, type, x.rows, x.rows ? x.stride : p->d, c.idx, c.qjl, c.gamma, c.norm, first, step, s);
    });
  });
}

// p, idx, qjl, gamma, norm, x_out
PyObject* dequantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 6, [&] {
    const tq_params* p = params(a[0]);
    const Rows x = matrix(a[5]);
    if (x.type != at::kFloat) throw NotPlain{};
    const Codes c = codes(p, a + 1, x.rows);
    void* const s = stream();
    return unlocked([&] {
      return tq_dequantize(p, c.idx, c.qjl, c.gamma, c.norm, x.rows, static_cast<float*>(x.ptr), x.rows ? x.stride : p->d, s);
    });
  });
}

// p, q, n_groups, q_per_group, idx, qjl, gamma, norm, n_per_group, scores, topk, topk_idx, topk_val
PyObject* score(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 13, [&] {
    const tq_params* p = params(a[0]);
    const Rows q = matrix(a[1]);
    const int32_t groups = integer32(a[2]), per_group = integer32(a[3]), topk = integer32(a[10]);
    const int64_t keys = integer(a[8]);
    if (q.type != at::kFloat || groups < 0 || per_group < 0 || topk < 0 || keys < 0 || keys > 0x7fffffff) throw NotPlain{};
    const int64_t nq = (int64_t)groups * per_group;
    if (q.rows < nq) throw NotPlain{};
    const Codes c = codes(p, a + 4, groups * keys);
    Rows s{nullptr, 0, 0, keys, at::kFloat};
    if (a[9] != Py_None) {
      s = matrix(a[9]);
      if (s.type != at::kFloat || s.rows < nq || s.cols < keys) throw NotPlain{};
      if (s.rows == 0) s.stride = keys;
    }
    int32_t* const ti = array<int32_t>(a[11], at::kInt, nq * topk);
    float* const tv = array<float>(a[12], at::kFloat, nq * topk);
    void* const st = stream();
    return unlocked([&] {
      return tq_score(p, static_cast<const float*>(q.ptr), q.rows ? q.stride : p->d, groups, per_group, c.idx, c.qjl, c.gamma, c.norm,
                      keys, static_cast<float*>(s.ptr), s.stride, topk, ti, tv, st);
    });
  });
}

// pk, pv, q, n_groups, q_per_group, k_codes, v_codes, n_per_group, scale, out, group_stride or None
PyObject* attend(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 11, [&] {
    const tq_params *pk = params(a[0]), *pv = params(a[1]);
    const Rows q = matrix(a[2]), out = matrix(a[9]);
    const int32_t groups = integer32(a[3]), per_group = integer32(a[4]);
    const int64_t keys = integer(a[7]), stride = a[10] == Py_None ? keys : integer(a[10]);
    if (q.type != at::kFloat || out.type != at::kFloat || !PyFloat_CheckExact(a[8])) throw NotPlain{};
    const float scale = (float)PyFloat_AS_DOUBLE(a[8]);
    Codes c[2];
    for (int i = 0; i < 2; ++i) {
      if (!PyTuple_CheckExact(a[5 + i]) || PyTuple_GET_SIZE(a[5 + i]) != 4) throw NotPlain{};
      PyObject* const arrays[4] = {PyTuple_GET_ITEM(a[5 + i], 0), PyTuple_GET_ITEM(a[5 + i], 1), PyTuple_GET_ITEM(a[5 + i], 2),
                                   PyTuple_GET_ITEM(a[5 + i], 3)};
      c[i] = codes(i == 0 ? pk : pv, arrays, 0);
    }
    if (pk->workspace_bytes < tq_attend_workspace_bytes(pk, pv, groups, per_group, keys)) throw NotPlain{};  // the caller grows it
    void* const s = stream();
    return unlocked([&] {
      return tq_attend_cache(pk, pv, static_cast<const float*>(q.ptr), q.rows ? q.stride : pk->d, groups, per_group, c[0].idx, c[0].qjl,
                             c[0].gamma, c[0].norm, c[1].idx, c[1].qjl, c[1].gamma, c[1].norm, keys, stride, scale,
                             static_cast<float*>(out.ptr), out.rows ? out.stride : pv->d, s);
    });
  });
}

#define TQ_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {TQ_METHOD(quantize_mse), TQ_METHOD(quantize_prod), TQ_METHOD(append), TQ_METHOD(dequantize),
                         TQ_METHOD(score), TQ_METHOD(attend), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tqcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tqcall(void) { return PyModule_Create(&module); }
