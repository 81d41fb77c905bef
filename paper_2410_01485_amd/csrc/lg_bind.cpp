// lg_bind.cpp — the tensor side of the binding as a CPython extension: checks the tensors of a call, takes their
// addresses and torch's current stream, and calls the C ABI.  Nothing here computes.
//
// A decode step of a small batch takes the GPU about 10 us; the same checks in Python took 6 us per call, so that the
// host was what a generation loop waited for.  Here they take well under one.
//
// The library is not linked: setup() receives the addresses of its entry points from the loader in binding.py (which
// may have loaded another build of it).  Every function takes its arguments by position (binding.py supplies names
// and defaults) and returns the lg_status of the call.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>
#include <string>
#include <vector>

#include "../../include/longgen_attn.h"

namespace {

struct PyFail {};  // the Python error indicator is set

// ---------------------------------------------------------------- the library's entry points
#define LG_ENTRIES(X)                                                                                           \
  X(lg_sparse_attn_fwd) X(lg_sparse_attn_bwd) X(lg_sparse_attn_fwd_varlen) X(lg_sparse_attn_bwd_varlen)         \
  X(lg_sparse_attn_decode) X(lg_sparse_attn_decode_cache) X(lg_sparse_attn_decode_cache_static)                 \
  X(lg_kv_ring_append) X(lg_sparse_attn_decode_paged) X(lg_kv_paged_append)
struct Entries {
#define X(name) decltype(&::name) name = nullptr;
  LG_ENTRIES(X)
#undef X
} lib;
PyObject* stream_getter = nullptr;  // torch._C._cuda_getCurrentRawStream

PyObject* setup(PyObject*, PyObject* args) {
  PyObject *table, *getter;
  if (!PyArg_ParseTuple(args, "O!O", &PyDict_Type, &table, &getter)) return nullptr;
#define X(name)                                                              \
  {                                                                          \
    PyObject* a = PyDict_GetItemString(table, #name);                        \
    if (!a) {                                                                \
      PyErr_SetString(PyExc_KeyError, #name);                                \
      return nullptr;                                                        \
    }                                                                        \
    lib.name = reinterpret_cast<decltype(lib.name)>(PyLong_AsVoidPtr(a));    \
    if (PyErr_Occurred()) return nullptr;                                    \
  }
  LG_ENTRIES(X)
#undef X
  Py_INCREF(getter);
  Py_XDECREF(stream_getter);
  stream_getter = getter;
  Py_RETURN_NONE;
}

// ---------------------------------------------------------------- arguments
const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "expected a torch tensor, got %s", Py_TYPE(o)->tp_name);
    throw PyFail();
  }
  return THPVariable_Unpack(o);
}

int integer(PyObject* o) {
  const long x = PyLong_AsLong(o);
  if (x == -1 && PyErr_Occurred()) throw PyFail();
  if (x != (long)(int)x) {
    PyErr_SetString(PyExc_OverflowError, "argument does not fit an int");
    throw PyFail();
  }
  return (int)x;
}

float number(PyObject* o) {
  const double x = PyFloat_AsDouble(o);
  if (x == -1.0 && PyErr_Occurred()) throw PyFail();
  return (float)x;
}

std::string shape_text(at::IntArrayRef s) {
  std::string t = "(";
  for (size_t x = 0; x < s.size(); ++x) t += (x ? ", " : "") + std::to_string(s[x]);
  return t + (s.size() == 1 ? ",)" : ")");
}

int64_t rank(const at::Tensor& t, int64_t dims) {
  if (t.dim() != dims) {
    PyErr_Format(PyExc_ValueError, "expected a tensor of %lld dimensions, got %s", (long long)dims,
                 shape_text(t.sizes()).c_str());
    throw PyFail();
  }
  return dims;
}

const char* type_name(at::ScalarType t) {
  switch (t) {
    case at::kFloat: return "torch.float32";
    case at::kBFloat16: return "torch.bfloat16";
    case at::kInt: return "torch.int32";
    case at::kHalf: return "torch.float16";
    case at::kDouble: return "torch.float64";
    default: return c10::toString(t);
  }
}

// t must be a contiguous device tensor of this shape and element type: the library reads every buffer of a call with
// the one dtype code it is given.  Returns its address.
void* checked(const at::Tensor& t, std::initializer_list<int64_t> shape, at::ScalarType type) {
  const at::IntArrayRef want(shape);
  if (!t.is_cuda() || !t.is_contiguous() || t.sizes() != want) {
    PyErr_Format(PyExc_ValueError, "expected a contiguous device tensor of shape %s, got %s", shape_text(want).c_str(),
                 shape_text(t.sizes()).c_str());
    throw PyFail();
  }
  if (t.scalar_type() != type) {
    PyErr_Format(PyExc_TypeError, "expected dtype %s, got %s", type_name(type), type_name(t.scalar_type()));
    throw PyFail();
  }
  return t.data_ptr();
}
void* checked(PyObject* o, std::initializer_list<int64_t> shape, at::ScalarType type) {
  return checked(tensor(o), shape, type);
}
float* lse_of(PyObject* o, std::initializer_list<int64_t> shape) {
  return o == Py_None ? nullptr : static_cast<float*>(checked(o, shape, at::kFloat));
}

int dtype_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return LG_F32;
  if (t.scalar_type() == at::kBFloat16) return LG_BF16;
  PyErr_Format(PyExc_TypeError, "unsupported dtype %s", type_name(t.scalar_type()));
  throw PyFail();
}

struct Workspace {
  void* p = nullptr;
  size_t bytes = 0;
};
Workspace workspace(PyObject* o) {
  Workspace w;
  if (o == Py_None) return w;
  const at::Tensor& t = tensor(o);
  if (!t.is_cuda() || !t.is_contiguous()) {
    PyErr_SetString(PyExc_TypeError, "the workspace must be a contiguous device tensor");
    throw PyFail();
  }
  w.p = t.data_ptr();
  w.bytes = t.nbytes();
  return w;
}

void* stream_of(const at::Tensor& t) {
  PyObject* dev = PyLong_FromLong(t.get_device());
  PyObject* r = dev ? PyObject_CallOneArg(stream_getter, dev) : nullptr;
  Py_XDECREF(dev);
  if (!r) throw PyFail();
  void* s = PyLong_AsVoidPtr(r);
  Py_DECREF(r);
  if (!s && PyErr_Occurred()) throw PyFail();
  return s;
}

// What every call ends with.
struct Tail {
  int dtype;
  float scale;
  void* stream;
};
Tail tail(const at::Tensor& t, PyObject* scale) { return {dtype_code(t), scale ? number(scale) : 0.f, stream_of(t)}; }

// Runs f without the interpreter lock: a launch can wait for room in the queue.
template <typename F>
PyObject* status(F&& f) {
  PyThreadState* s = PyEval_SaveThread();
  const int st = f();
  PyEval_RestoreThread(s);
  return PyLong_FromLong(st);
}

struct Pattern {
  int sink, window, block, stride;
};
Pattern pattern(PyObject* const* a) { return {integer(a[0]), integer(a[1]), integer(a[2]), integer(a[3])}; }

// Offsets of packed sequences: any sequence of integers.
std::vector<int> offsets(PyObject* o, int64_t total) {
  PyObject* f = PySequence_Fast(o, "cu_seqlens must be a sequence of integers");
  if (!f) throw PyFail();
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(f);
  std::vector<int> cu(n);
  bool ok = true;
  for (Py_ssize_t x = 0; x < n && ok; ++x) {
    PyObject* i = PyNumber_Long(PySequence_Fast_GET_ITEM(f, x));
    const long v = i ? PyLong_AsLong(i) : -1;
    ok = i && !(v == -1 && PyErr_Occurred());
    if (ok && v != (long)(int)v) {
      PyErr_SetString(PyExc_OverflowError, "cu_seqlens entry does not fit an int");
      ok = false;
    }
    if (ok) cu[x] = (int)v;
    Py_XDECREF(i);
  }
  Py_DECREF(f);
  if (!ok) throw PyFail();
  if (n < 2) {
    PyErr_SetString(PyExc_ValueError, "cu_seqlens needs at least two entries (one sequence)");
    throw PyFail();
  }
  if (cu[n - 1] != total) {
    PyErr_Format(PyExc_ValueError, "cu_seqlens ends at %d, the tensors hold %lld tokens", cu[n - 1], (long long)total);
    throw PyFail();
  }
  return cu;
}

// ---------------------------------------------------------------- the calls
#define LG_CALL(name, nargs)                                                                                       \
  PyObject* name##_impl(PyObject* const* a);                                                                       \
  PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n) {                                                    \
    if (n != (nargs)) {                                                                                            \
      PyErr_Format(PyExc_TypeError, #name " takes %d arguments, got %zd", (nargs), n);                             \
      return nullptr;                                                                                              \
    }                                                                                                              \
    try {                                                                                                          \
      return name##_impl(a);                                                                                       \
    } catch (const PyFail&) {                                                                                      \
    } catch (const std::exception& e) {                                                                            \
      PyErr_SetString(PyExc_RuntimeError, e.what());                                                               \
    }                                                                                                              \
    return nullptr;                                                                                                \
  }                                                                                                                \
  PyObject* name##_impl(PyObject* const* a)

// q k v out lse | sink window block stride scale
LG_CALL(fwd, 10) {
  const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]);
  rank(q, 4), rank(k, 4);
  const int64_t B = q.size(0), Hq = q.size(1), N = q.size(2), D = q.size(3), Hkv = k.size(1);
  const at::ScalarType t = q.scalar_type();
  void *pq = checked(q, {B, Hq, N, D}, t), *pk = checked(k, {B, Hkv, N, D}, t), *pv = checked(a[2], {B, Hkv, N, D}, t);
  void* po = checked(a[3], {B, Hq, N, D}, t);
  float* pl = lse_of(a[4], {B, Hq, N});
  const Pattern p = pattern(a + 5);
  const Tail z = tail(q, a[9]);
  return status([&] {
    return lib.lg_sparse_attn_fwd(pq, pk, pv, po, pl, B, Hq, Hkv, N, D, p.sink, p.window, p.block, p.stride,
                                  z.dtype, z.scale, z.stream);
  });
}

// q k v out lse dout dq dk dv workspace | sink window block stride scale
LG_CALL(bwd, 15) {
  const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]);
  rank(q, 4), rank(k, 4);
  const int64_t B = q.size(0), Hq = q.size(1), N = q.size(2), D = q.size(3), Hkv = k.size(1);
  const at::ScalarType t = q.scalar_type();
  const auto rows = {B, Hq, N, D}, keys = {B, Hkv, N, D};
  void *pq = checked(q, rows, t), *po = checked(a[3], rows, t);
  void *pg = checked(a[5], rows, t), *pdq = checked(a[6], rows, t);
  void *pk = checked(k, keys, t), *pv = checked(a[2], keys, t);
  void *pdk = checked(a[7], keys, t), *pdv = checked(a[8], keys, t);
  const float* pl = static_cast<float*>(checked(a[4], {B, Hq, N}, at::kFloat));
  const Workspace w = workspace(a[9]);
  const Pattern p = pattern(a + 10);
  const Tail z = tail(q, a[14]);
  return status([&] {
    return lib.lg_sparse_attn_bwd(pq, pk, pv, po, pl, pg, pdq, pdk, pdv, w.p, w.bytes, B, Hq, Hkv, N, D, p.sink,
                                  p.window, p.block, p.stride, z.dtype, z.scale, z.stream);
  });
}

// q k v out lse cu_seqlens | sink window block stride scale
LG_CALL(fwd_varlen, 11) {
  const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]);
  rank(q, 3), rank(k, 3);
  const int64_t Hq = q.size(0), T = q.size(1), D = q.size(2), Hkv = k.size(0);
  const at::ScalarType t = q.scalar_type();
  const std::vector<int> cu = offsets(a[5], T);
  void *pq = checked(q, {Hq, T, D}, t), *pk = checked(k, {Hkv, T, D}, t), *pv = checked(a[2], {Hkv, T, D}, t);
  void* po = checked(a[3], {Hq, T, D}, t);
  float* pl = lse_of(a[4], {Hq, T});
  const Pattern p = pattern(a + 6);
  const Tail z = tail(q, a[10]);
  return status([&] {
    return lib.lg_sparse_attn_fwd_varlen(pq, pk, pv, po, pl, cu.data(), (int)cu.size() - 1, Hq, Hkv, D, p.sink,
                                         p.window, p.block, p.stride, z.dtype, z.scale, z.stream);
  });
}

// q k v out lse dout dq dk dv workspace cu_seqlens | sink window block stride scale
LG_CALL(bwd_varlen, 16) {
  const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]);
  rank(q, 3), rank(k, 3);
  const int64_t Hq = q.size(0), T = q.size(1), D = q.size(2), Hkv = k.size(0);
  const at::ScalarType t = q.scalar_type();
  const std::vector<int> cu = offsets(a[10], T);
  const auto rows = {Hq, T, D}, keys = {Hkv, T, D};
  void *pq = checked(q, rows, t), *po = checked(a[3], rows, t);
  void *pg = checked(a[5], rows, t), *pdq = checked(a[6], rows, t);
  void *pk = checked(k, keys, t), *pv = checked(a[2], keys, t);
  void *pdk = checked(a[7], keys, t), *pdv = checked(a[8], keys, t);
  const float* pl = static_cast<float*>(checked(a[4], {Hq, T}, at::kFloat));
  const Workspace w = workspace(a[9]);
  const Pattern p = pattern(a + 11);
  const Tail z = tail(q, a[15]);
  return status([&] {
    return lib.lg_sparse_attn_bwd_varlen(pq, pk, pv, po, pl, pg, pdq, pdk, pdv, w.p, w.bytes, cu.data(),
                                         (int)cu.size() - 1, Hq, Hkv, D, p.sink, p.window, p.block, p.stride,
                                         z.dtype, z.scale, z.stream);
  });
}

// q k_cache v_cache out lse workspace N | sink window block stride scale
LG_CALL(decode, 12) {
  const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]);
  rank(q, 3), rank(k, 4);
  const int64_t B = q.size(0), Hq = q.size(1), D = q.size(2), Hkv = k.size(1);
  const at::ScalarType t = q.scalar_type();
  const Pattern p = pattern(a + 7);
  const int64_t C = (int64_t)p.sink + p.window;
  void *pq = checked(q, {B, Hq, D}, t), *pk = checked(k, {B, Hkv, C, D}, t), *pv = checked(a[2], {B, Hkv, C, D}, t);
  void* po = checked(a[3], {B, Hq, D}, t);
  float* pl = lse_of(a[4], {B, Hq});
  const Workspace w = workspace(a[5]);
  const int n_at = integer(a[6]);
  const Tail z = tail(q, a[11]);
  return status([&] {
    return lib.lg_sparse_attn_decode(pq, pk, pv, po, pl, w.p, w.bytes, B, Hq, Hkv, n_at, D, p.sink, p.window,
                                     p.block, p.stride, z.dtype, z.scale, z.stream);
  });
}

// q k_cache v_cache out lse workspace N | sink window block stride scale
LG_CALL(decode_cache, 12) {
  const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]);
  rank(q, 3), rank(k, 4);
  const int64_t B = q.size(0), Hq = q.size(1), D = q.size(2), Hkv = k.size(1), C = k.size(2);
  const at::ScalarType t = q.scalar_type();
  void *pq = checked(q, {B, Hq, D}, t), *pk = checked(k, {B, Hkv, C, D}, t), *pv = checked(a[2], {B, Hkv, C, D}, t);
  void* po = checked(a[3], {B, Hq, D}, t);
  float* pl = lse_of(a[4], {B, Hq});
  const Workspace w = workspace(a[5]);
  const Pattern p = pattern(a + 7);
  const int n_at = integer(a[6]);
  const Tail z = tail(q, a[11]);
  return status([&] {
    return lib.lg_sparse_attn_decode_cache(pq, pk, pv, po, pl, w.p, w.bytes, B, Hq, Hkv, n_at, D, p.sink, p.window,
                                           p.block, p.stride, C, z.dtype, z.scale, z.stream);
  });
}

// q k_cache v_cache out lse N | sink window block stride scale
LG_CALL(decode_cache_static, 11) {
  const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]);
  rank(q, 3), rank(k, 4);
  const int64_t B = q.size(0), Hq = q.size(1), D = q.size(2), Hkv = k.size(1), C = k.size(2);
  const at::ScalarType t = q.scalar_type();
  void *pq = checked(q, {B, Hq, D}, t), *pk = checked(k, {B, Hkv, C, D}, t), *pv = checked(a[2], {B, Hkv, C, D}, t);
  void* po = checked(a[3], {B, Hq, D}, t);
  float* pl = lse_of(a[4], {B, Hq});
  const Pattern p = pattern(a + 6);
  const int n_at = integer(a[5]);
  const Tail z = tail(q, a[10]);
  return status([&] {
    return lib.lg_sparse_attn_decode_cache_static(pq, pk, pv, po, pl, B, Hq, Hkv, n_at, D, p.sink, p.window,
                                                  p.block, p.stride, C, z.dtype, z.scale, z.stream);
  });
}

// k_new v_new k_cache v_cache pos | sink window block stride
LG_CALL(ring_append, 9) {
  const at::Tensor &k = tensor(a[0]), &kc = tensor(a[2]);
  rank(k, 4), rank(kc, 4);
  const int64_t B = k.size(0), Hkv = k.size(1), T = k.size(2), D = k.size(3), C = kc.size(2);
  const at::ScalarType t = k.scalar_type();
  void *pk = checked(k, {B, Hkv, T, D}, t), *pv = checked(a[1], {B, Hkv, T, D}, t);
  void *pkc = checked(kc, {B, Hkv, C, D}, t), *pvc = checked(a[3], {B, Hkv, C, D}, t);
  const Pattern p = pattern(a + 5);
  const int n_at = integer(a[4]);
  const Tail z = tail(k, nullptr);
  return status([&] {
    return lib.lg_kv_ring_append(pk, pv, pkc, pvc, B, Hkv, D, T, n_at, C, p.sink, p.window, p.block, p.stride,
                                 z.dtype, z.stream);
  });
}

// q k_pages v_pages page_table seq_lens out lse workspace n_max | sink window block stride scale
LG_CALL(decode_paged, 14) {
  const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &table = tensor(a[3]);
  rank(q, 3), rank(k, 4), rank(table, 2);
  const int64_t B = q.size(0), Hq = q.size(1), D = q.size(2);
  const int64_t pages = k.size(0), Hkv = k.size(1), ps = k.size(2), per_seq = table.size(1);
  const at::ScalarType t = q.scalar_type();
  void* pq = checked(q, {B, Hq, D}, t);
  void *pk = checked(k, {pages, Hkv, ps, D}, t), *pv = checked(a[2], {pages, Hkv, ps, D}, t);
  void* po = checked(a[5], {B, Hq, D}, t);
  const int32_t* pt = static_cast<int32_t*>(checked(table, {B, per_seq}, at::kInt));
  const int32_t* pn = static_cast<int32_t*>(checked(a[4], {B}, at::kInt));
  float* pl = lse_of(a[6], {B, Hq});
  const Workspace w = workspace(a[7]);
  const Pattern p = pattern(a + 9);
  const int n_at = integer(a[8]);
  const Tail z = tail(q, a[13]);
  return status([&] {
    return lib.lg_sparse_attn_decode_paged(pq, pk, pv, pt, pn, po, pl, w.p, w.bytes, B, Hq, Hkv, n_at, D, p.sink,
                                           p.window, p.block, p.stride, ps, per_seq, pages, z.dtype, z.scale,
                                           z.stream);
  });
}

// k_new v_new k_pages v_pages page_table positions n_max | sink window block stride
LG_CALL(paged_append, 11) {
  const at::Tensor &k = tensor(a[0]), &kp = tensor(a[2]), &table = tensor(a[4]);
  rank(k, 4), rank(kp, 4), rank(table, 2);
  const int64_t B = k.size(0), Hkv = k.size(1), T = k.size(2), D = k.size(3);
  const int64_t pages = kp.size(0), ps = kp.size(2), per_seq = table.size(1);
  const at::ScalarType t = k.scalar_type();
  void *pk = checked(k, {B, Hkv, T, D}, t), *pv = checked(a[1], {B, Hkv, T, D}, t);
  void *pkp = checked(kp, {pages, Hkv, ps, D}, t), *pvp = checked(a[3], {pages, Hkv, ps, D}, t);
  const int32_t* pt = static_cast<int32_t*>(checked(table, {B, per_seq}, at::kInt));
  const int32_t* pp = static_cast<int32_t*>(checked(a[5], {B}, at::kInt));
  const Pattern p = pattern(a + 7);
  const int n_at = integer(a[6]);
  const Tail z = tail(k, nullptr);
  return status([&] {
    return lib.lg_kv_paged_append(pk, pv, pkp, pvp, pt, pp, B, Hkv, D, T, n_at, p.sink, p.window, p.block,
                                  p.stride, ps, per_seq, pages, z.dtype, z.stream);
  });
}

PyMethodDef methods[] = {
    {"setup", setup, METH_VARARGS, "setup({entry point: address}, current raw stream of a device index)"},
#define M(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
    M(fwd), M(bwd), M(fwd_varlen), M(bwd_varlen), M(decode), M(decode_cache), M(decode_cache_static), M(ring_append),
    M(decode_paged), M(paged_append),
#undef M
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lg_bind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lg_bind() { return PyModule_Create(&module); }
