// The calls of a small problem from Python without the cost of marshalling them in Python: dfs_forward, the token orders and the staged calls
// of a quality check take their arguments straight from the objects.  A launch costs the host some 3 us and its kernel often less, so what bounds
// such calls is what Python does between two of them: some fifty attribute lookups of tensors and a ctypes call.  Measured (us, in Python ->
// here).  The host's time of a call in a burst of eight: refresh and reuse step of 256 fp32 tokens (one launch each) 9.7 -> 4.7 and 9.9 -> 5.0, token
// order 6.4 -> 3.9.  A call among others: token order of 75 600 or 64 tokens 6.2 -> 3.6, reuse step of 512 tokens x 8 heads, d = 64,
// 9.4 -> 7.3, of 256 fp32 tokens 9.2 -> 8.7; the refresh step of these stays at 12.4, which its kernel takes.
// A quality check in staged calls (nine of them and two of torch), 675 tokens x 2 heads, d = 64, 73 -> 53, 1 575 x 2 73 -> 62; larger ones
// take what their kernels take (2 625 x 4, d = 128, 111).
//
// The module holds the version of the torch it was built against, whose classes it reads: binding.py uses it with no other.
// A call goes to the library only if every argument is of the plain kind and passes every check of binding.py; else None is returned,
// nothing has happened, and binding.py does the call, or raises, in its own way.
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>

#include <cstring>

#include "../../include/dfsattn.h"

namespace {

PyObject* g_geom_type = nullptr;                    // binding.Geom, a ctypes structure with the layout of dfs_geom
PyObject *s_kv_idx, *s_kv_cnt, *s_mask, *s_k_head, *s_K_max;

struct NotPlain {};                                 // thrown where binding.py has to look at an argument

void need(bool ok) {
  if (!ok) throw NotPlain();
}

int to_int(PyObject* x) {
  need(PyLong_CheckExact(x));
  int overflow = 0;
  const long v = PyLong_AsLongAndOverflow(x, &overflow);
  need(!overflow && v == long(int(v)));
  return int(v);
}

double to_double(PyObject* x) {
  if (PyFloat_CheckExact(x)) return PyFloat_AS_DOUBLE(x);
  return double(to_int(x));
}

dfs_geom to_geom(PyObject* x) {
  need(reinterpret_cast<PyObject*>(Py_TYPE(x)) == g_geom_type);
  dfs_geom g;
  Py_buffer b;
  need(PyObject_GetBuffer(x, &b, PyBUF_SIMPLE) == 0);
  const bool fits = b.len == Py_ssize_t(sizeof(g));
  if (fits) std::memcpy(&g, b.buf, sizeof(g));
  PyBuffer_Release(&b);
  need(fits);
  return g;
}

// A contiguous device tensor of at least `numel` elements (of `type`, if one is given): its address.
void* to_ptr(PyObject* x, at::ScalarType type, int64_t numel, int64_t* bytes = nullptr) {
  need(THPVariable_CheckExact(x));
  const at::Tensor& t = THPVariable_Unpack(x);
  need(t.is_cuda() && t.is_contiguous() && (type == at::ScalarType::Undefined || t.scalar_type() == type) && t.numel() >= numel);
  if (bytes) *bytes = t.numel() * int64_t(t.element_size());
  return t.data_ptr();
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

struct Attr {                                       // an attribute, held while its address is in use
  PyObject* o;
  Attr(PyObject* from, PyObject* name) : o(PyObject_GetAttr(from, name)) { need(o != nullptr); }
  ~Attr() { Py_XDECREF(o); }
  Attr(const Attr&) = delete;
  void* ptr(at::ScalarType type, int64_t numel) const { return o == Py_None ? nullptr : to_ptr(o, type, numel); }
};

// Runs a call; None if an argument is not plain, else the library's status.
template <class F>
PyObject* guarded(F f) {
  int rc;
  try {
    rc = f();
  } catch (...) {                                   // NotPlain, or what torch throws about a tensor without memory
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  return PyLong_FromLong(rc);
}

PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> int {
    need(n == 15);
    const dfs_geom g = to_geom(a[0]);
    dfs_sizes s;
    need(dfs_geom_sizes(&g, &s) == DFS_OK);
    const int dtype = to_int(a[1]), mode = to_int(a[8]), refresh = PyObject_IsTrue(a[7]);
    need(refresh >= 0);
    const auto type = dtype == DFS_BF16 ? at::kBFloat16 : at::kFloat;
    const int64_t numel = int64_t(g.heads) * s.N * g.d, rows = int64_t(g.heads) * s.M;
    PyObject* st = a[11];
    const Attr kv_idx(st, s_kv_idx), kv_cnt(st, s_kv_cnt), mask(st, s_mask), k_head(st, s_k_head), K_max(st, s_K_max);
    dfs_mask_state m;
    m.K_max = to_int(K_max.o);
    m.kv_idx = static_cast<int32_t*>(kv_idx.ptr(at::kInt, rows * m.K_max));
    m.kv_cnt = static_cast<int32_t*>(kv_cnt.ptr(at::kInt, rows));
    m.mask = static_cast<uint8_t*>(mask.ptr(at::kByte, rows * s.M));
    m.k_head = static_cast<int32_t*>(k_head.ptr(at::kInt, g.heads));
    const void *q = to_ptr(a[2], type, numel), *k = to_ptr(a[3], type, numel), *v = to_ptr(a[4], type, numel);
    const auto* perm_pad = static_cast<const int32_t*>(to_ptr(a[5], at::kInt, s.N_pad));
    const auto* inv = static_cast<const int32_t*>(to_ptr(a[6], at::kInt, s.N));
    const double sparsity = to_double(a[9]), mass = to_double(a[10]);
    const float scale = float(to_double(a[12]));
    void* o = to_ptr(a[13], type, numel);
    int64_t ws_bytes = 0;
    void* ws = to_ptr(a[14], at::ScalarType::Undefined, 0, &ws_bytes);
    void* st_ = stream();
    PyThreadState* gil = PyEval_SaveThread();
    const int rc = dfs_forward(&g, dtype, q, k, v, perm_pad, inv, refresh, mode, sparsity, mass, &m, scale, o, ws, size_t(ws_bytes), st_);
    PyEval_RestoreThread(gil);
    return rc;
  });
}

PyObject* token_order(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> int {
    need(n == 6);
    const dfs_geom g = to_geom(a[0]);
    dfs_sizes s;
    need(dfs_geom_sizes(&g, &s) == DFS_OK);
    const int order = to_int(a[1]);
    auto* perm_pad = static_cast<int32_t*>(to_ptr(a[2], at::kInt, s.N_pad));
    auto* inv = static_cast<int32_t*>(to_ptr(a[3], at::kInt, s.N));
    auto* blk_valid = static_cast<int32_t*>(to_ptr(a[4], at::kInt, s.M));
    int64_t ws_bytes = 0;
    void* ws = to_ptr(a[5], at::ScalarType::Undefined, 0, &ws_bytes);
    void* st = stream();
    PyThreadState* gil = PyEval_SaveThread();
    const int rc = dfs_token_order(&g, order, perm_pad, inv, blk_valid, ws, size_t(ws_bytes), st);
    PyEval_RestoreThread(gil);
    return rc;
  });
}

// The staged calls.  Their arguments as binding.py passes them on, None where it takes None.
void* to_ptr_or_null(PyObject* x, at::ScalarType type, int64_t numel, int64_t* bytes = nullptr) {
  return x == Py_None ? nullptr : to_ptr(x, type, numel, bytes);
}
at::ScalarType tensor_type(int dtype) { return dtype == DFS_BF16 ? at::kBFloat16 : at::kFloat; }
struct Problem {
  dfs_geom g;
  dfs_sizes s;
  explicit Problem(PyObject* x) : g(to_geom(x)) { need(dfs_geom_sizes(&g, &s) == DFS_OK); }
  int64_t source() const { return int64_t(g.heads) * s.N * g.d; }
  int64_t ordered() const { return int64_t(g.heads) * s.N_pad * g.d; }
  int64_t scores() const { return int64_t(g.heads) * s.M_v * s.M_v; }
  int64_t rows() const { return int64_t(g.heads) * s.M; }
};
template <class F>
int without_gil(F f) {
  PyThreadState* gil = PyEval_SaveThread();
  const int rc = f();
  PyEval_RestoreThread(gil);
  return rc;
}

template <bool BACK>
PyObject* reorder(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> int {
    need(n == 5);
    const Problem p(a[0]);
    const int dtype = to_int(a[1]);
    const auto type = tensor_type(dtype);
    const void* x = to_ptr(a[2], type, BACK ? p.ordered() : p.source());
    const auto* index = static_cast<const int32_t*>(to_ptr(a[3], at::kInt, BACK ? p.s.N : p.s.N_pad));
    void *y = to_ptr(a[4], type, BACK ? p.source() : p.ordered()), *st = stream();
    return without_gil([&] { return BACK ? dfs_unperm(&p.g, dtype, x, index, y, st) : dfs_permute(&p.g, dtype, x, index, y, st); });
  });
}

PyObject* block_score(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> int {
    need(n == 6);
    const Problem p(a[0]);
    const int dtype = to_int(a[1]);
    const void *q = to_ptr(a[2], tensor_type(dtype), p.ordered()), *k = to_ptr(a[3], tensor_type(dtype), p.ordered());
    auto* score = static_cast<float*>(to_ptr(a[4], at::kFloat, p.scores()));
    int64_t ws_bytes = 0;
    void *ws = to_ptr(a[5], at::ScalarType::Undefined, 0, &ws_bytes), *st = stream();
    return without_gil([&] { return dfs_block_score(&p.g, dtype, q, k, score, ws, size_t(ws_bytes), st); });
  });
}

PyObject* select_mask(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> int {
    need(n == 11);
    const Problem p(a[0]);
    const auto* score = static_cast<const float*>(to_ptr(a[1], at::kFloat, p.scores()));
    const int mode = to_int(a[2]), K_max = to_int(a[8]);
    const double sparsity = to_double(a[3]), mass = to_double(a[4]);
    auto* mask = static_cast<uint8_t*>(to_ptr_or_null(a[5], at::kByte, p.rows() * p.s.M));
    auto *kv_idx = static_cast<int32_t*>(to_ptr(a[6], at::kInt, p.rows() * K_max)), *kv_cnt = static_cast<int32_t*>(to_ptr(a[7], at::kInt, p.rows()));
    auto* k_head = static_cast<int32_t*>(to_ptr_or_null(a[9], at::kInt, p.g.heads));
    int64_t ws_bytes = 0;
    void *ws = to_ptr_or_null(a[10], at::ScalarType::Undefined, 0, &ws_bytes), *st = stream();
    return without_gil([&] { return dfs_select_mask(&p.g, score, mode, sparsity, mass, mask, kv_idx, kv_cnt, K_max, k_head, ws, size_t(ws_bytes), st); });
  });
}

PyObject* sparse_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> int {
    need(n == 11);
    const Problem p(a[0]);
    const int dtype = to_int(a[1]), K_max = to_int(a[7]);
    const auto type = tensor_type(dtype);
    const void *q = to_ptr(a[2], type, p.ordered()), *k = to_ptr(a[3], type, p.ordered()), *v = to_ptr(a[4], type, p.ordered());
    const auto *kv_idx = static_cast<const int32_t*>(to_ptr(a[5], at::kInt, p.rows() * K_max)),
               *kv_cnt = static_cast<const int32_t*>(to_ptr(a[6], at::kInt, p.rows()));
    const float scale = float(to_double(a[8]));
    void* o = to_ptr(a[9], type, p.ordered());
    auto* lse = static_cast<float*>(to_ptr_or_null(a[10], at::kFloat, int64_t(p.g.heads) * p.s.N_pad));
    void* st = stream();
    return without_gil([&] { return dfs_sparse_attn_fwd(&p.g, dtype, q, k, v, kv_idx, kv_cnt, K_max, scale, o, lse, st); });
  });
}

PyObject* recall(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> int {
    need(n == 4);
    const Problem p(a[0]);
    const int64_t rows = int64_t(p.g.heads) * p.s.N_pad;
    const auto *kept = static_cast<const float*>(to_ptr(a[1], at::kFloat, rows)), *all = static_cast<const float*>(to_ptr(a[2], at::kFloat, rows));
    auto* out = static_cast<float*>(to_ptr(a[3], at::kFloat, p.g.heads));
    void* st = stream();
    return without_gil([&] { return dfs_recall(&p.g, kept, all, out, st); });
  });
}

PyObject* set_geom_type(PyObject*, PyObject* type) {
  Py_INCREF(type);
  g_geom_type = type;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(forward)), METH_FASTCALL, nullptr},
    {"token_order", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(token_order)), METH_FASTCALL, nullptr},
    {"permute", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(reorder<false>)), METH_FASTCALL, nullptr},
    {"unperm", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(reorder<true>)), METH_FASTCALL, nullptr},
    {"block_score", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(block_score)), METH_FASTCALL, nullptr},
    {"select_mask", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(select_mask)), METH_FASTCALL, nullptr},
    {"sparse_attn", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(sparse_attn)), METH_FASTCALL, nullptr},
    {"recall", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(recall)), METH_FASTCALL, nullptr},
    {"set_geom_type", set_geom_type, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
  s_kv_idx = PyUnicode_InternFromString("kv_idx");
  s_kv_cnt = PyUnicode_InternFromString("kv_cnt");
  s_mask = PyUnicode_InternFromString("mask");
  s_k_head = PyUnicode_InternFromString("k_head");
  s_K_max = PyUnicode_InternFromString("K_max");
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "torch_version", DFS_TORCH_VERSION) != 0) Py_CLEAR(m);
  return m;
}
