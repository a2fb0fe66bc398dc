// Python binding of the calls that sit in a model's loop (laq_evict, laq_decode_attention, laq_qcache_store)
// as a CPython extension: the marshalling of binding.py in C++.
//
// A small call is bound by the host: the kernels of one layer's step take a few microseconds, and what
// Python spends on unpacking tensors, filling ctypes structures and making output tensors took 10 us per
// decode call and 20 us per eviction; here it is 2 to 4.
//
// Every function takes exactly what its namesake in binding.py takes (positionally, defaults filled in
// there) and returns None for anything out of the ordinary -- a tensor of another type, device or layout,
// an argument that is not a plain number, anything that throws (no memory for an output, a tensor without an
// address) -- without having launched anything: binding.py then walks its own checks and raises what it always
// raised, of the type it always had.  An error of the library comes back as its (negative) code.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string.h>

#include <vector>

#include "laq.h"

namespace {

decltype(&laq_evict) fn_evict;
decltype(&laq_workspace_bytes) fn_workspace_bytes;
decltype(&laq_decode_attention) fn_decode_attention;
decltype(&laq_decode_workspace_bytes) fn_decode_workspace_bytes;
decltype(&laq_qcache_store) fn_qcache_store;
PyObject* get_device;      // torch._C._cuda_getDevice
PyObject* get_stream;      // torch._C._cuda_getCurrentRawStream

bool is_none(PyObject* o) { return o == Py_None; }
bool is_text(PyObject* o, const char* text) { return PyUnicode_Check(o) && PyUnicode_CompareWithASCIIString(o, text) == 0; }

// tensor on a GPU, or null
const at::Tensor* gpu_tensor(PyObject* o) {
  if (!THPVariable_Check(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.is_cuda() && t.layout() == at::kStrided ? &t : nullptr;
}

int dtype_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kBFloat16) return LAQ_BF16;
  if (t.scalar_type() == at::kFloat) return LAQ_F32;
  return -1;
}

bool aligned(const at::Tensor& t, uintptr_t to = 16) { return reinterpret_cast<uintptr_t>(t.data_ptr()) % to == 0; }

// a caller-supplied output: dense, of the type and on the device, large enough, aligned
const at::Tensor* output(PyObject* o, at::ScalarType type, int64_t numel, const at::Tensor& like) {
  const at::Tensor* t = gpu_tensor(o);
  if (!t || t->device() != like.device() || t->scalar_type() != type || !t->is_contiguous() || t->numel() < numel || !aligned(*t))
    return nullptr;
  return t;
}

bool as_int(PyObject* o, long long* v) {
  if (!PyLong_CheckExact(o)) return false;
  *v = PyLong_AsLongLong(o);
  if (*v == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return *v >= INT32_MIN && *v <= INT32_MAX;
}

// list or tuple of whole numbers
bool as_ints(PyObject* o, std::vector<int32_t>* out) {
  if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return false;
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
  PyObject** items = PySequence_Fast_ITEMS(o);
  out->resize(n);
  for (Py_ssize_t i = 0; i < n; ++i) {
    long long v;
    if (!as_int(items[i], &v)) return false;
    (*out)[i] = (int32_t)v;
  }
  return true;
}

// stream of the calling thread on the current device
bool current_stream(void** out) {
  PyObject* dev = PyObject_CallNoArgs(get_device);
  PyObject* st = dev ? PyObject_CallOneArg(get_stream, dev) : nullptr;
  Py_XDECREF(dev);
  if (!st) return false;
  *out = PyLong_AsVoidPtr(st);
  Py_DECREF(st);
  return !PyErr_Occurred();
}

at::Tensor make(at::IntArrayRef sizes, at::ScalarType type, const at::Tensor& like) {
  return at::empty(sizes, at::TensorOptions().dtype(type).device(like.device()));
}

PyObject* none() { Py_RETURN_NONE; }
// after a C++ exception: one that carries a Python exception (a dispatch mode raised it) leaves that set
PyObject* thrown() { return PyErr_Occurred() ? nullptr : none(); }

// rows of the packed outputs; false: a budget the library will refuse
bool packed_rows(const std::vector<int32_t>& budget, int64_t Hkv, int64_t L, int64_t* rows) {
  int64_t total = 0;
  for (const int32_t b : budget) {
    if (b < 1) return false;
    total += Hkv * (b < L ? b : L);
  }
  *rows = total;
  return true;
}

// evict(q_win, k, v, budget, pool_kernel, scale, scores, idx, k_out, v_out, ws, q_pos, keep, pool_mode,
//       want_scores, block_table, L, choose) -> (scores, idx, k_out, v_out) | error code | None
PyObject* evict(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  try {
    if (n_args != 18) return none();
    const at::Tensor *q = gpu_tensor(a[0]), *k = gpu_tensor(a[1]), *v = is_none(a[2]) ? nullptr : gpu_tensor(a[2]);
    if (!q || !k || (!v && !is_none(a[2])) || q->dim() != 4 || k->dim() != 4 || !q->is_contiguous() || k->stride(3) != 1) return none();
    const int dt = dtype_code(*k);
    if (dt < 0 || q->scalar_type() != k->scalar_type() || q->device() != k->device() || !aligned(*q) || !aligned(*k)) return none();
    laq_shape sh;
    memset(&sh, 0, sizeof sh);
    const int64_t n = q->size(0), Hkv = k->size(1), d = q->size(3);
    int64_t L = k->size(2);
    if (k->size(3) != d) return none();
    if (is_none(a[15])) {
      long long want_L;
      if (!is_none(a[16]) && (!as_int(a[16], &want_L) || want_L != L)) return none();
      if (k->size(0) != n) return none();
      if (!k->is_contiguous()) {
        sh.kv_stride_inst = k->stride(0);
        sh.kv_stride_head = k->stride(1);
        sh.kv_stride_row = k->stride(2);
      }
    } else {
      const at::Tensor* table = gpu_tensor(a[15]);
      long long want_L;
      if (!table || !as_int(a[16], &want_L) || want_L < 1) return none();
      const int64_t rows = k->size(2);
      L = want_L;
      if (table->device() != k->device() || table->scalar_type() != at::kInt || table->dim() != 2 || !table->is_contiguous() ||
          rows < 1 || rows % 256 || rows > INT32_MAX || table->size(0) != n || table->size(1) != (L + rows - 1) / rows)
        return none();
      if (k->stride(1) != rows * d || k->stride(2) != d) {
        sh.kv_stride_head = k->stride(1);
        sh.kv_stride_row = k->stride(2);
      }
      sh.block_table = table->data_ptr<int32_t>();
      sh.block_rows = (int32_t)rows;
      sh.kv_stride_block = k->stride(0);
    }
    if (n < 1 || n > INT32_MAX || q->size(1) > INT32_MAX || Hkv > INT32_MAX || L > INT32_MAX || q->size(2) > INT32_MAX) return none();
    std::vector<int32_t> budget, pos;
    int64_t rows = 0;
    long long pool, keep = -1;
    if (!as_ints(a[3], &budget) || (int64_t)budget.size() != n || !packed_rows(budget, Hkv, L, &rows) || !as_int(a[4], &pool)) return none();
    const double scale = PyFloat_CheckExact(a[5]) ? PyFloat_AS_DOUBLE(a[5]) : -1.0;
    if (!PyFloat_CheckExact(a[5])) return none();
    if (!is_none(a[11])) {
      if (!as_ints(a[11], &pos) || (int64_t)pos.size() != q->size(2)) return none();
      sh.q_pos = pos.data();
    }
    if (!is_none(a[12]) && !as_int(a[12], &keep)) return none();
    if (is_text(a[13], "max")) sh.pool_mode = LAQ_POOL_MAX;
    else if (is_text(a[13], "avg")) sh.pool_mode = LAQ_POOL_AVG;
    else return none();
    if (is_text(a[17], "auto")) sh.score_choice = LAQ_CHOOSE_AUTO;
    else if (is_text(a[17], "two-pass")) sh.score_choice = LAQ_CHOOSE_TWO_PASS;
    else if (is_text(a[17], "single-read")) sh.score_choice = LAQ_CHOOSE_SINGLE_READ;
    else return none();
    if (!PyBool_Check(a[14])) return none();
    if (v) {
      if (v->scalar_type() != k->scalar_type() || v->device() != k->device() || v->sizes() != k->sizes() ||
          v->strides() != k->strides() || !aligned(*v))
        return none();
    } else if (!is_none(a[9])) {
      return none();
    }
    sh.n_inst = (int32_t)n; sh.Hq = (int32_t)q->size(1); sh.Hkv = (int32_t)Hkv; sh.d = (int32_t)d; sh.L = (int32_t)L;
    sh.W = (int32_t)q->size(2); sh.dtype = dt; sh.scale = (float)scale; sh.keep = (int32_t)keep;

    // outputs: what the caller gave, else new ones
    at::Tensor made[5];
    const at::Tensor* out[5] = {};         // scores, idx, k_out, v_out, ws
    const at::ScalarType type[4] = {at::kFloat, at::kInt, k->scalar_type(), k->scalar_type()};
    const int64_t numel[4] = {n * Hkv * L, rows, rows * d, rows * d};
    for (int i = 0; i < 4; ++i)
      if (!is_none(a[6 + i]) && !(out[i] = output(a[6 + i], type[i], numel[i], *k))) return none();
    const size_t need = fn_workspace_bytes(&sh);
    if (need == 0) return none();
    if (!is_none(a[10])) {
      out[4] = gpu_tensor(a[10]);
      if (!out[4] || out[4]->device() != k->device() || !out[4]->is_contiguous() || !aligned(*out[4], 256)) return none();
    }
    if (!out[0] && a[14] == Py_True) out[0] = &(made[0] = make({n, Hkv, L}, at::kFloat, *k));
    if (!out[1]) out[1] = &(made[1] = make({rows}, at::kInt, *k));
    if (!out[2]) out[2] = &(made[2] = make({rows, d}, type[2], *k));
    if (v && !out[3]) out[3] = &(made[3] = make({rows, d}, type[3], *k));
    if (!out[4]) out[4] = &(made[4] = make({(int64_t)need}, at::kByte, *k));
    void* stream;
    if (!current_stream(&stream)) return nullptr;
    // (a tensor without memory throws when it is asked for its address: not where the GIL is released)
    int rc;
    const size_t ws_bytes = out[4]->numel() * out[4]->element_size();
    const void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v ? v->data_ptr() : nullptr;
    void* op[5];
    for (int i = 0; i < 5; ++i) op[i] = out[i] ? out[i]->data_ptr() : nullptr;
    Py_BEGIN_ALLOW_THREADS;
    rc = fn_evict(&sh, qp, kp, vp, budget.data(), (int)pool, static_cast<float*>(op[0]), static_cast<int32_t*>(op[1]), op[2],
                  op[3], op[4], ws_bytes, stream);
    Py_END_ALLOW_THREADS;
    if (rc != LAQ_OK) return PyLong_FromLong(rc);
    PyObject* res = PyTuple_New(4);
    if (!res) return nullptr;
    for (int i = 0; i < 4; ++i) {
      PyObject* o;
      if (!is_none(a[6 + i]) || !out[i]) {           // the caller's own, or no such output
        o = a[6 + i];
        Py_INCREF(o);
      } else {
        o = THPVariable_Wrap(std::move(made[i]));
        if (!o) {
          Py_DECREF(res);
          return nullptr;
        }
      }
      PyTuple_SET_ITEM(res, i, o);
    }
    return res;
  } catch (const std::exception&) {
    return thrown();
  }
}

// decode(q, k_c, v_c, budget, Hkv, L, scale, out, ws, split) -> out | error code | None
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  try {
    if (n_args != 10) return none();
    const at::Tensor *q = gpu_tensor(a[0]), *k = gpu_tensor(a[1]), *v = gpu_tensor(a[2]);
    if (!q || !k || !v || q->dim() != 3 || k->dim() != 2 || v->dim() != 2) return none();
    const int dt = dtype_code(*q);
    std::vector<int32_t> budget;
    long long Hkv, L;
    int64_t rows = 0;
    const int64_t n = q->size(0), Hq = q->size(1), d = q->size(2);
    if (dt < 0 || k->scalar_type() != q->scalar_type() || v->scalar_type() != q->scalar_type() || k->device() != q->device() ||
        v->device() != q->device() || !q->is_contiguous() || !k->is_contiguous() || !v->is_contiguous() || !as_ints(a[3], &budget) ||
        (int64_t)budget.size() != n || !as_int(a[4], &Hkv) || !as_int(a[5], &L) || Hkv < 1 || L < 1 || !packed_rows(budget, Hkv, L, &rows) ||
        k->size(0) != rows || k->size(1) != d || v->size(0) != rows || v->size(1) != d || !PyFloat_CheckExact(a[6]) || !PyBool_Check(a[9]) ||
        n < 1 || n > INT32_MAX || Hq > INT32_MAX)
      return none();
    laq_shape sh;
    memset(&sh, 0, sizeof sh);
    sh.n_inst = (int32_t)n; sh.Hq = (int32_t)Hq; sh.Hkv = (int32_t)Hkv; sh.d = (int32_t)d; sh.L = (int32_t)L; sh.W = 1; sh.dtype = dt;
    sh.scale = (float)PyFloat_AS_DOUBLE(a[6]);
    at::Tensor made, scratch;
    const at::Tensor *out = nullptr, *ws = nullptr;
    if (!is_none(a[7]) && !(out = output(a[7], at::kFloat, n * Hq * d, *q))) return none();
    if (a[9] == Py_True) {
      if (!is_none(a[8])) {
        if (!(ws = gpu_tensor(a[8]))) return none();
      } else if (const size_t need = fn_decode_workspace_bytes(&sh, budget.data())) {
        ws = &(scratch = make({(int64_t)need}, at::kByte, *q));
      }
    }
    if (!out) out = &(made = make({n, Hq, d}, at::kFloat, *q));
    void* stream;
    if (!current_stream(&stream)) return nullptr;
    int rc;
    const size_t ws_bytes = ws ? ws->numel() * ws->element_size() : 0;
    const void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr();
    void *op = out->data_ptr(), *wp = ws ? ws->data_ptr() : nullptr;
    Py_BEGIN_ALLOW_THREADS;
    rc = fn_decode_attention(&sh, qp, kp, vp, budget.data(), static_cast<float*>(op), wp, ws_bytes, stream);
    Py_END_ALLOW_THREADS;
    if (rc != LAQ_OK) return PyLong_FromLong(rc);
    if (!is_none(a[7])) {
      Py_INCREF(a[7]);
      return a[7];
    }
    return THPVariable_Wrap(std::move(made));
  } catch (const std::exception&) {
    return thrown();
  }
}

// qcache_store(q_cache, q_step, t) -> q_cache | error code | None
PyObject* qcache_store(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  try {
    if (n_args != 3) return none();
    const at::Tensor *c = gpu_tensor(a[0]), *q = gpu_tensor(a[1]);
    long long t;
    if (!c || !q || c->dim() != 4 || q->dim() != 3 || !c->is_contiguous() || !q->is_contiguous() || c->scalar_type() != q->scalar_type() ||
        c->device() != q->device() || q->size(0) != c->size(0) || q->size(1) != c->size(1) || q->size(2) != c->size(3) || !as_int(a[2], &t))
      return none();
    const int dt = dtype_code(*c);
    if (dt < 0 || c->size(0) < 1 || c->size(0) > INT32_MAX || c->size(1) > INT32_MAX || c->size(2) < 1 || c->size(2) > INT32_MAX) return none();
    laq_shape sh;
    memset(&sh, 0, sizeof sh);
    sh.n_inst = (int32_t)c->size(0); sh.Hq = sh.Hkv = (int32_t)c->size(1); sh.d = (int32_t)c->size(3);
    sh.L = sh.W = (int32_t)c->size(2); sh.dtype = dt;
    void* stream;
    if (!current_stream(&stream)) return nullptr;
    int rc;
    const void* qp = q->data_ptr();
    void* cp = c->data_ptr();
    Py_BEGIN_ALLOW_THREADS;
    rc = fn_qcache_store(&sh, qp, (int32_t)t, cp, stream);
    Py_END_ALLOW_THREADS;
    if (rc != LAQ_OK) return PyLong_FromLong(rc);
    Py_INCREF(a[0]);
    return a[0];
  } catch (const std::exception&) {
    return thrown();
  }
}

// bind(addresses of laq_evict, laq_workspace_bytes, laq_decode_attention, laq_decode_workspace_bytes, laq_qcache_store,
//      torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)
PyObject* bind(PyObject*, PyObject* args) {
  unsigned long long f[5];
  PyObject *dev, *st;
  if (!PyArg_ParseTuple(args, "KKKKKOO", &f[0], &f[1], &f[2], &f[3], &f[4], &dev, &st)) return nullptr;
  fn_evict = reinterpret_cast<decltype(fn_evict)>(f[0]);
  fn_workspace_bytes = reinterpret_cast<decltype(fn_workspace_bytes)>(f[1]);
  fn_decode_attention = reinterpret_cast<decltype(fn_decode_attention)>(f[2]);
  fn_decode_workspace_bytes = reinterpret_cast<decltype(fn_decode_workspace_bytes)>(f[3]);
  fn_qcache_store = reinterpret_cast<decltype(fn_qcache_store)>(f[4]);
  Py_INCREF(dev);
  Py_INCREF(st);
  get_device = dev;
  get_stream = st;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"evict", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(evict)), METH_FASTCALL, nullptr},
    {"decode", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode)), METH_FASTCALL, nullptr},
    {"qcache_store", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(qcache_store)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
