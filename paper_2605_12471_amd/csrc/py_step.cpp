// The Python binding's step in native code: what KvFoldCache.step() does for a call in its ordinary form, from the tensors' own fields
// instead of a dozen Python attributes.  A step was queued from Python in 9.3 us (two launches; 7.1 with one), of which the library and the HIP runtime
// take 5.9 (3.9), and the kernels of a decoding step less than the whole: one token on 1000 keys 7.1 us.
//
// step() answers None for whatever is not in that form -- other types, shapes, devices, layouts, tensors without storage, conflicting
// options, numbers out of range -- and the caller then goes the way of plain Python, which raises what it always has.
#include <Python.h>

#include <c10/core/ScalarType.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <cstdint>
#include <new>

#include "../../include/kvfold.h"

namespace {

struct Cache {
  decltype(&kvfold_step_ex) step_ex;
  decltype(&kvfold_step_noalloc) step_noalloc;
  decltype(&kvfold_step_rope) step_rope;
  decltype(&kvfold_step_window) step_window;
  kvfold_cache_t* handle;
  int64_t device, n_q_heads, n_kv_heads, head_dim;
  c10::ScalarType dtype;
};

// The tensor's memory if it is a plain one of this shape on the device, nullptr if not.
void* plain(PyObject* obj, const Cache& c, c10::ScalarType dtype, c10::IntArrayRef shape) {
  if (!THPVariable_CheckExact(obj)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(obj);
  if (!t.defined() || !t.has_storage() || t.layout() != c10::kStrided || !t.is_cuda() || t.get_device() != c.device || t.scalar_type() != dtype ||
      t.sizes() != shape || !t.is_contiguous())
    return nullptr;
  return t.data_ptr();
}

bool whole_number(PyObject* obj, int64_t lo, int64_t hi, int64_t* out) {
  if (!PyLong_CheckExact(obj)) return false;
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(obj, &overflow);
  if (overflow || v < lo || v > hi) return false;
  *out = v;
  return true;
}

void free_cache(PyObject* capsule) { delete static_cast<Cache*>(PyCapsule_GetPointer(capsule, "kvfold")); }

// bind(step_ex, step_noalloc, step_rope, step_window, handle, device, n_q_heads, n_kv_heads, head_dim, bf16): the addresses as integers
PyObject* bind(PyObject*, PyObject* args) {
  unsigned long long f[4], handle;
  long long device, hq, hkv, d;
  int bf16;
  if (!PyArg_ParseTuple(args, "KKKKKLLLLp", &f[0], &f[1], &f[2], &f[3], &handle, &device, &hq, &hkv, &d, &bf16)) return nullptr;
  Cache* c = new (std::nothrow) Cache;
  if (!c) return PyErr_NoMemory();
  c->step_ex = reinterpret_cast<decltype(c->step_ex)>(f[0]);
  c->step_noalloc = reinterpret_cast<decltype(c->step_noalloc)>(f[1]);
  c->step_rope = reinterpret_cast<decltype(c->step_rope)>(f[2]);
  c->step_window = reinterpret_cast<decltype(c->step_window)>(f[3]);
  c->handle = reinterpret_cast<kvfold_cache_t*>(handle);
  c->device = device;
  c->n_q_heads = hq;
  c->n_kv_heads = hkv;
  c->head_dim = d;
  c->dtype = bf16 ? c10::ScalarType::BFloat16 : c10::ScalarType::Float;
  PyObject* capsule = PyCapsule_New(c, "kvfold", free_cache);
  if (!capsule) delete c;
  return capsule;
}

// step(cache, layer, q, k_new, v_new, out, pos, lse, stream, rope, window, noalloc): the library's status, or None
PyObject* step(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  if (n_args != 12) {
    PyErr_SetString(PyExc_TypeError, "step: 12 arguments");
    return nullptr;
  }
  Cache* c = static_cast<Cache*>(PyCapsule_GetPointer(a[0], "kvfold"));
  if (!c) return nullptr;
  try {
    int64_t layer, pos, n_sink = 0, window = 0;
    if (!whole_number(a[1], INT32_MIN, INT32_MAX, &layer) || !whole_number(a[6], INT64_MIN, INT64_MAX, &pos)) Py_RETURN_NONE;
    if (!THPVariable_CheckExact(a[2])) Py_RETURN_NONE;
    const at::Tensor& qt = THPVariable_Unpack(a[2]);
    if (!qt.defined() || qt.dim() != 3) Py_RETURN_NONE;
    const int64_t n = qt.size(0);
    if (n > INT32_MAX) Py_RETURN_NONE;
    const int64_t wide[3] = {n, c->n_q_heads, c->head_dim}, narrow[3] = {n, c->n_kv_heads, c->head_dim}, per_head[2] = {c->n_q_heads, n}, angles[2] = {n, c->head_dim / 2};
    // (An empty tensor has no memory; the library's answer to it comes by the other way.)
    void *q = plain(a[2], *c, c->dtype, wide), *k = plain(a[3], *c, c->dtype, narrow), *v = plain(a[4], *c, c->dtype, narrow), *out = plain(a[5], *c, c->dtype, wide);
    if (!q || !k || !v || !out) Py_RETURN_NONE;
    float* lse = nullptr;
    if (a[7] != Py_None && !(lse = static_cast<float*>(plain(a[7], *c, c10::ScalarType::Float, per_head)))) Py_RETURN_NONE;
    void* stream;
    if (a[8] == Py_None) {
      stream = c10::hip::getCurrentHIPStream().stream();
    } else {
      int64_t s;
      if (!whole_number(a[8], 0, INT64_MAX, &s)) Py_RETURN_NONE;
      stream = reinterpret_cast<void*>(s);
    }
    const bool rope = a[9] != Py_None, win = a[10] != Py_None, noalloc = a[11] == Py_True;
    if (!noalloc && a[11] != Py_False) Py_RETURN_NONE;
    if ((int)rope + (int)win + (int)noalloc > 1) Py_RETURN_NONE;
    const float *cos = nullptr, *sin = nullptr;
    if (rope) {
      if (!PyTuple_CheckExact(a[9]) || PyTuple_GET_SIZE(a[9]) != 2) Py_RETURN_NONE;
      cos = static_cast<const float*>(plain(PyTuple_GET_ITEM(a[9], 0), *c, c10::ScalarType::Float, angles));
      sin = static_cast<const float*>(plain(PyTuple_GET_ITEM(a[9], 1), *c, c10::ScalarType::Float, angles));
      if (!cos || !sin) Py_RETURN_NONE;
    }
    if (win) {
      if (!PyTuple_CheckExact(a[10]) || PyTuple_GET_SIZE(a[10]) != 2 || !whole_number(PyTuple_GET_ITEM(a[10], 0), INT32_MIN, INT32_MAX, &n_sink) ||
          !whole_number(PyTuple_GET_ITEM(a[10], 1), INT64_MIN, INT64_MAX, &window))
        Py_RETURN_NONE;
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    if (win)
      rc = c->step_window(c->handle, (int)layer, q, k, v, (int32_t)n, pos, (int32_t)n_sink, window, out, lse, stream);
    else if (rope)
      rc = c->step_rope(c->handle, (int)layer, q, k, v, (int32_t)n, pos, cos, sin, out, lse, stream);
    else
      rc = (noalloc ? c->step_noalloc : c->step_ex)(c->handle, (int)layer, q, k, v, (int32_t)n, pos, out, lse, stream);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(rc);
  } catch (...) {
    Py_RETURN_NONE;  // (before anything was queued: the library throws nothing)
  }
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(step)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "kvfold_py_step", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_kvfold_py_step() {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
