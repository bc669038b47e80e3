// Host module of the package (imported as _host): the parts of the drivers that run between the
// caller and the launches on every pass or token, where a Python statement per layer or argument
// costs as much as a kernel.  Argument hand-over and tensor views only.
#include <Python.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <vector>

#include "cake_pass.h"

namespace {

// Releases the interpreter while the host launches or waits: with the device's queue full a launch waits too, and
// the program's other threads are to go on.
template <typename F>
int without_gil(F f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f();
  Py_END_ALLOW_THREADS
  return rc;
}

bool parse(PyObject* const* args, Py_ssize_t n, Py_ssize_t want, uint64_t* out) {
  if (n != want) {
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
    return false;
  }
  for (Py_ssize_t i = 0; i < n; ++i) {
    out[i] = PyLong_AsUnsignedLongLongMask(args[i]);
    if (PyErr_Occurred()) return false;
  }
  return true;
}
template <typename T> T* at(uint64_t x) { return reinterpret_cast<T*>(static_cast<uintptr_t>(x)); }

// pass_launch(pass, parts, ticket, stream) -> return code
PyObject* pass_launch(PyObject*, PyObject* const* args, Py_ssize_t n) {
  uint64_t a[4];
  if (!parse(args, n, 4, a)) return nullptr;
  return PyLong_FromLong(without_gil([&] { return cake_pass_launch(at<const cake_pass>(a[0]), (int32_t)a[1], (uint32_t)a[2], at<void>(a[3])); }));
}

// pass_place(pass, caps, tables, stream) -> return code
PyObject* pass_place(PyObject*, PyObject* const* args, Py_ssize_t n) {
  uint64_t a[4];
  if (!parse(args, n, 4, a)) return nullptr;
  return PyLong_FromLong(without_gil([&] { return cake_pass_place(at<const cake_pass>(a[0]), at<const int32_t>(a[1]), at<void*>(a[2]), at<void>(a[3])); }));
}

// wait_plan(mirror, ticket, stream) -> return code
PyObject* wait_plan(PyObject*, PyObject* const* args, Py_ssize_t n) {
  uint64_t a[3];
  if (!parse(args, n, 3, a)) return nullptr;
  return PyLong_FromLong(without_gil([&] { return cake_pass_wait_plan(at<const void>(a[0]), (uint32_t)a[1], at<void>(a[2])); }));
}

// stream_wait(stream) -> return code
PyObject* stream_wait(PyObject*, PyObject* const* args, Py_ssize_t n) {
  uint64_t a[1];
  if (!parse(args, n, 1, a)) return nullptr;
  return PyLong_FromLong(without_gil([&] { return cake_stream_wait(at<void>(a[0])); }));
}

// Calls that ask a tensor for anything turn the tensor library's exceptions into Python's (HANDLE_TH_ERRORS): a
// sparse tensor has no strides, one inside vmap no memory.

// A contiguous view of `base` at an element offset.  What Tensor.as_strided returns for a tensor that
// takes no part in autograd, made directly: 0.3 us instead of 2.
PyObject* view_of(const at::Tensor& base, int64_t offset, c10::IntArrayRef sizes) {
  auto impl = c10::make_intrusive<c10::TensorImpl>(c10::TensorImpl::VIEW, c10::Storage(base.storage()), base.key_set(), base.dtype());
  impl->set_storage_offset(base.storage_offset() + offset);
  impl->set_sizes_contiguous(sizes);
  return THPVariable_Wrap(at::Tensor(std::move(impl)));
}

// layer_views(pool_k, pool_v, pool_idx, pool_ind, keep, L, B, H_kv, S_w, d)
//   keep: address of int32 [L, B]
//   -> (idx, k, v, ind) lists of per-layer views: [B, H_kv, cap (+ S_w, d)], cap = max over b of keep,
//      the layers one after the other (the places cake_plan_eviction gives them)
PyObject* layer_views(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 10) {
    PyErr_SetString(PyExc_TypeError, "10 arguments expected");
    return nullptr;
  }
  for (int i = 0; i < 4; ++i)
    if (!THPVariable_Check(args[i])) {
      PyErr_SetString(PyExc_TypeError, "the pools must be tensors");
      return nullptr;
    }
  uint64_t a[6];
  if (!parse(args + 4, 6, 6, a)) return nullptr;
  const int32_t* keep = at<const int32_t>(a[0]);
  const int64_t L = (int64_t)a[1], B = (int64_t)a[2], H = (int64_t)a[3], s_w = (int64_t)a[4], d = (int64_t)a[5];
  const at::Tensor &pk = THPVariable_Unpack(args[0]), &pv = THPVariable_Unpack(args[1]);
  const at::Tensor &px = THPVariable_Unpack(args[2]), &pi = THPVariable_Unpack(args[3]);
  int64_t rows = 0;
  for (int64_t l = 0; l < L; ++l) rows += *std::max_element(keep + l * B, keep + (l + 1) * B);
  if (B * H * (rows + L * s_w) * d > std::min(pk.numel(), pv.numel()) || B * H * rows > std::min(px.numel(), pi.numel())) {
    PyErr_SetString(PyExc_ValueError, "the pools are smaller than the layers' rows");
    return nullptr;
  }
  PyObject* lists[4];
  for (auto& l : lists) l = PyList_New(L);
  int64_t before = 0;
  bool ok = lists[0] && lists[1] && lists[2] && lists[3];
  for (int64_t l = 0; ok && l < L; ++l) {
    const int64_t cap = *std::max_element(keep + l * B, keep + (l + 1) * B);
    const int64_t kv[4] = {B, H, cap + s_w, d}, ix[3] = {B, H, cap};
    const int64_t off_i = B * H * before, off_kv = B * H * (before + l * s_w) * d;
    PyObject* made[4] = {view_of(px, off_i, ix), view_of(pk, off_kv, kv), view_of(pv, off_kv, kv), view_of(pi, off_i, ix)};
    for (int i = 0; i < 4; ++i) {
      ok = ok && made[i] != nullptr;
      PyList_SET_ITEM(lists[i], l, made[i]);
    }
    before += cap;
  }
  PyObject* out = ok ? PyTuple_Pack(4, lists[0], lists[1], lists[2], lists[3]) : nullptr;
  for (auto& l : lists) Py_XDECREF(l);
  return out;
  END_HANDLE_TH_ERRORS
}

// decode_run(plan, q_new, k_new, v_new, stream) -> return code.  The tensors are [(layers,) B, heads, d] of the
// plan's rank with contiguous d, k_new and v_new alike.
PyObject* decode_run(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 5 || !THPVariable_Check(args[1]) || !THPVariable_Check(args[2]) || !THPVariable_Check(args[3])) {
    PyErr_SetString(PyExc_TypeError, "decode_run(plan, q_new, k_new, v_new, stream)");
    return nullptr;
  }
  uint64_t a[2];
  if (!parse(args, 1, 1, a) || !parse(args + 4, 1, 1, a + 1)) return nullptr;
  const at::Tensor &q = THPVariable_Unpack(args[1]), &k = THPVariable_Unpack(args[2]), &v = THPVariable_Unpack(args[3]);
  const int64_t dim = at<const cake_decode_plan>(a[0])->rank;
  if (q.dim() != dim || k.dim() != dim || v.dim() != dim || q.stride(dim - 1) != 1 || k.stride(dim - 1) != 1 ||
      v.strides() != k.strides()) {
    PyErr_SetString(PyExc_AssertionError, "q_new, k_new, v_new: [B, heads, d] (step) or [layers, B, heads, d] (step_all) with contiguous d, k_new and v_new alike");
    return nullptr;
  }
  const int64_t lead = dim - 3;
  const int64_t qs[3] = {lead ? q.stride(0) : 0, q.stride(lead), q.stride(lead + 1)};
  const int64_t ns[3] = {lead ? k.stride(0) : 0, k.stride(lead), k.stride(lead + 1)};
  const void *qp = q.data_ptr(), *kp = k.data_ptr(), *vp = v.data_ptr();
  return PyLong_FromLong(without_gil([&] { return cake_decode_run(at<const cake_decode_plan>(a[0]), qp, qs, kp, vp, ns, at<void>(a[1])); }));
  END_HANDLE_TH_ERRORS
}

// cascade_stage(cascade, m, q_win, k, v, indicator, stream) -> return code.  q_win, k, v are 4-d with contiguous d,
// v has k's strides.
PyObject* cascade_stage(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  bool ok = n == 7;
  for (int i = 2; ok && i < 6; ++i) ok = THPVariable_Check(args[i]);
  if (!ok) {
    PyErr_SetString(PyExc_TypeError, "cascade_stage(cascade, m, q_win, k, v, indicator, stream)");
    return nullptr;
  }
  uint64_t a[3];
  if (!parse(args, 2, 2, a) || !parse(args + 6, 1, 1, a + 2)) return nullptr;
  const at::Tensor &q = THPVariable_Unpack(args[2]), &k = THPVariable_Unpack(args[3]), &v = THPVariable_Unpack(args[4]),
                   &ind = THPVariable_Unpack(args[5]);
  const auto four = [](const at::Tensor& t) { return t.dim() == 4 && t.stride(3) == 1; };
  if (!four(q) || !four(k) || !four(v) || v.strides() != k.strides()) {
    PyErr_SetString(PyExc_AssertionError, "expect [B, H, rows, d] with contiguous d, k and v alike");
    return nullptr;
  }
  const void *qp = q.data_ptr(), *kp = k.data_ptr(), *vp = v.data_ptr();
  float* out = static_cast<float*>(ind.data_ptr());
  const int64_t qs[3] = {q.stride(0), q.stride(1), q.stride(2)}, ks[3] = {k.stride(0), k.stride(1), k.stride(2)};
  return PyLong_FromLong(without_gil([&] {
    return cake_cascade_stage(at<const cake_cascade>(a[0]), (int32_t)a[1], qp, kp, vp, out, qs, ks, at<void>(a[2]));
  }));
  END_HANDLE_TH_ERRORS
}

// cascade_gather(cascade, n_layers, pool_k, pool_v, stream) -> return code
PyObject* cascade_gather(PyObject*, PyObject* const* args, Py_ssize_t n) {
  uint64_t a[5];
  if (!parse(args, n, 5, a)) return nullptr;
  return PyLong_FromLong(without_gil([&] {
    return cake_cascade_gather(at<const cake_cascade>(a[0]), (int32_t)a[1], at<void>(a[2]), at<void>(a[3]), at<void>(a[4]));
  }));
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(name)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {METHOD(pass_launch), METHOD(pass_place), METHOD(wait_plan), METHOD(stream_wait), METHOD(layer_views), METHOD(decode_run),
                          METHOD(cascade_stage), METHOD(cascade_gather),
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host() { return PyModule_Create(&kModule); }
