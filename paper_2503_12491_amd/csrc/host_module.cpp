// Host module of the package (imported as _host): the parts of the drivers that run between the
// caller and the launches on every pass or token, where a Python statement per layer or argument
// costs as much as a kernel.  Argument hand-over and tensor views only.
#include <Python.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>

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

// session_stage(session, m, q_win, k, v, row_lse or None, indicator, ticket, stream): stage m of a session.
//   -> (admitted, return code, layers, K, V, indicator, position slabs): `layers`, those that were evicted into the
//   slabs, is None where there are none, the positions where they are not tracked.  The session's arrays are up to date.
PyObject* session_stage(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  bool ok = n == 9;
  for (int i = 2; ok && i < 7; ++i) ok = THPVariable_Check(args[i]) || (i == 5 && args[i] == Py_None);
  if (!ok) {
    PyErr_SetString(PyExc_TypeError, "session_stage(session, m, q_win, k, v, row_lse, indicator, ticket, stream)");
    return nullptr;
  }
  uint64_t a[4];
  if (!parse(args, 2, 2, a) || !parse(args + 7, 2, 2, a + 2)) return nullptr;
  const cake_session* s = at<const cake_session>(a[0]);
  const int64_t m = (int64_t)a[1];
  const uint32_t ticket = (uint32_t)a[2];
  void* stream = at<void>(a[3]);
  if (s == nullptr || m < 0 || m >= s->max_layers) {
    PyErr_SetString(PyExc_ValueError, "no session, or every layer has been admitted");
    return nullptr;
  }
  const at::Tensor &q = THPVariable_Unpack(args[2]), &k = THPVariable_Unpack(args[3]), &v = THPVariable_Unpack(args[4]),
                   &ind = THPVariable_Unpack(args[6]);
  const auto four = [](const at::Tensor& t) { return t.dim() == 4 && t.stride(3) == 1; };
  if (!four(q) || !four(k) || !four(v) || v.strides() != k.strides()) {
    PyErr_SetString(PyExc_AssertionError, "expect [B, H, rows, d] with contiguous d, k and v alike");
    return nullptr;
  }
  const float* lse = args[5] == Py_None ? nullptr : static_cast<const float*>(THPVariable_Unpack(args[5]).data_ptr());
  const void *qp = q.data_ptr(), *kp = k.data_ptr(), *vp = v.data_ptr();
  float* out = static_cast<float*>(ind.data_ptr());
  const int64_t qs[3] = {q.stride(0), q.stride(1), q.stride(2)}, ks[3] = {k.stride(0), k.stride(1), k.stride(2)};
  int rc = without_gil([&] {
    const int r = cake_session_scores(s, qp, kp, lse, out, qs, ks, ticket, stream);
    return r ? r : cake_session_wait(s, ticket, stream);
  });
  if (rc) return Py_BuildValue("iiOOOOO", 0, rc, Py_None, Py_None, Py_None, Py_None, Py_None);

  // layer m as it was handed over
  const int64_t B = s->shape.batch, L = s->max_layers, H = s->shape.n_kv_heads, d = s->shape.head_dim, w = s->shape.window,
                N = s->shape.seq_len, N_p = N - w;
  const double* got = static_cast<const double*>(s->mirror);
  for (int64_t b = 0; b < B; ++b) {
    s->pref[b * L + m] = got[b];
    s->hv[(b * L + m) * 2] = got[B + 2 * b];
    s->hv[(b * L + m) * 2 + 1] = got[B + 2 * b + 1];
    s->cur_len[m * B + b] = N_p;
  }
  const auto address = [](const void* p) { return (int64_t)reinterpret_cast<uintptr_t>(p); };
  s->k[m] = address(kp); s->v[m] = address(vp); s->ind[m] = address(out); s->pos[m] = 0;
  for (int i = 0; i < 3; ++i) s->strides[3 * m + i] = ks[i];
  s->cap[m] = N_p; s->off_kv[m] = s->off_i[m] = -1;
  const auto admitted = [](int code) { return Py_BuildValue("iiOOOOO", 1, code, Py_None, Py_None, Py_None, Py_None, Py_None); };

  // B^(m) of the layers seen so far, and the layers that it makes drop rows
  std::vector<int32_t> budget(m + 1), counts, cur, keep;
  for (int64_t b = 0; b < B; ++b) {
    if ((rc = cake_cascade_allocate(s->pref + b * L, (int32_t)(m + 1), s->total_budget, (int32_t)w, (int32_t)N, budget.data()))) return admitted(rc);
    for (int64_t l = 0; l <= m; ++l) s->budgets[l * B + b] = budget[l];
  }
  counts.assign(s->budgets, s->budgets + (m + 1) * B);
  cur.assign(s->cur_len, s->cur_len + (m + 1) * B);
  keep.resize(counts.size());
  if ((rc = cake_keep_counts(counts.data(), cur.data(), (int32_t)counts.size(), (int32_t)w, keep.data()))) return admitted(rc);
  std::vector<int64_t> layers, cap, off_kv, off_i;
  std::vector<int32_t> cl, kk;
  int64_t rows_kv = 0, rows_i = 0;
  for (int64_t l = 0; l <= m; ++l) {
    const int32_t *c = cur.data() + l * B, *n_keep = keep.data() + l * B;
    bool drops = false;
    for (int64_t b = 0; b < B; ++b) drops = drops || n_keep[b] < c[b];
    if (!drops) continue;
    layers.push_back(l);
    cap.push_back(*std::max_element(n_keep, n_keep + B));
    off_kv.push_back(rows_kv * B * H * d);
    off_i.push_back(rows_i * B * H);
    rows_kv += cap.back() + w;
    rows_i += std::max<int64_t>(cap.back(), 1);
    cl.insert(cl.end(), c, c + B);
    kk.insert(kk.end(), n_keep, n_keep + B);
  }
  const int32_t n_out = (int32_t)layers.size();
  if (n_out == 0) return admitted(0);

  // EVICT each of them: outputs carved from slabs of this stage
  const auto options = at::TensorOptions().device(k.device());
  const int64_t n_kv = rows_kv * B * H * d, n_i = rows_i * B * H;
  const at::Tensor k_slab = at::empty({n_kv}, options.dtype(k.dtype())), v_slab = at::empty({n_kv}, options.dtype(k.dtype())),
                   i_slab = at::empty({n_i}, options.dtype(at::kFloat)), idx_slab = at::empty({n_i}, options.dtype(at::kInt));
  // zero-filled: with a ragged batch the entries past a sequence's own count are never written
  at::Tensor p_slab;
  if (s->track_positions) p_slab = B > 1 ? at::zeros({n_i}, options.dtype(at::kInt)) : at::empty({n_i}, options.dtype(at::kInt));
  enum { kIndIn, kIdx, kKIn, kVIn, kKOut, kVOut, kIndOut, kPosIn, kPosOut, kRows };
  std::vector<uint64_t> words((size_t)kRows * n_out);
  std::vector<int64_t> strides;
  const int64_t eb = (int64_t)k.element_size();
  for (int32_t i = 0; i < n_out; ++i) {
    const int64_t l = layers[i];
    const auto put = [&](int row, int64_t x) { words[(size_t)row * n_out + i] = (uint64_t)x; };
    put(kIndIn, s->ind[l]); put(kKIn, s->k[l]); put(kVIn, s->v[l]); put(kPosIn, s->pos[l]);
    put(kIdx, address(idx_slab.data_ptr()) + off_i[i] * 4);
    put(kKOut, address(k_slab.data_ptr()) + off_kv[i] * eb);
    put(kVOut, address(v_slab.data_ptr()) + off_kv[i] * eb);
    put(kIndOut, address(i_slab.data_ptr()) + off_i[i] * 4);
    put(kPosOut, s->track_positions ? address(p_slab.data_ptr()) + off_i[i] * 4 : 0);
    strides.insert(strides.end(), s->strides + 3 * l, s->strides + 3 * l + 3);
  }
  cake_shape shape = s->shape;
  shape.n_layers = n_out;
  rc = without_gil([&] {
    if (int r = cake_write_words(s->tables, words.data(), kRows * n_out, stream)) return r;
    const auto row = [&](int r) { return s->tables + (size_t)r * n_out; };
    const auto in = [&](int r) { return const_cast<const void* const*>(row(r)); };
    const auto idx = reinterpret_cast<int32_t* const*>(row(kIdx));
    const auto ind_in = reinterpret_cast<const float* const*>(row(kIndIn));
    const auto ind_out = reinterpret_cast<float* const*>(row(kIndOut));
    if (int r = cake_select_topk(&shape, ind_in, cl.data(), kk.data(), idx, nullptr, 0, stream)) return r;
    return cake_compact_kv_positions(&shape, in(kKIn), in(kVIn), strides.data(), cl.data(), kk.data(), idx, ind_in, row(kKOut), row(kVOut), ind_out,
                                     s->track_positions ? reinterpret_cast<const int32_t* const*>(row(kPosIn)) : nullptr,
                                     s->track_positions ? reinterpret_cast<int32_t* const*>(row(kPosOut)) : nullptr, stream);
  });
  if (rc) return admitted(rc);
  PyObject* list = PyList_New(n_out);
  if (!list) return nullptr;
  for (int32_t i = 0; i < n_out; ++i) {
    const int64_t l = layers[i], rows = cap[i] + w;
    const auto word = [&](int row) { return (int64_t)words[(size_t)row * n_out + i]; };
    s->k[l] = word(kKOut); s->v[l] = word(kVOut); s->ind[l] = word(kIndOut); s->pos[l] = word(kPosOut);
    s->strides[3 * l] = H * rows * d; s->strides[3 * l + 1] = rows * d; s->strides[3 * l + 2] = d;
    s->cap[l] = cap[i]; s->off_kv[l] = off_kv[i]; s->off_i[l] = off_i[i];
    for (int64_t b = 0; b < B; ++b) s->cur_len[l * B + b] = kk[i * B + b];
    PyList_SET_ITEM(list, i, PyLong_FromLongLong(l));
  }
  PyObject* p = s->track_positions ? THPVariable_Wrap(p_slab) : (Py_INCREF(Py_None), Py_None);
  return Py_BuildValue("iiNNNNN", 1, 0, list, THPVariable_Wrap(k_slab), THPVariable_Wrap(v_slab), THPVariable_Wrap(i_slab), p);
  END_HANDLE_TH_ERRORS
}

// slab_views(slab, offsets, sizes) -> list of contiguous views of a slab, one per element offset and size tuple
PyObject* slab_views(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 3 || !THPVariable_Check(args[0]) || !PyList_Check(args[1]) || !PyList_Check(args[2]) || PyList_GET_SIZE(args[1]) != PyList_GET_SIZE(args[2])) {
    PyErr_SetString(PyExc_TypeError, "slab_views(slab, offsets, sizes)");
    return nullptr;
  }
  const at::Tensor& slab = THPVariable_Unpack(args[0]);
  const Py_ssize_t count = PyList_GET_SIZE(args[1]);
  PyObject* out = PyList_New(count);
  if (!out) return nullptr;
  for (Py_ssize_t i = 0; i < count; ++i) {
    const int64_t offset = PyLong_AsLongLong(PyList_GET_ITEM(args[1], i));
    PyObject* size = PyList_GET_ITEM(args[2], i);
    std::vector<int64_t> sizes;
    int64_t elements = 1;
    for (Py_ssize_t j = 0; PyTuple_Check(size) && j < PyTuple_GET_SIZE(size); ++j) {
      sizes.push_back(PyLong_AsLongLong(PyTuple_GET_ITEM(size, j)));
      elements *= sizes.back();
    }
    if (PyErr_Occurred() || offset < 0 || elements < 0 || sizes.empty() || offset + elements > slab.numel()) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a view outside the slab");
      Py_DECREF(out);
      return nullptr;
    }
    PyObject* view = view_of(slab, offset, sizes);
    if (!view) {
      Py_DECREF(out);
      return nullptr;
    }
    PyList_SET_ITEM(out, i, view);
  }
  return out;
  END_HANDLE_TH_ERRORS
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(name)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {METHOD(pass_launch), METHOD(pass_place), METHOD(wait_plan), METHOD(stream_wait), METHOD(layer_views), METHOD(decode_run),
                          METHOD(cascade_stage), METHOD(cascade_gather), METHOD(session_stage), METHOD(slab_views),
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host() { return PyModule_Create(&kModule); }
