// Native argument marshalling between torch tensors and the C ABI (mea.h): the
// ordinary case of attention.py's calls -- plain GPU tensors whose layout the
// kernels read in place -- as one call each.  Every function returns None for
// anything else, and for what the library refuses, before anything is launched;
// attention.py then takes its general path, which copies or raises.  A launch
// that fails is raised here, and not tried again.
//
// Why it exists: a training step on a small problem is bound by the host.
// Autograd runs the backward on a thread of its own, and each hand-over leaves
// the interpreter's working set cold, so the marshalling in Python, 52 us in a
// loop on one thread, took 178 us of every 1x1x256x256 forward + backward.
// The functions are found by address (init), so this module links to torch
// only and uses the library that _lib.load() loaded; errors are raised by
// _lib.check.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/hip/HIPStream.h>

#include <cmath>
#include <optional>

#include "../../include/mea.h"

namespace {

decltype(&mea_attention_fwd_workspace_size) g_fwd_ws;
decltype(&mea_attention_bwd_workspace_size) g_bwd_ws;
decltype(&mea_attention_fwd) g_fwd;
decltype(&mea_attention_bwd) g_bwd;
PyObject* g_check;  // check(name, status): raises what a status means

// A plain torch.Tensor or Parameter with storage on a GPU (no subclass, no
// functorch wrapper), or null.
const at::Tensor* gpu_tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.defined() && t.device().is_cuda() && t.layout() == at::kStrided && t.has_storage() ? &t : nullptr;
}

int dtype_code(at::ScalarType t) {
  return t == at::kFloat ? MEA_F32 : t == at::kHalf ? MEA_F16 : t == at::kBFloat16 ? MEA_BF16 : -1;
}

// Whether the kernels can read or write t ([B, H, n, features]) in place.
bool in_place(const at::Tensor& t) {
  if (t.dim() != 4 || t.stride(3) != 1 || reinterpret_cast<uintptr_t>(t.const_data_ptr()) % 16) return false;
  const int64_t unit = 16 / t.element_size();
  return t.stride(0) % unit == 0 && t.stride(1) % unit == 0 && t.stride(2) % unit == 0;
}

bool like(const at::Tensor& t, const at::Tensor& ref, at::ScalarType dtype) {
  return t.device() == ref.device() && t.scalar_type() == dtype && in_place(t);
}

mea_tensor_strides strides_of(const at::Tensor& t) { return {t.stride(0), t.stride(1), t.stride(2)}; }

// None, or an int32 [B] vector on q's device: its address in *out.
bool kv_len_ok(PyObject* o, const at::Device& dev, int64_t B, const int32_t** out) {
  *out = nullptr;
  if (o == Py_None) return true;
  const at::Tensor* t = gpu_tensor(o);
  if (!t || t->scalar_type() != at::kInt || t->device() != dev || t->dim() != 1 || t->size(0) != B ||
      !t->is_contiguous())
    return false;
  *out = static_cast<const int32_t*>(t->const_data_ptr());
  return true;
}

// Sizes, dtype, mask, scale and padding of a call; false: not the ordinary case.
bool problem(mea_problem* p, int64_t B, int64_t H, int64_t n_q, int64_t n_k, int64_t d, int64_t d_v, int dtype,
             PyObject* causal, PyObject* scale, PyObject* kv_len, const at::Device& dev, bool out_f32) {
  *p = mea_problem{};
  p->batch = B;
  p->heads = H;
  p->n_q = n_q;
  p->n_k = n_k;
  p->d = d;
  p->d_v = d_v == d ? 0 : d_v;
  p->dtype = dtype;
  const int c = PyObject_IsTrue(causal);
  p->causal = c;
  double s = d > 0 ? 1.0 / std::sqrt((double)d) : 0.0;
  if (scale != Py_None && c >= 0) s = PyFloat_AsDouble(scale);
  if (c < 0 || PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  p->scale = (float)s;
  p->out_f32 = out_f32 && dtype != MEA_F32;
  return kv_len_ok(kv_len, dev, B, &p->kv_len);
}

// Same-shape checks of [B, H, n_q, d], [B, H, n_k, d], [B, H, n_k, d_v].
bool qkv_shapes(const at::Tensor& q, const at::Tensor& k, const at::Tensor& v) {
  return q.size(0) == k.size(0) && q.size(1) == k.size(1) && q.size(3) == k.size(3) && k.size(0) == v.size(0) &&
         k.size(1) == v.size(1) && k.size(2) == v.size(2);
}

hipStream_t stream_of(const at::Device& dev) { return c10::hip::getCurrentHIPStream(dev.index()).stream(); }

at::Tensor workspace(size_t bytes, const at::Device& dev) {
  return at::empty({(int64_t)bytes}, at::TensorOptions().dtype(at::kByte).device(dev));
}

PyObject* none() { Py_RETURN_NONE; }

// The result of a call whose status is not MEA_OK: None where the library
// refused the arguments (it launches nothing then), else the error.
PyObject* failed(const char* name, mea_status st) {
  if (st == MEA_ERR_INVALID_ARG || st == MEA_ERR_UNSUPPORTED) return none();
  return PyObject_CallFunction(g_check, "si", name, (int)st);
}

// A new tuple of tensors; undefined ones are None.
PyObject* tuple_of(std::initializer_list<at::Tensor> ts) {
  PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
  Py_ssize_t i = 0;
  for (const at::Tensor& t : ts) {
    PyObject* o = t.defined() ? THPVariable_Wrap(t) : Py_NewRef(Py_None);
    PyTuple_SET_ITEM(r, i++, o);
  }
  return r;
}

// Allocates lse, o_lo and the workspace, and launches the forward (without the
// interpreter lock).  Returns the status.
mea_status launch_fwd(const mea_problem& p, const at::Tensor& q, const void* k, const void* v, void* o,
                      at::Tensor* lse, at::Tensor* o_lo, at::IntArrayRef lse_shape, at::IntArrayRef o_shape,
                      at::ScalarType out_dtype) {
  size_t bytes = 0;
  mea_status st = g_fwd_ws(&p, &bytes);
  if (st != MEA_OK) return st;
  const at::Device dev = q.device();
  if (lse) *lse = at::empty(lse_shape, at::TensorOptions().dtype(at::kFloat).device(dev));
  if (o_lo) *o_lo = at::empty(o_shape, at::TensorOptions().dtype(out_dtype).device(dev));
  at::Tensor ws;
  if (bytes) ws = workspace(bytes, dev);
  return g_fwd(&p, q.const_data_ptr(), k, v, o, lse ? static_cast<float*>(lse->mutable_data_ptr()) : nullptr,
               o_lo ? o_lo->mutable_data_ptr() : nullptr, bytes ? ws.mutable_data_ptr() : nullptr, bytes,
               stream_of(dev));
}

// fwd(q, k, v, causal, scale, need_lse, out, out_dtype, kv_len, residual):
// attention_fwd's result, or None.
PyObject* ext_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 10) return none();
  const at::Tensor *q = gpu_tensor(a[0]), *k = gpu_tensor(a[1]), *v = gpu_tensor(a[2]);
  if (!q || !k || !v) return none();
  const at::ScalarType dt = q->scalar_type();
  if (dtype_code(dt) < 0 || !in_place(*q) || !like(*k, *q, dt) || !like(*v, *q, dt) || !qkv_shapes(*q, *k, *v))
    return none();
  at::ScalarType out_dt = dt;
  if (a[7] != Py_None) {
    if (!THPDtype_Check(a[7])) return none();
    out_dt = reinterpret_cast<THPDtype*>(a[7])->scalar_type;
    if (out_dt != dt && out_dt != at::kFloat) return none();
  }
  const int64_t shape[4] = {q->size(0), q->size(1), q->size(2), v->size(3)};
  const at::Tensor* out = nullptr;
  if (a[6] != Py_None) {
    out = gpu_tensor(a[6]);
    if (!out || !like(*out, *q, out_dt) || out->sizes() != at::IntArrayRef(shape, 4)) return none();
  }
  const int need_lse = PyObject_IsTrue(a[5]), residual = PyObject_IsTrue(a[9]);
  mea_problem p;
  if (need_lse < 0 || residual < 0 ||
      !problem(&p, shape[0], shape[1], shape[2], k->size(2), q->size(3), shape[3], dtype_code(dt), a[3], a[4], a[8],
               q->device(), out_dt == at::kFloat)) {
    PyErr_Clear();
    return none();
  }
  at::Tensor o, lse, o_lo;
  mea_status st;
  {
    pybind11::gil_scoped_release no_gil;
    o = out ? *out : at::empty(at::IntArrayRef(shape, 4), at::TensorOptions().dtype(out_dt).device(q->device()));
    mea_strides ms = {};
    if (!q->is_contiguous() || !k->is_contiguous() || !v->is_contiguous() || !o.is_contiguous()) {
      ms.q = strides_of(*q);
      ms.k = strides_of(*k);
      ms.v = strides_of(*v);
      ms.o = strides_of(o);
      p.strides = &ms;
    }
    st = launch_fwd(p, *q, k->const_data_ptr(), v->const_data_ptr(), o.mutable_data_ptr(), need_lse ? &lse : nullptr,
                    residual && out_dt != at::kFloat ? &o_lo : nullptr, at::IntArrayRef(shape, 3),
                    at::IntArrayRef(shape, 4), out_dt);
  }
  if (st != MEA_OK) return failed("mea_attention_fwd", st);
  return residual ? tuple_of({o, lse, o_lo}) : tuple_of({o, lse});
  END_HANDLE_TH_ERRORS
}

mea_status launch_bwd(const mea_problem& p, const at::Tensor& q, const void* k, const void* v, const void* o,
                      const void* o_lo, const void* d_o, const at::Tensor& lse, void* dq, void* dk, void* dv) {
  size_t bytes = 0;
  const mea_status st = g_bwd_ws(&p, &bytes);
  if (st != MEA_OK) return st;
  at::Tensor ws = workspace(bytes, q.device());
  return g_bwd(&p, q.const_data_ptr(), k, v, o, o_lo, d_o, static_cast<const float*>(lse.const_data_ptr()), dq, dk, dv,
               ws.mutable_data_ptr(), bytes, stream_of(q.device()));
}

// The log-sum-exp of n_q rows per (batch, head).
bool lse_ok(const at::Tensor* t, const at::Device& dev, int64_t B, int64_t H, int64_t n_q) {
  return t && t->device() == dev && t->scalar_type() == at::kFloat && t->is_contiguous() && t->dim() == 3 &&
         t->size(0) == B && t->size(1) == H && t->size(2) == n_q;
}

// bwd(q, k, v, o, lse, do, causal, scale, need_dq, need_dkdv, out, kv_len,
// o_lo): attention_bwd's result, or None.
PyObject* ext_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 13) return none();
  const at::Tensor *q = gpu_tensor(a[0]), *k = gpu_tensor(a[1]), *v = gpu_tensor(a[2]), *o = gpu_tensor(a[3]),
                   *lse = gpu_tensor(a[4]), *d_o = gpu_tensor(a[5]);
  if (!q || !k || !v || !o || !lse || !d_o) return none();
  const at::ScalarType dt = q->scalar_type(), out_dt = o->scalar_type();
  if (dtype_code(dt) < 0 || (out_dt != dt && out_dt != at::kFloat) || !in_place(*q) || !like(*k, *q, dt) ||
      !like(*v, *q, dt) || !like(*o, *q, out_dt) || !like(*d_o, *q, out_dt) || !qkv_shapes(*q, *k, *v) ||
      !lse_ok(lse, q->device(), q->size(0), q->size(1), q->size(2)))
    return none();
  const int64_t shape[4] = {q->size(0), q->size(1), q->size(2), v->size(3)};
  const at::IntArrayRef o_shape(shape, 4);
  if (o->sizes() != o_shape || d_o->sizes() != o_shape) return none();
  const at::Tensor* o_lo = nullptr;
  if (a[12] != Py_None) {
    o_lo = gpu_tensor(a[12]);
    if (!o_lo || !like(*o_lo, *q, out_dt) || o_lo->sizes() != o_shape || !o_lo->is_contiguous()) return none();
  }
  const int need[2] = {PyObject_IsTrue(a[8]), PyObject_IsTrue(a[9])};
  // The gradients: given ones are checked, the others allocated.
  const at::Tensor* src[3] = {q, k, v};
  const at::Tensor* given[3] = {nullptr, nullptr, nullptr};
  if (a[10] != Py_None) {
    if (!PyTuple_CheckExact(a[10]) || PyTuple_GET_SIZE(a[10]) != 3) return none();
    for (int i = 0; i < 3; ++i) {
      PyObject* g = PyTuple_GET_ITEM(a[10], i);
      if (g == Py_None || need[i > 0] <= 0) continue;
      given[i] = gpu_tensor(g);
      if (!given[i] || !like(*given[i], *q, dt) || given[i]->sizes() != src[i]->sizes()) return none();
    }
  }
  mea_problem p;
  if (need[0] < 0 || need[1] < 0 || !(need[0] || need[1]) ||
      !problem(&p, shape[0], shape[1], shape[2], k->size(2), q->size(3), shape[3], dtype_code(dt), a[6], a[7], a[11],
               q->device(), out_dt == at::kFloat)) {
    PyErr_Clear();
    return none();
  }
  at::Tensor g[3];
  mea_status st;
  {
    pybind11::gil_scoped_release no_gil;
    bool contiguous = q->is_contiguous() && k->is_contiguous() && v->is_contiguous() && o->is_contiguous() &&
                      d_o->is_contiguous();
    for (int i = 0; i < 3; ++i) {
      if (!need[i > 0]) continue;
      g[i] = given[i] ? *given[i]
                      : at::empty(src[i]->sizes(), at::TensorOptions().dtype(dt).device(q->device()));
      contiguous = contiguous && g[i].is_contiguous();
    }
    mea_strides ms = {};
    if (!contiguous) {
      mea_tensor_strides* gs[3] = {&ms.dq, &ms.dk, &ms.dv};
      ms.q = strides_of(*q);
      ms.k = strides_of(*k);
      ms.v = strides_of(*v);
      ms.o = strides_of(*o);
      ms.d_o = strides_of(*d_o);
      for (int i = 0; i < 3; ++i)
        if (g[i].defined()) *gs[i] = strides_of(g[i]);
      p.strides = &ms;
    }
    auto ptr = [](at::Tensor& t) { return t.defined() ? t.mutable_data_ptr() : nullptr; };
    st = launch_bwd(p, *q, k->const_data_ptr(), v->const_data_ptr(), o->const_data_ptr(),
                    o_lo ? o_lo->const_data_ptr() : nullptr, d_o->const_data_ptr(), *lse, ptr(g[0]), ptr(g[1]),
                    ptr(g[2]));
  }
  if (st != MEA_OK) return failed("mea_attention_bwd", st);
  return tuple_of({g[0], g[1], g[2]});
  END_HANDLE_TH_ERRORS
}

// A contiguous packed projection [B, n, 3, H, d], or null.
const at::Tensor* packed_qkv(PyObject* o) {
  const at::Tensor* t = gpu_tensor(o);
  return t && t->dim() == 5 && t->size(2) == 3 && t->is_contiguous() && dtype_code(t->scalar_type()) >= 0 &&
                 t->size(4) % 16 == 0 && reinterpret_cast<uintptr_t>(t->const_data_ptr()) % 16 == 0
             ? t
             : nullptr;
}

// Address of q (0), k (1) or v (2) inside a packed projection.
char* packed_part(const at::Tensor& t, int i) {
  return static_cast<char*>(const_cast<void*>(t.const_data_ptr())) + i * t.size(3) * t.size(4) * t.element_size();
}

// packed_fwd(qkv, causal, scale, kv_len): (o [B, n, H, d], lse, o_lo), or None.
PyObject* ext_packed_fwd(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  const at::Tensor* t = n_args == 4 ? packed_qkv(a[0]) : nullptr;
  if (!t) return none();
  const int64_t B = t->size(0), n = t->size(1), H = t->size(3), d = t->size(4);
  const at::ScalarType dt = t->scalar_type();
  mea_problem p;
  if (!problem(&p, B, H, n, n, d, d, dtype_code(dt), a[1], a[2], a[3], t->device(), false)) return none();
  mea_strides ms = {};
  ms.q = ms.k = ms.v = mea_tensor_strides{n * 3 * H * d, d, 3 * H * d};
  ms.o = mea_tensor_strides{n * H * d, d, H * d};
  p.strides = &ms;
  at::Tensor o, lse, o_lo;
  mea_status st;
  {
    pybind11::gil_scoped_release no_gil;
    o = at::empty({B, n, H, d}, at::TensorOptions().dtype(dt).device(t->device()));
    st = launch_fwd(p, *t, packed_part(*t, 1), packed_part(*t, 2), o.mutable_data_ptr(), &lse,
                    dt != at::kFloat ? &o_lo : nullptr, {B, H, n}, {B, H, n, d}, dt);
  }
  if (st != MEA_OK) return failed("mea_attention_fwd", st);
  return tuple_of({o, lse, o_lo});
  END_HANDLE_TH_ERRORS
}

// packed_bwd(qkv, o, lse, o_lo, do, causal, scale, kv_len): the packed
// gradient, or None.  o and do are [B, n, H, d].
PyObject* ext_packed_bwd(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  const at::Tensor* t = n_args == 8 ? packed_qkv(a[0]) : nullptr;
  if (!t) return none();
  const at::Tensor *o = gpu_tensor(a[1]), *lse = gpu_tensor(a[2]), *d_o = gpu_tensor(a[4]);
  if (!o || !lse || !d_o) return none();
  const int64_t B = t->size(0), n = t->size(1), H = t->size(3), d = t->size(4);
  const at::ScalarType dt = t->scalar_type();
  const int64_t shape[4] = {B, n, H, d};
  const at::IntArrayRef o_shape(shape, 4);
  if (!like(*o, *t, dt) || !like(*d_o, *t, dt) || o->sizes() != o_shape || d_o->sizes() != o_shape ||
      !lse_ok(lse, t->device(), B, H, n))
    return none();
  const at::Tensor* o_lo = nullptr;
  if (a[3] != Py_None) {
    o_lo = gpu_tensor(a[3]);
    if (!o_lo || !like(*o_lo, *t, dt) || !o_lo->is_contiguous() || o_lo->numel() != o->numel()) return none();
  }
  mea_problem p;
  if (!problem(&p, B, H, n, n, d, d, dtype_code(dt), a[5], a[6], a[7], t->device(), false)) return none();
  auto bnh = [](const at::Tensor& x) { return mea_tensor_strides{x.stride(0), x.stride(2), x.stride(1)}; };
  mea_strides ms = {};
  ms.q = ms.k = ms.v = ms.dq = ms.dk = ms.dv = mea_tensor_strides{n * 3 * H * d, d, 3 * H * d};
  ms.o = bnh(*o);
  ms.d_o = bnh(*d_o);
  p.strides = &ms;
  at::Tensor g;
  mea_status st;
  {
    pybind11::gil_scoped_release no_gil;
    g = at::empty_like(*t);
    st = launch_bwd(p, *t, packed_part(*t, 1), packed_part(*t, 2), o->const_data_ptr(),
                    o_lo ? o_lo->const_data_ptr() : nullptr, d_o->const_data_ptr(), *lse, packed_part(g, 0),
                    packed_part(g, 1), packed_part(g, 2));
  }
  if (st != MEA_OK) return failed("mea_attention_bwd", st);
  return THPVariable_Wrap(g);
  END_HANDLE_TH_ERRORS
}

// init(check, fwd_workspace_size, bwd_workspace_size, fwd, bwd): _lib.check and
// the addresses of the library's entry points.
PyObject* ext_init(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 5) {
    PyErr_SetString(PyExc_TypeError, "init takes a function and four addresses");
    return nullptr;
  }
  void* f[4];
  for (int i = 0; i < 4; ++i) {
    f[i] = PyLong_AsVoidPtr(a[i + 1]);
    if (PyErr_Occurred()) return nullptr;
  }
  PyObject* old = g_check;
  g_check = Py_NewRef(a[0]);
  Py_XDECREF(old);
  g_fwd_ws = reinterpret_cast<decltype(g_fwd_ws)>(f[0]);
  g_bwd_ws = reinterpret_cast<decltype(g_bwd_ws)>(f[1]);
  g_fwd = reinterpret_cast<decltype(g_fwd)>(f[2]);
  g_bwd = reinterpret_cast<decltype(g_bwd)>(f[3]);
  Py_RETURN_NONE;
}

PyCFunction fast(PyObject* (*f)(PyObject*, PyObject* const*, Py_ssize_t)) {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f));
}

PyMethodDef methods[] = {
    {"init", fast(ext_init), METH_FASTCALL, nullptr},
    {"fwd", fast(ext_fwd), METH_FASTCALL, nullptr},
    {"bwd", fast(ext_bwd), METH_FASTCALL, nullptr},
    {"packed_fwd", fast(ext_packed_fwd), METH_FASTCALL, nullptr},
    {"packed_bwd", fast(ext_packed_bwd), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_ext", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_ext() { return PyModule_Create(&module); }
