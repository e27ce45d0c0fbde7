// The tensor-level calls of binding.py in native code: allocate the outputs, fill the descriptor, call the library on the
// current stream.  What bounds a small call is its host part, and most of that was interpreter time: building the
// descriptor, asking for the stream, a pointer per argument through ctypes.  Host us a call, through ctypes / here: decode of 32
// heads 12.0 / 4.7, fp32 prefill in one launch 17.8 / 7.3, bf16 prefill in two 23.1 / 10.7; the whole call where the GPU is the
// faster side: decode 12.0 / 5.3, three-branch step of 4 heads 12.0 / 7.7, B1 H4 L256 fp32 prefill 17.9 / 13.4.
//
// Only what a program ordinarily passes is served: tensors that are plain torch.Tensor objects, q on the GPU in fp32 or bf16
// and of the expected rank, no explicit stream, no torch mode.  For anything else a call returns None and binding.py takes its
// general path, which also raises the errors.  Like there, devices and types of the other tensors are the caller's business: they
// are handed on as the pointers they are.
// The library's functions are handed over as addresses (bind), so that there is one place that loads it.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>

#include "../../include/linattn.h"

namespace {

struct Library {
  decltype(&linattn_workspace_bytes) workspace_bytes = nullptr;
  decltype(&linattn_prefill) prefill = nullptr;
  decltype(&linattn_prefill_grouped) prefill_grouped = nullptr;
  decltype(&linattn_backward_workspace_bytes) backward_workspace_bytes = nullptr;
  decltype(&linattn_prefill_grouped_backward) prefill_grouped_backward = nullptr;
  decltype(&linattn_verify) verify = nullptr;
  decltype(&linattn_verify_grouped) verify_grouped = nullptr;
  decltype(&linattn_verify_tree) verify_tree = nullptr;
  decltype(&linattn_decode) decode = nullptr;
} lib;
PyObject *get_device = nullptr, *get_raw_stream = nullptr;   // torch._C._cuda_getDevice, _cuda_getCurrentRawStream

// a call's arguments that the native path takes; any `false` below means: the general path
bool tensor(PyObject* o, const at::Tensor*& t) {
  if (!THPVariable_CheckExact(o)) return false;
  t = &THPVariable_Unpack(o);
  return true;
}
bool tensor_or_none(PyObject* o, const at::Tensor*& t) {
  t = nullptr;
  return o == Py_None || tensor(o, t);
}
bool number(PyObject* o, double& x) {
  if (!PyFloat_CheckExact(o) && !PyLong_CheckExact(o)) return false;
  x = PyFloat_AsDouble(o);
  if (x == -1.0 && PyErr_Occurred()) { PyErr_Clear(); return false; }
  return true;
}
bool feature_map(PyObject* o, int32_t& phi) {
  if (!PyUnicode_CheckExact(o)) return false;
  if (PyUnicode_CompareWithASCIIString(o, "elu1") == 0) phi = LINATTN_PHI_ELU1;
  else if (PyUnicode_CompareWithASCIIString(o, "relu") == 0) phi = LINATTN_PHI_RELU;
  else return false;
  return true;
}
bool io_type(const at::Tensor& q, int32_t& io) {
  // (under a mode that watches torch's calls the allocations stay where it sees them)
  if (!q.is_cuda() || at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set()) return false;
  if (q.scalar_type() == at::kFloat) io = LINATTN_F32;
  else if (q.scalar_type() == at::kBFloat16) io = LINATTN_BF16;
  else return false;
  return true;
}
bool items(PyObject* o, Py_ssize_t n) { return PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == n; }
void* ptr(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }
template <typename T>
T* ptr_as(const at::Tensor* t) { return static_cast<T*>(ptr(t)); }

// the current stream of the current device; false with a Python error set
bool current_stream(void*& s) {
  PyObject* dev = PyObject_CallNoArgs(get_device);
  if (!dev) return false;
  PyObject* raw = PyObject_CallOneArg(get_raw_stream, dev);
  Py_DECREF(dev);
  if (!raw) return false;
  s = PyLong_AsVoidPtr(raw);
  Py_DECREF(raw);
  return !PyErr_Occurred();
}

// strides of dense [B,H,L,*] tensors unless given
linattn_desc make_desc(int64_t B, int64_t H, int64_t L, int64_t d, int64_t d_v, int64_t conv_k, int64_t chunk, int32_t io, int32_t phi,
                       double eps, const int64_t* sq = nullptr, const int64_t* sv = nullptr) {
  linattn_desc x{};
  x.B = (int32_t)B; x.H = (int32_t)H; x.d = (int32_t)d; x.conv_k = (int32_t)conv_k; x.chunk = (int32_t)chunk;
  x.io_dtype = io; x.phi = phi; x.eps = (float)eps;
  x.stride_b = sq ? sq[0] : H * L * d;
  x.stride_h = sq ? sq[1] : L * d;
  x.stride_t = sq ? sq[2] : d;
  if (d_v != d) {
    x.d_v = (int32_t)d_v;
    x.stride_b_v = sv ? sv[0] : H * L * d_v;
    x.stride_h_v = sv ? sv[1] : L * d_v;
    x.stride_t_v = sv ? sv[2] : d_v;
  }
  return x;
}

// the call itself, other threads running meanwhile (its arguments are made before)
struct OthersRun {
  PyThreadState* state = PyEval_SaveThread();
  ~OthersRun() { PyEval_RestoreThread(state); }
};
template <typename F, typename... A>
int without_gil(F f, A... a) {
  OthersRun r;
  return f(a...);
}
PyObject* out_or_status(int st, const at::Tensor& out) { return st == 0 ? THPVariable_Wrap(out) : PyLong_FromLong(st); }

// verify(q, k, v, conv_w, (S, z, hist), n_commit, eps, phi); decode has no n_commit
PyObject* step(PyObject* const* a, bool one) {
  const at::Tensor *q, *k, *v, *w, *S, *z, *hist, *n_commit = nullptr;
  double eps;
  int32_t phi, io;
  if (!tensor(a[0], q) || !tensor(a[1], k) || !tensor(a[2], v) || !tensor(a[3], w) || !items(a[4], 3) || !tensor(PyTuple_GET_ITEM(a[4], 0), S) ||
      !tensor(PyTuple_GET_ITEM(a[4], 1), z) || !tensor_or_none(PyTuple_GET_ITEM(a[4], 2), hist) || (!one && !tensor_or_none(a[5], n_commit)) ||
      !number(a[one ? 5 : 6], eps) || !feature_map(a[one ? 6 : 7], phi) || !io_type(*q, io) || w->dim() < 3 || v->dim() < 1 ||
      (one ? q->dim() < 3 : q->dim() != 4))
    Py_RETURN_NONE;
  const int64_t kk = one ? 1 : q->size(2);
  const linattn_desc x = make_desc(q->size(0), q->size(1), kk, q->size(-1), v->size(-1), w->size(2), 64, io, phi, eps);
  const at::Tensor out = at::empty_like(*v);
  void* s;
  if (!current_stream(s)) return nullptr;
  const int st = one ? without_gil(lib.decode, &x, ptr(q), ptr(k), ptr(v), ptr_as<float>(w), ptr_as<float>(S), ptr_as<float>(z), ptr(hist), ptr(&out), s)
                     : without_gil(lib.verify, &x, (int32_t)kk, ptr(q), ptr(k), ptr(v), ptr_as<float>(w), ptr_as<float>(S), ptr_as<float>(z), ptr(hist),
                                   ptr_as<int32_t>(n_commit), ptr(&out), s);
  return out_or_status(st, out);
}
PyObject* py_verify(PyObject*, PyObject* const* a, Py_ssize_t) {
  HANDLE_TH_ERRORS
  return step(a, false);
  END_HANDLE_TH_ERRORS
}
PyObject* py_decode(PyObject*, PyObject* const* a, Py_ssize_t) {
  HANDLE_TH_ERRORS
  return step(a, true);
  END_HANDLE_TH_ERRORS
}

// verify_tree(q, k, v, parent, conv_w, (S, z, hist), accept, eps, phi)
PyObject* py_verify_tree(PyObject*, PyObject* const* a, Py_ssize_t) {
  HANDLE_TH_ERRORS
  const at::Tensor *q, *k, *v, *w, *parent, *accept, *S, *z, *hist;
  double eps;
  int32_t phi, io;
  if (!tensor(a[0], q) || !tensor(a[1], k) || !tensor(a[2], v) || !tensor(a[3], parent) || !tensor(a[4], w) || !items(a[5], 3) ||
      !tensor(PyTuple_GET_ITEM(a[5], 0), S) || !tensor(PyTuple_GET_ITEM(a[5], 1), z) || !tensor_or_none(PyTuple_GET_ITEM(a[5], 2), hist) ||
      !tensor_or_none(a[6], accept) || !number(a[7], eps) || !feature_map(a[8], phi) || !io_type(*q, io) || q->dim() != 4 || w->dim() < 3)
    Py_RETURN_NONE;
  const int64_t n = q->size(2), d = q->size(3);
  const linattn_desc x = make_desc(q->size(0), q->size(1), n, d, d, w->size(2), 64, io, phi, eps);
  const at::Tensor out = at::empty_like(*q);
  void* s;
  if (!current_stream(s)) return nullptr;
  const int st = without_gil(lib.verify_tree, &x, (int32_t)n, ptr(q), ptr(k), ptr(v), ptr_as<int32_t>(parent), ptr_as<float>(w), ptr_as<float>(S), ptr_as<float>(z),
                           ptr(hist), ptr_as<int32_t>(accept), ptr(&out), s);
  return out_or_status(st, out);
  END_HANDLE_TH_ERRORS
}

// verify_grouped(q, k, v, conv_w, (S, z, hist, kwin, vwin, fill), alpha, n_commit, eps, phi)
PyObject* py_verify_grouped(PyObject*, PyObject* const* a, Py_ssize_t) {
  HANDLE_TH_ERRORS
  const at::Tensor *q, *k, *v, *w, *n_commit, *S, *z, *hist, *kwin, *vwin, *fill;
  double eps, alpha;
  int32_t phi, io;
  if (!tensor(a[0], q) || !tensor(a[1], k) || !tensor(a[2], v) || !tensor(a[3], w) || !items(a[4], 6) || !tensor(PyTuple_GET_ITEM(a[4], 0), S) ||
      !tensor(PyTuple_GET_ITEM(a[4], 1), z) || !tensor_or_none(PyTuple_GET_ITEM(a[4], 2), hist) || !tensor(PyTuple_GET_ITEM(a[4], 3), kwin) ||
      !tensor(PyTuple_GET_ITEM(a[4], 4), vwin) || !tensor(PyTuple_GET_ITEM(a[4], 5), fill) || !number(a[5], alpha) ||
      !tensor_or_none(a[6], n_commit) || !number(a[7], eps) || !feature_map(a[8], phi) || !io_type(*q, io) || q->dim() != 4 || w->dim() < 3)
    Py_RETURN_NONE;
  const int64_t kk = q->size(2), d = q->size(3);
  const linattn_desc x = make_desc(q->size(0), q->size(1), kk, d, d, w->size(2), 64, io, phi, eps);
  const at::Tensor out = at::empty_like(*q);
  void* s;
  if (!current_stream(s)) return nullptr;
  const int st = without_gil(lib.verify_grouped, &x, (int32_t)kk, (float)alpha, ptr(q), ptr(k), ptr(v), ptr_as<float>(w), ptr_as<float>(S), ptr_as<float>(z), ptr(hist),
                              ptr(kwin), ptr(vwin), ptr_as<int32_t>(fill), ptr_as<int32_t>(n_commit), ptr(&out), s);
  return out_or_status(st, out);
  END_HANDLE_TH_ERRORS
}

// prefill(q, k, v, conv_w, None or (S, z, hist), chunk, eps, want_state, phi, None or alpha) -> (out, (S, z, hist))
PyObject* py_prefill(PyObject*, PyObject* const* a, Py_ssize_t) {
  HANDLE_TH_ERRORS
  const at::Tensor *q, *k, *v, *w, *S_in = nullptr, *z_in = nullptr, *h_in = nullptr;
  double eps, chunk, alpha = 0.0;
  int32_t phi, io;
  const bool grouped = a[9] != Py_None;
  if (!tensor(a[0], q) || !tensor(a[1], k) || !tensor(a[2], v) || !tensor(a[3], w) || !PyLong_CheckExact(a[5]) || !number(a[5], chunk) ||
      !number(a[6], eps) || !PyBool_Check(a[7]) || !feature_map(a[8], phi) || (grouped && !number(a[9], alpha)) || !io_type(*q, io) || q->dim() != 4 ||
      k->dim() != 4 || v->dim() != 4 || w->dim() < 3 || !(chunk >= 0.0 && chunk < 1e9))
    Py_RETURN_NONE;
  if (a[4] != Py_None &&
      (!items(a[4], 3) || !tensor_or_none(PyTuple_GET_ITEM(a[4], 0), S_in) || !tensor_or_none(PyTuple_GET_ITEM(a[4], 1), z_in) ||
       !tensor_or_none(PyTuple_GET_ITEM(a[4], 2), h_in)))
    Py_RETURN_NONE;
  const int64_t B = q->size(0), H = q->size(1), L = q->size(2), d = q->size(3), d_v = v->size(3), Kc = w->size(2);
  const bool dense = q->is_contiguous() && k->is_contiguous() && v->is_contiguous();
  if (!dense && (q->stride(3) != 1 || v->stride(3) != 1 || k->strides() != q->strides() || (d_v == d && v->strides() != q->strides())))
    Py_RETURN_NONE;
  const linattn_desc x = make_desc(B, H, L, d, d_v, Kc, (int64_t)chunk, io, phi, eps, dense ? nullptr : q->strides().data(), dense ? nullptr : v->strides().data());
  const at::Tensor out = dense ? at::empty_like(*v) : at::empty_strided(v->sizes(), v->strides(), at::TensorOptions().dtype(v->dtype()).device(v->device()));
  const bool want_state = a[7] == Py_True;
  const auto on = at::TensorOptions().device(q->device());
  at::Tensor S, z, h, ws;
  if (want_state) {
    S = at::empty({B, H, d, d_v}, on.dtype(at::kFloat));
    z = at::empty({B, H, d}, on.dtype(at::kFloat));
    h = at::empty({B, H, Kc > 1 ? Kc - 1 : 0, d_v}, on.dtype(q->dtype()));
  }
  const size_t bytes = lib.workspace_bytes(&x, (int32_t)L);
  if (bytes) ws = at::empty({(int64_t)bytes}, on.dtype(at::kByte));
  void* s;
  if (!current_stream(s)) return nullptr;
  const at::Tensor *So = want_state ? &S : nullptr, *zo = want_state ? &z : nullptr, *ho = want_state ? &h : nullptr, *wp = bytes ? &ws : nullptr;
  const int st = grouped ? without_gil(lib.prefill_grouped, &x, (int32_t)L, (float)alpha, ptr(q), ptr(k), ptr(v), ptr_as<float>(w), ptr_as<float>(S_in), ptr_as<float>(z_in), ptr(h_in),
                                         ptr(&out), ptr_as<float>(So), ptr_as<float>(zo), ptr(ho), ptr(wp), bytes, s)
                   : without_gil(lib.prefill, &x, (int32_t)L, ptr(q), ptr(k), ptr(v), ptr_as<float>(w), ptr_as<float>(S_in), ptr_as<float>(z_in), ptr(h_in), ptr(&out),
                                 ptr_as<float>(So), ptr_as<float>(zo), ptr(ho), ptr(wp), bytes, s);
  if (st != 0) return PyLong_FromLong(st);
  if (!want_state) return Py_BuildValue("(N(OOO))", THPVariable_Wrap(out), Py_None, Py_None, Py_None);
  return Py_BuildValue("(N(NNN))", THPVariable_Wrap(out), THPVariable_Wrap(S), THPVariable_Wrap(z), THPVariable_Wrap(h));
  END_HANDLE_TH_ERRORS
}

// prefill_grouped_backward(q, k, v, conv_w, dout, alpha, eps, phi, group, want_dw) -> (dq, dk, dv, dw)
PyObject* py_backward(PyObject*, PyObject* const* a, Py_ssize_t) {
  HANDLE_TH_ERRORS
  const at::Tensor *q, *k, *v, *w, *dout;
  double alpha, eps, group;
  int32_t phi, io;
  if (!tensor(a[0], q) || !tensor(a[1], k) || !tensor(a[2], v) || !tensor(a[3], w) || !tensor(a[4], dout) || !number(a[5], alpha) || !number(a[6], eps) ||
      !feature_map(a[7], phi) || !PyLong_CheckExact(a[8]) || !number(a[8], group) || !PyBool_Check(a[9]) || !io_type(*q, io) || q->dim() != 4 || k->dim() != 4 ||
      v->dim() != 4 || dout->dim() != 4 || w->dim() < 3 || !(group >= 0.0 && group < 1e9))
    Py_RETURN_NONE;
  const int64_t B = q->size(0), H = q->size(1), L = q->size(2), d = q->size(3), Kc = w->size(2);
  const bool dense = q->is_contiguous() && k->is_contiguous() && v->is_contiguous() && dout->is_contiguous();
  if (!dense && (q->stride(3) != 1 || k->strides() != q->strides() || v->strides() != q->strides() || dout->strides() != q->strides()))
    Py_RETURN_NONE;
  const linattn_desc x = make_desc(B, H, L, d, d, Kc, (int64_t)group, io, phi, eps, dense ? nullptr : q->strides().data());
  const auto on = at::TensorOptions().device(q->device());
  auto rows = [&] { return dense ? at::empty_like(*q) : at::empty_strided(q->sizes(), q->strides(), on.dtype(q->dtype())); };
  const at::Tensor dq = rows(), dk = rows(), dv = rows();
  const bool want_dw = a[9] == Py_True;
  at::Tensor dw;
  if (want_dw) dw = at::empty({H, d, Kc}, on.dtype(at::kFloat));
  const size_t bytes = lib.backward_workspace_bytes(&x, (int32_t)L);
  const at::Tensor ws = at::empty({(int64_t)(bytes > 16 ? bytes : 16)}, on.dtype(at::kByte));
  void* s;
  if (!current_stream(s)) return nullptr;
  const int st = without_gil(lib.prefill_grouped_backward, &x, (int32_t)L, (float)alpha, ptr(q), ptr(k), ptr(v), ptr_as<float>(w), ptr(dout), ptr(&dq), ptr(&dk), ptr(&dv),
                                        ptr_as<float>(want_dw ? &dw : nullptr), ptr(&ws), bytes, s);
  if (st != 0) return PyLong_FromLong(st);
  if (!want_dw) return Py_BuildValue("(NNNO)", THPVariable_Wrap(dq), THPVariable_Wrap(dk), THPVariable_Wrap(dv), Py_None);
  return Py_BuildValue("(NNNN)", THPVariable_Wrap(dq), THPVariable_Wrap(dk), THPVariable_Wrap(dv), THPVariable_Wrap(dw));
  END_HANDLE_TH_ERRORS
}

// bind(addresses of the nine functions in the order of Library's members, _cuda_getDevice, _cuda_getCurrentRawStream)
PyObject* py_bind(PyObject*, PyObject* args) {
  unsigned long long p[9];
  PyObject *dev, *raw;
  if (!PyArg_ParseTuple(args, "KKKKKKKKKOO", p, p + 1, p + 2, p + 3, p + 4, p + 5, p + 6, p + 7, p + 8, &dev, &raw)) return nullptr;
  auto set = [](auto& f, unsigned long long x) { f = reinterpret_cast<std::decay_t<decltype(f)>>(static_cast<uintptr_t>(x)); };
  set(lib.workspace_bytes, p[0]); set(lib.prefill, p[1]); set(lib.prefill_grouped, p[2]);
  set(lib.backward_workspace_bytes, p[3]); set(lib.prefill_grouped_backward, p[4]);
  set(lib.verify, p[5]); set(lib.verify_grouped, p[6]); set(lib.verify_tree, p[7]); set(lib.decode, p[8]);
  Py_INCREF(dev);
  Py_INCREF(raw);
  Py_XSETREF(get_device, dev);
  Py_XSETREF(get_raw_stream, raw);
  Py_RETURN_NONE;
}

#define FAST(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST("verify", py_verify), FAST("decode", py_decode), FAST("verify_tree", py_verify_tree),
                         FAST("verify_grouped", py_verify_grouped), FAST("prefill", py_prefill), FAST("prefill_grouped_backward", py_backward),
                         {"bind", py_bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
