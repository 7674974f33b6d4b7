// The small stages' calls (rewards, rejection sampling, turn advantages) as one native step from Python: argument checks,
// output allocation and the C entry point.  Such a call is host time only (kernels of 2 to 4 us, at most a few KB of data):
// marshalled in Python, a rollout batch of 384 samples took 28.1 us for its three calls, so it takes 18.5.
//
// A function returns a tuple of outputs, or an int (the C entry point's error code), or None for whatever is not plainly in
// order (another type, dtype, layout or device, a dispatch or function mode): the caller then takes the general path, which
// accepts or refuses it.  The entry points' addresses come from the caller (bind), so that both paths call the same library.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>

#include <climits>

#include "../../include/pg_head.h"

namespace {

struct {
  decltype(&turn_reward) reward;
  decltype(&prs_retain) retain;
  decltype(&trloo_advantage) trloo;
  decltype(&grpo_advantage) grpo;
} g_entry;

PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  void* p[4];
  if (n != 4) { PyErr_SetString(PyExc_TypeError, "bind takes four addresses"); return nullptr; }
  for (int i = 0; i < 4; ++i) {
    p[i] = PyLong_AsVoidPtr(args[i]);
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
      return nullptr;
    }
  }
  g_entry.reward = reinterpret_cast<decltype(g_entry.reward)>(p[0]);
  g_entry.retain = reinterpret_cast<decltype(g_entry.retain)>(p[1]);
  g_entry.trloo = reinterpret_cast<decltype(g_entry.trloo)>(p[2]);
  g_entry.grpo = reinterpret_cast<decltype(g_entry.grpo)>(p[3]);
  Py_RETURN_NONE;
}

// Reads the arguments of one call; ok turns false at the first thing that the general path has to look at.
struct Reader {
  bool ok = true;
  c10::DeviceIndex device = -1;      // the current device
  Reader() {
    ok = g_entry.reward && !c10::impl::TorchDispatchModeTLS::any_modes_set() && at::impl::PythonTorchFunctionTLS::stack_len() == 0;
  }
  const at::Tensor* tensor(PyObject* o, at::ScalarType dtype, int64_t numel = -1) {
    if (!ok || !THPVariable_CheckExact(o)) { ok = false; return nullptr; }
    const at::Tensor& t = THPVariable_Unpack(o);
    ok = t.layout() == at::kStrided && t.has_storage() && t.is_cuda() && t.scalar_type() == dtype && t.is_contiguous() && (numel < 0 || t.numel() == numel);
    if (!ok) return nullptr;
    if (device < 0) device = c10::hip::current_device();
    ok = t.get_device() == device;
    return ok ? &t : nullptr;
  }
  const at::Tensor* optional(PyObject* o, at::ScalarType dtype, int64_t numel) { return o == Py_None ? nullptr : tensor(o, dtype, numel); }
  float real(PyObject* o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
    return (float)v;
  }
  bool flag(PyObject* o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) { PyErr_Clear(); ok = false; }
    return v > 0;
  }
  void* stream(PyObject* o) {        // a raw handle, or None: the current stream
    if (!ok) return nullptr;
    if (o == Py_None) return c10::hip::getCurrentHIPStream(device).stream();
    void* p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
    return p;
  }
};

template <typename T>
T* data(const at::Tensor* t) { return t ? static_cast<T*>(t->data_ptr()) : nullptr; }

at::Tensor output(at::IntArrayRef shape, at::ScalarType dtype, c10::DeviceIndex device) {
  return at::empty(shape, at::TensorOptions().dtype(dtype).device(at::Device(at::kCUDA, device)));
}
PyObject* wrap(at::Tensor& t) {
  if (t.defined()) return THPVariable_Wrap(std::move(t));
  Py_RETURN_NONE;
}
PyObject* result(int32_t rc, std::initializer_list<at::Tensor*> out) {
  if (rc != PG_OK) return PyLong_FromLong(rc);
  PyObject* r = PyTuple_New((Py_ssize_t)out.size());
  if (!r) return nullptr;
  Py_ssize_t i = 0;
  for (at::Tensor* t : out) {
    PyObject* o = wrap(*t);
    if (!o) { Py_DECREF(r); return nullptr; }
    PyTuple_SET_ITEM(r, i++, o);
  }
  return r;
}

// (correct, t_reference, t_kernel, t_generated | None, t_total | None, speedup_cap, want_pr, stream | None)
PyObject* stage_reward(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  Reader in;
  if (n_args != 8) Py_RETURN_NONE;
  const at::Tensor* correct = in.tensor(a[0], at::kByte);
  const int64_t n = correct ? correct->numel() : 0;
  const at::Tensor* ref = in.optional(a[1], at::kFloat, n);
  const at::Tensor* ker = in.optional(a[2], at::kFloat, n);
  const at::Tensor* gen = in.optional(a[3], at::kFloat, n);
  const at::Tensor* tot = in.optional(a[4], at::kFloat, n);
  const float cap = in.real(a[5]);
  const bool want_pr = in.flag(a[6]);
  void* stream = in.stream(a[7]);
  if (!in.ok) Py_RETURN_NONE;
  at::Tensor R = output({n}, at::kFloat, in.device), pr;
  if (want_pr) pr = output({n}, at::kFloat, in.device);
  float* const out[2] = {data<float>(&R), want_pr ? data<float>(&pr) : nullptr};
  int32_t rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_entry.reward(data<const uint8_t>(correct), data<const float>(ref), data<const float>(ker), data<const float>(gen), data<const float>(tot), n, cap, out[0],
                      out[1], stream);
  Py_END_ALLOW_THREADS
  return result(rc, {&R, &pr});
  END_HANDLE_TH_ERRORS
}

// (pr, valid | None, seed, tau, s, hard, want_p, stream | None)
PyObject* stage_retain(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  Reader in;
  if (n_args != 8) Py_RETURN_NONE;
  const at::Tensor* pr = in.tensor(a[0], at::kFloat);
  const int64_t n = pr ? pr->numel() : 0;
  const at::Tensor* valid = in.optional(a[1], at::kByte, n);
  if (!PyLong_CheckExact(a[2])) Py_RETURN_NONE;
  const unsigned long long seed = PyLong_AsUnsignedLongLongMask(a[2]);
  const float tau = in.real(a[3]), s = in.real(a[4]);
  const bool hard = in.flag(a[5]), want_p = in.flag(a[6]);
  void* stream = in.stream(a[7]);
  if (!in.ok) Py_RETURN_NONE;
  at::Tensor keep = output({n}, at::kByte, in.device), p;
  if (want_p) p = output({n}, at::kFloat, in.device);
  uint8_t* const k = data<uint8_t>(&keep);
  float* const q = want_p ? data<float>(&p) : nullptr;
  int32_t rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_entry.retain(data<const float>(pr), data<const uint8_t>(valid), n, tau, s, hard, seed, k, q, stream);
  Py_END_ALLOW_THREADS
  return result(rc, {&keep, &p});
  END_HANDLE_TH_ERRORS
}

// (rewards [P, K, Tmax], valid, gamma, want_returns, want_group_n, group_mean, stream | None)
PyObject* stage_advantage(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  Reader in;
  if (n_args != 7) Py_RETURN_NONE;
  const at::Tensor* rewards = in.tensor(a[0], at::kFloat);
  const at::Tensor* valid = in.tensor(a[1], at::kByte);
  const float gamma = in.real(a[2]);
  const bool want_ret = in.flag(a[3]), want_n = in.flag(a[4]), group_mean = in.flag(a[5]);
  void* stream = in.stream(a[6]);
  if (!in.ok || rewards->dim() != 3 || valid->sizes() != rewards->sizes()) Py_RETURN_NONE;
  const int64_t P = rewards->size(0), K = rewards->size(1), Tm = rewards->size(2);
  if (P > INT_MAX || K > INT_MAX || Tm > INT_MAX) Py_RETURN_NONE;
  at::Tensor adv = output({P, K, Tm}, at::kDouble, in.device), ret, group_n;
  if (want_ret) ret = output({P, K, Tm}, at::kDouble, in.device);
  if (want_n) group_n = output({P, Tm}, at::kInt, in.device);
  double* const out[2] = {want_ret ? data<double>(&ret) : nullptr, data<double>(&adv)};
  int* const gn = want_n ? data<int>(&group_n) : nullptr;
  int32_t rc;
  Py_BEGIN_ALLOW_THREADS
  rc = (group_mean ? g_entry.grpo : g_entry.trloo)(data<const float>(rewards), data<const uint8_t>(valid), (int32_t)P, (int32_t)K, (int32_t)Tm, gamma, out[0], out[1],
                                                   gn, stream);
  Py_END_ALLOW_THREADS
  return result(rc, {&adv, &ret, &group_n});
  END_HANDLE_TH_ERRORS
}


PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bind)), METH_FASTCALL, nullptr},
    {"turn_reward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(stage_reward)), METH_FASTCALL, nullptr},
    {"prs_retain", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(stage_retain)), METH_FASTCALL, nullptr},
    {"turn_advantage", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(stage_advantage)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_stage_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__stage_calls(void) { return PyModule_Create(&module); }
