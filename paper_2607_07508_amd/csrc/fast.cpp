// The per-token entry points' argument marshalling as a CPython module.
//
// These passes take 10 to 30 us on the GPU, as long as Python takes to check a call's
// five arrays, allocate its outputs and workspace and convert fifteen arguments (17 us
// of the surrogate's 36 us pass with its explained variance). Each function here does
// that for the plain case: exact torch.Tensor arguments on one GPU, contiguous, of the
// right types, no torch-function mode. It returns the outputs, or the library's status
// (an int) if the call failed, or None if anything is out of the ordinary, for which the
// Python code, which also holds every error message, takes the call.
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/sao.h"

namespace {

using at::ScalarType;

// The library's functions, resolved from the loaded library by bind().
struct Api {
  decltype(&sao_workspace_size) workspace_size;
  decltype(&sao_advantage) advantage;
  decltype(&sao_step_advantage) step_advantage;
  decltype(&sao_group_advantage) group_advantage;
  decltype(&sao_clipped_loss_store) clipped_loss_store;
  decltype(&sao_ppo_loss_store) ppo_loss_store;
  decltype(&sao_explained_variance_store) explained_variance_store;
};
Api g_api;
PyObject* g_current_stream = nullptr;  // device index -> stream handle

PyObject* none() { Py_RETURN_NONE; }

// What is not plain: the caller leaves the call to Python.
struct NotPlain {};

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw NotPlain{};
  return THPVariable_Unpack(o);
}

// One call: its device and arrays, checked as the binding's _vec does.
struct Call {
  at::Device dev;
  int64_t T;

  explicit Call(PyObject* first) : dev(at::kCPU) {
    if (at::impl::PythonTorchFunctionTLS::stack_len() != 0) throw NotPlain{};
    const at::Tensor& t = tensor(first);
    dev = t.device();
    if (!dev.is_cuda() || t.dim() < 1 || t.size(0) == 0) throw NotPlain{};
    T = t.size(0);
  }
  void* in(PyObject* o, ScalarType type, int64_t n) const {
    const at::Tensor& t = tensor(o);
    if (t.device() != dev || t.scalar_type() != type || !t.is_contiguous() || t.numel() < n) throw NotPlain{};
    return t.data_ptr();
  }
  template <class V>
  V* get(PyObject* o, int64_t n, bool optional = false) const {
    if (optional && o == Py_None) return nullptr;
    return static_cast<V*>(in(o, type_of(static_cast<V*>(nullptr)), n));
  }
  static ScalarType type_of(float*) { return at::kFloat; }
  static ScalarType type_of(uint8_t*) { return at::kByte; }
  static ScalarType type_of(int32_t*) { return at::kInt; }
  static ScalarType type_of(int64_t*) { return at::kLong; }
  static ScalarType type_of(double*) { return at::kDouble; }

  at::Tensor make(int64_t n, ScalarType type) const {
    return at::empty({n}, at::TensorOptions().dtype(type).device(dev));
  }
  // Workspace of `op`; its memory goes back to the stream's pool on return, as a Python
  // call's does.
  at::Tensor workspace(sao_op_t op) const {
    return make(static_cast<int64_t>(g_api.workspace_size(op, T, 1, 1, SAO_F32)), at::kByte);
  }
};

template <class V>
V* ptr(const at::Tensor& t) {
  return t.defined() ? static_cast<V*>(t.data_ptr()) : nullptr;
}

double number(PyObject* o) {
  const double x = PyFloat_AsDouble(o);
  if (x == -1.0 && PyErr_Occurred()) throw NotPlain{};
  return x;
}
int64_t integer(PyObject* o) {
  const long long x = PyLong_AsLongLong(o);
  if (x == -1 && PyErr_Occurred()) throw NotPlain{};
  return x;
}
bool truth(PyObject* o) {
  const int x = PyObject_IsTrue(o);
  if (x < 0) throw NotPlain{};
  return x != 0;
}
// torch's current stream of the device.
hipStream_t stream(const Call& c) {
  PyObject* index = PyLong_FromLong(c.dev.index());
  PyObject* o = index ? PyObject_CallFunctionObjArgs(g_current_stream, index, nullptr) : nullptr;
  Py_XDECREF(index);
  if (!o) throw NotPlain{};
  void* p = PyLong_AsVoidPtr(o);
  Py_DECREF(o);
  if (PyErr_Occurred()) throw NotPlain{};
  return static_cast<hipStream_t>(p);
}

// The outputs as a tuple (None for an undefined tensor), or the status if the call failed.
PyObject* result(sao_status_t status, std::initializer_list<at::Tensor> outs) {
  if (status != SAO_OK) return PyLong_FromLong(status);
  PyObject* t = PyTuple_New(static_cast<Py_ssize_t>(outs.size()));
  if (!t) return nullptr;
  Py_ssize_t i = 0;
  for (const at::Tensor& x : outs) {
    PyObject* o = x.defined() ? THPVariable_Wrap(x) : none();
    if (!o) {
      Py_DECREF(t);
      return nullptr;
    }
    PyTuple_SET_ITEM(t, i++, o);
  }
  return t;
}

// Runs f with C++ exceptions turned into None: the Python code then repeats the call and
// raises what it raises.
template <class F>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, F&& f) {
  if (n != want) return none();
  try {
    return f();
  } catch (const NotPlain&) {
  } catch (const std::exception&) {
  }
  PyErr_Clear();
  return none();
}

// Other threads run while the kernels are launched.
template <class F>
sao_status_t unlocked(F&& f) {
  sao_status_t s;
  Py_BEGIN_ALLOW_THREADS s = f();
  Py_END_ALLOW_THREADS return s;
}

// (values, rewards, mask, cu_seqlens, gamma, lam, alpha, status, want_count)
PyObject* py_advantage(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 9, [&]() -> PyObject* {
    const Call c(a[0]);
    const auto* v = c.get<float>(a[0], c.T);
    const auto* r = c.get<float>(a[1], c.T);
    const auto* m = c.get<uint8_t>(a[2], c.T);
    const at::Tensor& cu = tensor(a[3]);
    if (cu.dim() < 1 || cu.size(0) < 2) throw NotPlain{};
    const int64_t B = cu.size(0) - 1;
    const auto* pc = c.get<int32_t>(a[3], B + 1);
    const double gamma = number(a[4]), lam = number(a[5]), alpha = number(a[6]);
    auto* status = c.get<int32_t>(a[7], 1, true);
    const hipStream_t st = stream(c);
    const at::Tensor adv = c.make(c.T, at::kFloat), ret = c.make(c.T, at::kFloat);
    const at::Tensor cnt = truth(a[8]) ? c.make(1, at::kLong) : at::Tensor();
    const at::Tensor ws = c.workspace(SAO_OP_ADVANTAGE);
    const sao_status_t s = unlocked([&] {
      return g_api.advantage(v, r, m, pc, static_cast<int32_t>(B), c.T, gamma, lam, alpha, ptr<float>(adv),
                             ptr<float>(ret), ptr<int64_t>(cnt), status, ws.data_ptr(), ws.numel(), st);
    });
    return result(s, {adv, ret, cnt});
  });
}

// (values, rewards, mask, cu_seqlens, gamma, lam, alpha, form, status, want_last, want_count)
PyObject* py_step_advantage(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&]() -> PyObject* {
    const Call c(a[0]);
    const auto* v = c.get<float>(a[0], c.T);
    const auto* r = c.get<float>(a[1], c.T);
    const auto* m = c.get<uint8_t>(a[2], c.T);
    const at::Tensor& cu = tensor(a[3]);
    if (cu.dim() < 1 || cu.size(0) < 2) throw NotPlain{};
    const int64_t B = cu.size(0) - 1;
    const auto* pc = c.get<int32_t>(a[3], B + 1);
    const double gamma = number(a[4]), lam = number(a[5]), alpha = number(a[6]);
    const auto form = static_cast<sao_step_value_t>(integer(a[7]));
    auto* status = c.get<int32_t>(a[8], 1, true);
    const hipStream_t st = stream(c);
    const at::Tensor adv = c.make(c.T, at::kFloat), ret = c.make(c.T, at::kFloat);
    const at::Tensor last = truth(a[9]) ? c.make(c.T, at::kByte) : at::Tensor();
    const at::Tensor cnt = truth(a[10]) ? c.make(1, at::kLong) : at::Tensor();
    const at::Tensor ws = c.workspace(SAO_OP_STEP_ADVANTAGE);
    const sao_status_t s = unlocked([&] {
      return g_api.step_advantage(v, r, m, pc, static_cast<int32_t>(B), c.T, gamma, lam, alpha, form, ptr<float>(adv),
                                  ptr<float>(ret), ptr<uint8_t>(last), ptr<int64_t>(cnt), status, ws.data_ptr(),
                                  ws.numel(), st);
    });
    return result(s, {adv, ret, last, cnt});
  });
}

// (rewards, mask, cu_seqlens, group_size, eps_stab, status, want_count)
PyObject* py_group_advantage(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 7, [&]() -> PyObject* {
    const Call c(a[0]);
    const auto* r = c.get<float>(a[0], c.T);
    const auto* m = c.get<uint8_t>(a[1], c.T);
    const at::Tensor& cu = tensor(a[2]);
    if (cu.dim() < 1 || cu.size(0) < 2) throw NotPlain{};
    const int64_t B = cu.size(0) - 1;
    const auto* pc = c.get<int32_t>(a[2], B + 1);
    const int64_t group = integer(a[3]);
    if (group != static_cast<int32_t>(group)) throw NotPlain{};
    const double eps = number(a[4]);
    auto* status = c.get<int32_t>(a[5], 1, true);
    const hipStream_t st = stream(c);
    const at::Tensor adv = c.make(c.T, at::kFloat), reward = c.make(B, at::kDouble), traj = c.make(B, at::kDouble);
    const at::Tensor cnt = truth(a[6]) ? c.make(1, at::kLong) : at::Tensor();
    const at::Tensor ws = c.workspace(SAO_OP_GROUP_ADVANTAGE);
    const sao_status_t s = unlocked([&] {
      return g_api.group_advantage(r, m, pc, static_cast<int32_t>(B), c.T, static_cast<int32_t>(group), eps,
                                   ptr<float>(adv), ptr<double>(reward), ptr<double>(traj), ptr<int64_t>(cnt), status,
                                   ws.data_ptr(), ws.numel(), st);
    });
    return result(s, {adv, traj, reward, cnt});
  });
}

// (logp, logp_rollout, adv, mask, eps_low, eps_high, n_tokens): loss and counts start here
PyObject* py_clipped_loss(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 7, [&]() -> PyObject* {
    const Call c(a[0]);
    const auto* lp = c.get<float>(a[0], c.T);
    const auto* lro = c.get<float>(a[1], c.T);
    const auto* adv = c.get<float>(a[2], c.T);
    const auto* m = c.get<uint8_t>(a[3], c.T);
    const auto lo = static_cast<float>(number(a[4])), hi = static_cast<float>(number(a[5]));
    const auto* cnt = c.get<int64_t>(a[6], 1, true);
    const hipStream_t st = stream(c);
    const at::Tensor loss = c.make(2, at::kDouble), counts = c.make(5, at::kLong), g = c.make(c.T, at::kFloat),
                     flags = c.make(c.T, at::kByte), ws = c.workspace(SAO_OP_LOSS);
    const sao_status_t s = unlocked([&] {
      return g_api.clipped_loss_store(lp, lro, adv, m, c.T, lo, hi, cnt, ptr<double>(loss), ptr<float>(g),
                                      ptr<uint8_t>(flags), ptr<int64_t>(counts), ws.data_ptr(), ws.numel(), st);
    });
    return result(s, {loss, g, flags, counts});
  });
}

// (logp, logp_old, logp_behav, adv, mask, eps_low, eps_high, n_tokens): as above
PyObject* py_ppo_loss(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 8, [&]() -> PyObject* {
    const Call c(a[0]);
    const auto* lp = c.get<float>(a[0], c.T);
    const auto* old = c.get<float>(a[1], c.T);
    const auto* behav = c.get<float>(a[2], c.T, true);
    const auto* adv = c.get<float>(a[3], c.T);
    const auto* m = c.get<uint8_t>(a[4], c.T);
    const auto lo = static_cast<float>(number(a[5])), hi = static_cast<float>(number(a[6]));
    const auto* cnt = c.get<int64_t>(a[7], 1, true);
    const hipStream_t st = stream(c);
    const at::Tensor loss = c.make(1, at::kDouble), counts = c.make(5, at::kLong), g = c.make(c.T, at::kFloat),
                     flags = c.make(c.T, at::kByte), ws = c.workspace(SAO_OP_PPO_LOSS);
    const sao_status_t s = unlocked([&] {
      return g_api.ppo_loss_store(lp, old, behav, adv, m, c.T, lo, hi, cnt, ptr<double>(loss), ptr<float>(g),
                                  ptr<uint8_t>(flags), ptr<int64_t>(counts), ws.data_ptr(), ws.numel(), st);
    });
    return result(s, {loss, g, flags, counts});
  });
}

// (values, ret, mask): the moments start here
PyObject* py_explained_variance(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 3, [&]() -> PyObject* {
    const Call c(a[0]);
    const auto* v = c.get<float>(a[0], c.T);
    const auto* r = c.get<float>(a[1], c.T);
    const auto* m = c.get<uint8_t>(a[2], c.T);
    const hipStream_t st = stream(c);
    const at::Tensor moments = c.make(5, at::kDouble), ev = c.make(1, at::kDouble),
                     ws = c.workspace(SAO_OP_EXPLAINED_VARIANCE);
    const sao_status_t s = unlocked([&] {
      return g_api.explained_variance_store(v, r, m, c.T, ptr<double>(moments), ptr<double>(ev), ws.data_ptr(),
                                            ws.numel(), st);
    });
    return result(s, {ev, moments});
  });
}

// bind({name: address}, current_stream): the library's functions, and torch's.
PyObject* py_bind(PyObject*, PyObject* args) {
  PyObject *table, *current_stream;
  if (!PyArg_ParseTuple(args, "OO", &table, &current_stream)) return nullptr;
  auto set = [&](const char* name, auto& f) {
    PyObject* o = PyMapping_GetItemString(table, name);
    if (!o) return false;
    f = reinterpret_cast<std::remove_reference_t<decltype(f)>>(PyLong_AsVoidPtr(o));
    Py_DECREF(o);
    return f != nullptr && !PyErr_Occurred();
  };
  const bool all = set("sao_workspace_size", g_api.workspace_size) && set("sao_advantage", g_api.advantage) &&
                   set("sao_step_advantage", g_api.step_advantage) &&
                   set("sao_group_advantage", g_api.group_advantage) &&
                   set("sao_clipped_loss_store", g_api.clipped_loss_store) &&
                   set("sao_ppo_loss_store", g_api.ppo_loss_store) &&
                   set("sao_explained_variance_store", g_api.explained_variance_store);
  if (!all) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null function address");
    return nullptr;
  }
  Py_INCREF(current_stream);
  Py_XSETREF(g_current_stream, current_stream);
  Py_RETURN_NONE;
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyMethodDef method(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL, nullptr};
}

PyMethodDef g_methods[] = {
    {"bind", py_bind, METH_VARARGS, nullptr},
    method<py_advantage>("advantage"),
    method<py_step_advantage>("step_advantage"),
    method<py_group_advantage>("group_advantage"),
    method<py_clipped_loss>("clipped_loss"),
    method<py_ppo_loss>("ppo_loss"),
    method<py_explained_variance>("explained_variance"),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_fast", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// The torch version whose headers this was compiled with is the module's `torch`.
PyMODINIT_FUNC PyInit__fast() {
  PyObject* m = PyModule_Create(&g_module);
  if (m && PyModule_AddStringConstant(m, "torch", SAO_TORCH) < 0) Py_CLEAR(m);
  return m;
}
