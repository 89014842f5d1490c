// Python's way into the C ABI for the calls that a training step or a decode loop makes: tensors are taken apart, results
// and workspaces allocated and the library called without passing through ctypes and torch's Python functions (forward of
// two heads of 512 rows: 8.8 us of host time, of which the launch 3; 13.7 for the backward).  Argument marshalling only.
//
// Every function takes its arguments by position, None for a tensor to be allocated, and returns its results, or the
// library's status as an int where that is not RSA_OK.  What is allocated here are plain tensors.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <ATen/ops/zeros_like.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "rsa.h"

namespace {

struct Refused {};  // a Python error is set

// The arguments of one call.
struct Call {
  PyObject *const *args;
  rsa_desc *d = nullptr;
  Py_buffer view{};

  Call(PyObject *const *args_, Py_ssize_t n, Py_ssize_t want) : args(args_) {
    if (n != want) {
      PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
      throw Refused{};
    }
    // the descriptor is a ctypes structure, which exports its memory
    if (PyObject_GetBuffer(args[0], &view, PyBUF_SIMPLE) != 0) throw Refused{};
    if (view.len != (Py_ssize_t)sizeof(rsa_desc)) {
      PyErr_SetString(PyExc_TypeError, "not a descriptor");
      PyBuffer_Release(&view);
      throw Refused{};
    }
    d = static_cast<rsa_desc *>(view.buf);
  }
  ~Call() { PyBuffer_Release(&view); }
  Call(const Call &) = delete;

  bool given(int i) const { return args[i] != Py_None; }
  const at::Tensor &tensor(int i) const {
    if (!THPVariable_Check(args[i])) {
      PyErr_Format(PyExc_TypeError, "argument %d: a tensor expected, not %s", i, Py_TYPE(args[i])->tp_name);
      throw Refused{};
    }
    return THPVariable_Unpack(args[i]);
  }
  // ... of the GPU with a contiguous last index; other strides travel in the descriptor
  const at::Tensor &input(int i) const {
    const at::Tensor &t = tensor(i);
    if (!t.is_cuda() || t.dim() == 0 || t.stride(-1) != 1) {
      PyErr_Format(PyExc_AssertionError, "argument %d: a tensor of the GPU with a contiguous last index expected", i);
      throw Refused{};
    }
    return t;
  }
  template <class F> at::Tensor tensor_or(int i, F make) const { return given(i) ? tensor(i) : make(); }
};

void *ptr(const at::Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; }

at::Tensor bytes(size_t n, const at::Tensor &like) { return at::empty({(int64_t)n}, like.options().dtype(at::kByte)); }

PyObject *wrapped(std::initializer_list<at::Tensor> ts) {
  if (ts.size() == 1) return THPVariable_Wrap(*ts.begin());
  PyObject *r = PyTuple_New((Py_ssize_t)ts.size());
  if (!r) return nullptr;
  Py_ssize_t i = 0;
  for (const at::Tensor &t : ts) {
    PyObject *o = THPVariable_Wrap(t);
    if (!o) { Py_DECREF(r); return nullptr; }
    PyTuple_SET_ITEM(r, i++, o);
  }
  return r;
}

// The library call, on the current device's current stream and without the interpreter's lock (a launch may wait for a
// place in the queue).
template <class F> PyObject *finish(F call, std::initializer_list<at::Tensor> results) {
  void *stream = c10::hip::getCurrentHIPStream().stream();
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = call(stream);
  Py_END_ALLOW_THREADS
  return status == RSA_OK ? wrapped(results) : PyLong_FromLong(status);
}

template <PyObject *(*F)(Call &)> struct Entry {
  template <int N> static PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    try {
      Call c(args, n, N);
      return F(c);
    } catch (Refused) {
      return nullptr;
    }
    END_HANDLE_TH_ERRORS
  }
};

// workspace i of a pass of the attention: given, or what the descriptor asks for (nothing: none)
at::Tensor pass_workspace(const Call &c, int i, int pass, const at::Tensor &like, size_t &n) {
  if (c.given(i)) {
    const at::Tensor &t = c.tensor(i);
    n = (size_t)t.numel();
    return t;
  }
  n = rsa_workspace_bytes(c.d, pass);
  return n ? bytes(n, like) : at::Tensor();
}
at::Tensor workspace(const Call &c, int i, size_t need, const at::Tensor &like, size_t &n) {
  at::Tensor t = c.given(i) ? c.tensor(i) : bytes(need > 16 ? need : 16, like);
  n = (size_t)t.numel();
  return t;
}
at::Tensor row_terms(const at::Tensor &Q) {  // (Q may have fewer dimensions than the descriptor's four: taken as dense)
  return at::empty(Q.sizes().slice(0, Q.dim() < 3 ? Q.dim() : 3), Q.options().dtype(at::kFloat).memory_format(std::nullopt));
}
// The ranks' rows, as Python divides: a descriptor that the library will refuse gets there with any numbers in it.
int64_t rows_of(const rsa_desc *d) {
  if (d->N == 0) {
    PyErr_SetString(PyExc_ZeroDivisionError, "integer division or modulo by zero");
    throw Refused{};
  }
  int64_t chunk;
  if (d->N == -1) {
    chunk = (int64_t)(0 - (uint64_t)d->L);
  } else {
    chunk = d->L / d->N;
    if (d->L % d->N != 0 && (d->L < 0) != (d->N < 0)) --chunk;
  }
  return (int64_t)((uint64_t)((int64_t)d->rank_end - d->rank_begin) * (uint64_t)chunk);
}

// desc, Q, K, V, O, LSE, ws
PyObject *forward(Call &c) {
  const at::Tensor &Q = c.input(1), &K = c.input(2), &V = c.input(3);
  const at::Tensor O = c.tensor_or(4, [&] { return at::empty_like(Q); });
  const at::Tensor LSE = c.tensor_or(5, [&] { return row_terms(Q); });
  size_t n;
  const at::Tensor ws = pass_workspace(c, 6, 0, Q, n);
  return finish([&](void *st) {
    return rsa_forward(c.d, ptr(Q), ptr(K), ptr(V), ptr(O), static_cast<float *>(ptr(LSE)), ptr(ws), n, st); }, {O, LSE});
}

// desc, dO, Q, K, V, O, LSE, dQ, dK, dV, ws
PyObject *backward(Call &c) {
  const at::Tensor &dO = c.input(1), &Q = c.input(2), &K = c.input(3), &V = c.input(4), &O = c.input(5), &LSE = c.input(6);
  const at::Tensor dQ = c.tensor_or(7, [&] { return at::empty_like(Q); });
  const at::Tensor dK = c.tensor_or(8, [&] { return at::empty_like(K); });
  const at::Tensor dV = c.tensor_or(9, [&] { return at::empty_like(V); });
  size_t n;
  const at::Tensor ws = pass_workspace(c, 10, 1, Q, n);
  return finish([&](void *st) {
    return rsa_backward(c.d, ptr(dO), ptr(Q), ptr(K), ptr(V), ptr(O), static_cast<const float *>(ptr(LSE)), ptr(dQ), ptr(dK),
                        ptr(dV), ptr(ws), n, st); }, {dQ, dK, dV});
}

at::Tensor heads_like(const Call &c, const at::Tensor &X) {
  return at::empty({c.d->B, c.d->Z, rows_of(c.d), c.d->A}, X.options());
}
// desc, X, W, Q, K, V
PyObject *qkv_proj(Call &c) {
  const at::Tensor &X = c.tensor(1), &W = c.tensor(2);
  const int32_t H = (int32_t)X.size(-1);
  const auto make = [&] { return heads_like(c, X); };
  const at::Tensor Q = c.tensor_or(3, make), K = c.tensor_or(4, make), V = c.tensor_or(5, make);
  return finish([&](void *st) { return rsa_qkv_proj(c.d, H, ptr(X), ptr(W), ptr(Q), ptr(K), ptr(V), st); }, {Q, K, V});
}
// desc, O, Wo, Y
PyObject *out_proj(Call &c) {
  const at::Tensor &O = c.tensor(1), &Wo = c.tensor(2);
  const int32_t H = (int32_t)Wo.size(-1);
  const at::Tensor Y = c.tensor_or(3, [&] { return at::empty({O.size(0), O.size(2), H}, O.options()); });
  return finish([&](void *st) { return rsa_out_proj(c.d, H, ptr(O), ptr(Wo), ptr(Y), st); }, {Y});
}
// desc, dY, O, Wo, dO, dWo, ws
PyObject *out_proj_bwd(Call &c) {
  const at::Tensor &dY = c.tensor(1), &O = c.tensor(2), &Wo = c.tensor(3);
  const int32_t H = (int32_t)Wo.size(-1);
  const at::Tensor dO = c.tensor_or(4, [&] { return at::empty_like(O); });
  const at::Tensor dWo = c.tensor_or(5, [&] { return at::empty(Wo.sizes(), Wo.options().dtype(at::kFloat)); });
  size_t n;
  const at::Tensor ws = workspace(c, 6, rsa_proj_workspace_bytes(c.d, H), O, n);
  return finish([&](void *st) {
    return rsa_out_proj_bwd(c.d, H, ptr(dY), ptr(O), ptr(Wo), ptr(dO), static_cast<float *>(ptr(dWo)), ptr(ws), n, st); },
    {dO, dWo});
}
// desc, dQ, dK, dV, X, W, dX, dW, ws
PyObject *qkv_proj_bwd(Call &c) {
  const at::Tensor &dQ = c.tensor(1), &dK = c.tensor(2), &dV = c.tensor(3), &X = c.tensor(4), &W = c.tensor(5);
  const int32_t H = (int32_t)X.size(-1);
  const at::Tensor dX = c.tensor_or(6, [&] { return at::empty_like(X); });
  const at::Tensor dW = c.tensor_or(7, [&] { return at::empty(W.sizes(), W.options().dtype(at::kFloat)); });
  size_t n;
  const at::Tensor ws = workspace(c, 8, rsa_proj_workspace_bytes(c.d, H), X, n);
  return finish([&](void *st) {
    return rsa_qkv_proj_bwd(c.d, H, ptr(dQ), ptr(dK), ptr(dV), ptr(X), ptr(W), ptr(dX), static_cast<float *>(ptr(dW)), ptr(ws),
                            n, st); }, {dX, dW});
}
// desc, X, E, Xp, ws
PyObject *linformer_project(Call &c) {
  const at::Tensor &X = c.tensor(1), &E = c.tensor(2);
  const int32_t Kp = (int32_t)E.size(1);
  const at::Tensor Xp = c.tensor_or(3, [&] { return at::empty({X.size(0), X.size(1), Kp, X.size(3)}, X.options()); });
  size_t n;
  const at::Tensor ws = workspace(c, 4, rsa_linformer_workspace_bytes(c.d, Kp), X, n);
  return finish([&](void *st) { return rsa_linformer_project(c.d, Kp, ptr(X), ptr(E), ptr(Xp), ptr(ws), n, st); }, {Xp});
}
// desc, Q, Kp, Vp, O, LSE
PyObject *linformer_forward(Call &c) {
  const at::Tensor &Q = c.tensor(1), &Kp = c.tensor(2), &Vp = c.tensor(3);
  const at::Tensor O = c.tensor_or(4, [&] { return at::empty_like(Q); });
  const at::Tensor LSE = c.tensor_or(5, [&] { return row_terms(Q); });
  return finish([&](void *st) {
    return rsa_linformer_forward(c.d, (int32_t)Kp.size(2), ptr(Q), ptr(Kp), ptr(Vp), ptr(O), static_cast<float *>(ptr(LSE)), st); },
    {O, LSE});
}
// desc, dO, Q, Kp, Vp, O, LSE, dQ, dKp, dVp, ws
PyObject *linformer_backward(Call &c) {
  const at::Tensor &dO = c.tensor(1), &Q = c.tensor(2), &Kp = c.tensor(3), &Vp = c.tensor(4), &O = c.tensor(5), &LSE = c.tensor(6);
  const int32_t kp = (int32_t)Kp.size(2);
  const at::Tensor dQ = c.tensor_or(7, [&] { return at::empty_like(Q); });
  const at::Tensor dKp = c.tensor_or(8, [&] { return at::empty_like(Kp); });
  const at::Tensor dVp = c.tensor_or(9, [&] { return at::empty_like(Vp); });
  size_t n;
  const at::Tensor ws = workspace(c, 10, rsa_linformer_workspace_bytes(c.d, kp), Q, n);
  return finish([&](void *st) {
    return rsa_linformer_backward(c.d, kp, ptr(dO), ptr(Q), ptr(Kp), ptr(Vp), ptr(O), static_cast<const float *>(ptr(LSE)),
                                  ptr(dQ), ptr(dKp), ptr(dVp), ptr(ws), n, st); }, {dQ, dKp, dVp});
}
// desc, dXp, X, E, dX, dE: the rows of the descriptor's ranks; a new tensor is zero elsewhere (with all ranks every row is
// written: zeroing both first costs as much as a fifth of the kernels' traffic)
PyObject *linformer_project_bwd(Call &c) {
  const at::Tensor &dXp = c.tensor(1), &X = c.tensor(2), &E = c.tensor(3);
  const bool all = c.d->rank_begin == 0 && c.d->rank_end == c.d->N;
  const at::Tensor dX = c.tensor_or(4, [&] { return all ? at::empty_like(X) : at::zeros_like(X); });
  const at::Tensor dE = c.tensor_or(5, [&] {
    const auto o = E.options().dtype(at::kFloat);
    return all ? at::empty_like(E, o, at::MemoryFormat::Contiguous) : at::zeros_like(E, o, at::MemoryFormat::Contiguous);
  });
  return finish([&](void *st) {
    return rsa_linformer_project_bwd(c.d, (int32_t)E.size(1), ptr(dXp), ptr(X), ptr(E), ptr(dX), static_cast<float *>(ptr(dE)), st); },
    {dX, dE});
}

template <PyObject *(*F)(Call &), int N> PyMethodDef method(const char *name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&Entry<F>::template call<N>)), METH_FASTCALL, nullptr};
}

}  // namespace

PyMODINIT_FUNC PyInit__binding(void);
PyMODINIT_FUNC PyInit__binding(void) {
  static PyMethodDef table[] = {
      method<forward, 7>("forward"), method<backward, 11>("backward"), method<qkv_proj, 6>("qkv_proj"),
      method<out_proj, 4>("out_proj"), method<out_proj_bwd, 7>("out_proj_bwd"), method<qkv_proj_bwd, 9>("qkv_proj_bwd"),
      method<linformer_project, 5>("linformer_project"), method<linformer_forward, 6>("linformer_forward"),
      method<linformer_backward, 11>("linformer_backward"), method<linformer_project_bwd, 6>("linformer_project_bwd"),
      {nullptr, nullptr, 0, nullptr}};
  static PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, table, nullptr, nullptr, nullptr, nullptr};
  return PyModule_Create(&module);
}
