// Native argument marshalling of the Python binding for the calls that take a list of problems: one
// decoding step passes 64 problems of four tensors, an adapter step 256 parameters, and reading those
// tensors attribute by attribute from Python took 145 and 350 us a call, several times the GPU's work.
// Each function checks and raises exactly as its caller documents and returns the library's status.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ops/empty.h>

#include <vector>

#include "attt.h"

namespace {

// A Python error is set; unwinds to the module function's handler.
struct PyError {};

[[noreturn]] void raise(PyObject* type, const char* fmt, const char* arg = "") {
  PyErr_Format(type, fmt, arg);
  throw PyError{};
}

// What a call reads, held until it returns: the problems, and the tensors that their mappings hand out.
// Only then may the allocator give their memory to the call's own workspace, whatever the caller's
// objects do meanwhile (a sequence may make its problems on access).
struct Held {
  std::vector<PyObject*> v;
  ~Held() {
    for (PyObject* o : v) Py_DECREF(o);
  }
  PyObject* keep(PyObject* o) {  // takes over the caller's reference
    if (!o) throw PyError{};
    try {
      v.push_back(o);
    } catch (...) {
      Py_DECREF(o);
      throw;
    }
    return o;
  }
};

// The problems of a call: a tuple of their own. Like len(), this refuses what has no length (a generator).
PyObject* list(Held& held, PyObject* seq) {
  const Py_ssize_t n = PyObject_Size(seq);
  if (n < 0) throw PyError{};
  held.v.reserve(1 + 8 * (size_t)n);
  return held.keep(PySequence_Tuple(seq));
}

// A mapping's entry; nullptr when `optional` and absent.
PyObject* item(Held& held, PyObject* map, PyObject* key, bool optional = false) {
  if (PyDict_CheckExact(map)) {
    PyObject* v = PyDict_GetItemWithError(map, key);
    if (v) {
      Py_INCREF(v);
      return held.keep(v);
    }
    if (optional && !PyErr_Occurred()) return nullptr;
    if (!PyErr_Occurred()) PyErr_SetObject(PyExc_KeyError, key);
    throw PyError{};
  }
  return held.keep(optional ? PyObject_CallMethod(map, "get", "O", key) : PyObject_GetItem(map, key));
}

const at::Tensor& tensor(PyObject* o, const char* name) {
  if (!THPVariable_Check(o)) raise(PyExc_TypeError, "%s must be a tensor", name);
  return THPVariable_Unpack(o);
}

const at::Tensor& device_tensor(PyObject* o, const char* name) {
  const at::Tensor& t = tensor(o, name);
  if (!t.is_cuda() || !t.is_contiguous()) raise(PyExc_ValueError, "%s must be a contiguous device tensor", name);
  return t;
}

int64_t dim(const at::Tensor& t, int64_t d) {
  if (d >= t.dim()) raise(PyExc_IndexError, "tuple index out of range");
  return t.size(d);
}

PyObject *k_x, *k_dy, *k_A, *k_B, *k_dA, *k_dB, *k_y, *k_scale, *k_param, *k_grad, *k_param_bf16;

// What float() takes, a number's text too; a TypeError for the rest.
float number(Held& held, PyObject* o) {
  PyObject* f = PyNumber_Float(o);
  if (!f && PyErr_ExceptionMatches(PyExc_ValueError)) PyErr_Format(PyExc_TypeError, "%R is not a number", o);
  return (float)PyFloat_AS_DOUBLE(held.keep(f));
}

float scale_of(Held& held, PyObject* map) { return number(held, item(held, map, k_scale)); }

// The library plans, launches and, the first time, loads its code: other Python threads run meanwhile. The
// tensors stay held, and nothing of Python is touched.
template <class F>
auto without_gil(F f) {
  struct Released {
    PyThreadState* state = PyEval_SaveThread();
    ~Released() { PyEval_RestoreThread(state); }
  } released;
  return f();
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

std::vector<attt_lora_problem> lora_problems(Held& held, PyObject* seq, bool check, at::ScalarType* dt, at::Device* dev) {
  PyObject* f = list(held, seq);
  const Py_ssize_t n = PyTuple_GET_SIZE(f);
  std::vector<attt_lora_problem> v(n);
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject* p = PyTuple_GET_ITEM(f, i);
    auto get = [&](PyObject* key, const char* name) -> const at::Tensor& {
      PyObject* o = item(held, p, key);
      return check ? device_tensor(o, name) : tensor(o, name);
    };
    const at::Tensor &x = get(k_x, "x"), &dy = get(k_dy, "dy"), &A = get(k_A, "A"), &B = get(k_B, "B"),
                     &dA = get(k_dA, "dA"), &dB = get(k_dB, "dB");
    if (i == 0 && dt) *dt = x.scalar_type();
    if (i == 0 && dev) *dev = x.device();
    v[i] = {x.data_ptr(), dy.data_ptr(), A.data_ptr(), B.data_ptr(), static_cast<float*>(dA.data_ptr()),
            static_cast<float*>(dB.data_ptr()), dim(x, 0), dim(x, 1), dim(dy, 1), (int32_t)dim(A, 0), scale_of(held, p)};
  }
  return v;
}

// lora_workspace_size(problems, dtype) -> (status, bytes)
PyObject* lora_workspace_size(PyObject* args) {
  Held held;
  PyObject* seq;
  int dtype;
  if (!PyArg_ParseTuple(args, "Oi", &seq, &dtype)) throw PyError{};
  const auto v = lora_problems(held, seq, false, nullptr, nullptr);
  size_t need = 0;
  const attt_status st = without_gil([&] { return attt_lora_workspace_size(v.data(), (int32_t)v.size(), dtype, &need); });
  return Py_BuildValue("in", (int)st, (Py_ssize_t)need);
}

// lora_grad(problems, workspace or None) -> status
PyObject* lora_grad(PyObject* args) {
  Held held;
  PyObject *seq, *ws_obj;
  if (!PyArg_ParseTuple(args, "OO", &seq, &ws_obj)) throw PyError{};
  at::ScalarType dt = at::kFloat;
  at::Device dev(at::kCPU);
  const auto v = lora_problems(held, seq, true, &dt, &dev);
  if (v.empty()) return PyLong_FromLong(ATTT_OK);
  if (dt != at::kFloat && dt != at::kBFloat16)
    raise(PyExc_TypeError, "unsupported dtype torch.%s (float32 or bfloat16)", c10::toString(dt));
  const int32_t dtype = dt == at::kBFloat16 ? ATTT_BF16 : ATTT_F32;
  size_t need = 0;
  attt_status st = without_gil([&] { return attt_lora_workspace_size(v.data(), (int32_t)v.size(), dtype, &need); });
  if (st) return PyLong_FromLong(st);
  at::Tensor ws;
  if (ws_obj != Py_None) ws = tensor(ws_obj, "workspace");
  void* s = stream();
  st = without_gil([&] {
    if (!ws.defined() || ws.numel() < (int64_t)need)
      ws = at::empty({(int64_t)(need > 256 ? need : 256)}, at::TensorOptions().dtype(at::kByte).device(dev));
    return attt_lora_grad(v.data(), (int32_t)v.size(), dtype, ws.data_ptr(), (size_t)ws.numel(), s);
  });
  return PyLong_FromLong(st);
}

// lora_sgd_step(params, lr, zero_grad) -> status
PyObject* lora_sgd_step(PyObject* args) {
  Held held;
  PyObject *seq, *lr_obj;
  int zero;
  if (!PyArg_ParseTuple(args, "OOp", &seq, &lr_obj, &zero)) throw PyError{};
  const float lr = number(held, lr_obj);
  PyObject* f = list(held, seq);
  const Py_ssize_t n = PyTuple_GET_SIZE(f);
  std::vector<attt_lora_param> v(n);
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject* p = PyTuple_GET_ITEM(f, i);
    const at::Tensor &P = device_tensor(item(held, p, k_param), "param"), &G = device_tensor(item(held, p, k_grad), "grad");
    if (P.scalar_type() != at::kFloat || G.scalar_type() != at::kFloat || G.numel() != P.numel())
      raise(PyExc_ValueError, "param and grad must be float32 tensors of equal size");
    void* copy = nullptr;
    PyObject* b = item(held, p, k_param_bf16, true);
    if (b && b != Py_None) {
      const at::Tensor& Pb = device_tensor(b, "param_bf16");
      if (Pb.scalar_type() != at::kBFloat16 || Pb.numel() != P.numel())
        raise(PyExc_ValueError, "param_bf16 must be a bfloat16 tensor of the param's size");
      copy = Pb.data_ptr();
    }
    v[i] = {static_cast<float*>(P.data_ptr()), static_cast<float*>(G.data_ptr()), copy, P.numel()};
  }
  void* s = stream();
  return PyLong_FromLong(without_gil([&] { return attt_lora_sgd_step(v.data(), (int32_t)n, lr, zero, s); }));
}

// lora_forward(problems) -> status
PyObject* lora_forward(PyObject* args) {
  Held held;
  PyObject* seq;
  if (!PyArg_ParseTuple(args, "O", &seq)) throw PyError{};
  PyObject* f = list(held, seq);
  const Py_ssize_t n = PyTuple_GET_SIZE(f);
  std::vector<attt_lora_fwd_problem> v(n);
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject* p = PyTuple_GET_ITEM(f, i);
    auto get = [&](PyObject* key, const char* name) -> const at::Tensor& {
      const at::Tensor& t = device_tensor(item(held, p, key), name);
      if (t.scalar_type() != at::kBFloat16 || t.dim() != 2) raise(PyExc_ValueError, "%s must be a 2-D bfloat16 tensor", name);
      return t;
    };
    const at::Tensor &x = get(k_x, "x"), &y = get(k_y, "y"), &A = get(k_A, "A"), &B = get(k_B, "B");
    v[i] = {x.data_ptr(), y.data_ptr(), A.data_ptr(), B.data_ptr(), x.size(0), x.size(1), y.size(1), (int32_t)A.size(0),
            scale_of(held, p)};
  }
  void* s = stream();
  return PyLong_FromLong(without_gil([&] { return attt_lora_forward(v.data(), (int32_t)n, s); }));
}

// lora_hot_swap(pairs) -> status
PyObject* lora_hot_swap(PyObject* args) {
  Held held;
  PyObject* seq;
  if (!PyArg_ParseTuple(args, "O", &seq)) throw PyError{};
  PyObject* f = list(held, seq);
  const Py_ssize_t n = PyTuple_GET_SIZE(f);
  std::vector<attt_lora_swap_item> v(n);
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject* pair = held.keep(PySequence_Tuple(PyTuple_GET_ITEM(f, i)));
    if (PyTuple_GET_SIZE(pair) != 2) raise(PyExc_ValueError, "a pair must be (src, dst)");
    const at::Tensor &src = device_tensor(PyTuple_GET_ITEM(pair, 0), "src"),
                     &dst = device_tensor(PyTuple_GET_ITEM(pair, 1), "dst");
    if (src.scalar_type() != at::kFloat || dst.scalar_type() != at::kBFloat16 || src.numel() != dst.numel())
      raise(PyExc_ValueError, "src must be float32 and dst bfloat16 of the same numel");
    v[i] = {static_cast<const float*>(src.data_ptr()), dst.data_ptr(), src.numel()};
  }
  void* s = stream();
  return PyLong_FromLong(without_gil([&] { return attt_lora_hot_swap(v.data(), (int32_t)n, s); }));
}

// No C++ exception leaves a module function; torch's become the Python errors they are elsewhere (its
// OutOfMemoryError among them).
template <PyObject* (*Fn)(PyObject*)>
PyObject* guarded(PyObject*, PyObject* args) {
  HANDLE_TH_ERRORS
  try {
    return Fn(args);
  } catch (const PyError&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

PyMethodDef kMethods[] = {{"lora_workspace_size", guarded<lora_workspace_size>, METH_VARARGS, nullptr},
                          {"lora_grad", guarded<lora_grad>, METH_VARARGS, nullptr},
                          {"lora_sgd_step", guarded<lora_sgd_step>, METH_VARARGS, nullptr},
                          {"lora_forward", guarded<lora_forward>, METH_VARARGS, nullptr},
                          {"lora_hot_swap", guarded<lora_hot_swap>, METH_VARARGS, nullptr},
                          {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_binding", "argument marshalling of libattt.so's list calls", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
  struct {
    PyObject** at;
    const char* name;
  } keys[] = {{&k_x, "x"},   {&k_dy, "dy"}, {&k_A, "A"},         {&k_B, "B"},         {&k_dA, "dA"},   {&k_dB, "dB"},
              {&k_y, "y"},   {&k_scale, "scale"}, {&k_param, "param"}, {&k_grad, "grad"}, {&k_param_bf16, "param_bf16"}};
  for (auto& k : keys)
    if (!(*k.at = PyUnicode_InternFromString(k.name))) return nullptr;
  return PyModule_Create(&kModule);
}
