// Calls whose way through Python takes longer than the kernel behind them, as a Python extension on torch's own tensors.
//
// tsd_accept_commit_static is one launch of some 4 us.  Through ctypes, with its outputs allocated by torch.empty, a call took 10.5 us: three
// allocations and a view 5.4, the arguments' conversion and the launch 3.5.  From here 8 series of 4 x 16 take 6.2 us, 1024 of
// 6 x 96 6.5, the kernel's own time; on inputs that were not read just before 10.7 -> 6.9 and 10.2 -> 8.8.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

// tsd_accept_commit_static (tsd.h), handed over by the binding that loaded the library
using AcceptFn = int (*)(const float*, const float*, const float*, const int32_t*, int32_t, int32_t, int32_t, float, float, float, uint64_t,
                         uint32_t, int32_t*, float*, float*, float*, void*);
AcceptFn accept_fn = nullptr;

// A contiguous tensor of its own over `whole`'s memory from element `offset` on.
at::Tensor over(const at::Tensor& whole, at::IntArrayRef sizes, int64_t offset) {
  at::Tensor t = at::detail::make_tensor<c10::TensorImpl>(c10::Storage(whole.storage()), whole.key_set(), whole.dtype());
  t.unsafeGetTensorImpl()->set_sizes_contiguous(sizes);
  t.unsafeGetTensorImpl()->set_storage_offset(offset);
  return t;
}

const at::Tensor* tensor(PyObject* o, const char* name) {
  if (THPVariable_Check(o)) return &THPVariable_Unpack(o);
  PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
  return nullptr;
}

// (lib's function address)
PyObject* bind(PyObject*, PyObject* address) {
  void* p = PyLong_AsVoidPtr(address);
  if (!p && PyErr_Occurred()) return nullptr;
  accept_fn = reinterpret_cast<AcceptFn>(p);
  Py_RETURN_NONE;
}

// X, mu_q, mu_p, rounds or None, sigma_p, sigma_q, fallback_r, seed, flags, want_taps -> (status, n_acc, commit, ell, logu)
PyObject* accept_commit_static(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 10 || !accept_fn) {
    PyErr_SetString(PyExc_TypeError, "accept_commit_static takes ten arguments, after bind()");
    return nullptr;
  }
  const at::Tensor *X = tensor(args[0], "X"), *mu_q = X ? tensor(args[1], "mu_q") : nullptr, *mu_p = mu_q ? tensor(args[2], "mu_p") : nullptr;
  if (!mu_p) return nullptr;
  const at::Tensor* rounds = nullptr;
  if (args[3] != Py_None && !(rounds = tensor(args[3], "rounds"))) return nullptr;
  const double sigma_p = PyFloat_AsDouble(args[4]), sigma_q = PyFloat_AsDouble(args[5]), fallback_r = PyFloat_AsDouble(args[6]);
  const uint64_t seed = PyLong_AsUnsignedLongLongMask(args[7]);
  const uint32_t flags = (uint32_t)PyLong_AsUnsignedLongMask(args[8]);
  const int taps = PyObject_IsTrue(args[9]);
  if (PyErr_Occurred()) return nullptr;
  try {
    if (X->dim() != 3) {
      PyErr_Format(PyExc_ValueError, "X must be [B, K, P], has %d dimensions", (int)X->dim());
      return nullptr;
    }
    if (!X->device().has_index()) {  // (a tensor that is not on a GPU, whose pointer must not reach a kernel)
      PyErr_Format(PyExc_ValueError, "Expected a cuda device, but got: %s", X->device().str().c_str());
      return nullptr;
    }
    const int64_t B = X->size(0), K = X->size(1), P = X->size(2);
    const auto f32 = at::TensorOptions().dtype(at::kFloat).device(X->device());
    // (the kernel writes every entry: nothing to fill beforehand)
    // (the two taps in one allocation.  Not the counts with them: torch.save refuses tensors of two types over one memory, and a kept count
    // would keep the taps.)
    at::Tensor n_acc = at::empty({B}, f32.dtype(at::kInt)), commit = at::empty({B, K + 1, P}, f32), ell, logu;
    if (taps) {
      const at::Tensor both = at::empty({2, B, K}, f32);
      ell = over(both, {B, K}, 0);
      logu = over(both, {B, K}, B * K);
    }
    auto at_of = [](const at::Tensor& t) { return static_cast<float*>(t.data_ptr()); };
    const float *x = at_of(*X), *q = at_of(*mu_q), *p = at_of(*mu_p);
    const int32_t* r = rounds ? static_cast<int32_t*>(rounds->data_ptr()) : nullptr;
    void* stream = c10::hip::getCurrentHIPStream(X->device().index()).stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = accept_fn(x, q, p, r, (int32_t)B, (int32_t)K, (int32_t)P, (float)sigma_p, (float)sigma_q, (float)fallback_r, seed, flags,
                   static_cast<int32_t*>(n_acc.data_ptr()), at_of(commit), taps ? at_of(ell) : nullptr, taps ? at_of(logu) : nullptr, stream);
    Py_END_ALLOW_THREADS
    PyObject* out = PyTuple_New(5);
    if (!out) return nullptr;
    PyTuple_SET_ITEM(out, 0, PyLong_FromLong(rc));
    PyTuple_SET_ITEM(out, 1, THPVariable_Wrap(n_acc));
    PyTuple_SET_ITEM(out, 2, THPVariable_Wrap(commit));
    for (int i = 0; i < 2; ++i) {
      PyObject* o = taps ? THPVariable_Wrap(i ? logu : ell) : Py_None;
      if (!taps) Py_INCREF(Py_None);
      PyTuple_SET_ITEM(out, 3 + i, o);
    }
    return out;
  } catch (const std::exception&) {
    torch::translate_exception_to_python(std::current_exception());  // (torch.OutOfMemoryError among them)
    return nullptr;
  }
}

PyMethodDef methods[] = {{"bind", bind, METH_O, "the address of tsd_accept_commit_static"},
                         {"accept_commit_static", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(accept_commit_static)), METH_FASTCALL,
                          "see binding.accept_commit_static"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_calls() { return PyModule_Create(&module); }
