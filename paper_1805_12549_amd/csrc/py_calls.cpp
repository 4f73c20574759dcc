// The calls a program makes per forward pass, as a Python extension: what binding.py does with ctypes, without the interpreter's part of it.
//
// One image through ResNet-18 was 22 launches of 3 to 9 us each (19 now); with tensors, workspace and arguments handled in Python a call took 5.0 us of host time
// (7.8 where it allocates its output, 11.6 with bitmap and counts too) beside the 2.7 us of a launch, and the GPU waited for the host.
//
// Only what a plain call needs is here.  A call with anything else - a tensor subclass, an active __torch_function__ mode, symbolic sizes, an argument
// that is no tensor - returns None, and binding.py takes it.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "cg_calls.h"
#include "cg_conv.h"

namespace {

// A layer as its calls see it; the handle is binding.py's, which drops this object before it destroys the handle.
struct Layer {
  PyObject_HEAD
  cg_conv* handle;
  int64_t ho, wo, c_out, words;
  at::ScalarType y_type;
};

// memory of the caching allocator that belongs to one stream, given back at the end of the call: it then serves later work of the same stream only, and
// under capture it is the graph's own
struct Scratch {
  void* ptr = nullptr;
  Scratch(size_t bytes, hipStream_t stream) {
    if (bytes) ptr = c10::hip::HIPCachingAllocator::raw_alloc_with_stream(bytes, stream);
  }
  ~Scratch() {
    if (ptr) c10::hip::HIPCachingAllocator::raw_delete(ptr);
  }
};

struct WithoutGil {
  PyThreadState* state = PyEval_SaveThread();
  ~WithoutGil() { PyEval_RestoreThread(state); }
};

extern PyTypeObject layer_type;

bool plain_tensor(PyObject* o) { return THPVariable_CheckExact(o); }

// an output argument: True (allocate), False / None (leave out), a tensor; anything else: false
bool wanted(PyObject* o, bool& make, at::Tensor& given) {
  if (o == Py_True) {
    make = true;
  } else if (o != Py_False && o != Py_None) {
    if (!plain_tensor(o)) return false;
    given = THPVariable_Unpack(o);
  }
  return true;
}

// forward(layer, stream, x, residual, y, bitmap, counts): (y, bitmap, counts); an error code; None: not a plain call
PyObject* forward(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  if (n_args != 7) {
    PyErr_SetString(PyExc_TypeError, "forward takes seven arguments");
    return nullptr;
  }
  if (Py_TYPE(args[0]) != &layer_type) {
    PyErr_SetString(PyExc_TypeError, "forward's first argument is a Layer");
    return nullptr;
  }
  const Layer* const l = (const Layer*)args[0];
  PyObject *const stream_arg = args[1], *const residual_arg = args[3], *const y_arg = args[4];
  if (at::impl::torch_function_mode_enabled() || !plain_tensor(args[2])) Py_RETURN_NONE;
  if (residual_arg != Py_None && !plain_tensor(residual_arg)) Py_RETURN_NONE;
  if (y_arg != Py_None && !plain_tensor(y_arg)) Py_RETURN_NONE;
  bool make_bitmap = false, make_counts = false;
  at::Tensor residual, y, bitmap, counts;
  if (!wanted(args[5], make_bitmap, bitmap) || !wanted(args[6], make_counts, counts)) Py_RETURN_NONE;
  const at::Tensor& x = THPVariable_Unpack(args[2]);
  if (x.unsafeGetTensorImpl()->has_symbolic_sizes_strides() || x.dim() == 0) Py_RETURN_NONE;
  if (residual_arg != Py_None) residual = THPVariable_Unpack(residual_arg);
  if (y_arg != Py_None) y = THPVariable_Unpack(y_arg);
  hipStream_t stream;
  if (stream_arg == Py_None) {
    stream = c10::hip::getCurrentHIPStream().stream();
  } else {
    PyObject* const address = PyObject_GetAttrString(stream_arg, "cuda_stream");
    if (!address) return nullptr;
    stream = (hipStream_t)PyLong_AsVoidPtr(address);
    Py_DECREF(address);
    if (PyErr_Occurred()) return nullptr;
  }
  int rc;
  {
    const WithoutGil released;
    const int64_t n = x.size(0), ho = l->ho, wo = l->wo, c = l->c_out;
    const at::TensorOptions here = at::TensorOptions().device(x.device());
    if (!y.defined()) y = at::empty_strided({n, ho, wo, c}, {ho * wo * c, wo * c, c, 1}, here.dtype(l->y_type));
    if (make_bitmap) bitmap = at::empty_strided({n * ho * wo, l->words}, {l->words, 1}, here.dtype(at::kInt));
    if (make_counts) counts = at::empty({2 + n * c}, here.dtype(at::kInt));
    const size_t need = cg_conv_call_scratch_bytes(l->handle, (int32_t)n, bitmap.defined(), counts.defined());
    const Scratch scratch(need, stream);
    rc = cg_conv_call(l->handle, (int32_t)n, x.data_ptr(), residual.defined() ? residual.data_ptr() : nullptr, y.data_ptr(),
                      bitmap.defined() ? (uint32_t*)bitmap.data_ptr() : nullptr, counts.defined() ? (uint32_t*)counts.data_ptr() : nullptr,
                      scratch.ptr, need, stream);
  }
  if (rc != CG_OK) return PyLong_FromLong(rc);
  PyObject* const out = PyTuple_New(3);
  if (!out) return nullptr;
  const auto put = [&](int at, PyObject* given, bool made, const at::Tensor& t) {
    PyObject* o = made ? THPVariable_Wrap(t) : t.defined() ? given : Py_None;
    if (!made) Py_INCREF(o);
    PyTuple_SET_ITEM(out, at, o);
  };
  put(0, y_arg, y_arg == Py_None, y);
  put(1, args[5], make_bitmap, bitmap);
  put(2, args[6], make_counts, counts);
  return out;
  END_HANDLE_TH_ERRORS
}

// empty_bf16(like, sizes ...): a contiguous bf16 tensor on the device of `like`; None: not a plain tensor
PyObject* empty_bf16(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  if (n_args < 2 || n_args > 5) {
    PyErr_SetString(PyExc_TypeError, "empty_bf16 takes a tensor and one to four sizes");
    return nullptr;
  }
  if (at::impl::torch_function_mode_enabled() || !plain_tensor(args[0])) Py_RETURN_NONE;
  const at::Tensor& like = THPVariable_Unpack(args[0]);
  int64_t sizes[4];
  for (Py_ssize_t i = 1; i < n_args; ++i) {
    sizes[i - 1] = PyLong_AsLongLong(args[i]);
    if (sizes[i - 1] == -1 && PyErr_Occurred()) return nullptr;
  }
  at::Tensor t;
  {
    const WithoutGil released;
    t = at::empty(at::IntArrayRef(sizes, n_args - 1), at::TensorOptions().device(like.device()).dtype(at::kBFloat16));
  }
  return THPVariable_Wrap(t);
  END_HANDLE_TH_ERRORS
}

int layer_init(PyObject* self, PyObject* args, PyObject*) {
  Layer* const l = (Layer*)self;
  unsigned long long handle;
  long long ho, wo, c_out;
  int out_dtype;
  if (!PyArg_ParseTuple(args, "KLLLi", &handle, &ho, &wo, &c_out, &out_dtype)) return -1;
  l->handle = (cg_conv*)handle;
  l->ho = ho;
  l->wo = wo;
  l->c_out = c_out;
  l->words = (c_out + 31) / 32;
  l->y_type = out_dtype == CG_F32 ? at::kFloat : out_dtype == CG_BF16 ? at::kBFloat16 : out_dtype == CG_I8 ? at::kChar : at::kInt;
  return 0;
}

PyTypeObject layer_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyMethodDef methods[] = {
    {"forward", (PyCFunction)(void (*)(void))forward, METH_FASTCALL, "forward(layer, stream, x, residual, y, bitmap, counts)"},
    {"empty_bf16", (PyCFunction)(void (*)(void))empty_bf16, METH_FASTCALL, "empty_bf16(like, *sizes)"},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", "Forward calls without the interpreter's part of them.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
  layer_type.tp_name = "_calls.Layer";
  layer_type.tp_basicsize = sizeof(Layer);
  layer_type.tp_flags = Py_TPFLAGS_DEFAULT;
  layer_type.tp_doc = "Layer(handle, ho, wo, c_out, out_dtype)";
  layer_type.tp_new = PyType_GenericNew;
  layer_type.tp_init = layer_init;
  if (PyType_Ready(&layer_type) < 0) return nullptr;
  PyObject* const m = PyModule_Create(&module);
  if (!m) return nullptr;
  // (torch's objects are read as this version lays them out)
  if (PyModule_AddStringConstant(m, "torch_version", CG_TORCH_VERSION) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  Py_INCREF(&layer_type);
  if (PyModule_AddObject(m, "Layer", (PyObject*)&layer_type) < 0) {
    Py_DECREF(&layer_type);
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
