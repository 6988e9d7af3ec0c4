// Argument marshalling of the step entry points for the calls a training loop makes: plain tensors on the current device, with the
// workspace and the result handed over.  A short step is bound by the host, and of its time in Python most went into looking at the
// tensors.  Python / here, us a call, back to back: fused step of 4 fp32 rows, d = 1000 7.2 / 4.8 (the kernel's time), in buffers of their
// own 10.8 / 4.8, clipped 11.0 / 7.6; 32 rows in buffers of their own 21 / 7.8, 512 rows 190 / 55.
// Every function returns the library's code, or None for a call that it does not take, before anything is enqueued: the caller then goes
// through the checks in Python, which also word the exceptions.  Whatever is taken here passes those checks.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "normtest.h"

namespace {

struct Refused {};   // thrown where Python has to look

PyObject* raw_stream = nullptr;   // torch._C._cuda_getCurrentRawStream
PyObject* hyper_type = nullptr;
PyObject* shard_type = nullptr;
PyObject* parameter_type = nullptr;

// The tensor behind an argument: torch.Tensor itself or a Parameter, no other subclass, which may be anything.
const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o) && (PyObject*)Py_TYPE(o) != parameter_type) throw Refused();
  return THPVariable_Unpack(o);
}

struct Where {
  c10::Device device = c10::Device(c10::DeviceType::CPU);
  int64_t d = 0;
};

// The current device's tensors only: the library launches there.
void check_device(const at::Tensor& t) {
  if (!t.is_cuda() || c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getDevice() != t.device()) throw Refused();
}

int dtype_of(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return NT_F32;
  if (t.scalar_type() == at::kBFloat16) return NT_BF16;
  throw Refused();
}

// w, m, v, the mean: contiguous float32 vectors of at least d elements beside the gradients, or None where that may be.
float* vector_of(PyObject* o, const Where& at_, bool required) {
  if (o == Py_None && !required) return nullptr;
  const at::Tensor& t = tensor(o);
  if (t.scalar_type() != at::kFloat || t.device() != at_.device || !t.is_contiguous() || t.numel() < at_.d) throw Refused();
  return (float*)t.data_ptr();
}

int64_t integer(PyObject* o) {
  if (!PyLong_CheckExact(o)) throw Refused();
  const long long x = PyLong_AsLongLong(o);
  if (x == -1 && PyErr_Occurred()) throw Refused();
  return x;
}

// Address of a ctypes structure; the argument holds it while the call runs.
template <class T>
const T* structure(PyObject* o, PyObject* type) {
  if ((PyObject*)Py_TYPE(o) != type) throw Refused();
  Py_buffer view;
  if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Refused();
  const T* p = view.len == (Py_ssize_t)sizeof(T) ? (const T*)view.buf : nullptr;
  PyBuffer_Release(&view);
  if (!p) throw Refused();
  return p;
}
const nt_shard_info* shard_of(PyObject* o) { return o == Py_None ? nullptr : structure<nt_shard_info>(o, shard_type); }

void* stream_of(const c10::Device& device) {
  PyObject* index = PyLong_FromLong(device.index());
  PyObject* handle = index ? PyObject_CallOneArg(raw_stream, index) : nullptr;
  Py_XDECREF(index);
  if (!handle) throw Refused();
  void* st = PyLong_AsVoidPtr(handle);
  Py_DECREF(handle);
  if (!st && PyErr_Occurred()) throw Refused();
  return st;
}

template <class F>
F* entry(PyObject* o) {
  void* p = PyLong_Check(o) ? PyLong_AsVoidPtr(o) : nullptr;
  if (!p) throw Refused();
  return (F*)p;
}

struct Bytes {
  void* data;
  size_t size;
};
Bytes bytes_of(PyObject* o) {
  const at::Tensor& t = tensor(o);
  return {t.data_ptr(), (size_t)(t.numel() * t.element_size())};
}

// (J, ld) tensor whose rows are the gradients; d: the argument, None for all columns.
struct Matrix {
  const void* data;
  int64_t J, ld;
  int dtype;
  Where at_;
};
Matrix matrix_of(PyObject* grads, PyObject* d) {
  const at::Tensor& g = tensor(grads);
  check_device(g);
  if (g.dim() != 2 || (g.size(1) > 1 && g.stride(1) != 1)) throw Refused();
  Matrix m;
  m.J = g.size(0);
  m.ld = m.J > 1 ? g.stride(0) : g.size(1);
  m.dtype = dtype_of(g);
  m.data = g.data_ptr();
  m.at_ = {g.device(), d == Py_None ? g.size(1) : integer(d)};
  return m;
}

// CALL with the interpreter released, as ctypes does.
template <class CALL>
PyObject* enqueue(CALL call) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

template <class BODY>
PyObject* guarded(Py_ssize_t given, Py_ssize_t wanted, BODY body) {
  if (given != wanted) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    return body();
  } catch (const Refused&) {
  } catch (const std::exception&) {
  }
  PyErr_Clear();
  Py_RETURN_NONE;
}

// step(entry, grads, w, m, v, hyper, d, shard, gbar_out, workspace, result)
PyObject* step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&] {
    auto* f = entry<decltype(normtest_step)>(a[0]);
    const Matrix g = matrix_of(a[1], a[6]);
    float *w = vector_of(a[2], g.at_, false), *m = vector_of(a[3], g.at_, false), *v = vector_of(a[4], g.at_, false);
    const nt_hyper* hyper = structure<nt_hyper>(a[5], hyper_type);
    const nt_shard_info* shard = shard_of(a[7]);
    float* gbar = vector_of(a[8], g.at_, false);
    const Bytes ws = bytes_of(a[9]);
    nt_result* res = (nt_result*)bytes_of(a[10]).data;
    void* st = stream_of(g.at_.device);
    return enqueue([&] { return f(g.data, (nt_dtype)g.dtype, g.J, g.at_.d, g.ld, w, m, v, gbar, hyper, shard, ws.data, ws.size, res, st); });
  });
}

// step_clipped(entry, grads, w, m, v, gbar_buf, max_norm, hyper, d, shard, workspace, result)
PyObject* step_clipped(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 12, [&] {
    auto* f = entry<decltype(normtest_step_clipped)>(a[0]);
    const Matrix g = matrix_of(a[1], a[8]);
    float *w = vector_of(a[2], g.at_, true), *m = vector_of(a[3], g.at_, true), *v = vector_of(a[4], g.at_, true);
    float* gbar = vector_of(a[5], g.at_, true);
    if (!PyFloat_CheckExact(a[6])) throw Refused();
    const double max_norm = PyFloat_AS_DOUBLE(a[6]);
    const nt_hyper* hyper = structure<nt_hyper>(a[7], hyper_type);
    const nt_shard_info* shard = shard_of(a[9]);
    const Bytes ws = bytes_of(a[10]);
    nt_result* res = (nt_result*)bytes_of(a[11]).data;
    void* st = stream_of(g.at_.device);
    return enqueue([&] {
      return f(g.data, (nt_dtype)g.dtype, g.J, g.at_.d, g.ld, w, m, v, gbar, max_norm, hyper, shard, ws.data, ws.size, res, st);
    });
  });
}

// step_rows(entry, rows, w, m, v, hyper, d, table, shard, gbar_out, workspace, result); rows: a list or tuple
PyObject* step_rows(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 12, [&] {
    auto* f = entry<decltype(normtest_step_rows)>(a[0]);
    if (!PyList_CheckExact(a[1]) && !PyTuple_CheckExact(a[1])) throw Refused();
    const Py_ssize_t J = PySequence_Fast_GET_SIZE(a[1]);
    if (J < 1) throw Refused();
    PyObject** rows = PySequence_Fast_ITEMS(a[1]);
    const at::Tensor& first = tensor(rows[0]);
    check_device(first);
    const int dtype = dtype_of(first);
    int64_t shortest = INT64_MAX;
    for (Py_ssize_t j = 0; j < J; ++j) {
      const at::Tensor& r = tensor(rows[j]);
      if (r.scalar_type() != first.scalar_type() || r.device() != first.device() || r.dim() != 1 || !r.is_contiguous()) throw Refused();
      if (r.numel() < shortest) shortest = r.numel();
    }
    const Where at_ = {first.device(), a[6] == Py_None ? shortest : integer(a[6])};
    if (shortest < at_.d) throw Refused();
    float *w = vector_of(a[2], at_, false), *m = vector_of(a[3], at_, false), *v = vector_of(a[4], at_, false);
    const nt_hyper* hyper = structure<nt_hyper>(a[5], hyper_type);
    at::Tensor table = tensor(a[7]);
    if (!table.is_cuda()) throw Refused();
    const nt_shard_info* shard = shard_of(a[8]);
    float* gbar = vector_of(a[9], at_, false);
    const Bytes ws = bytes_of(a[10]);
    nt_result* res = (nt_result*)bytes_of(a[11]).data;
    void* st = stream_of(at_.device);
    const void* const* entries = (const void* const*)table.data_ptr();
    // the kernels read the table: its memory stays until they have
    table.record_stream(c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getStream(at_.device));
    return enqueue([&] { return f(entries, (nt_dtype)dtype, J, at_.d, w, m, v, gbar, hyper, shard, ws.data, ws.size, res, st); });
  });
}

// adamw_gbar(entry, gbar, w, m, v, hyper, grad_scale, d, result)
PyObject* adamw_gbar(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 9, [&] {
    auto* f = entry<decltype(normtest_adamw_gbar)>(a[0]);
    const at::Tensor& g = tensor(a[1]);
    check_device(g);
    const Where at_ = {g.device(), a[7] == Py_None ? g.numel() : integer(a[7])};
    float *gbar = vector_of(a[1], at_, true), *w = vector_of(a[2], at_, true), *m = vector_of(a[3], at_, true);
    float* v = vector_of(a[4], at_, true);
    const nt_hyper* hyper = structure<nt_hyper>(a[5], hyper_type);
    if (!PyFloat_CheckExact(a[6])) throw Refused();
    const double scale = PyFloat_AS_DOUBLE(a[6]);
    const nt_result* res = a[8] == Py_None ? nullptr : (const nt_result*)bytes_of(a[8]).data;
    void* st = stream_of(at_.device);
    return enqueue([&] { return f(gbar, at_.d, w, m, v, hyper, scale, res, st); });
  });
}

// layer_stats(entry, grads, layer_offsets, workspace, need, d, layers); grads: the (J, ld) tensor; need(gdtype, J, d, flags): bytes of the
// workspace the step needed, an entry of the library too
PyObject* layer_stats(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 7, [&] {
    auto* f = entry<decltype(normtest_layer_stats)>(a[0]);
    const Matrix g = matrix_of(a[1], a[5]);
    const at::Tensor& offsets = tensor(a[2]);
    if (offsets.scalar_type() != at::kLong || offsets.device() != g.at_.device || offsets.dim() != 1 || !offsets.is_contiguous() ||
        offsets.numel() < 2 || offsets.numel() > (1 << 24))
      throw Refused();
    const int32_t L = (int32_t)offsets.numel() - 1;
    if (tensor(a[3]).device() != g.at_.device) throw Refused();
    const Bytes ws = bytes_of(a[3]), layers = bytes_of(a[6]);
    if (ws.size < entry<decltype(normtest_workspace_bytes_for)>(a[4])((nt_dtype)g.dtype, g.J, g.at_.d, NT_DO_STATS)) throw Refused();
    if (layers.size < (size_t)L * sizeof(nt_layer_stats)) throw Refused();
    void* st = stream_of(g.at_.device);
    const int64_t* off = (const int64_t*)offsets.data_ptr();
    return enqueue([&] { return f(g.data, 0, (nt_dtype)g.dtype, g.J, g.at_.d, g.ld, off, L, ws.data, (nt_layer_stats*)layers.data, st); });
  });
}

// init(nt_hyper, nt_shard_info, torch.nn.Parameter, torch._C._cuda_getCurrentRawStream)
PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 4, [&]() -> PyObject* {
    PyObject** to[4] = {&hyper_type, &shard_type, &parameter_type, &raw_stream};
    for (int k = 0; k < 4; ++k) {
      Py_INCREF(a[k]);
      Py_XSETREF(*to[k], a[k]);
    }
    Py_RETURN_NONE;
  });
}

#define FAST(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(init),       FAST(step),        FAST(step_clipped), FAST(step_rows),
                         FAST(adamw_gbar), FAST(layer_stats), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_callpath", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__callpath() { return PyModule_Create(&module); }
