// The host path of binding.gemm / gemm_static / grouped_gemm: reads the tensors' pointers and strides, makes the output and
// the workspace where the caller brought none, and calls the C entry point on the current stream.  Host code only; the
// entry points come in as addresses (bind), so that this file knows the C ABI and nothing else of the library.
//
// A decode step's kernel lasts a few microseconds and its launch costs about 2.7 us of host time; what the caller spends
// around it has to stay below that.  The same marshalling through ctypes took 8.5 - 11 us per call (the stream lookup
// alone 3 us, the output tensor 1.8 us, the foreign call 1 us), which is what a one-row product then took whatever its
// kernel did.
//
// Every function returns the output tensor, a negative ccq_status as an int, or None when an argument is not of the plain
// kind handled here; the Python code then goes through its general path, which checks and reports.  What PyTorch throws on
// the way reaches Python as PyTorch's own exception (torch.OutOfMemoryError from an allocation, which a serving loop catches
// to shrink its batch).
#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <Python.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <optional>

#include "ccq.h"

namespace {

struct Entry {
  decltype(&ccq_gemm) gemm = nullptr;
  decltype(&ccq_gemm_workspace_bytes) gemm_workspace = nullptr;
  decltype(&ccq_gemm_static) gemm_static = nullptr;
  decltype(&ccq_grouped_gemm) grouped = nullptr;
  decltype(&ccq_grouped_workspace_bytes) grouped_workspace = nullptr;
} entry;

struct Names {
  PyObject *desc, *codes, *scales, *alpha, *ssup, *E;
} names;

// The ccq_weight behind weight.desc (a ctypes structure).
class Descriptor {
 public:
  explicit Descriptor(PyObject* weight) {
    PyObject* d = PyObject_GetAttr(weight, names.desc);
    if (d && PyObject_GetBuffer(d, &view_, PyBUF_SIMPLE) == 0) {
      if (view_.len == (Py_ssize_t)sizeof(ccq_weight)) w = static_cast<const ccq_weight*>(view_.buf);
      held_ = true;
    }
    Py_XDECREF(d);   // (the view keeps its object)
    if (!w) PyErr_Clear();
  }
  ~Descriptor() {
    if (held_) PyBuffer_Release(&view_);
  }
  const ccq_weight* w = nullptr;

 private:
  Py_buffer view_;
  bool held_ = false;
};

// (A subclass may have an idea of its own of what its attributes are: the general path asks it.)
const at::Tensor* tensor(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

// Outputs and workspaces are made past PyTorch's dispatcher.  Where someone looks on there (a TorchDispatchMode, a
// functorch transform) the general path makes them, through it.
bool looked_on() { return c10::impl::dispatch_mode_enabled() || c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode); }

bool plain_bf16(const at::Tensor* t) { return t && t->dim() == 2 && t->scalar_type() == at::kBFloat16 && t->is_cuda() && t->stride(1) == 1; }

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// bf16 [rows][N] whose row stride is a multiple of 8 elements, as the entry points require.
at::Tensor new_output(int64_t rows, int64_t N, c10::Device device) {
  const int64_t ld = (N + 7) / 8 * 8;
  at::Tensor y = at::detail::empty_cuda({rows, ld}, at::kBFloat16, device, std::nullopt);
  if (ld != N) {
    const int64_t size[2] = {rows, N}, stride[2] = {ld, 1};
    y.unsafeGetTensorImpl()->set_sizes_and_strides(at::IntArrayRef(size, 2), at::IntArrayRef(stride, 2));
  }
  return y;
}

// Gives up the interpreter lock, as a foreign call through ctypes and torch.empty do: an allocation can wait for the device,
// a launch for room in its queue, and other threads run meanwhile.  Nothing of Python is touched inside.
class Unlocked {
 public:
  Unlocked() : state_(PyEval_SaveThread()) {}
  ~Unlocked() { PyEval_RestoreThread(state_); }
  Unlocked(const Unlocked&) = delete;
  Unlocked& operator=(const Unlocked&) = delete;

 private:
  PyThreadState* state_;
};

struct Workspace {
  at::Tensor held;
  void* ptr = nullptr;
  int64_t bytes = 0;
  bool of(PyObject* given) {
    const at::Tensor* t = tensor(given);
    if (!t) return false;
    ptr = t->data_ptr();
    bytes = (int64_t)t->nbytes();
    return true;
  }
  void make(int64_t need, c10::Device device) {
    if (need <= 0) return;
    held = at::detail::empty_cuda({need}, at::kByte, device, std::nullopt);
    ptr = held.data_ptr();
    bytes = need;
  }
};

PyObject* answer(int rc, PyObject* given, at::Tensor&& made) {
  if (rc != CCQ_OK) return PyLong_FromLong(rc);
  if (given == Py_None) return THPVariable_Wrap(std::move(made));
  Py_INCREF(given);
  return given;
}

PyObject* general() { Py_RETURN_NONE; }

// gemm(weight, x, out or None, workspace or None)
PyObject* call_gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 4 || !entry.gemm || looked_on()) return general();
  const at::Tensor *x = tensor(a[1]), *y = tensor(a[2]);
  if (!plain_bf16(x) || (a[2] != Py_None && (!y || y->dim() != 2))) return general();
  Descriptor d(a[0]);
  if (!d.w) return general();
  const int64_t M = x->size(0);
  if (M > INT32_MAX) return general();
  Workspace ws;
  if (a[3] != Py_None && !ws.of(a[3])) return general();
  const int64_t need = a[3] == Py_None ? entry.gemm_workspace(d.w, (int32_t)M) : 0;
  if (need < 0) return general();
  at::Tensor made;
  int rc;
  {
    Unlocked u;
    if (!y) y = &(made = new_output(M, d.w->N, x->device()));
    ws.make(need, x->device());
    rc = entry.gemm(d.w, x->data_ptr(), (int32_t)M, x->stride(0), y->data_ptr(), y->stride(0), ws.ptr, ws.bytes, current_stream());
  }
  return answer(rc, a[2], std::move(made));
  END_HANDLE_TH_ERRORS
}

// gemm_static(weight, x, out)
PyObject* call_gemm_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 3 || !entry.gemm_static || looked_on()) return general();
  const at::Tensor *x = tensor(a[1]), *y = tensor(a[2]);
  if (!plain_bf16(x) || !plain_bf16(y)) return general();
  Descriptor d(a[0]);
  if (!d.w) return general();
  const int64_t M = x->size(0);
  if (M > INT32_MAX || y->size(0) != M || y->size(1) != d.w->N) return general();
  int rc;
  {
    Unlocked u;
    rc = entry.gemm_static(d.w, x->data_ptr(), (int32_t)M, x->stride(0), y->data_ptr(), y->stride(0), current_stream());
  }
  return answer(rc, a[2], at::Tensor());
  END_HANDLE_TH_ERRORS
}

// Byte stride between the experts of one array of a stacked weight, 0 where there is none.
bool expert_stride(PyObject* weight, PyObject* name, int64_t* out, bool* there = nullptr) {
  PyObject* o = PyObject_GetAttr(weight, name);
  if (!o) {
    PyErr_Clear();
    return false;
  }
  const at::Tensor* t = tensor(o);
  const bool ok = t ? t->dim() >= 1 : o == Py_None;
  *out = t && ok ? t->stride(0) * (int64_t)t->element_size() : 0;
  if (there) *there = t != nullptr;
  Py_DECREF(o);
  return ok;
}

// The host copy of the expert offsets: a contiguous array of at least n int32.
class HostOffsets {
 public:
  HostOffsets(PyObject* given, int64_t n) {
    held_ = PyObject_GetBuffer(given, &view_, PyBUF_CONTIG_RO | PyBUF_FORMAT) == 0;
    if (!held_) PyErr_Clear();
    else if (view_.itemsize == 4 && view_.format && view_.format[0] == 'i' && view_.format[1] == 0 && view_.len >= (Py_ssize_t)(4 * n))
      offsets = static_cast<const int32_t*>(view_.buf);
  }
  ~HostOffsets() {
    if (held_) PyBuffer_Release(&view_);
  }
  const int32_t* offsets = nullptr;

 private:
  Py_buffer view_;
  bool held_ = false;
};

// grouped_gemm(weight, x, sorted_rows, expert_offsets, host offsets (a contiguous int32 array) or None, out or None, workspace or None)
PyObject* call_grouped(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 7 || !entry.grouped || looked_on()) return general();
  const at::Tensor *x = tensor(a[1]), *rows = tensor(a[2]), *offs = tensor(a[3]), *y = tensor(a[5]);
  if (!plain_bf16(x) || !rows || !offs || rows->scalar_type() != at::kInt || offs->scalar_type() != at::kInt) return general();
  if (a[5] != Py_None && (!y || y->dim() != 2)) return general();
  Descriptor d(a[0]);
  if (!d.w) return general();
  PyObject* e = PyObject_GetAttr(a[0], names.E);
  const long E = e ? PyLong_AsLong(e) : -1;
  Py_XDECREF(e);
  if (PyErr_Occurred()) PyErr_Clear();
  if (E <= 0 || E > INT32_MAX) return general();
  int64_t cs, ss, ab, sup;
  bool has_alpha;
  if (!expert_stride(a[0], names.codes, &cs) || !expert_stride(a[0], names.scales, &ss) || !expert_stride(a[0], names.alpha, &ab, &has_alpha) ||
      !expert_stride(a[0], names.ssup, &sup))
    return general();
  if (!has_alpha) ab = 2 * sup;   // (the super scales' stride is half of that of the fp32 arrays)
  std::optional<HostOffsets> host;
  if (a[4] != Py_None) {
    host.emplace(a[4], E + 1);
    if (!host->offsets) return general();
  }
  const int64_t P = rows->numel();
  if (P > INT32_MAX || x->size(0) > INT32_MAX) return general();
  Workspace ws;
  if (a[6] != Py_None && !ws.of(a[6])) return general();
  const int64_t need = a[6] == Py_None ? entry.grouped_workspace(d.w, (int32_t)E, (int32_t)P) : 0;
  at::Tensor made;
  int rc;
  {
    Unlocked u;
    if (!y) y = &(made = new_output(P, d.w->N, x->device()));
    ws.make(need, x->device());
    rc = entry.grouped(d.w, (int32_t)E, cs, ss, ab, x->data_ptr(), (int32_t)x->size(0), x->stride(0), static_cast<const int32_t*>(rows->data_ptr()), (int32_t)P,
                       static_cast<const int32_t*>(offs->data_ptr()), host ? host->offsets : nullptr, y->data_ptr(), y->stride(0), ws.ptr, ws.bytes,
                       current_stream());
  }
  return answer(rc, a[5], std::move(made));
  END_HANDLE_TH_ERRORS
}

// bind(addresses of ccq_gemm, ccq_gemm_workspace_bytes, ccq_gemm_static, ccq_grouped_gemm, ccq_grouped_workspace_bytes)
PyObject* call_bind(PyObject*, PyObject* args) {
  unsigned long long p[5];
  if (!PyArg_ParseTuple(args, "KKKKK", &p[0], &p[1], &p[2], &p[3], &p[4])) return nullptr;
  entry.gemm = reinterpret_cast<decltype(entry.gemm)>(p[0]);
  entry.gemm_workspace = reinterpret_cast<decltype(entry.gemm_workspace)>(p[1]);
  entry.gemm_static = reinterpret_cast<decltype(entry.gemm_static)>(p[2]);
  entry.grouped = reinterpret_cast<decltype(entry.grouped)>(p[3]);
  entry.grouped_workspace = reinterpret_cast<decltype(entry.grouped_workspace)>(p[4]);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", call_bind, METH_VARARGS, "addresses of the C entry points"},
    {"gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call_gemm)), METH_FASTCALL, nullptr},
    {"gemm_static", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call_gemm_static)), METH_FASTCALL, nullptr},
    {"grouped_gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call_grouped)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ccq_call", "host path of the multiply entry points", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__ccq_call() {
  names.desc = PyUnicode_InternFromString("desc");
  names.codes = PyUnicode_InternFromString("codes");
  names.scales = PyUnicode_InternFromString("scales");
  names.alpha = PyUnicode_InternFromString("alpha");
  names.ssup = PyUnicode_InternFromString("ssup");
  names.E = PyUnicode_InternFromString("E");
  return PyModule_Create(&module);
}
