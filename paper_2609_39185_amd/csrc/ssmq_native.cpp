// ssmq_native.cpp -- argument marshalling of the per-token calls for CPython: from
// torch tensors and integers to the C ABI of include/ssmq.h, without building ctypes
// objects for each argument (through ctypes a call with eleven tensors takes 6 to 7 us
// of host time before the launch, more than the kernels of the small layers take: 1536
// Mamba-1 channels, conv1d_update and state_update, 17.0 us per token; this way 8.1).
//
// Each function takes plain positional arguments and returns the ABI's status, or None
// for a call that it leaves to the ctypes path: any argument that is not an exact
// torch.Tensor (or int, bool, None), lives outside the GPU, is not contiguous, has no
// storage of its own (transforms, fake tensors) or has another shape or element size
// than the call needs. That path then accepts or rejects the call as it always does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include <cstdint>

#include "ssmq.h"

namespace {

// A call that the ctypes path has to take.
struct Unhandled {};

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw Unhandled{};
  const at::Tensor& t = THPVariable_Unpack(o);
  const c10::DispatchKeySet wrapped({c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                     c10::DispatchKey::Functionalize, c10::DispatchKey::Python});
  if (!t.defined() || t.key_set().has_any(wrapped) || !t.has_storage() || !t.is_cuda() || !t.is_contiguous())
    throw Unhandled{};
  return t;
}

void* pointer(PyObject* o) { return o == Py_None ? nullptr : tensor(o).mutable_data_ptr(); }
float* floats(PyObject* o) { return static_cast<float*>(pointer(o)); }

uint64_t integer(PyObject* o) {  // modulo 2^64, as ctypes fields take their integers
  if (!PyLong_Check(o)) throw Unhandled{};
  return PyLong_AsUnsignedLongLongMask(o);
}
int32_t int32(PyObject* o) { return static_cast<int32_t>(static_cast<uint32_t>(integer(o))); }
uint32_t uint32(PyObject* o) { return static_cast<uint32_t>(integer(o)); }
bool truth(PyObject* o) {
  if (o != Py_True && o != Py_False) throw Unhandled{};
  return o == Py_True;
}

// The stream's handle: the caller's, or torch's current stream of the tensor's device.
void* stream_of(PyObject* o, const at::Tensor& t) {
  if (o != Py_None) return reinterpret_cast<void*>(integer(o));
  return static_cast<void*>(c10::hip::getCurrentHIPStream(t.get_device()).stream());
}

struct Format {
  int64_t entries;  // per element of the code tensor
  int64_t bytes;    // of that element
};
Format format_of(int32_t f) {
  switch (f) {
    case SSMQ_FP16: case SSMQ_BF16: return {1, 2};
    case SSMQ_FP32: return {1, 4};
    case SSMQ_INT4: return {2, 1};
    default: return {1, 1};
  }
}

template <typename Call>
PyObject* handled(Call&& call) {
  try {
    return call();
  } catch (...) {  // Unhandled, or torch refusing an access: the ctypes path decides
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

template <typename Launch>
PyObject* launched(Launch&& launch) {
  ssmq_status st;
  Py_BEGIN_ALLOW_THREADS
  st = launch();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// state, scale, x, dt, A, B, C, D, y, rule, format, dither_block, scale_group, seed, layer,
// step, entry_base, fp32_state, dt_bias, dt_softplus, z, stream handle or None
PyObject* state_update(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return handled([&]() -> PyObject* {
    if (n != 22) throw Unhandled{};
    const at::Tensor &state = tensor(v[0]), &A = tensor(v[4]), &B = tensor(v[5]);
    ssmq_qparams q{int32(v[9]), int32(v[10]), int32(v[11]), int32(v[12]), uint32(v[13]), uint32(v[14]),
                   uint32(v[15]), truth(v[17]) ? SSMQ_FLAG_FP32_STATE : 0u, integer(v[16])};
    if (state.dim() != 4 || B.dim() < 2) throw Unhandled{};
    const Format f = format_of(q.format);
    int64_t dstate = state.size(3);
    if (q.flags != 0) {
      if (state.scalar_type() != at::kFloat) throw Unhandled{};
    } else {
      if (static_cast<int64_t>(state.element_size()) != f.bytes) throw Unhandled{};
      dstate *= f.entries;
    }
    const int64_t most = INT32_MAX;
    if (state.size(1) > most || state.size(2) > most || dstate > most || B.size(1) > most) throw Unhandled{};
    const ssmq_dims d{state.size(0), static_cast<int32_t>(state.size(1)), static_cast<int32_t>(state.size(2)),
                      static_cast<int32_t>(dstate), static_cast<int32_t>(B.size(1)), A.dim() == 2 ? 1 : 0};
    const ssmq_step_opts opts{floats(v[18]), truth(v[19]) ? 1 : 0, 0, floats(v[20])};
    void* const st = pointer(v[0]);
    float *const scale = floats(v[1]), *const y = floats(v[8]);
    const float *const x = floats(v[2]), *const dt = floats(v[3]), *const a = floats(v[4]), *const b = floats(v[5]),
                *const c = floats(v[6]), *const D = floats(v[7]);
    void* const stream = stream_of(v[21], state);
    return launched([&] { return ssmq_state_update_ex(&d, &q, &opts, st, scale, x, dt, a, b, c, D, y, stream); });
  });
}

// conv_state, x, weight, bias, out, act, stream handle or None
PyObject* conv1d_update(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return handled([&]() -> PyObject* {
    if (n != 7) throw Unhandled{};
    const at::Tensor& state = tensor(v[0]);
    if (state.dim() != 3 || state.size(1) > INT32_MAX || state.size(2) > INT32_MAX) throw Unhandled{};
    const int64_t batch = state.size(0);
    const int32_t channels = static_cast<int32_t>(state.size(1)), width = static_cast<int32_t>(state.size(2));
    float *const st = floats(v[0]), *const out = floats(v[4]);
    const float *const x = floats(v[1]), *const w = floats(v[2]), *const bias = floats(v[3]);
    const int32_t act = truth(v[5]) ? 1 : 0;
    void* const stream = stream_of(v[6], state);
    return launched([&] { return ssmq_conv1d_update(batch, channels, width, st, x, w, bias, act, out, stream); });
  });
}

// h, codes, scale, rule, format, head_size, dither_block, scale_group, seed, layer, step,
// entry_base, stream handle or None
PyObject* requantize(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return handled([&]() -> PyObject* {
    if (n != 13) throw Unhandled{};
    const at::Tensor &h = tensor(v[0]), &codes = tensor(v[1]);
    const ssmq_qparams q{int32(v[3]), int32(v[4]), int32(v[6]), int32(v[7]), uint32(v[8]), uint32(v[9]),
                         uint32(v[10]), 0u, integer(v[11])};
    const Format f = format_of(q.format);
    if (codes.numel() * f.entries != h.numel() || static_cast<int64_t>(codes.element_size()) != f.bytes)
      throw Unhandled{};
    const int64_t entries = h.numel(), head_size = static_cast<int64_t>(integer(v[5]));
    const float* const src = floats(v[0]);
    void* const dst = pointer(v[1]);
    float* const scale = floats(v[2]);
    void* const stream = stream_of(v[12], h);
    return launched([&] { return ssmq_requantize(&q, entries, head_size, src, dst, scale, stream); });
  });
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyCFunction fastcall() {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F));
}

PyMethodDef kMethods[] = {
    {"state_update", fastcall<state_update>(), METH_FASTCALL, nullptr},
    {"conv1d_update", fastcall<conv1d_update>(), METH_FASTCALL, nullptr},
    {"requantize", fastcall<requantize>(), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", "Per-token calls of libssmq.so on torch tensors.", -1,
                       kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

#define SSMQ_STR_(v) #v
#define SSMQ_STR(v) SSMQ_STR_(v)

PyMODINIT_FUNC PyInit__native() {
  PyObject* const m = PyModule_Create(&kModule);
  // What the importer compares: torch's tensor layout and CPython's are compiled in.
  if (m && PyModule_AddStringConstant(m, "BUILT_FOR",
                                      "torch " SSMQ_TORCH_VERSION ", Python " SSMQ_STR(PY_MAJOR_VERSION) "." SSMQ_STR(
                                          PY_MINOR_VERSION)) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
