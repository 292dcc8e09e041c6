// Argument marshalling of the decode step as native code.  A step of few sequences takes the GPU less time than the same checks
// took in Python: the smallest step 8.1 us a call, 4.5 from here, of which the launch itself is 2.6; with a workspace from
// torch.empty 9.8, from the allocator here 5 (one sequence, 4 KV heads, W = 512, where the kernel is the bound: 9.8 -> 9.15).
//
// decode_step(q, k_new, v_new, pos, k_ring, v_ring, state, gamma_swa, gamma_rla, softmax_scale, rms_eps, out, feature_map)
// returns the output; None when the arguments are not plainly what the step takes (the caller's Python path then converts
// or raises as it always did), and a status as an int when the library refuses the call.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>

#include "rattn.h"

namespace {

typedef rattn_status (*step_fn)(const rattn_decode_params*, const void*, const void*, const void*, const int32_t*, void*, void*,
                                float*, const float*, const float*, void*, void*, size_t, void*);
typedef rattn_status (*bytes_fn)(const rattn_decode_params*, size_t*);
step_fn g_step = nullptr;
bytes_fn g_bytes = nullptr;

// bind(address of rattn_decode_step_ws, address of rattn_decode_workspace_bytes) of the loaded library
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 2) return PyErr_Format(PyExc_TypeError, "bind takes two addresses");
  g_step = (step_fn)PyLong_AsVoidPtr(args[0]);
  g_bytes = (bytes_fn)PyLong_AsVoidPtr(args[1]);
  if (PyErr_Occurred()) return nullptr;
  Py_RETURN_NONE;
}

// a plain tensor on device `dev`, contiguous, of type `dt` and `nd` dimensions
bool plain(const at::Tensor& t, int dev, at::ScalarType dt, int nd) {
  return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.get_device() == dev && t.scalar_type() == dt && t.dim() == nd &&
         t.is_contiguous() && t.has_storage();
}
bool shaped(const at::Tensor& t, int64_t a, int64_t b, int64_t c) { return t.size(0) == a && t.size(1) == b && t.size(2) == c; }

// The interpreter lock is free while one of these lives, as in a ctypes call
struct NoGil {
  PyThreadState* state = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(state); }
};

PyObject* step(PyObject* const* args) {
  const at::Tensor* t[7];
  for (int i = 0; i < 7; ++i) {
    if (!THPVariable_CheckExact(args[i])) Py_RETURN_NONE;
    t[i] = &THPVariable_Unpack(args[i]);
  }
  const at::Tensor &q = *t[0], &kn = *t[1], &vn = *t[2], &pos = *t[3], &kr = *t[4], &vr = *t[5], &state = *t[6];
  const at::ScalarType dt = q.scalar_type();
  const int dev = q.is_cuda() ? q.get_device() : -1;
  if ((dt != at::kFloat && dt != at::kBFloat16) || dev < 0 || dev != c10::hip::current_device()) Py_RETURN_NONE;
  if (!plain(q, dev, dt, 3) || !plain(kn, dev, dt, 3) || !plain(vn, dev, dt, 3) || !plain(pos, dev, at::kInt, 1) ||
      !plain(kr, dev, dt, 4) || !plain(vr, dev, dt, 4) || !plain(state, dev, at::kFloat, 4))
    Py_RETURN_NONE;
  const int64_t N = q.size(0), Hq = q.size(1), D = q.size(2), Hkv = kr.size(1), W = kr.size(2);
  if (!shaped(kn, N, Hkv, D) || !shaped(vn, N, Hkv, D) || pos.size(0) != N || !shaped(kr, N, Hkv, W) || kr.size(3) != D ||
      !shaped(vr, N, Hkv, W) || vr.size(3) != D || !shaped(state, N, Hkv, D) || state.size(3) != D)
    Py_RETURN_NONE;
  if (N > INT32_MAX || Hq > INT32_MAX || Hkv > INT32_MAX || D > INT32_MAX || W > INT32_MAX) Py_RETURN_NONE;
  const float* gain[2] = {nullptr, nullptr};
  for (int i = 0; i < 2; ++i) {
    PyObject* a = args[7 + i];
    if (a == Py_None) continue;
    if (!THPVariable_CheckExact(a)) Py_RETURN_NONE;
    const at::Tensor& g = THPVariable_Unpack(a);
    if (!plain(g, dev, at::kFloat, 2) || g.size(0) != Hq || g.size(1) != D) Py_RETURN_NONE;
    gain[i] = (const float*)g.data_ptr();
  }
  if (!PyFloat_CheckExact(args[9]) || !PyFloat_CheckExact(args[10]) || !PyUnicode_CheckExact(args[12])) Py_RETURN_NONE;
  rattn_decode_params p;
  p.N = (int32_t)N; p.Hq = (int32_t)Hq; p.Hkv = (int32_t)Hkv; p.D = (int32_t)D; p.window = (int32_t)W;
  p.dtype = dt == at::kFloat ? RATTN_F32 : RATTN_BF16;
  p.softmax_scale = (float)PyFloat_AS_DOUBLE(args[9]);
  p.rms_eps = (float)PyFloat_AS_DOUBLE(args[10]);
  if (PyUnicode_CompareWithASCIIString(args[12], "softmax") == 0) p.feature_map = RATTN_PHI_SOFTMAX;
  else if (PyUnicode_CompareWithASCIIString(args[12], "relu") == 0) p.feature_map = RATTN_PHI_RELU;
  else if (PyUnicode_CompareWithASCIIString(args[12], "identity") == 0) p.feature_map = RATTN_PHI_IDENTITY;
  else Py_RETURN_NONE;
  // The result as an object ahead of the step: behind it nothing may fail, since a caller that is told so would step again and
  // fold the evicted token into the state twice
  THPObjectPtr result;
  void* o;
  if (args[11] == Py_None) {
    at::Tensor fresh = at::empty_like(q);
    o = fresh.data_ptr();
    result = THPVariable_Wrap(std::move(fresh));
    if (!result) return nullptr;
  } else {
    if (!THPVariable_CheckExact(args[11])) Py_RETURN_NONE;
    const at::Tensor& out = THPVariable_Unpack(args[11]);   // the step writes N Hq D elements of it, whatever its shape
    if (!plain(out, dev, dt, out.dim()) || out.numel() < q.numel()) Py_RETURN_NONE;
    o = out.data_ptr();
    Py_INCREF(args[11]);
    result = args[11];
  }
  const void *qp = q.data_ptr(), *knp = kn.data_ptr(), *vnp = vn.data_ptr();
  void *posp = pos.data_ptr(), *krp = kr.data_ptr(), *vrp = vr.data_ptr(), *sp = state.data_ptr();
  rattn_status s;
  {
    NoGil others_run;   // the allocator may wait for the device, a launch for room in the stream's queue
    size_t bytes = 0;
    s = g_bytes(&p, &bytes);
    if (s == RATTN_OK) {
      c10::DataPtr ws;   // from the caching allocator, on the current stream: back in its pool when the step is enqueued
      if (bytes > 0) ws = c10::hip::HIPCachingAllocator::get()->allocate(bytes);
      void* stream = (void*)c10::hip::getCurrentHIPStream((c10::DeviceIndex)dev).stream();
      s = g_step(&p, qp, knp, vnp, (const int32_t*)posp, krp, vrp, (float*)sp, gain[0], gain[1], o, ws.get(), bytes, stream);
    }
  }
  return s == RATTN_OK ? result.release() : PyLong_FromLong(s);
}

PyObject* decode_step(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 13 || !g_step) return PyErr_Format(PyExc_TypeError, "decode_step takes 13 arguments, after bind");
  try {
    return step(args);
  } catch (const std::exception&) {   // (an allocation that failed, a tensor without memory: as the Python path says it)
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
  }
}

PyMethodDef g_methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {"decode_step", (PyCFunction)(void (*)(void))decode_step, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&g_module); }
