// Argument checks and calls of the per-step entry points for the Python
// binding (module _bifattn_bind).
//
// A decode step of a small layer is bound by the host: checking its tensors
// attribute by attribute in Python takes 6.5 us and the whole call 10.3 us,
// where the GPU needs 4.9 us for it. Caller makes the same checks on the
// tensor objects themselves (well under 1 us).
//
// A method returns the library's status, or None when it does not take the
// call: any tensor that is not exactly what the plan expects, and any tensor
// that is not an ordinary one (a subclass with its own dispatch, a wrapped or
// non-strided tensor). The binding then goes through its Python checks, which
// raise the specific error or make the call themselves, so what is accepted
// and what is refused does not depend on this file.
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <cstdint>

#include "bifattn.h"

namespace {

typedef bifattn_status_t (*decode_fn)(bifattn_plan_t, const void*, const void*, const void*,
                                      const void*, const void*, const int32_t*, const float*,
                                      const float*, float*, hipStream_t);
typedef bifattn_status_t (*append_fn)(bifattn_plan_t, const void*, const void*, void*, void*,
                                      int32_t*, hipStream_t);

struct Caller {
  PyObject_HEAD
  decode_fn decode;
  append_fn append;
  bifattn_plan_t plan;
  PyObject* current_stream;  // callable: device index -> raw stream of the calling thread
  PyObject* device_obj;      // the plan's device index as a Python int
  int device;
  int64_t b, h, g, d, m_c, m_d, n;
  int kv;
};

// The tensor's implementation, or null when this file does not take it.
const at::Tensor* plain(PyObject* o, int device) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || t.get_device() != device)
    return nullptr;
  const c10::DispatchKeySet keys = t.key_set();
  if (keys.has_any(c10::python_ks) || keys.has(c10::DispatchKey::FuncTorchBatched) ||
      keys.has(c10::DispatchKey::FuncTorchGradWrapper) ||
      keys.has(c10::DispatchKey::Functionalize) || !t.has_storage())
    return nullptr;
  return &t;
}

bool shaped(const at::Tensor& t, std::initializer_list<int64_t> shape) {
  return t.sizes().equals(c10::IntArrayRef(shape.begin(), shape.size())) && t.is_contiguous();
}

// Device pointer of a tensor of this dtype and shape in *ptr.
bool take(PyObject* o, const Caller* C, at::ScalarType type, std::initializer_list<int64_t> shape,
          void** ptr) {
  const at::Tensor* t = plain(o, C->device);
  if (!t || t->scalar_type() != type || !shaped(*t, shape)) return false;
  *ptr = t->data_ptr();
  return true;
}

bool take_cache(PyObject* o, const Caller* C, std::initializer_list<int64_t> shape, void** ptr) {
  const at::Tensor* t = plain(o, C->device);
  if (!t || !shaped(*t, shape)) return false;
  const at::ScalarType s = t->scalar_type();
  const bool byte = s == at::kByte || s == at::kChar;
  const bool ok = C->kv == BIFATTN_KV_BF16   ? s == at::kBFloat16
                  : C->kv == BIFATTN_KV_INT4 ? byte
                                             : byte || s == at::kFloat8_e4m3fn;
  if (!ok) return false;
  *ptr = t->data_ptr();
  return true;
}

bool take_scale(PyObject* o, const Caller* C, void** ptr) {
  *ptr = nullptr;
  return o == Py_None || take(o, C, at::kFloat, {C->g}, ptr);
}

// The stream argument: None for the current stream of the plan's device, or
// a raw stream as a Python int. False with no Python error set otherwise.
bool take_stream(PyObject* o, const Caller* C, hipStream_t* stream) {
  PyObject* raw = o;
  if (o == Py_None) {
    raw = PyObject_CallOneArg(C->current_stream, C->device_obj);
    if (!raw) {
      PyErr_Clear();
      return false;
    }
  } else if (!PyLong_CheckExact(o)) {
    return false;
  }
  void* p = PyLong_AsVoidPtr(raw);
  if (raw != o) Py_DECREF(raw);
  if (!p && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  *stream = static_cast<hipStream_t>(p);
  return true;
}

int64_t cols(const Caller* C) { return C->kv == BIFATTN_KV_INT4 ? C->d / 2 : C->d; }

// decode(q, Kc, Vc, Kd, Vd, decode_lens, k_scale, v_scale, out, stream)
PyObject* caller_decode(PyObject* self, PyObject* const* a, Py_ssize_t nargs) {
  const Caller* C = reinterpret_cast<const Caller*>(self);
  if (nargs != 10) {
    PyErr_SetString(PyExc_TypeError, "decode takes 10 arguments");
    return nullptr;
  }
  void *q, *Kc, *Vc, *Kd, *Vd, *lens, *ks, *vs, *out;
  hipStream_t stream = nullptr;
  try {
    const int64_t w = cols(C);
    const bool flat = C->n == 1 && THPVariable_CheckExact(a[0]) && THPVariable_Unpack(a[0]).dim() == 3;
    const bool qo = flat ? take(a[0], C, at::kBFloat16, {C->b, C->h, C->d}, &q) &&
                               take(a[8], C, at::kFloat, {C->b, C->h, C->d}, &out)
                         : take(a[0], C, at::kBFloat16, {C->b, C->h, C->n, C->d}, &q) &&
                               take(a[8], C, at::kFloat, {C->b, C->h, C->n, C->d}, &out);
    if (!qo || !take_cache(a[1], C, {C->g, C->m_c, w}, &Kc) ||
        !take_cache(a[2], C, {C->g, C->m_c, w}, &Vc) ||
        !take_cache(a[3], C, {C->b, C->g, C->m_d, w}, &Kd) ||
        !take_cache(a[4], C, {C->b, C->g, C->m_d, w}, &Vd) ||
        !take(a[5], C, at::kInt, {C->b}, &lens) || !take_scale(a[6], C, &ks) ||
        !take_scale(a[7], C, &vs) || !take_stream(a[9], C, &stream))
      Py_RETURN_NONE;
  } catch (...) {  // nothing C++ throws passes into the interpreter
    Py_RETURN_NONE;
  }
  bifattn_status_t st;
  Py_BEGIN_ALLOW_THREADS
  st = C->decode(C->plan, q, Kc, Vc, Kd, Vd, static_cast<const int32_t*>(lens),
                 static_cast<const float*>(ks), static_cast<const float*>(vs),
                 static_cast<float*>(out), stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// append(k_new, v_new, Kd, Vd, decode_lens, stream)
PyObject* caller_append(PyObject* self, PyObject* const* a, Py_ssize_t nargs) {
  const Caller* C = reinterpret_cast<const Caller*>(self);
  if (nargs != 6) {
    PyErr_SetString(PyExc_TypeError, "append takes 6 arguments");
    return nullptr;
  }
  void *k, *v, *Kd, *Vd, *lens;
  hipStream_t stream = nullptr;
  try {
    const int64_t w = cols(C);
    if (!take_cache(a[0], C, {C->b, C->g, C->n, w}, &k) ||
        !take_cache(a[1], C, {C->b, C->g, C->n, w}, &v) ||
        !take_cache(a[2], C, {C->b, C->g, C->m_d, w}, &Kd) ||
        !take_cache(a[3], C, {C->b, C->g, C->m_d, w}, &Vd) ||
        !take(a[4], C, at::kInt, {C->b}, &lens) || !take_stream(a[5], C, &stream))
      Py_RETURN_NONE;
  } catch (...) {
    Py_RETURN_NONE;
  }
  bifattn_status_t st;
  Py_BEGIN_ALLOW_THREADS
  st = C->append(C->plan, k, v, Kd, Vd, static_cast<int32_t*>(lens), stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// Caller(decode, append, plan, current_stream, device, b, h, g, d, m_c, m_d, n, kv):
// the entry points and the plan as addresses.
PyObject* caller_new(PyTypeObject* type, PyObject* args, PyObject*) {
  unsigned long long decode, append, plan;
  PyObject* cs;
  int device, kv;
  long long b, h, g, d, m_c, m_d, n;
  if (!PyArg_ParseTuple(args, "KKKOiLLLLLLLi", &decode, &append, &plan, &cs, &device, &b, &h, &g,
                        &d, &m_c, &m_d, &n, &kv))
    return nullptr;
  Caller* C = reinterpret_cast<Caller*>(type->tp_alloc(type, 0));
  if (!C) return nullptr;
  C->device_obj = PyLong_FromLong(device);
  if (!C->device_obj) {
    Py_DECREF(C);
    return nullptr;
  }
  Py_INCREF(cs);
  C->current_stream = cs;
  C->decode = reinterpret_cast<decode_fn>(static_cast<uintptr_t>(decode));
  C->append = reinterpret_cast<append_fn>(static_cast<uintptr_t>(append));
  C->plan = reinterpret_cast<bifattn_plan_t>(static_cast<uintptr_t>(plan));
  C->device = device;
  C->b = b, C->h = h, C->g = g, C->d = d, C->m_c = m_c, C->m_d = m_d, C->n = n;
  C->kv = kv;
  return reinterpret_cast<PyObject*>(C);
}

void caller_dealloc(PyObject* self) {
  Caller* C = reinterpret_cast<Caller*>(self);
  Py_XDECREF(C->current_stream);
  Py_XDECREF(C->device_obj);
  Py_TYPE(self)->tp_free(self);
}

PyMethodDef caller_methods[] = {
    {"decode", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(caller_decode)),
     METH_FASTCALL, "status of bifattn_decode_scaled, or None when the call is not taken"},
    {"append", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(caller_append)),
     METH_FASTCALL, "status of bifattn_append_kv, or None when the call is not taken"},
    {nullptr, nullptr, 0, nullptr}};

PyTypeObject caller_type = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_bifattn_bind", nullptr, -1, nullptr,
                          nullptr,               nullptr,          nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bifattn_bind() {
  caller_type.tp_name = "_bifattn_bind.Caller";
  caller_type.tp_basicsize = sizeof(Caller);
  caller_type.tp_flags = Py_TPFLAGS_DEFAULT;
  caller_type.tp_new = caller_new;
  caller_type.tp_dealloc = caller_dealloc;
  caller_type.tp_methods = caller_methods;
  if (PyType_Ready(&caller_type) < 0) return nullptr;
  PyObject* m = PyModule_Create(&module_def);
  if (!m) return nullptr;
  Py_INCREF(&caller_type);
  if (PyModule_AddObject(m, "Caller", reinterpret_cast<PyObject*>(&caller_type)) < 0) {
    Py_DECREF(&caller_type);
    Py_DECREF(m);
    return nullptr;
  }
  // The tensor layouts read above are this version's.
  if (PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
