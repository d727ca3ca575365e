// CPython side of the three entry points that a program calls once per layer and token: tensors and descriptors to plain
// pointers, then the C ABI.  A small call lasts as long on the host as on the GPU, and of its 9.63 us there (a decode of two
// launches, issued one after the other) ctypes and the interpreter took 4: thirteen argument conversions, three references,
// seven address look-ups and a struct, each an object of its own.  So it takes 6.86, of which the launches are 4.8.  No arithmetic, no state but the handles that bind()
// leaves; addresses are asked of the tensors at every call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "lra_attn.h"

namespace {

decltype(&lra_attn_decode) g_decode;
decltype(&lra_attn_prefill) g_prefill;
decltype(&lra_cache_append) g_append;
const lra_tuning* g_tuning;
PyTypeObject *g_shape_type, *g_cache_type;
PyObject *g_get_device, *g_get_stream, *g_is_initialized;  // torch's current device and its stream's handle; whether the GPU is in use
PyObject *s_data_ptr, *s_size, *s_nbytes, *s_cuda_stream, *s_zero, *s_one;

// The address of a tensor's first element (None: no address).
bool address(PyObject* t, void** p) {
  *p = nullptr;
  if (t == Py_None) return true;
  PyObject* v = PyObject_CallMethodNoArgs(t, s_data_ptr);
  if (!v) return false;
  *p = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  return !(*p == nullptr && PyErr_Occurred());
}

// What a 32-bit field takes from a Python number: int(x), its low bits.
bool int32(PyObject* o, int32_t* x) {
  PyObject* v = PyLong_CheckExact(o) ? Py_NewRef(o) : PyNumber_Long(o);
  if (!v) return false;
  *x = static_cast<int32_t>(PyLong_AsUnsignedLongMask(v));
  Py_DECREF(v);
  return !PyErr_Occurred();
}

bool size(PyObject* t, PyObject* dim, int32_t* x) {
  PyObject* v = PyObject_CallMethodOneArg(t, s_size, dim);
  if (!v) return false;
  const bool ok = int32(v, x);
  Py_DECREF(v);
  return ok;
}

bool workspace(PyObject* t, void** p, size_t* bytes) {
  *p = nullptr;
  *bytes = 0;
  if (t == Py_None) return true;
  if (!address(t, p)) return false;
  PyObject* v = PyObject_GetAttr(t, s_nbytes);
  if (!v) return false;
  *bytes = PyLong_AsSize_t(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}

// The handle of the given stream, or of the current one (the null stream is NULL either way).
bool stream_handle(PyObject* stream, void** p) {
  PyObject* v;
  if (stream != Py_None) {
    v = PyObject_GetAttr(stream, s_cuda_stream);
  } else {
    // (the GPU not in use yet, or not usable in this process: torch starts it, or says why not)
    PyObject* up = PyObject_CallNoArgs(g_is_initialized);
    if (!up) return false;
    const int yes = PyObject_IsTrue(up);
    Py_DECREF(up);
    if (yes < 0) return false;
    if (!yes) {
      PyObject* cuda = PyImport_ImportModule("torch.cuda");
      PyObject* cur = cuda ? PyObject_CallMethod(cuda, "current_stream", nullptr) : nullptr;
      v = cur ? PyObject_GetAttr(cur, s_cuda_stream) : nullptr;
      Py_XDECREF(cur);
      Py_XDECREF(cuda);
    } else {
      PyObject* dev = PyObject_CallNoArgs(g_get_device);
      v = dev ? PyObject_CallOneArg(g_get_stream, dev) : nullptr;
      Py_XDECREF(dev);
    }
  }
  if (!v) return false;
  *p = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  return !(*p == nullptr && PyErr_Occurred());
}

// A ctypes struct's memory, held while the call runs.
struct Struct {
  Py_buffer view{};
  bool held = false;
  bool open(PyObject* o, PyTypeObject* type) {
    if (!PyObject_TypeCheck(o, type)) {
      PyErr_Format(PyExc_TypeError, "expected %s, not %s", type->tp_name, Py_TYPE(o)->tp_name);
      return false;
    }
    held = PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) == 0;
    return held;
  }
  template <typename T> const T* as() const { return static_cast<const T*>(view.buf); }
  ~Struct() {
    if (held) PyBuffer_Release(&view);
  }
};

bool arity(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "expected %zd arguments, not %zd", want, n);
  return false;
}

// decode(shape, cache, b_k, b_v, n_adapters, q, query_adapter, seq_query_start, max_queries_per_seq, out, workspace, stream)
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Struct sh, c;
  lra_adapters ad{};
  void *b_k, *b_v, *q, *qa, *sqs, *out, *ws, *st;
  size_t ws_bytes;
  int32_t n_queries, mq;
  if (!arity(n, 12) || !sh.open(a[0], g_shape_type) || !c.open(a[1], g_cache_type) || !address(a[2], &b_k) || !address(a[3], &b_v) ||
      !int32(a[4], &ad.n_adapters) || !workspace(a[10], &ws, &ws_bytes) || !address(a[5], &q) || !address(a[6], &qa) ||
      !address(a[7], &sqs) || !size(a[5], s_zero, &n_queries) || !int32(a[8], &mq) || !address(a[9], &out) || !stream_handle(a[11], &st))
    return nullptr;
  ad.b_k = b_k;
  ad.b_v = b_v;
  lra_status status;
  Py_BEGIN_ALLOW_THREADS
  status = g_decode(sh.as<lra_shape>(), c.as<lra_cache>(), &ad, q, static_cast<const int32_t*>(qa), static_cast<const int32_t*>(sqs),
                    n_queries, mq, out, ws, ws_bytes, g_tuning, st);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

// prefill(shape, cache, b_k, b_v, n_adapters, q, seq_index, adapter_index, out, workspace, stream)
PyObject* prefill(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Struct sh, c;
  lra_adapters ad{};
  void *b_k, *b_v, *q, *out, *ws, *st;
  size_t ws_bytes;
  int32_t n_new, seq, adapter;
  if (!arity(n, 11) || !sh.open(a[0], g_shape_type) || !c.open(a[1], g_cache_type) || !address(a[2], &b_k) || !address(a[3], &b_v) ||
      !int32(a[4], &ad.n_adapters) || !workspace(a[9], &ws, &ws_bytes) || !address(a[5], &q) || !int32(a[6], &seq) || !int32(a[7], &adapter) ||
      !size(a[5], s_zero, &n_new) || !address(a[8], &out) || !stream_handle(a[10], &st))
    return nullptr;
  ad.b_k = b_k;
  ad.b_v = b_v;
  lra_status status;
  Py_BEGIN_ALLOW_THREADS
  status = g_prefill(sh.as<lra_shape>(), c.as<lra_cache>(), &ad, q, seq, adapter, n_new, out, ws, ws_bytes, g_tuning, st);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

// append(shape, cache, w, rope_theta, x, seq_index, workspace, stream); x and w dense, of one width (the caller has checked)
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Struct sh, c;
  lra_projection proj{};
  void *w, *x, *ws, *st;
  size_t ws_bytes;
  int32_t n_new, seq;
  if (!arity(n, 8) || !address(a[2], &w) || !size(a[2], s_one, &proj.d_model)) return nullptr;
  const double theta = PyFloat_AsDouble(a[3]);
  if ((theta == -1.0 && PyErr_Occurred()) || !workspace(a[6], &ws, &ws_bytes) || !sh.open(a[0], g_shape_type) ||
      !c.open(a[1], g_cache_type) || !address(a[4], &x) || !int32(a[5], &seq) || !size(a[4], s_zero, &n_new) || !stream_handle(a[7], &st))
    return nullptr;
  proj.w = w;
  proj.rope_theta = static_cast<float>(theta);
  lra_status status;
  Py_BEGIN_ALLOW_THREADS
  status = g_append(sh.as<lra_shape>(), c.as<lra_cache>(), &proj, x, seq, n_new, ws, ws_bytes, g_tuning, st);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

// bind(decode, prefill, append, tuning: addresses; LraShape, LraCache; current device, its raw stream, is_initialized: callables)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arity(n, 9)) return nullptr;
  void* p[4];
  for (int i = 0; i < 4; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no address");
      return nullptr;
    }
  }
  if (!PyType_Check(a[4]) || !PyType_Check(a[5])) {
    PyErr_SetString(PyExc_TypeError, "expected the two struct types");
    return nullptr;
  }
  g_decode = reinterpret_cast<decltype(g_decode)>(p[0]);
  g_prefill = reinterpret_cast<decltype(g_prefill)>(p[1]);
  g_append = reinterpret_cast<decltype(g_append)>(p[2]);
  g_tuning = static_cast<const lra_tuning*>(p[3]);
  g_shape_type = reinterpret_cast<PyTypeObject*>(Py_NewRef(a[4]));  // (held for good, like the library)
  g_cache_type = reinterpret_cast<PyTypeObject*>(Py_NewRef(a[5]));
  g_get_device = Py_NewRef(a[6]);
  g_get_stream = Py_NewRef(a[7]);
  g_is_initialized = Py_NewRef(a[8]);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bind)), METH_FASTCALL, nullptr},
    {"decode", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode)), METH_FASTCALL, nullptr},
    {"prefill", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(prefill)), METH_FASTCALL, nullptr},
    {"append", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(append)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lra_pycall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lra_pycall() {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_size = PyUnicode_InternFromString("size");
  s_nbytes = PyUnicode_InternFromString("nbytes");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  s_zero = PyLong_FromLong(0);
  s_one = PyLong_FromLong(1);
  if (!s_data_ptr || !s_size || !s_nbytes || !s_cuda_stream || !s_zero || !s_one) return nullptr;
  return PyModule_Create(&module);
}
