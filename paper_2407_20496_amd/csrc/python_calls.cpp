// Python calls of the per-product and per-layer entry points of libhinm (include/hinm.h): argument marshalling only.
//
// A decode-sized product runs 4 .. 10 us on the GPU, and building the shape structure, converting seventeen arguments
// and asking for the current stream in interpreted code took 6 .. 7 us of the calling thread: calls in a row were bound by that.
// Here a call costs about a microsecond besides the launch itself.  binding.py hands over the addresses of the entry
// points of the library it has loaded, so this module links to nothing; the interpreter lock is released around
// every library call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <vector>

#include "hinm.h"

namespace {

decltype(&hinm_pack) f_pack;
decltype(&hinm_prepare) f_prepare;
decltype(&hinm_spmm) f_spmm;
decltype(&hinm_spmm_vectors) f_spmm_vectors;
decltype(&hinm_spmm_prepared) f_spmm_prepared;
decltype(&hinm_chain) f_chain;

PyObject* g_dtype_code;      // any accepted dtype -> HINM_F16 / HINM_BF16
PyObject* g_current_stream;  // () -> raw pointer of the current stream or None; used until a source is set
PyObject* g_get_device;      // () -> current device, and
PyObject* g_raw_stream;      // (device) -> raw pointer of its current stream
PyObject* s_data_ptr;
PyObject* s_cuda_stream;
PyObject* s_f16;
PyObject* s_bf16;
PyObject* s_layer[12];

// The low 64 bits, as ctypes converts integers: sizes use all of them (2**64 - 1 for "any").
bool to_i64(PyObject* o, int64_t* out) {
  if (PyLong_Check(o)) {
    *out = (int64_t)PyLong_AsUnsignedLongLongMask(o);
  } else {
    PyObject* n = PyNumber_Long(o);
    if (!n) return false;
    *out = (int64_t)PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
  }
  return !(*out == -1 && PyErr_Occurred());
}

// None -> NULL, an integer is the address, anything else has data_ptr()
bool to_ptr(PyObject* o, void** out) {
  if (o == Py_None) {
    *out = nullptr;
    return true;
  }
  PyObject* n = nullptr;
  if (!PyLong_Check(o)) {
    n = PyObject_CallMethodNoArgs(o, s_data_ptr);
    if (!n) return false;
    o = n;
  }
  *out = PyLong_AsVoidPtr(o);
  Py_XDECREF(n);
  return !(*out == nullptr && PyErr_Occurred());
}

bool to_stream(PyObject* o, void** out) {
  if (o != Py_None && !PyLong_Check(o)) {
    PyObject* n = PyObject_GetAttr(o, s_cuda_stream);
    if (!n) return false;
    const bool ok = to_ptr(n, out);
    Py_DECREF(n);
    return ok;
  }
  if (o != Py_None) return to_ptr(o, out);
  PyObject* raw;
  if (g_raw_stream) {
    PyObject* device = PyObject_CallNoArgs(g_get_device);
    if (!device) return false;
    raw = PyObject_CallOneArg(g_raw_stream, device);
    Py_DECREF(device);
  } else {
    raw = PyObject_CallOneArg(g_current_stream, Py_None);
  }
  if (!raw) return false;
  const bool ok = to_ptr(raw, out);
  Py_DECREF(raw);
  return ok;
}

bool to_dtype(PyObject* o, int32_t* out) {
  if (o == s_f16) {
    *out = HINM_F16;
    return true;
  }
  if (o == s_bf16) {
    *out = HINM_BF16;
    return true;
  }
  PyObject* code = PyObject_CallOneArg(g_dtype_code, o);
  if (!code) return false;
  int64_t v;
  const bool ok = to_i64(code, &v);
  Py_DECREF(code);
  *out = (int32_t)v;
  return ok;
}

// M, K, V, Kv, dtype
bool to_shape(PyObject* const* a, hinm_shape* s) {
  int64_t m, k, v, kv;
  if (!to_i64(a[0], &m) || !to_i64(a[1], &k) || !to_i64(a[2], &v) || !to_i64(a[3], &kv) || !to_dtype(a[4], &s->dtype))
    return false;
  s->M = (int32_t)m;
  s->K = (int32_t)k;
  s->V = (int32_t)v;
  s->Kv = (int32_t)kv;
  return true;
}

bool takes(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "%zd arguments where %zd are wanted", n, want);
  return false;
}

template <class Call>
PyObject* status_of(Call call) {
  hinm_status st;
  Py_BEGIN_ALLOW_THREADS
  st = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong((long)st);
}

// (M, K, V, Kv, dtype, W, vals, nm_idx, vec_idx, workspace, workspace_bytes, stream)
PyObject* pack(PyObject*, PyObject* const* a, Py_ssize_t n) {
  hinm_shape s;
  void* p[5];
  void* stream;
  int64_t bytes;
  if (!takes(n, 12) || !to_shape(a, &s)) return nullptr;
  for (int i = 0; i < 5; ++i)
    if (!to_ptr(a[5 + i], &p[i])) return nullptr;
  if (!to_i64(a[10], &bytes) || !to_stream(a[11], &stream)) return nullptr;
  return status_of([&] {
    return f_pack(&s, p[0], p[1], static_cast<uint8_t*>(p[2]), static_cast<int32_t*>(p[3]), p[4], (size_t)bytes, stream);
  });
}

// (M, K, V, Kv, dtype, vals, nm_idx, vec_idx, pi_in, pi_out, prepared, prepared_bytes, stream)
PyObject* prepare(PyObject*, PyObject* const* a, Py_ssize_t n) {
  hinm_shape s;
  void* p[6];
  void* stream;
  int64_t bytes;
  if (!takes(n, 13) || !to_shape(a, &s)) return nullptr;
  for (int i = 0; i < 6; ++i)
    if (!to_ptr(a[5 + i], &p[i])) return nullptr;
  if (!to_i64(a[11], &bytes) || !to_stream(a[12], &stream)) return nullptr;
  return status_of([&] {
    return f_prepare(&s, p[0], static_cast<uint8_t*>(p[1]), static_cast<int32_t*>(p[2]), static_cast<int32_t*>(p[3]),
                     static_cast<int32_t*>(p[4]), p[5], (size_t)bytes, stream);
  });
}

// (M, K, V, Kv, dtype, N, vals, nm_idx, vec_idx, pi_in, pi_out, X, ldx, Y, ldy, flags, workspace, workspace_bytes, stream)
PyObject* spmm(PyObject*, PyObject* const* a, Py_ssize_t n) {
  hinm_shape s;
  void *p[6], *y, *ws, *stream;
  int64_t cols, ldx, ldy, flags, bytes;
  if (!takes(n, 19) || !to_shape(a, &s) || !to_i64(a[5], &cols)) return nullptr;
  for (int i = 0; i < 6; ++i)
    if (!to_ptr(a[6 + i], &p[i])) return nullptr;
  if (!to_i64(a[12], &ldx) || !to_ptr(a[13], &y) || !to_i64(a[14], &ldy) || !to_i64(a[15], &flags) || !to_ptr(a[16], &ws) ||
      !to_i64(a[17], &bytes) || !to_stream(a[18], &stream))
    return nullptr;
  return status_of([&] {
    return f_spmm(&s, (int32_t)cols, p[0], static_cast<uint8_t*>(p[1]), static_cast<int32_t*>(p[2]),
                  static_cast<int32_t*>(p[3]), static_cast<int32_t*>(p[4]), p[5], ldx, y, ldy, (uint32_t)flags, ws,
                  (size_t)bytes, stream);
  });
}

// (M, K, V, Kv, dtype, N, vals_v, vec_idx, pi_in, pi_out, X, ldx, Y, ldy, flags, stream)
PyObject* spmm_vectors(PyObject*, PyObject* const* a, Py_ssize_t n) {
  hinm_shape s;
  void *p[5], *y, *stream;
  int64_t cols, ldx, ldy, flags;
  if (!takes(n, 16) || !to_shape(a, &s) || !to_i64(a[5], &cols)) return nullptr;
  for (int i = 0; i < 5; ++i)
    if (!to_ptr(a[6 + i], &p[i])) return nullptr;
  if (!to_i64(a[11], &ldx) || !to_ptr(a[12], &y) || !to_i64(a[13], &ldy) || !to_i64(a[14], &flags) ||
      !to_stream(a[15], &stream))
    return nullptr;
  return status_of([&] {
    return f_spmm_vectors(&s, (int32_t)cols, p[0], static_cast<int32_t*>(p[1]), static_cast<int32_t*>(p[2]),
                          static_cast<int32_t*>(p[3]), p[4], ldx, y, ldy, (uint32_t)flags, stream);
  });
}

// (M, K, V, Kv, dtype, N, prepared, X, ldx, Y, ldy, flags, workspace, workspace_bytes, stream)
PyObject* spmm_prepared(PyObject*, PyObject* const* a, Py_ssize_t n) {
  hinm_shape s;
  void *prepared, *x, *y, *ws, *stream;
  int64_t cols, ldx, ldy, flags, bytes;
  if (!takes(n, 15) || !to_shape(a, &s) || !to_i64(a[5], &cols) || !to_ptr(a[6], &prepared) || !to_ptr(a[7], &x) ||
      !to_i64(a[8], &ldx) || !to_ptr(a[9], &y) || !to_i64(a[10], &ldy) || !to_i64(a[11], &flags) || !to_ptr(a[12], &ws) ||
      !to_i64(a[13], &bytes) || !to_stream(a[14], &stream))
    return nullptr;
  return status_of([&] {
    return f_spmm_prepared(&s, (int32_t)cols, prepared, x, ldx, y, ldy, (uint32_t)flags, ws, (size_t)bytes, stream);
  });
}

// one attribute of a layer, converted
template <class Convert, class T>
bool field(PyObject* layer, int which, Convert convert, T* out) {
  PyObject* o = PyObject_GetAttr(layer, s_layer[which]);
  if (!o) return false;
  const bool ok = convert(o, out);
  Py_DECREF(o);
  return ok;
}

// (layers, N, X, ldx, Y, ldy, scratch, scratch_bytes, stream)
PyObject* chain(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!takes(n, 9)) return nullptr;
  if (PyObject_Size(a[0]) < 0) return nullptr;  // an iterator that is used up by one pass is no sequence of layers
  PyObject* seq = PySequence_Fast(a[0], "layers must be a sequence");
  if (!seq) return nullptr;
  const Py_ssize_t count = PySequence_Fast_GET_SIZE(seq);
  std::vector<hinm_layer> layers;
  layers.reserve((size_t)count + 1);  // an address also for a chain of no layers, which is an error of shape
  layers.resize((size_t)count);
  bool ok = true;
  for (Py_ssize_t i = 0; i < count && ok; ++i) {
    PyObject* l = PySequence_Fast_GET_ITEM(seq, i);
    hinm_layer& d = layers[(size_t)i];
    int64_t v[4], flags = 0;
    void *vals, *nm, *vec, *pin, *pout, *prep;
    for (int q = 0; q < 4 && ok; ++q) ok = field(l, q, to_i64, &v[q]);
    ok = ok && field(l, 4, to_dtype, &d.shape.dtype) && field(l, 5, to_ptr, &vals) && field(l, 6, to_ptr, &nm) &&
         field(l, 7, to_ptr, &vec) && field(l, 8, to_ptr, &pin) && field(l, 9, to_ptr, &pout) &&
         field(l, 10, to_i64, &flags) && field(l, 11, to_ptr, &prep);
    if (!ok) break;
    d.shape.M = (int32_t)v[0];
    d.shape.K = (int32_t)v[1];
    d.shape.V = (int32_t)v[2];
    d.shape.Kv = (int32_t)v[3];
    d.vals = vals;
    d.nm_idx = static_cast<uint8_t*>(nm);
    d.vec_idx = static_cast<int32_t*>(vec);
    d.pi_in = static_cast<int32_t*>(pin);
    d.pi_out = static_cast<int32_t*>(pout);
    d.flags = (uint32_t)flags;
    d.prepared = prep;
  }
  Py_DECREF(seq);
  void *x, *y, *scratch, *stream;
  int64_t cols, ldx, ldy, bytes;
  if (!ok || !to_i64(a[1], &cols) || !to_ptr(a[2], &x) || !to_i64(a[3], &ldx) || !to_ptr(a[4], &y) || !to_i64(a[5], &ldy) ||
      !to_ptr(a[6], &scratch) || !to_i64(a[7], &bytes) || !to_stream(a[8], &stream))
    return nullptr;
  return status_of([&] {
    return f_chain((int32_t)count, layers.data(), (int32_t)cols, x, ldx, y, ldy, scratch, (size_t)bytes, stream);
  });
}

// (addresses in the order below, dtype_code, current_stream)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* f[6];
  if (!takes(n, 8)) return nullptr;
  for (int i = 0; i < 6; ++i)
    if (!to_ptr(a[i], &f[i])) return nullptr;
  f_pack = reinterpret_cast<decltype(f_pack)>(f[0]);
  f_prepare = reinterpret_cast<decltype(f_prepare)>(f[1]);
  f_spmm = reinterpret_cast<decltype(f_spmm)>(f[2]);
  f_spmm_vectors = reinterpret_cast<decltype(f_spmm_vectors)>(f[3]);
  f_spmm_prepared = reinterpret_cast<decltype(f_spmm_prepared)>(f[4]);
  f_chain = reinterpret_cast<decltype(f_chain)>(f[5]);
  Py_INCREF(a[6]);
  Py_XSETREF(g_dtype_code, a[6]);
  Py_INCREF(a[7]);
  Py_XSETREF(g_current_stream, a[7]);
  Py_RETURN_NONE;
}

// (get_device, raw_stream): from now on the current stream is asked for directly
PyObject* set_stream_source(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!takes(n, 2)) return nullptr;
  Py_INCREF(a[0]);
  Py_XSETREF(g_get_device, a[0]);
  Py_INCREF(a[1]);
  Py_XSETREF(g_raw_stream, a[1]);
  Py_RETURN_NONE;
}

#define HINM_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {HINM_METHOD(pack),    HINM_METHOD(prepare), HINM_METHOD(spmm), HINM_METHOD(spmm_vectors),
                         HINM_METHOD(spmm_prepared), HINM_METHOD(chain), HINM_METHOD(bind), HINM_METHOD(set_stream_source),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  s_f16 = PyUnicode_InternFromString("f16");
  s_bf16 = PyUnicode_InternFromString("bf16");
  const char* names[12] = {"M", "K", "V", "Kv", "dtype", "vals", "nm_idx", "vec_idx", "pi_in", "pi_out", "flags", "prepared"};
  for (int i = 0; i < 12; ++i) s_layer[i] = PyUnicode_InternFromString(names[i]);
  return PyModule_Create(&module);
}
