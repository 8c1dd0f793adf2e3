// The cache calls of the C ABI as CPython functions.  A restore or an insertion is a dozen calls whose kernels take 3 to
// 9 us each, and marshalling through ctypes took as long as the launch itself.  Only what a serving program passes is
// taken here: tensors or None, Python ints and floats, a list or tuple of ints as long as the entry.  Anything else
// raises TypeError before the library is called, and the binding marshals the call itself.
// The functions are called by address (bind), so that there is one copy of the library and of its error text.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <climits>
#include <cstdint>

#include "../../include/flexdenoise.h"

namespace {

decltype(&fc_cache_stitch) g_stitch;
decltype(&fc_cache_decompress) g_decompress;
decltype(&fc_cache_alpha) g_alpha;
decltype(&fc_cache_frame_similarity) g_similarity;
PyObject* g_data_ptr;                                    // "data_ptr"

bool refuse() {
  PyErr_SetString(PyExc_TypeError, "not a plain argument");
  return false;
}

bool to_ll(PyObject* o, long long* out) {
  if (!PyLong_CheckExact(o)) return refuse();
  *out = PyLong_AsLongLong(o);
  if (*out == -1 && PyErr_Occurred()) { PyErr_Clear(); return refuse(); }
  return true;
}
bool to_int(PyObject* o, int32_t* out) {
  long long v;
  if (!to_ll(o, &v)) return false;
  if (v < INT32_MIN || v > INT32_MAX) return refuse();
  *out = (int32_t)v;
  return true;
}
bool to_address(PyObject* o, void** out) {               // a stream's handle, or None
  *out = nullptr;
  if (o == Py_None) return true;
  if (!PyLong_CheckExact(o)) return refuse();
  *out = PyLong_AsVoidPtr(o);
  if (!*out && PyErr_Occurred()) { PyErr_Clear(); return refuse(); }
  return true;
}
bool to_ptr(PyObject* o, void** out) {                   // a tensor, or None
  *out = nullptr;
  if (o == Py_None) return true;
  PyObject* args[1] = {o};
  PyObject* v = PyObject_VectorcallMethod(g_data_ptr, args, 1 | PY_VECTORCALL_ARGUMENTS_OFFSET, nullptr);
  if (!v) {
    if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return false;
    PyErr_Clear();
    return refuse();
  }
  const bool ok = to_address(v, out);
  Py_DECREF(v);
  return ok;
}

template <typename F>
PyObject* status(F call) {
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}
bool arity(Py_ssize_t n, Py_ssize_t want) { return n == want && g_stitch ? true : refuse(); }

// x_obj, x_bg, m_obj, m_bg, out, pixels, channels, stream
PyObject* stitch(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *p[5], *stream;
  long long pixels;
  int32_t channels;
  if (!arity(n, 8)) return nullptr;
  for (int i = 0; i < 5; ++i)
    if (!to_ptr(a[i], &p[i])) return nullptr;
  if (!to_ll(a[5], &pixels) || !to_int(a[6], &channels) || !to_address(a[7], &stream)) return nullptr;
  return status([&] {
    return g_stitch((const float*)p[0], (const float*)p[1], (const uint8_t*)p[2], (const uint8_t*)p[3], (float*)p[4], pixels, channels, stream);
  });
}

// first, diff_base, n_base, alpha, extra, n_extra, src, frames, frame_elems, out, stream
PyObject* decompress(PyObject*, PyObject* const* a, Py_ssize_t n) {
  constexpr int kCodes = 256;                            // more frames than the library takes are refused by it either way
  void *first, *diff, *extra, *out, *stream;
  int32_t n_base, n_extra, frames, codes[kCodes];
  long long elems;
  if (!arity(n, 11)) return nullptr;
  if (!to_ptr(a[0], &first) || !to_ptr(a[1], &diff) || !to_int(a[2], &n_base)) return nullptr;
  if (!PyFloat_CheckExact(a[3])) { refuse(); return nullptr; }
  const float alpha = (float)PyFloat_AS_DOUBLE(a[3]);
  if (!to_ptr(a[4], &extra) || !to_int(a[5], &n_extra) || !to_int(a[7], &frames) || !to_ll(a[8], &elems) ||
      !to_ptr(a[9], &out) || !to_address(a[10], &stream))
    return nullptr;
  const bool list = PyList_CheckExact(a[6]);
  if (frames < 1 || frames > kCodes || (!list && !PyTuple_CheckExact(a[6])) || PySequence_Fast_GET_SIZE(a[6]) != frames) {
    refuse();
    return nullptr;
  }
  PyObject** items = PySequence_Fast_ITEMS(a[6]);
  for (int t = 0; t < frames; ++t)
    if (!to_int(items[t], &codes[t])) return nullptr;
  return status([&] {
    return g_decompress((const float*)first, (const float*)diff, n_base, alpha, (const float*)extra, n_extra, codes, frames, elems, (float*)out, stream);
  });
}

// first_s, keys_s, diff_base, n_base, frame_elems, alpha_out, workspace, workspace_bytes, stream
PyObject* alpha(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *first, *keys, *diff, *out, *ws, *stream;
  int32_t n_base;
  long long elems, bytes;
  if (!arity(n, 9)) return nullptr;
  if (!to_ptr(a[0], &first) || !to_ptr(a[1], &keys) || !to_ptr(a[2], &diff) || !to_int(a[3], &n_base) || !to_ll(a[4], &elems) ||
      !to_ptr(a[5], &out) || !to_ptr(a[6], &ws) || !to_ll(a[7], &bytes) || !to_address(a[8], &stream))
    return nullptr;
  if (bytes < 0) { refuse(); return nullptr; }
  return status([&] {
    return g_alpha((const float*)first, (const float*)keys, (const float*)diff, n_base, elems, (float*)out, ws, (size_t)bytes, stream);
  });
}

// frames_dev, frames, frame_elems, sim, workspace, workspace_bytes, stream
PyObject* similarity(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *dev, *sim, *ws, *stream;
  int32_t frames;
  long long elems, bytes;
  if (!arity(n, 7)) return nullptr;
  if (!to_ptr(a[0], &dev) || !to_int(a[1], &frames) || !to_ll(a[2], &elems) || !to_ptr(a[3], &sim) || !to_ptr(a[4], &ws) ||
      !to_ll(a[5], &bytes) || !to_address(a[6], &stream))
    return nullptr;
  if (bytes < 0) { refuse(); return nullptr; }
  return status([&] { return g_similarity((const float*)dev, frames, elems, (float*)sim, ws, (size_t)bytes, stream); });
}

// addresses of the four functions, in the order of their declarations above
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* p[4];
  if (n != 4) { refuse(); return nullptr; }
  for (int i = 0; i < 4; ++i)
    if (!to_address(a[i], &p[i])) return nullptr;
  g_stitch = (decltype(g_stitch))p[0];
  g_decompress = (decltype(g_decompress))p[1];
  g_alpha = (decltype(g_alpha))p[2];
  g_similarity = (decltype(g_similarity))p[3];
  Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {"fc_cache_stitch", (PyCFunction)(void (*)(void))stitch, METH_FASTCALL, nullptr},
    {"fc_cache_decompress", (PyCFunction)(void (*)(void))decompress, METH_FASTCALL, nullptr},
    {"fc_cache_alpha", (PyCFunction)(void (*)(void))alpha, METH_FASTCALL, nullptr},
    {"fc_cache_frame_similarity", (PyCFunction)(void (*)(void))similarity, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall(void) {
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  return g_data_ptr ? PyModule_Create(&g_module) : nullptr;
}
