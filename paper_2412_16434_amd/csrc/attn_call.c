// The attention call's argument checks and marshalling, compiled: what binding.py's prefix_prefill_attn does with some fifty
// attribute reads and a ctypes call, 3.6 of the 9.2 us that a call of one launch kept the host busy.  Only the ordinary call is
// taken (no stream or tuning argument, every tensor as the entry point wants it); for anything else, and for every error, the
// answer is None and the general path decides, so that there is one place that says what is wrong.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "symph.h"

typedef int32_t (*attn_fn)(const symph_kv_cache*, int32_t, const void*, const void*, const void*, void*, const int32_t*,
                           const int32_t*, const int32_t*, int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, float, void*,
                           int64_t, void*);

// Set once, by bind()
static attn_fn entry;
static PyObject *t_bf16, *t_fp32, *t_int32, *raw_stream, *get_device;
static PyObject *s_dtype, *s_shape, *s_is_cuda, *s_is_contiguous, *s_data_ptr, *s_stride, *s_numel, *s_element_size;

static PyObject* bind(PyObject* self, PyObject* args) {
  unsigned long long address;
  PyObject *a, *b, *c, *d, *e;
  (void)self;
  if (!PyArg_ParseTuple(args, "KOOOOO", &address, &a, &b, &c, &d, &e)) return NULL;
  Py_INCREF(a), Py_INCREF(b), Py_INCREF(c), Py_INCREF(d), Py_INCREF(e);
  Py_XDECREF(t_bf16), Py_XDECREF(t_fp32), Py_XDECREF(t_int32), Py_XDECREF(raw_stream), Py_XDECREF(get_device);
  t_bf16 = a, t_fp32 = b, t_int32 = c, raw_stream = d, get_device = e;
  entry = (attn_fn)(uintptr_t)address;
  Py_RETURN_NONE;
}

// Each of these returns 1, or 0 where the general path has to look (an exception may be set; the caller clears it).
static int as_int(PyObject* o, int64_t* out) {
  if (!o || !PyLong_CheckExact(o)) return 0;
  *out = PyLong_AsLongLong(o);
  return !(*out == -1 && PyErr_Occurred());
}
static int as_int32(PyObject* o, int32_t* out) {
  int64_t v;
  if (!as_int(o, &v) || v < INT32_MIN || v > INT32_MAX) return 0;
  *out = (int32_t)v;
  return 1;
}
static int method_int(PyObject* t, PyObject* name, int64_t* out) {
  PyObject* r = PyObject_CallMethodNoArgs(t, name);
  const int ok = as_int(r, out);
  Py_XDECREF(r);
  return ok;
}
static int attr_is(PyObject* t, PyObject* name, PyObject* want) {
  PyObject* r = PyObject_GetAttr(t, name);
  const int ok = r == want;
  Py_XDECREF(r);
  return ok;
}
static int dims(PyObject* t, PyObject* name, int call, int n, int64_t* out) {  // the n values of .shape / .stride()
  PyObject* r = call ? PyObject_CallMethodNoArgs(t, name) : PyObject_GetAttr(t, name);
  int ok = r && PyTuple_Check(r) && PyTuple_GET_SIZE(r) == n;
  for (int i = 0; ok && i < n; ++i) ok = as_int(PyTuple_GET_ITEM(r, i), out + i);
  Py_XDECREF(r);
  return ok;
}
// On the device, contiguous, of the element type (NULL: any)
static int dense(PyObject* t, PyObject* dtype, void** ptr) {
  if (!attr_is(t, s_is_cuda, Py_True) || (dtype && !attr_is(t, s_dtype, dtype))) return 0;
  PyObject* r = PyObject_CallMethodNoArgs(t, s_is_contiguous);
  const int ok = r == Py_True;
  Py_XDECREF(r);
  int64_t p;
  if (!ok || !method_int(t, s_data_ptr, &p)) return 0;
  *ptr = (void*)(uintptr_t)p;
  return 1;
}

// (k_pool, v_pool, layer, q, k_new, v_new, out, cu_new_lens, prefix_lens, block_table, max_new_len, max_prefix_len, scale,
// workspace) -> status or None
enum { kKPool, kVPool, kLayer, kQ, kKNew, kVNew, kOut, kCu, kLens, kTable, kMaxNew, kMaxPrefix, kScale, kWorkspace, kArgs };

static int gather(PyObject* const* a, symph_kv_cache* c, int32_t* ints, float* scale, void** ptrs, int64_t* ws_bytes,
                  void** stream) {
  int64_t pool[5], strides[5], q[3], o[3], kn[3], vn[3], v;
  PyObject* dt = PyObject_GetAttr(a[kKPool], s_dtype);
  Py_XDECREF(dt);  // (torch's dtypes live as long as the module)
  if (dt != t_bf16 && dt != t_fp32) return 0;
  if (!dims(a[kKPool], s_shape, 0, 5, pool) || !dims(a[kKPool], s_stride, 1, 5, strides)) return 0;
  for (int i = 0; i < 5; ++i)
    if (pool[i] > INT32_MAX) return 0;
  if (!method_int(a[kKPool], s_data_ptr, &v)) return 0;
  c->k_base = (void*)(uintptr_t)v;
  if (!method_int(a[kVPool], s_data_ptr, &v)) return 0;
  c->v_base = (void*)(uintptr_t)v;
  c->layer_stride = strides[0], c->block_stride = strides[1];
  c->n_layers = (int32_t)pool[0], c->n_blocks = (int32_t)pool[1], c->block_size = (int32_t)pool[2];
  c->n_kv_heads = (int32_t)pool[3], c->head_dim = (int32_t)pool[4];
  c->dtype = dt == t_bf16 ? SYMPH_BF16 : SYMPH_FP32;

  if (!dims(a[kQ], s_shape, 0, 3, q) || !dims(a[kOut], s_shape, 0, 3, o) || !dims(a[kKNew], s_shape, 0, 3, kn) ||
      !dims(a[kVNew], s_shape, 0, 3, vn))
    return 0;
  for (int i = 0; i < 3; ++i)
    if (q[i] != o[i] || kn[i] != vn[i] || q[i] > INT32_MAX) return 0;
  if (!dense(a[kQ], dt, ptrs + 0) || !dense(a[kKNew], dt, ptrs + 1) || !dense(a[kVNew], dt, ptrs + 2) ||
      !dense(a[kOut], dt, ptrs + 3) || !dense(a[kCu], t_int32, ptrs + 4) || !dense(a[kLens], t_int32, ptrs + 5))
    return 0;
  int64_t table[2] = {0, 0}, sessions;
  ptrs[6] = NULL;
  if (a[kTable] != Py_None &&
      (!dims(a[kTable], s_shape, 0, 2, table) || table[1] > INT32_MAX || !dense(a[kTable], t_int32, ptrs + 6)))
    return 0;
  if (!dims(a[kLens], s_shape, 0, 1, &sessions) || sessions > INT32_MAX) return 0;
  ints[1] = (int32_t)table[1], ints[2] = (int32_t)sessions, ints[3] = (int32_t)q[1], ints[4] = (int32_t)q[0];
  if (!as_int32(a[kLayer], ints) || !as_int32(a[kMaxNew], ints + 5) || !as_int32(a[kMaxPrefix], ints + 6)) return 0;
  if (!PyFloat_CheckExact(a[kScale])) return 0;
  *scale = (float)PyFloat_AS_DOUBLE(a[kScale]);
  ptrs[7] = NULL;
  *ws_bytes = 0;
  if (a[kWorkspace] != Py_None) {
    int64_t n, e;
    if (!dense(a[kWorkspace], NULL, ptrs + 7) || !method_int(a[kWorkspace], s_numel, &n) ||
        !method_int(a[kWorkspace], s_element_size, &e))
      return 0;
    *ws_bytes = n * e;
  }
  // the current stream of the current device
  PyObject* device = PyObject_CallNoArgs(get_device);
  PyObject* raw = device ? PyObject_CallOneArg(raw_stream, device) : NULL;
  const int ok = raw && PyLong_Check(raw);
  if (ok) *stream = PyLong_AsVoidPtr(raw);
  Py_XDECREF(raw);
  Py_XDECREF(device);
  return ok && !PyErr_Occurred();
}

static PyObject* attn(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  (void)self;
  symph_kv_cache c;
  int32_t ints[7], status;  // layer, table stride, sessions, query heads, tokens, max_new_len, max_prefix_len
  float scale;
  void *ptrs[8], *stream;
  int64_t ws_bytes;
  if (n != kArgs || !entry || !gather(a, &c, ints, &scale, ptrs, &ws_bytes, &stream)) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  Py_BEGIN_ALLOW_THREADS
  status = entry(&c, ints[0], ptrs[0], ptrs[1], ptrs[2], ptrs[3], ptrs[4], ptrs[5], ptrs[6], ints[1], ints[2], ints[3], ints[4],
                 ints[5], ints[6], scale, ptrs[7], ws_bytes, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

static PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, "bind(address of the entry point, bfloat16, float32, int32, raw stream of a device, current device)"},
    {"attn", (PyCFunction)(void (*)(void))attn, METH_FASTCALL, "status of the call, or None where the general path has to make it"},
    {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_attn_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__attn_call(void) {
  s_dtype = PyUnicode_InternFromString("dtype");
  s_shape = PyUnicode_InternFromString("shape");
  s_is_cuda = PyUnicode_InternFromString("is_cuda");
  s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_stride = PyUnicode_InternFromString("stride");
  s_numel = PyUnicode_InternFromString("numel");
  s_element_size = PyUnicode_InternFromString("element_size");
  if (!s_dtype || !s_shape || !s_is_cuda || !s_is_contiguous || !s_data_ptr || !s_stride || !s_numel || !s_element_size)
    return NULL;
  return PyModule_Create(&module);
}
