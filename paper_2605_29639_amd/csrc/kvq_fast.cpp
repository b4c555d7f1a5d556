// The calls of a serving step without Python between the arguments and the library: kv_quant_write,
// paged_decode_attn(_prefix), blocks_export and blocks_import of kvq.py, for arguments in the form a serving loop gives them (plain tensors
// and plain ints).  What this module does not accept (None is returned), or the library refuses from its arguments,
// it leaves to kvq.py, whose checks and errors are the binding's, and nothing has been launched; an error of
// the runtime or of the debug checks is the call's answer, and kvq.py raises it.
// One sequence of 600 tokens, int8, write and attention, host time a step: through ctypes 17.1 us, here 7.7
// (with a second attention launch, the reduce, 20.2 and 10.7: a launch takes 3); its kernels take 10.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "../../include/kvq.h"

namespace {

decltype(&kv_quant_write) g_write = nullptr;
decltype(&paged_decode_attn) g_attn = nullptr;
decltype(&paged_decode_attn_prefix) g_attn_prefix = nullptr;
decltype(&kvq_blocks_export) g_export = nullptr;
decltype(&kvq_blocks_import) g_import = nullptr;
decltype(&kvq_cache_bytes) g_cache_bytes = nullptr;
decltype(&kvq_scales_bytes) g_scales_bytes = nullptr;
PyObject* g_get_device = nullptr;  // torch._C._cuda_getDevice
PyObject* g_get_stream = nullptr;  // torch._C._cuda_getCurrentRawStream
PyObject* g_desc_type = nullptr;   // kvq.CacheDesc

// A plain contiguous device tensor of the type, or nullptr.  (A subclass may stand for something else.)
const at::Tensor* plain(PyObject* o, at::ScalarType type) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || t.scalar_type() != type || t.layout() != at::kStrided || !t.has_storage() || !t.is_cuda() ||
      !t.is_contiguous() || t.numel() == 0)
    return nullptr;
  return &t;
}

// (other objects that lend a buffer of a descriptor's size are none)
bool get_desc(PyObject* o, kvq_cache_desc_t* desc) {
  Py_buffer view;
  if ((PyObject*)Py_TYPE(o) != g_desc_type || PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
    PyErr_Clear();
    return false;
  }
  const bool ok = view.len == (Py_ssize_t)sizeof(*desc);
  if (ok) memcpy(desc, view.buf, sizeof(*desc));
  PyBuffer_Release(&view);
  return ok;
}

bool get_int(PyObject* o, int32_t* out) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long v = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow != 0 || v < INT32_MIN || v > INT32_MAX) return false;
  *out = (int32_t)v;
  return true;
}

// the given stream handle, or that of the current stream of the current device
bool get_stream(PyObject* o, void** stream) {
  PyObject* handle = nullptr;
  if (o == Py_None) {
    PyObject* device = PyObject_CallNoArgs(g_get_device);
    if (device) handle = PyObject_CallOneArg(g_get_stream, device);
    Py_XDECREF(device);
  } else if (PyLong_CheckExact(o)) {
    handle = o;
    Py_INCREF(handle);
  }
  if (handle) *stream = PyLong_AsVoidPtr(handle);
  Py_XDECREF(handle);
  if (!handle || PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}

// cache and scales of the sizes the library reports for the descriptor (an unquantized cache has no scales)
bool get_pool(PyObject* cache, PyObject* scales, const kvq_cache_desc_t& desc, void** cache_ptr, float** scales_ptr) {
  const at::Tensor* c = plain(cache, at::kByte);
  if (!c || (size_t)c->numel() != g_cache_bytes(&desc)) return false;
  const size_t bytes = g_scales_bytes(&desc);
  *cache_ptr = c->data_ptr();
  *scales_ptr = nullptr;
  if (bytes == 0) return THPVariable_CheckExact(scales) && THPVariable_Unpack(scales).scalar_type() == at::kFloat &&
                         THPVariable_Unpack(scales).numel() == 0;
  const at::Tensor* s = plain(scales, at::kFloat);
  if (!s || (size_t)s->numel() * sizeof(float) != bytes) return false;
  *scales_ptr = (float*)s->data_ptr();
  return true;
}

// (tensors that only stand for others, under vmap say, throw where their memory is asked for: kvq.py asks
// again and raises)
template <PyObject* (*CALL)(PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject*, PyObject* const* a, Py_ssize_t n) {
  try {
    return CALL(a, n);
  } catch (const std::exception&) {
    Py_RETURN_NONE;
  }
}

// write(k, v, slot_mapping, cache, scales, desc, stream) -> return code, or None
PyObject* fast_write(PyObject* const* a, Py_ssize_t n) {
  kvq_cache_desc_t desc;
  void *cache, *stream;
  float* scales;
  if (n != 7 || !g_write || !get_desc(a[5], &desc)) Py_RETURN_NONE;
  const at::Tensor *k = plain(a[0], at::kBFloat16), *v = plain(a[1], at::kBFloat16), *slots = plain(a[2], at::kLong);
  if (!k || !v || !slots || k->dim() != 3 || slots->dim() != 1 || k->size(0) > INT32_MAX || k->size(1) != desc.num_kv_heads ||
      k->size(2) != desc.head_dim || v->sizes() != k->sizes() || slots->size(0) != k->size(0))
    Py_RETURN_NONE;
  if (!get_pool(a[3], a[4], desc, &cache, &scales) || !get_stream(a[6], &stream)) Py_RETURN_NONE;
  int rc;
  const void *kp = k->data_ptr(), *vp = v->data_ptr();
  const int64_t* sp = (const int64_t*)slots->data_ptr();
  const int32_t tokens = (int32_t)k->size(0);
  Py_BEGIN_ALLOW_THREADS
  rc = g_write(kp, vp, sp, tokens, cache, scales, &desc, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// attn(q, cache, scales, desc, block_tables, seq_lens, q_len, max_seq_len, sm_scale, out, workspace,
//      chunk_tokens, stream, shared_prefix_tokens) -> return code, or None
PyObject* fast_attn(PyObject* const* a, Py_ssize_t n) {
  kvq_cache_desc_t desc;
  void *cache, *stream;
  float* scales;
  int32_t q_len, max_len, chunk, prefix;
  if (n != 14 || !g_attn || !get_desc(a[3], &desc)) Py_RETURN_NONE;
  const at::Tensor *q = plain(a[0], at::kBFloat16), *tables = plain(a[4], at::kInt), *lens = plain(a[5], at::kInt),
                   *out = plain(a[9], at::kFloat), *ws = plain(a[10], at::kByte);
  if (!q || !tables || !lens || !out || !ws || !get_int(a[6], &q_len) || !get_int(a[7], &max_len) ||
      !PyFloat_CheckExact(a[8]) || !get_int(a[11], &chunk) || !get_int(a[13], &prefix))
    Py_RETURN_NONE;
  if (lens->dim() != 1 || q->dim() != 3 || lens->size(0) > INT32_MAX || q->size(0) != lens->size(0) * q_len ||
      q->size(2) != desc.head_dim || q->size(1) > INT32_MAX || out->sizes() != q->sizes() || tables->dim() != 2 ||
      tables->size(0) != lens->size(0) || tables->size(1) > INT32_MAX)
    Py_RETURN_NONE;
  if (!get_pool(a[1], a[2], desc, &cache, &scales) || !get_stream(a[12], &stream)) Py_RETURN_NONE;
  int rc;
  const void* qp = q->data_ptr();
  const int32_t *tp = (const int32_t*)tables->data_ptr(), *lp = (const int32_t*)lens->data_ptr();
  const int32_t cols = (int32_t)tables->size(1), batch = (int32_t)lens->size(0), heads = (int32_t)q->size(1);
  const float scale = (float)PyFloat_AS_DOUBLE(a[8]);
  float* op = (float*)out->data_ptr();
  void* wp = ws->data_ptr();
  const size_t held = (size_t)ws->numel();
  Py_BEGIN_ALLOW_THREADS
  rc = prefix ? g_attn_prefix(qp, cache, scales, &desc, tp, cols, lp, batch, q_len, heads, max_len, scale, chunk, prefix,
                              op, wp, held, stream)
              : g_attn(qp, cache, scales, &desc, tp, cols, lp, batch, q_len, heads, max_len, scale, chunk, op, wp, held,
                       stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// A plain contiguous tensor on the device or in pinned host memory, or an empty one (a null pointer).
bool get_area(PyObject* o, at::ScalarType type, void** ptr) {
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || t.scalar_type() != type || t.layout() != at::kStrided || !t.has_storage() || !t.is_contiguous())
    return false;
  *ptr = nullptr;
  if (t.numel() == 0) return true;
  if (!t.is_cuda() && !t.is_pinned()) return false;
  *ptr = t.data_ptr();
  return true;
}

// move(out of the pool, cache, scales, desc, block_ids, packed_cache, packed_scales, stream) -> return code, or None
PyObject* fast_move(PyObject* const* a, Py_ssize_t n) {
  kvq_cache_desc_t desc;
  void *stream, *packed, *packed_scales;
  if (n != 8 || !g_write || !get_desc(a[3], &desc)) Py_RETURN_NONE;
  const at::Tensor *cache = plain(a[1], at::kByte), *scales = plain(a[2], at::kFloat), *ids = plain(a[4], at::kInt);
  if (!cache || !ids || ids->numel() > INT32_MAX || (!scales && g_scales_bytes(&desc) != 0)) Py_RETURN_NONE;
  if (!scales && (!THPVariable_CheckExact(a[2]) || THPVariable_Unpack(a[2]).scalar_type() != at::kFloat ||
                  THPVariable_Unpack(a[2]).numel() != 0))
    Py_RETURN_NONE;
  if (!get_area(a[5], at::kByte, &packed) || !get_area(a[6], at::kFloat, &packed_scales) || !get_stream(a[7], &stream))
    Py_RETURN_NONE;
  int rc;
  const bool out = a[0] == Py_True;
  void* cp = cache->data_ptr();
  float* sp = scales ? (float*)scales->data_ptr() : nullptr;
  const int32_t *ip = (const int32_t*)ids->data_ptr(), num = (int32_t)ids->numel();
  Py_BEGIN_ALLOW_THREADS
  rc = out ? g_export(cp, sp, &desc, ip, num, packed, (float*)packed_scales, stream)
           : g_import(packed, (const float*)packed_scales, &desc, ip, num, cp, sp, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// bind(addresses of the seven library functions, _cuda_getDevice, _cuda_getCurrentRawStream, CacheDesc)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 10) {
    PyErr_SetString(PyExc_TypeError, "bind takes seven addresses, two callables and a type");
    return nullptr;
  }
  void* p[7];
  for (int i = 0; i < 7; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred()) return nullptr;
  }
  g_cache_bytes = (decltype(g_cache_bytes))p[0];
  g_scales_bytes = (decltype(g_scales_bytes))p[1];
  g_attn = (decltype(g_attn))p[2];
  g_attn_prefix = (decltype(g_attn_prefix))p[3];
  g_export = (decltype(g_export))p[5];
  g_import = (decltype(g_import))p[6];
  Py_INCREF(a[7]);
  Py_INCREF(a[8]);
  Py_INCREF(a[9]);
  g_get_device = a[7];
  g_get_stream = a[8];
  g_desc_type = a[9];
  g_write = (decltype(g_write))p[4];
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"write", (PyCFunction)(void (*)(void))guarded<fast_write>, METH_FASTCALL, nullptr},
                         {"attn", (PyCFunction)(void (*)(void))guarded<fast_attn>, METH_FASTCALL, nullptr},
                         {"move", (PyCFunction)(void (*)(void))guarded<fast_move>, METH_FASTCALL, nullptr},
                         {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_kvq_fast", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__kvq_fast() { return PyModule_Create(&module); }
