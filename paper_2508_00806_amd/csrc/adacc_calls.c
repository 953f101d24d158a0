// The calls of the Python binding that programs make in their inner loops, marshalled in C: the fields of a method, the addresses
// and sizes of the tensors and the current stream go straight to the library's C functions.  What these functions do not
// take (other objects than the binding's own and torch tensors) they leave, with a TypeError and before the
// library is called, to the binding's general way.
// (Host time of a call beside the launch, [20, 1024] STD: compression 1.5 us by ctypes, restoration 1.8; 0.6 and 0.5 like this.)
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "adacc.h"

// ---- what bind() is given: the library's functions, torch's types and the way to its current stream
typedef int (*CompressCall)(const adacc_method *, const void *, uint64_t, void *, uint64_t, adacc_workspace *, void *);
typedef int (*DecompressCall)(const adacc_method *, const void *, uint64_t, uint64_t, void *, int, void *);
typedef int (*MaskCall)(const void *, uint64_t, void *, void *);
typedef int (*ChannelCompressCall)(const adacc_channel_method *, const void *, uint64_t, uint32_t, void *, uint64_t, void *, uint64_t, void *);
typedef int (*ChannelDecompressCall)(const adacc_channel_method *, const void *, uint64_t, uint64_t, uint32_t, void *, int, void *);
typedef int (*ChannelwiseCompressCall)(uint32_t, uint32_t, uint32_t, const void *, uint64_t, uint32_t, void *, uint64_t, void *, uint64_t, void *);
typedef int (*ChannelwiseDecompressCall)(uint32_t, uint32_t, const void *, uint64_t, uint64_t, uint32_t, void *, int, void *);

static CompressCall compress_call;
static DecompressCall decompress_call;
static MaskCall mask_pack_call, mask_unpack_call;
static ChannelCompressCall channel_compress_call;
static ChannelDecompressCall channel_decompress_call;
static ChannelwiseCompressCall channelwise_compress_call;
static ChannelwiseDecompressCall channelwise_decompress_call;
static PyObject *f32_type, *bf16_type, *f16_type, *initialised, *current_device, *raw_stream, *general_stream;

enum { KIND, BITS, QUANT_GROUP, ASYM, SCALE_RULE, OUTLIER_MODE, STAT_GROUP, THRESH, TOPK, MAX_OUTLIERS, DTYPE, Z_THRESH, MAX_CHANNELS,
       DATA_PTR, NUMEL, ELEMENT_SIZE, CUDA_STREAM, NAMES };
static const char *const spelled[NAMES] = {"kind", "bits", "quant_group", "asym", "scale_rule", "outlier_mode", "stat_group", "thresh", "topk",
                                           "max_outliers", "dtype", "z_thresh", "max_channels", "data_ptr", "numel", "element_size", "cuda_stream"};
static PyObject *names[NAMES];

// Every conversion returns 0 with an exception set where it fails.
static int to_u64(PyObject *o, uint64_t *out) {
  if (!PyLong_Check(o)) { PyErr_SetString(PyExc_TypeError, "an int is needed"); return 0; }
  *out = (uint64_t)PyLong_AsUnsignedLongLongMask(o);
  return 1;
}
static int field_u32(PyObject *o, int name, uint32_t *out) {
  uint64_t v = 0;
  PyObject *f = PyObject_GetAttr(o, names[name]);
  if (!f) return 0;
  const int ok = to_u64(f, &v);
  Py_DECREF(f);
  *out = (uint32_t)v;
  return ok;
}
static int field_f32(PyObject *o, int name, float *out) {
  PyObject *f = PyObject_GetAttr(o, names[name]);
  if (!f) return 0;
  const double v = PyFloat_AsDouble(f);
  Py_DECREF(f);
  if (v == -1.0 && PyErr_Occurred()) return 0;
  *out = (float)v;
  return 1;
}
static int method_u64(PyObject *o, int name, uint64_t *out) {  // o.name()
  PyObject *r = PyObject_CallMethodNoArgs(o, names[name]);
  if (!r) return 0;
  const int ok = to_u64(r, out);
  Py_DECREF(r);
  return ok;
}
static int address(PyObject *o, void **out) {
  uint64_t v = 0;
  if (o != Py_None && !(PyLong_Check(o) ? to_u64(o, &v) : method_u64(o, DATA_PTR, &v))) return 0;
  *out = (void *)(uintptr_t)v;
  return 1;
}
static int size_in_bytes(PyObject *o, uint64_t *out) {
  uint64_t n, each;
  if (!method_u64(o, NUMEL, &n) || !method_u64(o, ELEMENT_SIZE, &each)) return 0;
  *out = n * each;
  return 1;
}
static int count_of(PyObject *given, PyObject *tensor, uint64_t *out) {
  return given == Py_None ? method_u64(tensor, NUMEL, out) : to_u64(given, out);
}
// the given stream, or the current one of the current device
static int stream_of(PyObject *o, void **out) {
  uint64_t v = 0;
  int ok = 0;
  PyObject *r = NULL;
  if (o != Py_None) {
    if (PyLong_Check(o)) return address(o, out);
    r = PyObject_GetAttr(o, names[CUDA_STREAM]);
  } else {
    PyObject *up = PyObject_CallNoArgs(initialised);
    if (!up) return 0;
    const int yes = PyObject_IsTrue(up);
    Py_DECREF(up);
    if (yes > 0) {
      PyObject *dev = PyObject_CallNoArgs(current_device);
      if (!dev) return 0;
      r = PyObject_CallOneArg(raw_stream, dev);
      Py_DECREF(dev);
    } else if (yes == 0) {
      r = PyObject_CallOneArg(general_stream, Py_None);
    }
  }
  if (!r) return 0;
  ok = to_u64(r, &v);
  Py_DECREF(r);
  *out = (void *)(uintptr_t)v;
  return ok;
}
static int method_of(PyObject *m, adacc_method *out) {
  return field_u32(m, KIND, &out->kind) && field_u32(m, BITS, &out->bits) && field_u32(m, QUANT_GROUP, &out->quant_group) &&
         field_u32(m, ASYM, &out->asym) && field_u32(m, SCALE_RULE, &out->scale_rule) && field_u32(m, OUTLIER_MODE, &out->outlier_mode) &&
         field_u32(m, STAT_GROUP, &out->stat_group) && field_f32(m, THRESH, &out->thresh) && field_u32(m, TOPK, &out->topk) &&
         field_u32(m, MAX_OUTLIERS, &out->max_outliers) && field_u32(m, DTYPE, &out->dtype);
}
static int channel_method_of(PyObject *m, adacc_channel_method *out) {
  return field_u32(m, BITS, &out->bits) && field_u32(m, QUANT_GROUP, &out->quant_group) && field_u32(m, ASYM, &out->asym) &&
         field_u32(m, SCALE_RULE, &out->scale_rule) && field_f32(m, Z_THRESH, &out->z_thresh) &&
         field_u32(m, MAX_CHANNELS, &out->max_channels) && field_u32(m, DTYPE, &out->dtype);
}
// the output's element type: binary32, or the 16-bit format that the method names
static int output_type(PyObject *dst, uint32_t dtype, int *out) {
  PyObject *t = PyObject_GetAttr(dst, names[DTYPE]);
  if (!t) return 0;
  const int wide = t == f32_type, own = t == (dtype == ADACC_DTYPE_F16 ? f16_type : bf16_type);
  Py_DECREF(t);
  if (!wide && !own) { PyErr_SetString(PyExc_TypeError, "another output type"); return 0; }
  *out = wide ? ADACC_DST_F32 : ADACC_DST_16;
  return 1;
}
static int arguments(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return 1;
  PyErr_SetString(PyExc_TypeError, "another number of arguments");
  return 0;
}
#define CALL(expr)                          \
  int rc;                                   \
  Py_BEGIN_ALLOW_THREADS rc = (expr);       \
  Py_END_ALLOW_THREADS return PyLong_FromLong(rc)

// (method, src, blob, address of the workspace or None, numel or None, stream or None)
static PyObject *compress(PyObject *self, PyObject *const *a, Py_ssize_t n) {
  adacc_method m;
  void *src, *blob, *ws, *stream;
  uint64_t numel, bytes;
  if (!arguments(n, 6) || !method_of(a[0], &m) || !address(a[1], &src) || !address(a[2], &blob) || !address(a[3], &ws) ||
      !count_of(a[4], a[1], &numel) || !size_in_bytes(a[2], &bytes) || !stream_of(a[5], &stream)) return NULL;
  CALL(compress_call(&m, src, numel, blob, bytes, (adacc_workspace *)ws, stream));
}
// (method, blob, dst, numel or None, stream or None)
static PyObject *decompress(PyObject *self, PyObject *const *a, Py_ssize_t n) {
  adacc_method m;
  void *blob, *dst, *stream;
  uint64_t numel, bytes;
  int type;
  if (!arguments(n, 5) || !method_of(a[0], &m) || !output_type(a[2], m.dtype, &type) || !address(a[1], &blob) || !address(a[2], &dst) ||
      !count_of(a[3], a[2], &numel) || !size_in_bytes(a[1], &bytes) || !stream_of(a[4], &stream)) return NULL;
  CALL(decompress_call(&m, blob, bytes, numel, dst, type, stream));
}
// (mask, bits, n or None, stream or None); ADACC_ESIZE where one of them is too small
static PyObject *mask(PyObject *const *a, Py_ssize_t n, int pack) {
  void *bytes, *bits, *stream;
  uint64_t count, have_bytes, have_bits;
  if (!arguments(n, 4) || !address(a[0], &bytes) || !address(a[1], &bits) || !count_of(a[2], a[0], &count) ||
      !size_in_bytes(a[0], &have_bytes) || !size_in_bytes(a[1], &have_bits) || !stream_of(a[3], &stream)) return NULL;
  if (have_bits < count / 8u + (count % 8u != 0u) || have_bytes < count) return PyLong_FromLong(ADACC_ESIZE);
  CALL(pack ? mask_pack_call(bytes, count, bits, stream) : mask_unpack_call(bits, count, bytes, stream));
}
static PyObject *mask_pack(PyObject *self, PyObject *const *a, Py_ssize_t n) { return mask(a, n, 1); }
static PyObject *mask_unpack(PyObject *self, PyObject *const *a, Py_ssize_t n) { return mask(a, n, 0); }
// (method, src, tokens, hidden, blob, workspace, stream or None)
static PyObject *channel_compress(PyObject *self, PyObject *const *a, Py_ssize_t n) {
  adacc_channel_method m;
  void *src, *blob, *ws, *stream;
  uint64_t tokens, hidden, bytes, room;
  if (!arguments(n, 7) || !channel_method_of(a[0], &m) || !address(a[1], &src) || !to_u64(a[2], &tokens) || !to_u64(a[3], &hidden) ||
      !address(a[4], &blob) || !size_in_bytes(a[4], &bytes) || !address(a[5], &ws) || !size_in_bytes(a[5], &room) ||
      !stream_of(a[6], &stream)) return NULL;
  CALL(channel_compress_call(&m, src, tokens, (uint32_t)hidden, blob, bytes, ws, room, stream));
}
// (method, blob, tokens, hidden, dst, stream or None)
static PyObject *channel_decompress(PyObject *self, PyObject *const *a, Py_ssize_t n) {
  adacc_channel_method m;
  void *blob, *dst, *stream;
  uint64_t tokens, hidden, bytes;
  int type;
  if (!arguments(n, 6) || !channel_method_of(a[0], &m) || !output_type(a[4], m.dtype, &type) || !address(a[1], &blob) ||
      !size_in_bytes(a[1], &bytes) || !to_u64(a[2], &tokens) || !to_u64(a[3], &hidden) || !address(a[4], &dst) ||
      !stream_of(a[5], &stream)) return NULL;
  CALL(channel_decompress_call(&m, blob, bytes, tokens, (uint32_t)hidden, dst, type, stream));
}
// (bits, scale rule, format, src, tokens, hidden, blob, workspace, stream or None)
static PyObject *channelwise_compress(PyObject *self, PyObject *const *a, Py_ssize_t n) {
  void *src, *blob, *ws, *stream;
  uint64_t bits, rule, format, tokens, hidden, bytes, room;
  if (!arguments(n, 9) || !to_u64(a[0], &bits) || !to_u64(a[1], &rule) || !to_u64(a[2], &format) || !address(a[3], &src) ||
      !to_u64(a[4], &tokens) || !to_u64(a[5], &hidden) || !address(a[6], &blob) || !size_in_bytes(a[6], &bytes) || !address(a[7], &ws) ||
      !size_in_bytes(a[7], &room) || !stream_of(a[8], &stream)) return NULL;
  CALL(channelwise_compress_call((uint32_t)bits, (uint32_t)rule, (uint32_t)format, src, tokens, (uint32_t)hidden, blob, bytes, ws, room, stream));
}
// (bits, format, blob, tokens, hidden, dst, output type, stream or None)
static PyObject *channelwise_decompress(PyObject *self, PyObject *const *a, Py_ssize_t n) {
  void *blob, *dst, *stream;
  uint64_t bits, format, tokens, hidden, bytes, type;
  if (!arguments(n, 8) || !to_u64(a[0], &bits) || !to_u64(a[1], &format) || !address(a[2], &blob) || !size_in_bytes(a[2], &bytes) ||
      !to_u64(a[3], &tokens) || !to_u64(a[4], &hidden) || !address(a[5], &dst) || !to_u64(a[6], &type) || !stream_of(a[7], &stream)) return NULL;
  CALL(channelwise_decompress_call((uint32_t)bits, (uint32_t)format, blob, bytes, tokens, (uint32_t)hidden, dst, (int)type, stream));
}

// bind(addresses of the eight functions, float32, bfloat16, float16, is_initialized, current device, raw stream, general stream)
static PyObject *bind(PyObject *self, PyObject *const *a, Py_ssize_t n) {
  uint64_t f[8];
  PyObject **kept[7] = {&f32_type, &bf16_type, &f16_type, &initialised, &current_device, &raw_stream, &general_stream};
  if (!arguments(n, 15)) return NULL;
  for (int i = 0; i < 8; ++i)
    if (!to_u64(a[i], &f[i])) return NULL;
  compress_call = (CompressCall)(uintptr_t)f[0];
  decompress_call = (DecompressCall)(uintptr_t)f[1];
  mask_pack_call = (MaskCall)(uintptr_t)f[2];
  mask_unpack_call = (MaskCall)(uintptr_t)f[3];
  channel_compress_call = (ChannelCompressCall)(uintptr_t)f[4];
  channel_decompress_call = (ChannelDecompressCall)(uintptr_t)f[5];
  channelwise_compress_call = (ChannelwiseCompressCall)(uintptr_t)f[6];
  channelwise_decompress_call = (ChannelwiseDecompressCall)(uintptr_t)f[7];
  for (int i = 0; i < 7; ++i) {
    Py_INCREF(a[8 + i]);
    Py_XSETREF(*kept[i], a[8 + i]);
  }
  Py_RETURN_NONE;
}

#define ENTRY(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, NULL}
static PyMethodDef functions[] = {ENTRY(bind), ENTRY(compress), ENTRY(decompress), ENTRY(mask_pack), ENTRY(mask_unpack), ENTRY(channel_compress),
                                  ENTRY(channel_decompress), ENTRY(channelwise_compress), ENTRY(channelwise_decompress), {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, functions, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__calls(void) {
  for (int i = 0; i < NAMES; ++i)
    if (!names[i] && !(names[i] = PyUnicode_InternFromString(spelled[i]))) return NULL;
  return PyModule_Create(&module);
}
