/* Marshalling of the Python binding's per-step calls: tensor -> device address, shape struct -> pointer, the
 * current stream, then the C entry point, with the interpreter lock released.  With ctypes a step of one
 * launch took 8.3 us of host time (two launches: 12.4 us), here it takes 4.4 us (7.2 us), most of it the launches;
 * a step of 600 tokens that is waited for came down from 24.9 to 21.0 us.  No arithmetic, no validation: libfasa does that.
 *
 * Module functions take positional arguments in the order of include/fasa.h and return the status code.  An
 * address argument is None (NULL), an int, or an object with data_ptr() (a torch tensor); anything else goes to the Python
 * function handed to bind().  The last argument, the stream, is None for torch's current one. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <dlfcn.h>

#include "fasa.h"

static PyObject *s_data_ptr, *s_cuda_stream; /* interned method and attribute names */
static PyObject *f_address;                  /* Python: address of anything else */
static PyObject *f_device, *f_raw_stream;    /* torch._C: current device, its current stream */
static PyObject *t_shape, *t_paging;         /* the binding's ctypes structures */
static PyObject* f_refuse;                   /* Python: raises what ctypes raises for another object in their place */

/* The conversions below leave *ok = 0 and an exception behind when they fail, and do nothing once that has
 * happened: the first argument that is refused is the one reported. */
static void* address(PyObject* x, int* ok) {
  if (!*ok || x == Py_None) return NULL;
  PyObject* v;
  if (PyLong_Check(x)) {
    v = x;
    Py_INCREF(v);
  } else {
    v = PyObject_CallMethodNoArgs(x, s_data_ptr);
    if (!v) {
      if (!PyErr_ExceptionMatches(PyExc_AttributeError)) { *ok = 0; return NULL; }
      PyErr_Clear();
      v = PyObject_CallOneArg(f_address, x);
      if (!v) { *ok = 0; return NULL; }
    }
  }
  void* p = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  if (!p && PyErr_Occurred()) *ok = 0;
  return p;
}

static void* stream_of(PyObject* x, int* ok) {
  PyObject* v;
  if (!*ok) return NULL;
  if (x == Py_None) {
    PyObject* dev = PyObject_CallNoArgs(f_device);
    if (!dev) { *ok = 0; return NULL; }
    v = PyObject_CallOneArg(f_raw_stream, dev);
    Py_DECREF(dev);
  } else if (PyLong_Check(x)) {
    v = x;
    Py_INCREF(v);
  } else {
    v = PyObject_GetAttr(x, s_cuda_stream);
    if (!v && PyErr_ExceptionMatches(PyExc_AttributeError)) { PyErr_Clear(); v = PyNumber_Long(x); }
  }
  if (!v) { *ok = 0; return NULL; }
  void* p = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  if (!p && PyErr_Occurred()) *ok = 0;
  return p;
}

/* memory of a ctypes structure of that type (it exports its own bytes) */
static void* structure(PyObject* x, PyObject* type, int* ok) {
  Py_buffer b;
  if (!*ok) return NULL;
  if (!PyObject_TypeCheck(x, (PyTypeObject*)type)) {
    PyObject* r = PyObject_CallFunctionObjArgs(f_refuse, x, type, NULL);
    if (r) { Py_DECREF(r); PyErr_SetString(PyExc_TypeError, "wrong structure"); }
    *ok = 0;
    return NULL;
  }
  if (PyObject_GetBuffer(x, &b, PyBUF_SIMPLE) != 0) { *ok = 0; return NULL; }
  void* p = b.buf;
  PyBuffer_Release(&b); /* x is alive for the length of the call: it is one of its arguments */
  return p;
}

/* integers as ctypes converts them: anything with __index__ (numpy's integers too), reduced to the type's width */
static unsigned long int_bits(PyObject* x, int* ok) {
  if (!*ok) return 0;
  const unsigned long n = PyLong_AsUnsignedLongMask(x);
  if (n == (unsigned long)-1 && PyErr_Occurred()) *ok = 0;
  return n;
}
static size_t bytes_of(PyObject* x, int* ok) { return (size_t)int_bits(x, ok); }
static int32_t int_of(PyObject* x, int* ok) { return (int32_t)int_bits(x, ok); }

#define SHAPE(i) ((const fasa_shape*)structure(a[i], t_shape, &ok))
#define PAGING(i) ((const fasa_paging*)structure(a[i], t_paging, &ok))
#define P(i) address(a[i], &ok)
#define I(i) int_of(a[i], &ok)
#define Z(i) bytes_of(a[i], &ok)
#define STREAM(i) stream_of(a[i], &ok)

/* ENTRY(name, number of arguments, parameter list of the C function, declarations, arguments of the call) */
#define ENTRY(name, nargs, decls, ...)                                                                        \
  static __typeof__(&fasa_##name) p_##name;                                                                   \
  static PyObject* py_##name(PyObject* self, PyObject* const* a, Py_ssize_t n) {                               \
    (void)self;                                                                                               \
    if (n != nargs) { PyErr_SetString(PyExc_TypeError, #name ": wrong number of arguments"); return NULL; }   \
    int ok = 1, rc;                                                                                           \
    decls;                                                                                                    \
    if (!ok) return NULL;                                                                                     \
    Py_BEGIN_ALLOW_THREADS rc = p_##name(__VA_ARGS__);                                                        \
    Py_END_ALLOW_THREADS return PyLong_FromLong(rc);                                                          \
  }

#define STEP_DECLS(o)                                                                                         \
  void *q = P(o), *K = P(o + 1), *V = P(o + 2), *Kp = P(o + 3), *fc = P(o + 4), *kn = P(o + 5), *vn = P(o + 6)

ENTRY(pack_kcache, 7, const fasa_shape* s = SHAPE(0); void* K = P(1); void* fc = P(2); void* Kp = P(3);
      int32_t n0 = I(4); int32_t n1 = I(5); void* st = STREAM(6), s, K, fc, Kp, n0, n1, st)
ENTRY(score, 6, const fasa_shape* s = SHAPE(0); void* q = P(1); void* Kp = P(2); void* fc = P(3); float* S = P(4);
      void* st = STREAM(5), s, q, Kp, fc, S, st)
ENTRY(topk, 6, const fasa_shape* s = SHAPE(0); float* S = P(1); int32_t* T = P(2); void* ws = P(3); size_t z = Z(4);
      void* st = STREAM(5), s, S, T, ws, z, st)
ENTRY(sparse_attend, 9, const fasa_shape* s = SHAPE(0); void* q = P(1); void* K = P(2); void* V = P(3); int32_t* T = P(4);
      float* O = P(5); void* ws = P(6); size_t z = Z(7); void* st = STREAM(8), s, q, K, V, T, O, ws, z, st)
ENTRY(dense_attend, 8, const fasa_shape* s = SHAPE(0); void* q = P(1); void* K = P(2); void* V = P(3); float* O = P(4);
      void* ws = P(5); size_t z = Z(6); void* st = STREAM(7), s, q, K, V, O, ws, z, st)
ENTRY(decode_step, 14, const fasa_shape* s = SHAPE(0); STEP_DECLS(1); float* S = P(8); int32_t* T = P(9); float* O = P(10);
      void* ws = P(11); size_t z = Z(12); void* st = STREAM(13), s, q, K, V, Kp, fc, kn, vn, S, T, O, ws, z, st)
ENTRY(decode_step_static, 12, const fasa_shape* s = SHAPE(0); STEP_DECLS(1); float* S = P(8); int32_t* T = P(9);
      float* O = P(10); void* st = STREAM(11), s, q, K, V, Kp, fc, kn, vn, S, T, O, st)
ENTRY(decode_step_ragged, 16, const fasa_shape* s = SHAPE(0); STEP_DECLS(1); int32_t* nc = P(8); int32_t* bu = P(9);
      float* S = P(10); int32_t* T = P(11); float* O = P(12); void* ws = P(13); size_t z = Z(14); void* st = STREAM(15),
      s, q, K, V, Kp, fc, kn, vn, nc, bu, S, T, O, ws, z, st)
ENTRY(pack_kcache_paged, 8, const fasa_shape* s = SHAPE(0); const fasa_paging* pg = PAGING(1); void* K = P(2);
      void* fc = P(3); void* Kp = P(4); int32_t n0 = I(5); int32_t n1 = I(6); void* st = STREAM(7),
      s, pg, K, fc, Kp, n0, n1, st)
ENTRY(decode_step_paged, 17, const fasa_shape* s = SHAPE(0); const fasa_paging* pg = PAGING(1); STEP_DECLS(2);
      int32_t* nc = P(9); int32_t* bu = P(10); float* S = P(11); int32_t* T = P(12); float* O = P(13); void* ws = P(14);
      size_t z = Z(15); void* st = STREAM(16), s, pg, q, K, V, Kp, fc, kn, vn, nc, bu, S, T, O, ws, z, st)
ENTRY(offload_decode_step, 16, const fasa_shape* s = SHAPE(0); void* q = P(1); void* Kp = P(2); void* fc = P(3);
      void* Kh = P(4); void* Vh = P(5); void* kn = P(6); void* vn = P(7); float* S = P(8); int32_t* T = P(9);
      float* O = P(10); void* ws = P(11); size_t z = Z(12); void* sg = P(13); size_t zs = Z(14); void* st = STREAM(15),
      s, q, Kp, fc, Kh, Vh, kn, vn, S, T, O, ws, z, sg, zs, st)
ENTRY(contextual_agreement, 8, const fasa_shape* s = SHAPE(0); void* q = P(1); void* Kp = P(2); int32_t k = I(3);
      float* ca = P(4); void* ws = P(5); size_t z = Z(6); void* st = STREAM(7), s, q, Kp, k, ca, ws, z, st)

/* bind(library path, address function, current device function, raw stream function, shape type, paging type, refusal) */
static PyObject* py_bind(PyObject* self, PyObject* args) {
  (void)self;
  const char* path;
  PyObject *adr, *dev, *raw, *shape, *paging, *refuse;
  if (!PyArg_ParseTuple(args, "sOOOO!O!O", &path, &adr, &dev, &raw, &PyType_Type, &shape, &PyType_Type, &paging, &refuse))
    return NULL;
  void* h = dlopen(path, RTLD_NOW); /* the copy that is loaded already */
  if (!h) { PyErr_SetString(PyExc_ImportError, dlerror()); return NULL; }
#define BIND(name)                                                                             \
  if (!(p_##name = (__typeof__(&fasa_##name))dlsym(h, "fasa_" #name))) {                       \
    PyErr_SetString(PyExc_ImportError, "fasa_" #name " is not in the library");                \
    return NULL;                                                                               \
  }
  BIND(pack_kcache) BIND(score) BIND(topk) BIND(sparse_attend) BIND(dense_attend) BIND(decode_step)
  BIND(decode_step_static) BIND(decode_step_ragged) BIND(pack_kcache_paged) BIND(decode_step_paged)
  BIND(offload_decode_step) BIND(contextual_agreement)
  Py_INCREF(adr); Py_INCREF(dev); Py_INCREF(raw); Py_INCREF(shape); Py_INCREF(paging); Py_INCREF(refuse);
  Py_XSETREF(f_address, adr);
  Py_XSETREF(f_device, dev);
  Py_XSETREF(f_raw_stream, raw);
  Py_XSETREF(t_shape, shape);
  Py_XSETREF(t_paging, paging);
  Py_XSETREF(f_refuse, refuse);
  Py_RETURN_NONE;
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {
    {"bind", py_bind, METH_VARARGS, NULL},
    METHOD(pack_kcache), METHOD(score), METHOD(topk), METHOD(sparse_attend), METHOD(dense_attend),
    METHOD(decode_step), METHOD(decode_step_static), METHOD(decode_step_ragged), METHOD(pack_kcache_paged),
    METHOD(decode_step_paged), METHOD(offload_decode_step), METHOD(contextual_agreement),
    {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__pycall(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!s_data_ptr || !s_cuda_stream) return NULL;
  return PyModule_Create(&module);
}
