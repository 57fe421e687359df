// Python calls of the two decisions (block_boundary, select_parallel of dlm.h) without ctypes.  Their kernels take a few microseconds,
// so a call is bound by what marshalling its arguments costs the host: 2.7 and 4.8 us through ctypes with packed arrays, 1.2 and 2.1 here.
// Only plain arguments are taken: lists or tuples of ints that fit 32 bits, each at least as long as the first, numbers, tensors.
// Anything else returns None before anything is launched, and the caller goes the ctypes way, which takes every other form that has
// enough entries and refuses the rest.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "../../include/dlm.h"

#define MAX_SEQS 32

static int (*g_boundary)(const float*, const float*, const int32_t*, const int32_t*, const int32_t*, int, const dlm_boundary_params*, int32_t*, float*,
                         float*, void*);
static int (*g_select)(const void*, int, int, const float*, const float*, const int32_t*, int32_t*, const int32_t*, const int32_t*, const int32_t*, int,
                       int, const dlm_select_params*, int, uint8_t*, int32_t*, float*, void*);
static PyObject *g_f32, *g_bf16, *s_data_ptr, *s_size, *s_dtype, *g_minus_one;

// Each returns 0 for an argument that is not plain (with no error set).
static int to_int(PyObject* o, int32_t* out) {
  int overflow;
  if (!PyLong_Check(o)) return 0;
  const long v = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow || v < INT32_MIN || v > INT32_MAX) return 0;
  *out = (int32_t)v;
  return 1;
}
static int to_float(PyObject* o, float* out) {
  if (!PyFloat_CheckExact(o)) return 0;
  const double v = PyFloat_AS_DOUBLE(o);
  *out = (float)v;
  return (*out - *out == 0.f) || v - v != 0.;  // (a finite value that overflows is the other way's error)
}
static int to_ptr(PyObject* o, void** out) {  // a tensor, or None
  if (o == Py_None) {
    *out = NULL;
    return 1;
  }
  PyObject* r = PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (!r) {
    PyErr_Clear();
    return 0;
  }
  *out = PyLong_Check(r) ? PyLong_AsVoidPtr(r) : NULL;
  const int ok = PyLong_Check(r) && !PyErr_Occurred();
  Py_DECREF(r);
  PyErr_Clear();
  return ok;
}
// an array of at least n entries (n < 0: as many as there are); -1: not plain, else its first n entries and their number
static int to_ints(PyObject* o, int n, int32_t* out) {
  PyObject** item;
  Py_ssize_t len;
  if (PyList_CheckExact(o)) {
    item = ((PyListObject*)o)->ob_item;
    len = PyList_GET_SIZE(o);
  } else if (PyTuple_CheckExact(o)) {
    item = ((PyTupleObject*)o)->ob_item;
    len = PyTuple_GET_SIZE(o);
  } else {
    return -1;
  }
  if (n < 0) n = len <= MAX_SEQS ? (int)len : -1;
  if (n < 0 || len < n) return -1;
  for (int i = 0; i < n; ++i)
    if (!to_int(item[i], out + i)) return -1;
  return n;
}

// boundary(I, H, win_start, win_len, cold, L_out, S_out, margin_out, lam, l_min, smooth_radius, norm_mode, rule, stream) -> status or None
static PyObject* boundary(PyObject* self, PyObject* const* a, Py_ssize_t n_args) {
  int32_t start[MAX_SEQS], len[MAX_SEQS], cold[MAX_SEQS];
  void *I, *H, *L, *S, *margin;
  dlm_boundary_params p;
  if (n_args != 14 || !g_boundary) Py_RETURN_NONE;
  const int n = to_ints(a[2], -1, start);
  if (n < 0 || to_ints(a[3], n, len) < 0 || (a[4] != Py_None && to_ints(a[4], n, cold) < 0)) Py_RETURN_NONE;
  if (!to_float(a[8], &p.lambda) || !to_int(a[9], &p.l_min) || !to_int(a[10], &p.smooth_radius) || !to_int(a[11], &p.norm_mode) || !to_int(a[12], &p.rule))
    Py_RETURN_NONE;
  if (!to_ptr(a[0], &I) || !to_ptr(a[1], &H) || !to_ptr(a[5], &L) || !to_ptr(a[6], &S) || !to_ptr(a[7], &margin)) Py_RETURN_NONE;
  void* stream = PyLong_AsVoidPtr(a[13]);
  if (PyErr_Occurred()) return NULL;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_boundary((const float*)I, (const float*)H, start, len, a[4] == Py_None ? NULL : cold, n, &p, (int32_t*)L, (float*)S, (float*)margin, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// select(logits, lse, conf, argmax, tokens, row_start, tok_start, block_len, mask_id, tau_low, tau_high, gamma, mode, selected_out,
//        n_selected_out, apply_tokens, margin_out, stream) -> status or None
static PyObject* select_(PyObject* self, PyObject* const* a, Py_ssize_t n_args) {
  int32_t row[MAX_SEQS], tok[MAX_SEQS], len[MAX_SEQS], mask_id, vocab, apply;
  void *z, *lse, *conf, *argmax, *tokens, *sel, *nsel, *margin;
  dlm_select_params p;
  if (n_args != 18 || !g_select) Py_RETURN_NONE;
  const int n = to_ints(a[5], -1, row);
  if (n < 0 || to_ints(a[6], n, tok) < 0 || to_ints(a[7], n, len) < 0 || !to_int(a[8], &mask_id) || !to_int(a[15], &apply)) Py_RETURN_NONE;
  if (!to_float(a[9], &p.tau_low) || !to_float(a[10], &p.tau_high) || !to_float(a[11], &p.gamma) || !to_int(a[12], &p.mode)) Py_RETURN_NONE;
  if (a[0] == Py_None || !to_ptr(a[0], &z) || !to_ptr(a[1], &lse) || !to_ptr(a[2], &conf) || !to_ptr(a[3], &argmax) || !to_ptr(a[4], &tokens) ||
      !to_ptr(a[13], &sel) || !to_ptr(a[14], &nsel) || !to_ptr(a[16], &margin))
    Py_RETURN_NONE;
  PyObject* dtype = PyObject_GetAttr(a[0], s_dtype);
  PyObject* cols = dtype ? PyObject_CallMethodOneArg(a[0], s_size, g_minus_one) : NULL;
  const int code = dtype == g_bf16 ? DLM_BF16 : dtype == g_f32 ? DLM_F32 : -1;
  const int ok = cols && code >= 0 && to_int(cols, &vocab);
  Py_XDECREF(dtype);
  Py_XDECREF(cols);
  if (!ok) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  void* stream = PyLong_AsVoidPtr(a[17]);
  if (PyErr_Occurred()) return NULL;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_select(z, vocab, code, (const float*)lse, (const float*)conf, (const int32_t*)argmax, (int32_t*)tokens, row, tok, len, n, mask_id, &p, apply,
                (uint8_t*)sel, (int32_t*)nsel, (float*)margin, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// bind(address of block_boundary, address of select_parallel, torch.float32, torch.bfloat16)
static PyObject* bind(PyObject* self, PyObject* const* a, Py_ssize_t n_args) {
  if (n_args != 4) {
    PyErr_SetString(PyExc_TypeError, "bind takes four arguments");
    return NULL;
  }
  void *b = PyLong_AsVoidPtr(a[0]), *s = PyLong_AsVoidPtr(a[1]);
  if (PyErr_Occurred()) return NULL;
  *(void**)&g_boundary = b;
  *(void**)&g_select = s;
  Py_INCREF(a[2]);
  Py_INCREF(a[3]);
  Py_XSETREF(g_f32, a[2]);
  Py_XSETREF(g_bf16, a[3]);
  Py_RETURN_NONE;
}

static PyMethodDef methods[] = {{"boundary", (PyCFunction)(void (*)(void))boundary, METH_FASTCALL, "block_boundary"},
                                {"select", (PyCFunction)(void (*)(void))select_, METH_FASTCALL, "select_parallel"},
                                {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, "the library's entry points and torch's types"},
                                {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_decisions", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__decisions(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_size = PyUnicode_InternFromString("size");
  s_dtype = PyUnicode_InternFromString("dtype");
  g_minus_one = PyLong_FromLong(-1);
  if (!s_data_ptr || !s_size || !s_dtype || !g_minus_one) return NULL;
  return PyModule_Create(&module);
}
