/* The two calls of a decode step without the interpreter between the checks: the same checks of every tensor that
 * binding._ptr makes (that it is one, type, place, contiguity, size), made through the tensor's own attributes, and the call itself.  A
 * check that fails, or an argument of an unexpected kind, returns None: the caller then takes the Python path, which
 * says what is wrong.  Nothing is kept between calls but the names, the types and the two entry points. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "../../include/kvr.h"

typedef int32_t (*step_fn)(const kvr_desc*, const void*, const void*, const int32_t*, void*, void*, int32_t*, int32_t,
                           const float*, int64_t, int32_t, int32_t, int32_t*, int32_t*, int32_t*, int32_t, int32_t*,
                           int32_t*, int32_t, void*, void*, void*);
typedef int32_t (*attend_fn)(const kvr_desc*, const void*, const void*, const void*, const int32_t*, int32_t,
                             const void*, const void*, const int32_t*, const int32_t*, int32_t, float*, float*, int64_t,
                             void*, size_t, const kvr_attend_opts*, void*);

static PyObject *n_dtype, *n_is_cuda, *n_is_contiguous, *n_numel, *n_data_ptr;
static PyObject *t_f32, *t_bf16, *t_i32, *t_u8, *t_tensor;
static step_fn f_step;
static attend_fn f_attend;

static int integer(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return 0;
  *v = PyLong_AsLongLong(o);
  return !(*v == -1 && PyErr_Occurred());
}

static int asked(PyObject* t, PyObject* name, int64_t* v) {          /* an integer method without arguments */
  PyObject* r = PyObject_CallMethodNoArgs(t, name);
  const int ok = r && integer(r, v);
  Py_XDECREF(r);
  return ok;
}

static int truth(PyObject* r) {
  const int yes = r == Py_True;
  Py_XDECREF(r);
  return yes;
}

/* device address of a contiguous tensor of that type with at least `need` elements; numel may be null */
static int tensor(PyObject* t, PyObject* dtype, int64_t need, int none_ok, void** p, int64_t* numel) {
  int64_t n, a;
  *p = NULL;
  if (t == Py_None) return none_ok;
  if (PyObject_IsInstance(t, t_tensor) != 1) return 0;
  PyObject* dt = PyObject_GetAttr(t, n_dtype);
  const int same = dt == dtype;
  Py_XDECREF(dt);
  if (!same || !truth(PyObject_GetAttr(t, n_is_cuda)) || !truth(PyObject_CallMethodNoArgs(t, n_is_contiguous))) return 0;
  if (!asked(t, n_numel, &n) || n < need || !asked(t, n_data_ptr, &a)) return 0;
  *p = (void*)(uintptr_t)a;
  if (numel) *numel = n;
  return 1;
}

/* The products of sizes that the checks form stay within 64 bits: the descriptor's are what the library takes at most, every
 * count fits 32 bits.  Others go to the Python checks, whose integers have no end. */
static int sizes_fit(const kvr_desc* d, const int64_t* count, int n) {
  const int64_t U = (int64_t)d->batch * d->n_kv_heads, H = (int64_t)d->batch * d->n_q_heads;
  if (U > 65535 || H > 8 * 65535 || d->head_dim != KVR_HEAD_DIM || d->r > KVR_MAX_ROWS || d->w > 65536) return 0;
  for (int i = 0; i < n; ++i)
    if (count[i] != (int32_t)count[i]) return 0;
  return 1;
}

static PyObject* refuse(void) {
  PyErr_Clear();
  Py_RETURN_NONE;
}

static PyObject* setup(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  int64_t s, t;
  if (n != 7 || !integer(a[0], &s) || !integer(a[1], &t)) return PyErr_Format(PyExc_TypeError, "setup");
  f_step = (step_fn)(uintptr_t)s;
  f_attend = (attend_fn)(uintptr_t)t;
  for (int i = 2; i < 7; ++i) Py_INCREF(a[i]);
  t_f32 = a[2]; t_bf16 = a[3]; t_i32 = a[4]; t_u8 = a[5]; t_tensor = a[6];
  Py_RETURN_NONE;
}

/* desc address, stream, then the arguments of binding.kvr_step_update behind desc */
static PyObject* step_update(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  int64_t da, st, ret_cap, n_cap, n_recent, k_cand, evict_cap, vague_cap;
  void *kn, *vn, *nc, *kr, *vr, *rp, *sc, *es, *ep, *ne, *vp, *nv, *sk, *sv;
  if (n != 22 || !f_step || !integer(a[0], &da) || !integer(a[1], &st) || !integer(a[8], &ret_cap) || !integer(a[10], &n_cap) ||
      !integer(a[11], &n_recent) || !integer(a[12], &k_cand) || !integer(a[16], &evict_cap) || !integer(a[19], &vague_cap))
    return refuse();
  const kvr_desc* d = (const kvr_desc*)(uintptr_t)da;
  if (!sizes_fit(d, (int64_t[]){ret_cap, n_cap, n_recent, k_cand, evict_cap, vague_cap}, 6)) return refuse();
  PyObject* dt = d->dtype == KVR_F32 ? t_f32 : t_bf16;
  const int64_t U = (int64_t)d->batch * d->n_kv_heads, D = d->head_dim, S = (int64_t)d->r * d->w * D;
  if (!tensor(a[2], dt, U * D, 0, &kn, 0) || !tensor(a[3], dt, U * D, 0, &vn, 0) || !tensor(a[4], t_i32, d->batch, 0, &nc, 0) ||
      !tensor(a[5], dt, U * ret_cap * D, 0, &kr, 0) || !tensor(a[6], dt, U * ret_cap * D, 0, &vr, 0) ||
      !tensor(a[7], t_i32, U * ret_cap, 0, &rp, 0) || !tensor(a[9], t_f32, U * n_cap, 0, &sc, 0) ||
      !tensor(a[13], t_i32, U * evict_cap, 0, &es, 0) || !tensor(a[14], t_i32, U * evict_cap, 0, &ep, 0) ||
      !tensor(a[15], t_i32, U, 0, &ne, 0) || !tensor(a[17], t_i32, U * vague_cap, 1, &vp, 0) || !tensor(a[18], t_i32, U, 1, &nv, 0) ||
      !tensor(a[20], dt, U * S, 0, &sk, 0) || !tensor(a[21], dt, U * S, 0, &sv, 0))
    return refuse();
  int32_t rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f_step(d, kn, vn, nc, kr, vr, rp, (int32_t)ret_cap, sc, n_cap, (int32_t)n_recent, (int32_t)k_cand, es, ep, ne,
              (int32_t)evict_cap, vp, nv, (int32_t)vague_cap, sk, sv, (void*)(uintptr_t)st);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

/* desc address, stream, address of the options (0: none), then the arguments of binding.kvr_attend_decode from q to ws */
static PyObject* attend_decode(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  int64_t da, st, op, ret_cap, n_cap, vague_cap, wb = 0;
  void *q, *kr, *vr, *rp, *sk, *sv, *vp, *nv, *out, *sc, *ws;
  if (n != 17 || !f_attend || !integer(a[0], &da) || !integer(a[1], &st) || !integer(a[2], &op) || !integer(a[7], &ret_cap) ||
      !integer(a[12], &vague_cap) || !integer(a[15], &n_cap))
    return refuse();
  const kvr_desc* d = (const kvr_desc*)(uintptr_t)da;
  if (!sizes_fit(d, (int64_t[]){ret_cap, vague_cap, n_cap}, 3)) return refuse();
  PyObject* dt = d->dtype == KVR_F32 ? t_f32 : t_bf16;
  const int64_t U = (int64_t)d->batch * d->n_kv_heads, D = d->head_dim, S = (int64_t)d->r * d->w * D, H = (int64_t)d->batch * d->n_q_heads;
  if (!tensor(a[3], dt, H * D, 0, &q, 0) || !tensor(a[4], dt, U * ret_cap * D, 0, &kr, 0) ||
      !tensor(a[5], dt, U * ret_cap * D, 0, &vr, 0) || !tensor(a[6], t_i32, U * ret_cap, 1, &rp, 0) ||
      !tensor(a[8], dt, U * S, 1, &sk, 0) || !tensor(a[9], dt, U * S, 1, &sv, 0) || !tensor(a[10], t_i32, U * vague_cap, 1, &vp, 0) ||
      !tensor(a[11], t_i32, U, 1, &nv, 0) || !tensor(a[13], t_f32, H * D, 0, &out, 0) || !tensor(a[14], t_f32, U * n_cap, 1, &sc, 0) ||
      !tensor(a[16], t_u8, 0, 0, &ws, &wb))
    return refuse();
  int32_t rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f_attend(d, q, kr, vr, rp, (int32_t)ret_cap, sk, sv, vp, nv, (int32_t)vague_cap, out, sc, n_cap, ws, (size_t)wb,
                (const kvr_attend_opts*)(uintptr_t)op, (void*)(uintptr_t)st);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

static PyMethodDef methods[] = {{"setup", (PyCFunction)(void*)setup, METH_FASTCALL, 0},
                                {"step_update", (PyCFunction)(void*)step_update, METH_FASTCALL, 0},
                                {"attend_decode", (PyCFunction)(void*)attend_decode, METH_FASTCALL, 0},
                                {0, 0, 0, 0}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_kvr_fast", 0, -1, methods, 0, 0, 0, 0};

PyMODINIT_FUNC PyInit__kvr_fast(void) {
  n_dtype = PyUnicode_InternFromString("dtype");
  n_is_cuda = PyUnicode_InternFromString("is_cuda");
  n_is_contiguous = PyUnicode_InternFromString("is_contiguous");
  n_numel = PyUnicode_InternFromString("numel");
  n_data_ptr = PyUnicode_InternFromString("data_ptr");
  return PyModule_Create(&module);
}
