// Argument marshalling of the calls that a program issues for every task
// (submit, store_create, store_release, part_none, part_tiling), for the
// Python binding.  A task costs the library about 1 us; building its ctypes
// structures in Python cost three to four times that, which bounded every
// small program (pricing 1000 options, 28 tasks over as many new stores:
// 138.8 us a pass through ctypes, 48.7 us here).
//
// Each function takes the common argument forms only (lists or tuples of
// plain ints, floats and names; exact types) and returns None for anything
// else, without a call made: the binding then marshals the call through
// ctypes, whose conversions and errors stay the only ones.  As with ctypes,
// the interpreter lock is released during the call (it may compile a kernel,
// wait for the device or call back for memory).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

#include "dfx.h"

namespace {

struct Calls {
  int (*submit)(dfx_ctx*, const dfx_task*);
  int (*store_create)(dfx_ctx*, int32_t, const int64_t*, int32_t, dfx_store*);
  int (*store_release)(dfx_ctx*, dfx_store);
  int (*proj_identity)(dfx_ctx*, int32_t, dfx_proj*);
  int (*part_none)(dfx_ctx*, dfx_part*);
  int (*part_tiling)(dfx_ctx*, int32_t, const int64_t*, const int64_t*, dfx_proj, dfx_part*);
} g_call = {};
PyObject *g_ops = nullptr, *g_priv = nullptr, *g_dtypes = nullptr;   // name -> int

constexpr Py_ssize_t MAX_ARGS = 16, MAX_IMM = 8;

bool is_seq(PyObject* o) { return PyList_CheckExact(o) || PyTuple_CheckExact(o); }
Py_ssize_t seq_len(PyObject* o) { return PyList_CheckExact(o) ? PyList_GET_SIZE(o) : PyTuple_GET_SIZE(o); }
PyObject* seq_item(PyObject* o, Py_ssize_t i) {
  return PyList_CheckExact(o) ? PyList_GET_ITEM(o, i) : PyTuple_GET_ITEM(o, i);
}

// A plain int that fits, or false (no error left set).
bool int64_of(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  *v = PyLong_AsLongLongAndOverflow(o, &over);
  return over == 0;
}
bool int32_of(PyObject* o, int32_t* v) {
  int64_t w;
  if (!int64_of(o, &w) || w < INT32_MIN || w > INT32_MAX) return false;
  *v = (int32_t)w;
  return true;
}
// A plain int, or a name of `names`.
bool code_of(PyObject* o, PyObject* names, int32_t* v) {
  if (!PyUnicode_CheckExact(o)) return int32_of(o, v);
  PyObject* x = PyDict_GetItem(names, o);   // (borrowed)
  return x && int32_of(x, v);
}
bool ints_of(PyObject* o, int64_t* v, Py_ssize_t limit, Py_ssize_t* n) {
  if (!is_seq(o)) return false;
  *n = seq_len(o);
  if (*n > limit) return false;
  for (Py_ssize_t i = 0; i < *n; ++i)
    if (!int64_of(seq_item(o, i), v + i)) return false;
  return true;
}
bool ctx_of(PyObject* o, dfx_ctx** c) {
  if (!PyLong_CheckExact(o)) return false;
  *c = (dfx_ctx*)PyLong_AsVoidPtr(o);
  if (!PyErr_Occurred()) return true;
  PyErr_Clear();
  return false;
}

// submit(ctx, op, launch, args, imm) -> status
PyObject* m_submit(PyObject*, PyObject* const* a, Py_ssize_t na) {
  dfx_ctx* c;
  int32_t op;
  int64_t launch[DFX_MAX_DIM];
  dfx_arg args[MAX_ARGS];
  double imm[MAX_IMM];
  Py_ssize_t nd;
  if (na != 5 || !ctx_of(a[0], &c) || !code_of(a[1], g_ops, &op) || !ints_of(a[2], launch, DFX_MAX_DIM, &nd) ||
      !is_seq(a[3]) || !is_seq(a[4]))
    Py_RETURN_NONE;
  const Py_ssize_t n = seq_len(a[3]), ni = seq_len(a[4]);
  if (n > MAX_ARGS || ni > MAX_IMM) Py_RETURN_NONE;
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject* t = seq_item(a[3], i);
    int64_t store;
    int32_t part, priv;
    if (!is_seq(t) || seq_len(t) != 3 || !int64_of(seq_item(t, 0), &store) || !int32_of(seq_item(t, 1), &part) ||
        !code_of(seq_item(t, 2), g_priv, &priv))
      Py_RETURN_NONE;
    args[i].store = store;
    args[i].part = part;
    args[i].priv = priv;
  }
  for (Py_ssize_t i = 0; i < ni; ++i) {
    PyObject* x = seq_item(a[4], i);
    if (!PyFloat_CheckExact(x)) Py_RETURN_NONE;
    imm[i] = PyFloat_AS_DOUBLE(x);
  }
  dfx_task t;
  t.op = (uint32_t)op;
  t.ndim = (int32_t)nd;
  t.launch = launch;
  t.nargs = (int32_t)n;
  t.args = args;
  t.nimm = (int32_t)ni;
  t.imm = imm;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_call.submit(c, &t);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// store_create(ctx, shape, dtype) -> handle (positive) or status (negative)
PyObject* m_store_create(PyObject*, PyObject* const* a, Py_ssize_t na) {
  dfx_ctx* c;
  int64_t shape[DFX_MAX_DIM];
  int32_t dtype;
  Py_ssize_t nd;
  if (na != 3 || !ctx_of(a[0], &c) || !ints_of(a[1], shape, DFX_MAX_DIM, &nd) || !code_of(a[2], g_dtypes, &dtype))
    Py_RETURN_NONE;
  dfx_store out = 0;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_call.store_create(c, (int32_t)nd, shape, dtype, &out);
  Py_END_ALLOW_THREADS
  return PyLong_FromLongLong(rc ? rc : (long long)out);
}

// store_release(ctx, store) -> status
PyObject* m_store_release(PyObject*, PyObject* const* a, Py_ssize_t na) {
  dfx_ctx* c;
  int64_t s;
  if (na != 2 || !ctx_of(a[0], &c) || !int64_of(a[1], &s)) Py_RETURN_NONE;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_call.store_release(c, s);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// part_none(ctx) -> handle or status (negative)
PyObject* m_part_none(PyObject*, PyObject* const* a, Py_ssize_t na) {
  dfx_ctx* c;
  if (na != 1 || !ctx_of(a[0], &c)) Py_RETURN_NONE;
  dfx_part out = 0;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_call.part_none(c, &out);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc ? rc : out);
}

// part_tiling(ctx, tile) -> handle or status (negative): identity projection, no offset
PyObject* m_part_tiling(PyObject*, PyObject* const* a, Py_ssize_t na) {
  dfx_ctx* c;
  int64_t tile[DFX_MAX_DIM];
  const int64_t off[DFX_MAX_DIM] = {};
  Py_ssize_t nd;
  if (na != 2 || !ctx_of(a[0], &c) || !ints_of(a[1], tile, DFX_MAX_DIM, &nd)) Py_RETURN_NONE;
  dfx_proj proj = 0;
  dfx_part out = 0;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_call.proj_identity(c, (int32_t)nd, &proj);
  if (!rc) rc = g_call.part_tiling(c, (int32_t)nd, tile, off, proj, &out);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc ? rc : out);
}

// bind(addresses of the six calls, ops, priv, dtypes)
PyObject* m_bind(PyObject*, PyObject* args) {
  unsigned long long f[6];
  PyObject *ops, *priv, *dtypes;
  if (!PyArg_ParseTuple(args, "(KKKKKK)O!O!O!", f, f + 1, f + 2, f + 3, f + 4, f + 5, &PyDict_Type, &ops, &PyDict_Type,
                        &priv, &PyDict_Type, &dtypes))
    return nullptr;
  g_call.submit = (decltype(g_call.submit))(uintptr_t)f[0];
  g_call.store_create = (decltype(g_call.store_create))(uintptr_t)f[1];
  g_call.store_release = (decltype(g_call.store_release))(uintptr_t)f[2];
  g_call.proj_identity = (decltype(g_call.proj_identity))(uintptr_t)f[3];
  g_call.part_none = (decltype(g_call.part_none))(uintptr_t)f[4];
  g_call.part_tiling = (decltype(g_call.part_tiling))(uintptr_t)f[5];
  Py_INCREF(ops);
  Py_INCREF(priv);
  Py_INCREF(dtypes);
  Py_XSETREF(g_ops, ops);
  Py_XSETREF(g_priv, priv);
  Py_XSETREF(g_dtypes, dtypes);
  Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))m_##name, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {FAST(submit), FAST(store_create), FAST(store_release), FAST(part_none), FAST(part_tiling),
                           {"bind", m_bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&g_module); }
