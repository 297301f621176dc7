// Calls of the C ABI from Python without ctypes: the module _kvt_call.
//
// A small call (a decoding step of one agent, a short message) is bound by
// the host: building the ctypes structs and arrays of one call and handing
// its arguments over took about as long as the launches themselves.  These
// functions take plain integers (addresses and sizes that the Python side has
// checked), build the structs on the C stack and call the entry point, whose
// address the Python side passes, with the GIL released, as ctypes does.
// Smallest turn of the package's workloads (append + extend): 24.5 us of host
// time per pass with ctypes, 14.4 us with this module (the binding also asks torch
// for the raw stream handle instead of a stream object).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>
#include <string.h>

#include "kvt.h"

namespace {

// One length array, copied when it is taken: `convert` of the next one may run
// Python code that changes this one.  A list or tuple of Python ints or a
// contiguous int32 buffer is read directly, anything else through `convert`.
struct Lengths {
  int32_t* values = nullptr;
  Py_ssize_t n = 0;
  ~Lengths() { PyMem_Free(values); }
  bool take(PyObject* x, PyObject* convert) {
    int got = load(x);
    if (got != 0) return got > 0;
    PyObject* a = PyObject_CallOneArg(convert, x);
    if (a == nullptr) return false;
    got = load(a);
    Py_DECREF(a);
    if (got == 0) PyErr_SetString(PyExc_TypeError, "lengths must convert to int32 arrays");
    return got > 0;
  }

 private:
  bool room(Py_ssize_t count) {
    n = count;
    values = static_cast<int32_t*>(PyMem_Malloc(count > 0 ? (size_t)count * sizeof(int32_t) : 1));
    if (values == nullptr) PyErr_NoMemory();
    return values != nullptr;
  }
  // 1: taken; 0: neither a list of ints nor an int32 buffer; -1: exception
  // set.  No Python code runs between a look at x and the copy of its values.
  int load(PyObject* x) {
    if (PyList_CheckExact(x) || PyTuple_CheckExact(x)) {
      const Py_ssize_t count = PySequence_Fast_GET_SIZE(x);
      for (Py_ssize_t i = 0; i < count; ++i)
        if (!PyLong_CheckExact(PySequence_Fast_GET_ITEM(x, i))) return 0;
      if (!room(count)) return -1;
      for (Py_ssize_t i = 0; i < count; ++i) {
        int over = 0;
        const long v = PyLong_AsLongAndOverflow(PySequence_Fast_GET_ITEM(x, i), &over);
        if (v == -1 && PyErr_Occurred()) return -1;
        if (over != 0 || v < INT32_MIN || v > INT32_MAX) {
          PyErr_SetString(PyExc_OverflowError, "length or block id outside the int32 range");
          return -1;
        }
        values[i] = (int32_t)v;
      }
      return 1;
    }
    Py_buffer view;
    if (!PyObject_CheckBuffer(x)) return 0;
    if (PyObject_GetBuffer(x, &view, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) {
      PyErr_Clear();
      return 0;
    }
    const char* f = view.format;
    if (f != nullptr && (f[0] == '<' || f[0] == '=' || f[0] == '@')) ++f;
    int got = 0;
    if (f != nullptr && f[0] == 'i' && f[1] == 0 && view.itemsize == 4) {
      got = room(view.len / 4) ? 1 : -1;
      if (got == 1 && n > 0) memcpy(values, view.buf, (size_t)n * sizeof(int32_t));
    }
    PyBuffer_Release(&view);
    return got;
  }
};

// pack(prefix, suffix or None, convert) -> (bytes, tokens): prefix_len then
// suffix_len as int32, and the sum of suffix_len (None: one new token each).
PyObject* pack(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != 3) {
    PyErr_SetString(PyExc_TypeError, "pack(prefix, suffix, convert)");
    return nullptr;
  }
  Lengths p, s;
  if (!p.take(args[0], args[2])) return nullptr;
  const bool ones = args[1] == Py_None;
  if (!ones && !s.take(args[1], args[2])) return nullptr;
  if (!ones && s.n < p.n) {
    PyErr_SetString(PyExc_ValueError, "fewer suffix lengths than prefix lengths");
    return nullptr;
  }
  const Py_ssize_t ns = ones ? p.n : s.n;
  PyObject* out = PyBytes_FromStringAndSize(nullptr, (p.n + ns) * 4);
  if (out == nullptr) return nullptr;
  int32_t* d = reinterpret_cast<int32_t*>(PyBytes_AS_STRING(out));
  if (p.n > 0) memcpy(d, p.values, (size_t)p.n * sizeof(int32_t));
  if (!ones && ns > 0) memcpy(d + p.n, s.values, (size_t)ns * sizeof(int32_t));
  for (Py_ssize_t i = 0; ones && i < ns; ++i) d[p.n + i] = 1;
  long long total = 0;
  for (Py_ssize_t i = 0; i < ns; ++i) total += d[p.n + i];
  return Py_BuildValue("(NnL)", out, p.n, total);
}

// The arguments every call starts with: entry point, the pool (k, v, blocks,
// kv-heads, head_dim, dtype), the packed lengths and their count, the block
// table (device address, columns) and its host copy (an int32 buffer or None).
constexpr Py_ssize_t kHead = 12;
struct Head {
  void* fn;
  kvt_pool pool;
  kvt_seqs seqs;
  Py_buffer host;
  bool has_host = false;
  ~Head() {
    if (has_host) PyBuffer_Release(&host);
  }
};

bool integer(PyObject* o, long long* v) {
  *v = PyLong_AsLongLong(o);
  return !(*v == -1 && PyErr_Occurred());
}
bool address(PyObject* o, void** v) {
  if (o == Py_None) {
    *v = nullptr;
    return true;
  }
  *v = PyLong_AsVoidPtr(o);
  return !(*v == nullptr && PyErr_Occurred());
}
bool int32(PyObject* o, int32_t* v) {
  long long x;
  if (!integer(o, &x)) return false;
  if (x < INT32_MIN || x > INT32_MAX) {
    PyErr_SetString(PyExc_OverflowError, "argument outside the int32 range");
    return false;
  }
  *v = (int32_t)x;
  return true;
}

bool head(PyObject* const* a, Head* h) {
  long long nb, n;
  void* table;
  if (!address(a[0], &h->fn) || !address(a[1], &h->pool.k) || !address(a[2], &h->pool.v) || !integer(a[3], &nb) ||
      !int32(a[4], &h->pool.num_kv_heads) || !int32(a[5], &h->pool.head_dim) || !int32(a[6], &h->pool.dtype) ||
      !integer(a[8], &n) || !address(a[9], &table) || !int32(a[10], &h->seqs.max_blocks))
    return false;
  h->pool.num_blocks = nb;
  if (h->fn == nullptr || !PyBytes_CheckExact(a[7]) || n < 0 || n > INT32_MAX ||
      PyBytes_GET_SIZE(a[7]) < (Py_ssize_t)(2 * n * 4)) {
    PyErr_SetString(PyExc_TypeError, "bad entry point or packed lengths");
    return false;
  }
  const int32_t* d = reinterpret_cast<const int32_t*>(PyBytes_AS_STRING(a[7]));
  h->seqs.num_seqs = (int32_t)n;
  h->seqs.prefix_len = d;
  h->seqs.suffix_len = d + n;
  h->seqs.block_table = reinterpret_cast<const int32_t*>(table);
  h->seqs.block_table_host = nullptr;
  if (a[11] != Py_None) {
    if (PyObject_GetBuffer(a[11], &h->host, PyBUF_C_CONTIGUOUS) != 0) return false;
    h->has_host = true;
    if (h->host.itemsize != 4 || (long long)(h->host.len / 4) < n * (long long)h->seqs.max_blocks) {
      PyErr_SetString(PyExc_ValueError, "the block table's host copy is too small");
      return false;
    }
    h->seqs.block_table_host = reinterpret_cast<const int32_t*>(h->host.buf);
  }
  return true;
}

bool count_is(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
  return false;
}

// append(head..., k_new, v_new, stream) -> status
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Head h;
  void *kn, *vn, *stream;
  if (!count_is(n, kHead + 3) || !head(a, &h) || !address(a[kHead], &kn) || !address(a[kHead + 1], &vn) ||
      !address(a[kHead + 2], &stream))
    return nullptr;
  kvt_status st;
  Py_BEGIN_ALLOW_THREADS
  st = reinterpret_cast<decltype(&kvt_append_kv)>(h.fn)(&h.pool, &h.seqs, kn, vn, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// workspace(head..., num_q_heads[, shared_len, mode]) -> bytes
PyObject* workspace(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Head h;
  int32_t hq, shared = 0, mode = 0;
  const bool cascade = n == kHead + 3;
  if (!(cascade || count_is(n, kHead + 1)) || !head(a, &h) || !int32(a[kHead], &hq)) return nullptr;
  if (cascade && (!int32(a[kHead + 1], &shared) || !int32(a[kHead + 2], &mode))) return nullptr;
  size_t need;
  Py_BEGIN_ALLOW_THREADS
  need = cascade ? reinterpret_cast<decltype(&kvt_cascade_workspace_bytes_ex)>(h.fn)(&h.pool, &h.seqs, shared, mode, hq)
                 : reinterpret_cast<decltype(&kvt_extend_workspace_bytes)>(h.fn)(&h.pool, &h.seqs, hq);
  Py_END_ALLOW_THREADS
  return PyLong_FromSize_t(need);
}

// attend(head..., q, num_q_heads, scale, out, lse, workspace, workspace_bytes,
// stream[, shared_len, mode]) -> status
PyObject* attend(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Head h;
  void *q, *out, *lse, *ws, *stream;
  int32_t hq, shared = 0, mode = 0;
  long long ws_bytes;
  const bool cascade = n == kHead + 10;
  if (!(cascade || count_is(n, kHead + 8)) || !head(a, &h) || !address(a[kHead], &q) || !int32(a[kHead + 1], &hq))
    return nullptr;
  const double scale = PyFloat_AsDouble(a[kHead + 2]);
  if (scale == -1.0 && PyErr_Occurred()) return nullptr;
  if (!address(a[kHead + 3], &out) || !address(a[kHead + 4], &lse) || !address(a[kHead + 5], &ws) ||
      !integer(a[kHead + 6], &ws_bytes) || !address(a[kHead + 7], &stream))
    return nullptr;
  if (cascade && (!int32(a[kHead + 8], &shared) || !int32(a[kHead + 9], &mode))) return nullptr;
  kvt_status st;
  float* l = reinterpret_cast<float*>(lse);
  Py_BEGIN_ALLOW_THREADS
  st = cascade ? reinterpret_cast<decltype(&kvt_cascade_extend_attention_ex)>(h.fn)(
                     &h.pool, &h.seqs, shared, mode, q, hq, (float)scale, out, l, ws, (size_t)ws_bytes, stream)
               : reinterpret_cast<decltype(&kvt_extend_attention)>(h.fn)(&h.pool, &h.seqs, q, hq, (float)scale, out,
                                                                         l, ws, (size_t)ws_bytes, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

#define FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f))
PyMethodDef methods[] = {{"pack", FAST(pack), METH_FASTCALL, nullptr},
                         {"append", FAST(append), METH_FASTCALL, nullptr},
                         {"workspace", FAST(workspace), METH_FASTCALL, nullptr},
                         {"attend", FAST(attend), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_kvt_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__kvt_call(void) { return PyModule_Create(&module); }
