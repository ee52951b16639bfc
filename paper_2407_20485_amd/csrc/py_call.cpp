// Argument marshalling of the calls that a serving loop makes: pointers of torch tensors, the cache struct, the
// current stream, and the C entry point, in one C function per call.  A generation step of a few heads takes
// the GPU 7 us and a launch takes the host 2.8, so what the interpreter spends around it counts: 32 heads x 205 slots,
// binding.py's call through ctypes 5.9 us, here 4.1.
//
// Only the plain case is taken: torch.Tensor itself or None for a pointer, int and float themselves for numbers,
// binding.Cache itself for the cache.  Anything else (subclasses, addresses, structs, numpy numbers, values that do not fit)
// returns -1 before anything is done, and binding.py goes through ctypes, whose conversions and errors then apply.
#include <Python.h>

#include <exception>

#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include "../../include/a2sf.h"

namespace {

PyObject *g_cache_type, *g_f32, *g_bf16, *g_raw_stream, *g_get_device;  // set once, by init
PyObject *n_k, *n_v, *n_scores, *n_pos, *n_len, *n_G, *n_capacity, *n_d, *n_dtype;

// Each reader: true if `x` is of the plain kind.
bool tensor(PyObject* x, const at::Tensor** t) {
  if (!THPVariable_CheckExact(x)) return false;
  *t = &THPVariable_Unpack(x);
  return true;
}
bool pointer(PyObject* x, void** p) {
  const at::Tensor* t;
  if (x == Py_None) { *p = nullptr; return true; }
  if (!tensor(x, &t)) return false;
  *p = t->data_ptr();  // (throws for a tensor without storage)
  return true;
}
bool number(PyObject* x, int32_t* v) {
  if (!PyLong_CheckExact(x)) return false;
  int over = 0;
  const long long l = PyLong_AsLongLongAndOverflow(x, &over);
  *v = (int32_t)l;
  return !over && l == *v;
}
bool number(PyObject* x, float* v) {
  if (!PyFloat_CheckExact(x)) return false;
  *v = (float)PyFloat_AS_DOUBLE(x);
  return true;
}
struct Owned {  // a new reference, given back
  PyObject* p;
  ~Owned() { Py_XDECREF(p); }
};
template <typename F>
bool attribute(PyObject* x, PyObject* name, F read) {
  const Owned a{PyObject_GetAttr(x, name)};
  if (!a.p) { PyErr_Clear(); return false; }
  return read(a.p);
}
bool cache_struct(PyObject* x, a2sf_cache* c) {
  if ((PyObject*)Py_TYPE(x) != g_cache_type) return false;
  const auto data = [&](PyObject* name, void** p) {
    return attribute(x, name, [&](PyObject* a) { return a != Py_None && pointer(a, p); });
  };
  const auto field = [&](PyObject* name, int32_t* v) { return attribute(x, name, [&](PyObject* a) { return number(a, v); }); };
  return data(n_k, &c->k) && data(n_v, &c->v) && data(n_scores, (void**)&c->scores) && data(n_pos, (void**)&c->pos) &&
         data(n_len, (void**)&c->len) && field(n_G, &c->G) && field(n_capacity, &c->capacity) && field(n_d, &c->d) &&
         attribute(x, n_dtype, [&](PyObject* a) {
           c->dtype = a == g_f32 ? A2SF_F32 : A2SF_BF16;
           return a == g_f32 || a == g_bf16;
         });
}
bool workspace(PyObject* x, PyObject* bytes, void** p, size_t* n) {
  const at::Tensor* t = nullptr;
  if (x != Py_None && !tensor(x, &t)) return false;
  *p = t ? t->data_ptr() : nullptr;
  if (bytes == Py_None) {
    *n = t ? t->nbytes() : 0;
    return true;
  }
  if (!PyLong_CheckExact(bytes)) return false;
  int over = 0;
  const long long l = PyLong_AsLongLongAndOverflow(bytes, &over);
  *n = (size_t)l;
  return !over && l >= 0;
}
// torch's current stream of the current device; `any` is an argument of the call: with a tensor on the GPU torch is initialised
bool stream(PyObject* x, PyObject* any, void** st) {
  const at::Tensor* t;
  if (x != Py_None || !g_raw_stream || !tensor(any, &t) || !t->is_cuda()) return false;
  const Owned dev{PyObject_CallNoArgs(g_get_device)};
  const Owned raw{dev.p ? PyObject_CallOneArg(g_raw_stream, dev.p) : nullptr};
  if (!raw.p) { PyErr_Clear(); return false; }
  *st = PyLong_AsVoidPtr(raw.p);
  return true;
}

// Runs the body of a call; C++ exceptions (a tensor without storage) become Python's.
template <typename F>
PyObject* guarded(F body) {
  try {
    const int status = body();
    return PyErr_Occurred() ? nullptr : PyLong_FromLong(status);
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}
template <typename F>
int without_gil(F call) {
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = call();
  Py_END_ALLOW_THREADS
  return status;
}
bool expects(Py_ssize_t got, Py_ssize_t want) {
  if (got != want) PyErr_Format(PyExc_TypeError, "%zd arguments, not %zd", want, got);
  return got == want;
}

// (entry point, q, k_new, v_new, t_pos, cache, group or None, alpha, select, recent, o, mode, workspace, workspace_bytes, stream)
PyObject* decode_step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!expects(n, 15)) return nullptr;
  return guarded([&] {
    void *q, *k, *v, *o, *ws, *st, *fn = PyLong_AsVoidPtr(a[0]);
    int32_t t_pos, group = 1, mode;
    a2sf_budget b;
    float alpha;
    size_t bytes;
    a2sf_cache c;
    if (!(fn && pointer(a[1], &q) && pointer(a[2], &k) && pointer(a[3], &v) && number(a[4], &t_pos) && cache_struct(a[5], &c) &&
          (a[6] == Py_None || number(a[6], &group)) && number(a[7], &alpha) && number(a[8], &b.select) &&
          number(a[9], &b.recent) && pointer(a[10], &o) && number(a[11], &mode) && workspace(a[12], a[13], &ws, &bytes) &&
          stream(a[14], a[1], &st)))
      return -1;
    return without_gil([&]() -> int {
      if (a[6] == Py_None) return ((decltype(&a2sf_decode_step))fn)(q, k, v, t_pos, &c, alpha, b, mode, o, ws, bytes, st);
      return ((decltype(&a2sf_decode_step_gqa))fn)(q, k, v, t_pos, &c, group, alpha, b, mode, o, ws, bytes, st);
    });
  });
}

// (entry point, q, k, v, n, group or None, alpha, select, recent, cache, o, scores_full, workspace, workspace_bytes, stream)
PyObject* prefill(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!expects(n, 15)) return nullptr;
  return guarded([&] {
    void *q, *k, *v, *o, *full, *ws, *st, *fn = PyLong_AsVoidPtr(a[0]);
    int32_t rows, group = 1;
    a2sf_budget b;
    float alpha;
    size_t bytes;
    a2sf_cache c;
    if (!(fn && pointer(a[1], &q) && pointer(a[2], &k) && pointer(a[3], &v) && number(a[4], &rows) &&
          (a[5] == Py_None || number(a[5], &group)) && number(a[6], &alpha) && number(a[7], &b.select) &&
          number(a[8], &b.recent) && cache_struct(a[9], &c) && pointer(a[10], &o) && pointer(a[11], &full) &&
          workspace(a[12], a[13], &ws, &bytes) && stream(a[14], a[1], &st)))
      return -1;
    return without_gil([&]() -> int {
      if (a[5] == Py_None) return ((decltype(&a2sf_prefill))fn)(q, k, v, rows, alpha, b, &c, o, (float*)full, ws, bytes, st);
      return ((decltype(&a2sf_prefill_gqa))fn)(q, k, v, rows, group, alpha, b, &c, o, (float*)full, ws, bytes, st);
    });
  });
}

// (entry point, q, k, v, m, pos0, group or None, alpha, select, recent, cache, o, workspace, workspace_bytes, stream)
PyObject* prefill_chunk(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!expects(n, 15)) return nullptr;
  return guarded([&] {
    void *q, *k, *v, *o, *ws, *st, *fn = PyLong_AsVoidPtr(a[0]);
    int32_t m, pos0, group = 1;
    a2sf_budget b;
    float alpha;
    size_t bytes;
    a2sf_cache c;
    if (!(fn && pointer(a[1], &q) && pointer(a[2], &k) && pointer(a[3], &v) && number(a[4], &m) && number(a[5], &pos0) &&
          (a[6] == Py_None || number(a[6], &group)) && number(a[7], &alpha) && number(a[8], &b.select) &&
          number(a[9], &b.recent) && cache_struct(a[10], &c) && pointer(a[11], &o) && workspace(a[12], a[13], &ws, &bytes) &&
          stream(a[14], a[1], &st)))
      return -1;
    return without_gil([&]() -> int {
      if (a[6] == Py_None) return ((decltype(&a2sf_prefill_chunk))fn)(q, k, v, m, pos0, alpha, b, &c, o, ws, bytes, st);
      return ((decltype(&a2sf_prefill_chunk_gqa))fn)(q, k, v, m, pos0, group, alpha, b, &c, o, ws, bytes, st);
    });
  });
}

// (binding.Cache, torch.float32, torch.bfloat16, function device -> current raw stream or None, function -> current device)
PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!expects(n, 5)) return nullptr;
  PyObject** const to[] = {&g_cache_type, &g_f32, &g_bf16, &g_raw_stream, &g_get_device};
  for (int i = 0; i < 5; ++i) {
    Py_XDECREF(*to[i]);
    *to[i] = a[i] == Py_None ? nullptr : a[i];
    Py_XINCREF(*to[i]);
  }
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"init", (PyCFunction)(void (*)())init, METH_FASTCALL, nullptr},
                         {"decode_step", (PyCFunction)(void (*)())decode_step, METH_FASTCALL, nullptr},
                         {"prefill", (PyCFunction)(void (*)())prefill, METH_FASTCALL, nullptr},
                         {"prefill_chunk", (PyCFunction)(void (*)())prefill_chunk, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

#define A2SF_STR_(x) #x
#define A2SF_STR(x) A2SF_STR_(x)
PyMODINIT_FUNC PyInit__call() {
  PyObject** const names[] = {&n_k, &n_v, &n_scores, &n_pos, &n_len, &n_G, &n_capacity, &n_d, &n_dtype};
  const char* const text[] = {"k", "v", "scores", "pos", "len", "G", "capacity", "d", "dtype"};
  for (int i = 0; i < 9; ++i)
    if (!*names[i] && !(*names[i] = PyUnicode_InternFromString(text[i]))) return nullptr;
  PyObject* m = PyModule_Create(&module);
  // (binding.py does without the extension where these are not the ones that run)
  const char* const built_for = "torch " TORCH_VERSION ", Python " A2SF_STR(PY_MAJOR_VERSION) "." A2SF_STR(PY_MINOR_VERSION);
  if (m && PyModule_AddStringConstant(m, "built_for", built_for) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
