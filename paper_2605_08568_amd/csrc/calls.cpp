// The calls of a step as functions of a CPython module (_calls): the same functions and argument order as in parse.h, without ctypes between them.
// A step of a short prompt is eight launches of 2 us, and ctypes took as long as they do: 2-3 us to convert sixteen arguments, 1-2 us for
// every parse_layer / parse_patterns built field by field.  Here an argument is converted by its C type:
//   pointer          None or an object with data_ptr() (a tensor); an integer only for the two handles, the cache's and (last) the stream's
//   parse_layer *, parse_patterns *    an object with the structure's fields as attributes; in the calls of several layers (SEVERAL) a sequence
//                    of up to four of them
//   void *const *    a sequence of up to four tensors
//   int32_t, size_t  an integer (the low bits, as ctypes does);  float  a number
// Nothing is kept from one call for the next.  The interpreter's lock is released around the call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "parse.h"

namespace {

PyObject *s_data_ptr, *s_n, *s_m, *s_R, *s_G, *s_dtype, *s_layout, *s_Vt, *s_Ut, *s_Vt_S, *s_Ut_S, *s_subsets, *s_subset_stride, *s_n_patterns, *s_k,
    *s_Vt_shared, *s_Ut_shared, *s_n_shared, *s_schedule;

bool to_int(PyObject *o, int64_t *v) {
  if (PyLong_Check(o)) {
    *v = (int64_t)PyLong_AsUnsignedLongLongMask(o);
  } else {                                   // numpy integers and the like
    PyObject *i = PyNumber_Index(o);
    if (!i) return false;
    *v = (int64_t)PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
  }
  return !(*v == -1 && PyErr_Occurred());
}

// Never an integer: a count in the place of a tensor would be read as a device address.
bool to_tensor(PyObject *o, void **p) {
  PyObject *r = PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (!r) return false;
  int64_t v;
  const bool ok = to_int(r, &v);
  Py_DECREF(r);
  if (ok) *p = (void *)(intptr_t)v;
  return ok;
}

bool to_pointer(PyObject *o, void **p) {
  if (o == Py_None) { *p = nullptr; return true; }
  return to_tensor(o, p);
}

bool to_handle(PyObject *o, void **p) {
  if (o == Py_None) { *p = nullptr; return true; }
  int64_t v;
  if (!to_int(o, &v)) return false;
  *p = (void *)(intptr_t)v;
  return true;
}

bool int_field(PyObject *o, PyObject *name, int32_t *v) {
  PyObject *a = PyObject_GetAttr(o, name);
  if (!a) return false;
  int64_t w;
  const bool ok = to_int(a, &w);
  Py_DECREF(a);
  if (ok) *v = (int32_t)w;
  return ok;
}

template <class T>
bool pointer_field(PyObject *o, PyObject *name, T **p, bool (*to)(PyObject *, void **) = to_pointer) {
  PyObject *a = PyObject_GetAttr(o, name);
  if (!a) return false;
  void *v;
  const bool ok = to(a, &v);
  Py_DECREF(a);
  if (ok) *p = (T *)v;
  return ok;
}

bool to_struct(PyObject *o, parse_layer *l) {
  return int_field(o, s_n, &l->n) && int_field(o, s_m, &l->m) && int_field(o, s_R, &l->R) && int_field(o, s_G, &l->G) && int_field(o, s_dtype, &l->dtype) &&
         int_field(o, s_layout, &l->layout) && pointer_field(o, s_Vt, &l->Vt, to_tensor) &&
         pointer_field(o, s_Ut, &l->Ut, to_tensor);
}
bool to_struct(PyObject *o, parse_patterns *p) {
  return pointer_field(o, s_Vt_S, &p->Vt_S) && pointer_field(o, s_Ut_S, &p->Ut_S) && pointer_field(o, s_subsets, &p->subsets) &&
         int_field(o, s_subset_stride, &p->subset_stride) && int_field(o, s_n_patterns, &p->n_patterns) && int_field(o, s_k, &p->k) &&
         pointer_field(o, s_Vt_shared, &p->Vt_shared) && pointer_field(o, s_Ut_shared, &p->Ut_shared) && int_field(o, s_n_shared, &p->n_shared) &&
         int_field(o, s_schedule, &p->schedule);
}
bool to_struct(PyObject *o, void **p) { return to_tensor(o, p); }

constexpr Py_ssize_t kMost = 4;              // layers of a call

// One argument: what it is converted into, and what is handed to the call.  More than kMost layers reach the library as as many structures
// as it looks at before it refuses the call.
template <class T, bool SEVERAL, class = void>
struct Arg;
template <class T, bool SEVERAL>
struct Arg<T, SEVERAL, std::enable_if_t<std::is_integral_v<T>>> {
  T v;
  bool set(PyObject *o) { int64_t w; if (!to_int(o, &w)) return false; v = (T)w; return true; }
  T get() { return v; }
};
template <bool SEVERAL>
struct Arg<float, SEVERAL> {
  float v;
  bool set(PyObject *o) { const double d = PyFloat_AsDouble(o); v = (float)d; return !(d == -1.0 && PyErr_Occurred()); }
  float get() { return v; }
};
template <class T>
struct One {
  T v;
  bool set(PyObject *o) { return to_struct(o, &v); }
  T *get() { return &v; }
};
template <class T>
struct Many {
  T v[kMost] = {};                           // what a short sequence leaves out is zero, which the library refuses
  bool set(PyObject *o) {
    PyObject *seq = PySequence_Tuple(o);       // its own: an attribute's getter may change a list
    if (!seq) return false;
    bool ok = true;
    for (Py_ssize_t i = 0; ok && i < PyTuple_GET_SIZE(seq) && i < kMost; ++i) ok = to_struct(PyTuple_GET_ITEM(seq, i), &v[i]);
    Py_DECREF(seq);
    return ok;
  }
  T *get() { return v; }
};
template <bool SEVERAL> struct Arg<const parse_layer *, SEVERAL> : std::conditional_t<SEVERAL, Many<parse_layer>, One<parse_layer>> {};
template <bool SEVERAL> struct Arg<const parse_patterns *, SEVERAL> : std::conditional_t<SEVERAL, Many<parse_patterns>, One<parse_patterns>> {};
template <> struct Arg<void *const *, true> : Many<void *> {};
template <class T, bool SEVERAL>
struct Arg<T *, SEVERAL> {
  void *v;
  bool set(PyObject *o) { return to_pointer(o, &v); }
  T *get() { return (T *)v; }
};
struct Handle {
  void *v;
  bool set(PyObject *o) { return to_handle(o, &v); }
  void *get() { return v; }
};
template <bool SEVERAL>
struct Arg<parse_cache *, SEVERAL> {
  void *v;
  bool set(PyObject *o) { return to_handle(o, &v); }
  parse_cache *get() { return (parse_cache *)v; }
};
template <bool SEVERAL, size_t I, class... A>              // the last argument of every call is its stream
using ArgOf = std::conditional_t<I + 1 == sizeof...(A), Handle, Arg<std::tuple_element_t<I, std::tuple<A...>>, SEVERAL>>;

template <auto F, bool SEVERAL>
struct Call;
template <class... A, int (*F)(A...), bool SEVERAL>
struct Call<F, SEVERAL> {
  template <size_t... I>
  static PyObject *run(PyObject *const *args, std::index_sequence<I...>) {
    static_assert(std::is_same_v<std::tuple_element_t<sizeof...(A) - 1, std::tuple<A...>>, parse_stream>);
    std::tuple<ArgOf<SEVERAL, I, A...>...> v;
    if (!(std::get<I>(v).set(args[I]) && ...)) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = F(std::get<I>(v).get()...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
  }
  static PyObject *py(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != (Py_ssize_t)sizeof...(A)) {
      PyErr_Format(PyExc_TypeError, "%zd arguments given, %zd expected", n, (Py_ssize_t)sizeof...(A));
      return nullptr;
    }
    return run(args, std::index_sequence_for<A...>{});
  }
};

#define CALL_OF(f, several) {#f, (PyCFunction)(void (*)(void))Call<&f, several>::py, METH_FASTCALL, nullptr}
#define CALL(f) CALL_OF(f, false)
#define CALL_SEVERAL(f) CALL_OF(f, true)
PyMethodDef methods[] = {
    CALL(parse_pool), CALL(parse_route), CALL(parse_route_shared), CALL(parse_route_ranks), CALL(parse_cache_lookup_or_route),
    CALL(parse_bucket_patterns), CALL(parse_bucket_and_plan), CALL(parse_prefill_plan), CALL(parse_pack_patterns), CALL(parse_pack_new_entries),
    CALL(parse_pack_ranks), CALL(parse_lowrank_forward), CALL(parse_lowrank_prefill_planned), CALL_SEVERAL(parse_lowrank_prefill_multi),
    CALL_SEVERAL(parse_lowrank_decode_planned), CALL_SEVERAL(parse_lowrank_decode_multi), CALL(parse_router_grad),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
  const struct { PyObject **to; const char *name; } names[] = {
      {&s_data_ptr, "data_ptr"}, {&s_n, "n"}, {&s_m, "m"}, {&s_R, "R"}, {&s_G, "G"}, {&s_dtype, "dtype"}, {&s_layout, "layout"}, {&s_Vt, "Vt"}, {&s_Ut, "Ut"},
      {&s_Vt_S, "Vt_S"}, {&s_Ut_S, "Ut_S"}, {&s_subsets, "subsets"}, {&s_subset_stride, "subset_stride"}, {&s_n_patterns, "n_patterns"}, {&s_k, "k"},
      {&s_Vt_shared, "Vt_shared"}, {&s_Ut_shared, "Ut_shared"}, {&s_n_shared, "n_shared"}, {&s_schedule, "schedule"}};
  for (const auto &n : names)
    if (!(*n.to = PyUnicode_InternFromString(n.name))) return nullptr;
  return PyModule_Create(&module);
}
