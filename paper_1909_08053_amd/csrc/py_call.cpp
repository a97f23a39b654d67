// CPython module beside the C-ABI library: the entry points that a step calls, taking what the Python binding has in hand (ctypes
// structures, torch tensors, lists of them).  In Python the marshalling was 69 of the 178 us of host time of a step of 40 launches, which
// now takes 149; the launches themselves are some 3 us each.  No arithmetic, no state: an argument is checked (on the GPU,
// contiguous) and passed on.  By the parameter's type:
//   mlm_dims*, mlm_dropout*   a ctypes structure (the latter or None)
//   any other pointer         a tensor or None; as the last parameter the stream: None (torch's current one) or an integer
//   array of pointers         a sequence of tensors; the int32_t behind it is their number and takes no argument
//   size_t                    the bytes of the tensor ahead of it; takes no argument
//   int32_t                   an integer
// Every function returns the entry point's status.
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>
#include <tuple>
#include <type_traits>
#include <vector>
#include "mlm_shard.h"

namespace {

struct PythonError {};                 // a Python exception is set

struct Arguments {
  PyObject* const* arg;
  Py_ssize_t n, at = 0;
  size_t bytes = 0;                    // of the last tensor
  int32_t count = 0;
  bool counted = false;                // the next int32_t is `count`
  std::vector<const void*> pointers;

  PyObject* next() {
    if (at >= n) {
      PyErr_SetString(PyExc_TypeError, "too few arguments");
      throw PythonError();
    }
    return arg[at++];
  }
  void* tensor(PyObject* o) {
    if (o == Py_None) {
      bytes = 0;
      return nullptr;
    }
    if (!THPVariable_Check(o)) {
      PyErr_Format(PyExc_TypeError, "expected a tensor, not %s", Py_TYPE(o)->tp_name);
      throw PythonError();
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) {
      PyErr_SetString(PyExc_ValueError, "expected a contiguous CUDA tensor");
      throw PythonError();
    }
    bytes = t.nbytes();
    return t.data_ptr();
  }
  void* structure(PyObject* o, size_t size) {
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw PythonError();
    void* p = view.buf;                // (the structure lives as long as the caller's reference to it)
    const bool ok = (size_t)view.len == size;
    PyBuffer_Release(&view);
    if (!ok) {
      PyErr_SetString(PyExc_TypeError, "wrong structure");
      throw PythonError();
    }
    return p;
  }
  long long integer(PyObject* o) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw PythonError();
    return v;
  }
};

template <typename P, bool LAST>
P convert(Arguments& a) {
  if constexpr (std::is_same_v<P, const mlm_dims*>) {
    return (P)a.structure(a.next(), sizeof(mlm_dims));
  } else if constexpr (std::is_same_v<P, const mlm_dropout*>) {
    PyObject* o = a.next();
    return o == Py_None ? nullptr : (P)a.structure(o, sizeof(mlm_dropout));
  } else if constexpr (std::is_same_v<P, const void* const*>) {
    PyObject* seq = PySequence_Fast(a.next(), "expected a sequence of tensors");
    if (!seq) throw PythonError();
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
    a.pointers.assign(n > 0 ? n : 1, nullptr);
    try {
      for (Py_ssize_t i = 0; i < n; ++i) a.pointers[i] = a.tensor(PySequence_Fast_GET_ITEM(seq, i));
    } catch (...) {
      Py_DECREF(seq);
      throw;
    }
    Py_DECREF(seq);
    a.count = (int32_t)n;
    a.counted = true;
    return a.pointers.data();
  } else if constexpr (LAST && std::is_same_v<P, void*>) {
    PyObject* o = a.next();
    if (o == Py_None) return (void*)c10::hip::getCurrentHIPStream().stream();
    PyObject* i = PyNumber_Long(o);
    if (!i) throw PythonError();
    const uintptr_t v = (uintptr_t)PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    return (void*)v;
  } else if constexpr (std::is_pointer_v<P>) {
    return (P)a.tensor(a.next());
  } else if constexpr (std::is_same_v<P, size_t>) {
    return a.bytes;
  } else {
    static_assert(std::is_same_v<P, int32_t>, "a parameter type without a rule");
    if (a.counted) {
      a.counted = false;
      return a.count;
    }
    return (int32_t)a.integer(a.next());
  }
}

template <typename... P, size_t... I>
int call(int (*f)(P...), Arguments& a, std::index_sequence<I...>) {
  const std::tuple<P...> t{convert<P, I + 1 == sizeof...(P)>(a)...};       // (braces: in order)
  if (a.at != a.n) {
    PyErr_SetString(PyExc_TypeError, "too many arguments");
    throw PythonError();
  }
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = std::apply(f, t);
  Py_END_ALLOW_THREADS
  return rc;
}
template <typename... P> int call(int (*f)(P...), Arguments& a) { return call(f, a, std::index_sequence_for<P...>()); }

template <auto F>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  try {
    Arguments a{args, n};
    return PyLong_FromLong(call(F, a));
  } catch (const PythonError&) {
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}

#define MLM_ENTRY(name) {#name, (PyCFunction)(void (*)(void))entry<&name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    MLM_ENTRY(mlm_layernorm_fwd), MLM_ENTRY(mlm_layernorm_bwd), MLM_ENTRY(mlm_combine), MLM_ENTRY(mlm_combine_dropout),
    MLM_ENTRY(mlm_combine_layernorm_fwd), MLM_ENTRY(mlm_combine_layernorm_bwd), MLM_ENTRY(mlm_combine_layernorm_fwd_dropout),
    MLM_ENTRY(mlm_combine_layernorm_bwd_dropout), MLM_ENTRY(mlm_colsum), MLM_ENTRY(mlm_colsum_noalloc), MLM_ENTRY(mlm_deferred_sums_begin),
    MLM_ENTRY(mlm_deferred_sums_flush), MLM_ENTRY(mlm_attn_shard_fwd), MLM_ENTRY(mlm_attn_shard_bwd), MLM_ENTRY(mlm_attn_shard_fwd_dropout),
    MLM_ENTRY(mlm_attn_shard_bwd_dropout), MLM_ENTRY(mlm_attn_shard_bwd_input), MLM_ENTRY(mlm_mlp_shard_fwd), MLM_ENTRY(mlm_mlp_shard_bwd),
    MLM_ENTRY(mlm_mlp_shard_bwd_input), MLM_ENTRY(mlm_layer_shard_wgrads), MLM_ENTRY(mlm_vocab_ce_shard_fwd), MLM_ENTRY(mlm_vocab_ce_merge),
    MLM_ENTRY(mlm_vocab_ce_shard_bwd), MLM_ENTRY(mlm_embed_shard_fwd), MLM_ENTRY(mlm_embed_shard_bwd), MLM_ENTRY(mlm_embed_bwd_replicated),
    MLM_ENTRY(mlm_rows_gather), MLM_ENTRY(mlm_rows_scatter), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_mlm_call", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__mlm_call(void) { return PyModule_Create(&module); }
