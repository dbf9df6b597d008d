// Python entry points of libhgnn.so: one function per C entry point that enqueues work, with the C arguments in their order
// except for the stream (the current one of the current device) and the byte sizes (those of the tensor in front of them).
// Tensors become device pointers, None becomes NULL; a tensor that is not a contiguous device tensor is refused. The result is
// the C function's code. Everything else (names, defaults, error texts) is in binding.py.
//
// Why native: a call of the library is two or three launches of 3-4 us, and marshalling its 5 to 26 arguments in Python took
// 5-11 us on top (current stream 3 us, 0.3 us per tensor, the size of a buffer as much again), for which the GPU waited in small
// batches. embed_fwd, one launch, 7.2 -> 3.0 us; forward pass of one molecule, seven calls and 16 launches, 92 -> 59 us (60 as a
// HIP graph); reverse pass of a crystal's conservative forces, 260 -> 117 us of the host.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>
#include <tuple>
#include <type_traits>

#include "../../include/hgnn.h"

namespace {

struct Args {
  PyObject* const* v;
  Py_ssize_t n;
  Py_ssize_t at = 0;
  size_t bytes = 0;   // of the tensor taken last
  bool ok = true;     // false: a Python error is set
};

template <class T>
T take(Args& a) {
  if constexpr (std::is_same_v<T, size_t>) {
    return a.bytes;
  } else {
    if (!a.ok) return T{};
    if (a.at >= a.n) {
      PyErr_SetString(PyExc_TypeError, "too few arguments");
      a.ok = false;
      return T{};
    }
    PyObject* o = a.v[a.at++];
    if constexpr (std::is_pointer_v<T>) {
      a.bytes = 0;
      if (o == Py_None) return nullptr;
      if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "argument %zd: expected a tensor or None, got %s", a.at, Py_TYPE(o)->tp_name);
        a.ok = false;
        return nullptr;
      }
      const at::Tensor& t = THPVariable_Unpack(o);
      if (!t.is_cuda() || !t.is_contiguous()) {
        PyErr_SetString(PyExc_AssertionError, "libhgnn takes contiguous device tensors");
        a.ok = false;
        return nullptr;
      }
      a.bytes = t.nbytes();
      return static_cast<T>(t.data_ptr());
    } else if constexpr (std::is_floating_point_v<T>) {
      const double x = PyFloat_AsDouble(o);
      if (x == -1.0 && PyErr_Occurred()) a.ok = false;
      return static_cast<T>(x);
    } else {
      static_assert(std::is_integral_v<T>);
      PyObject* k = PyNumber_Index(o);
      const long long x = k ? PyLong_AsLongLong(k) : -1;
      Py_XDECREF(k);
      if (x == -1 && PyErr_Occurred()) a.ok = false;
      return static_cast<T>(x);
    }
  }
}

// arguments in order, then the call without the interpreter lock (two of the functions wait for the stream)
template <class R, class... A>
bool run(R (*fn)(void*, A...), PyObject* const* v, Py_ssize_t n, R& result) {
  try {
    Args a{v, n};
    std::tuple<A...> t{take<A>(a)...};   // (braces: left to right)
    if (!a.ok) return false;
    if (a.at != n) {
      PyErr_SetString(PyExc_TypeError, "too many arguments");
      return false;
    }
    void* st = c10::hip::getCurrentHIPStream().stream();
    Py_BEGIN_ALLOW_THREADS
    result = std::apply([&](A... x) { return fn(st, x...); }, t);
    Py_END_ALLOW_THREADS
    return true;
  } catch (const std::exception& e) {   // a tensor without storage, no device
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return false;
  }
}

template <auto Fn>
PyObject* call(PyObject*, PyObject* const* v, Py_ssize_t n) {
  int32_t code = 0;
  return run(Fn, v, n, code) ? PyLong_FromLong(code) : nullptr;
}

// the number of edges (which no code is: they are negative), or the code
int64_t count_edges(void* st, int32_t N, int32_t G, const float* pos, const int32_t* graph_off, const float* cell,
                    const uint8_t* pbc, float rc, void* ws, size_t ws_bytes, int32_t* row_ptr) {
  int64_t E = 0;
  const int32_t code = hgnn_radius_graph_count(st, N, G, pos, graph_off, cell, pbc, rc, ws, ws_bytes, row_ptr, &E);
  return code != HGNN_OK ? code : E;
}
PyObject* call_count(PyObject*, PyObject* const* v, Py_ssize_t n) {
  int64_t E = 0;
  return run(&count_edges, v, n, E) ? PyLong_FromLongLong(E) : nullptr;
}

#define ENTRY(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&call<&hgnn_##name>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"radius_graph_count", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&call_count)), METH_FASTCALL, nullptr},
    ENTRY(radius_graph_fill),
    ENTRY(embed_fwd), ENTRY(embed_bwd), ENTRY(embed_bwd_static),
    ENTRY(mp_layer_fwd), ENTRY(mp_layer_bwd), ENTRY(mp_layer_attr_fwd), ENTRY(mp_layer_attr_bwd),
    ENTRY(edge_rbf), ENTRY(edge_rbf_bwd), ENTRY(edge_geometry_fwd), ENTRY(edge_geometry_bwd),
    ENTRY(pool_by_graph_fwd), ENTRY(pool_by_graph_bwd),
    ENTRY(multihead_plan), ENTRY(multihead_decode_fwd), ENTRY(multihead_decode_bwd),
    ENTRY(multihead_deep_fwd), ENTRY(multihead_deep_bwd),
    ENTRY(adamw_step),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Python entry points of libhgnn.so", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
