// Python binding of libdkv.so's stage calls: tensors, integers and descriptors to the C types of include/dkv.h.
//
// A decoder calls once per layer and token, and its calls are as long as their preparation on the host: 12.3 us a call
// through ctypes against 10 us of the two kernels it launches. Here the conversions are generated from the functions' own
// types: a pointer takes None, an address or whatever has data_ptr(), an array of pointers a sequence of the latter, the last
// parameter of every call is its stream. The GIL is given up around the call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/dkv.h"

namespace {

PyObject *s_data_ptr, *s_cuda_stream, *s_shape, *s_stride, *s_element_size, *s_zero;
PyObject *current_device, *current_raw_stream;      // torch.cuda.current_device, torch._C._cuda_getCurrentRawStream
PyObject* desc_type;                                // dkv.dkv_desc, see use_desc

// The conversions return false with a Python error set.
bool tensor_address(PyObject* o, uintptr_t& out) {
  PyObject* v = PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (v == nullptr) return false;
  out = (uintptr_t)PyLong_AsUnsignedLongLongMask(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}

// A tensor, None or an address: a plain int (True is none).
bool to_address(PyObject* o, uintptr_t& out) {
  if (o == Py_None) {
    out = 0;
    return true;
  }
  if (!PyLong_CheckExact(o)) return tensor_address(o, out);
  out = (uintptr_t)PyLong_AsUnsignedLongLongMask(o);
  return !PyErr_Occurred();
}

bool to_integer(PyObject* o, unsigned long long& out) {
  if (PyFloat_Check(o)) {
    PyErr_SetString(PyExc_TypeError, "an integer is required, not a float");
    return false;
  }
  if (PyLong_Check(o)) {
    out = PyLong_AsUnsignedLongLongMask(o);
    return !PyErr_Occurred();
  }
  PyObject* v = PyNumber_Index(o);
  if (v == nullptr) return false;
  out = PyLong_AsUnsignedLongLongMask(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}

// The stream of a call: an address, an object with one, or (None) torch's current stream.
bool to_stream(PyObject* o, uintptr_t& out) {
  PyObject* v = nullptr;
  if (PyLong_Check(o)) {
    v = o;
    Py_INCREF(v);
  } else if (o == Py_None) {
    if (current_raw_stream == nullptr) {
      PyObject *cuda = PyImport_ImportModule("torch.cuda"), *c = cuda ? PyImport_ImportModule("torch._C") : nullptr;
      if (c != nullptr && current_device == nullptr) current_device = PyObject_GetAttrString(cuda, "current_device");
      if (current_device != nullptr) current_raw_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
      Py_XDECREF(cuda);
      Py_XDECREF(c);
      if (current_raw_stream == nullptr) return false;
    }
    PyObject* dev = PyObject_CallNoArgs(current_device);
    if (dev == nullptr) return false;
    v = PyObject_CallOneArg(current_raw_stream, dev);
    Py_DECREF(dev);
  } else {
    v = PyObject_GetAttr(o, s_cuda_stream);
  }
  if (v == nullptr) return false;
  out = (uintptr_t)PyLong_AsUnsignedLongLongMask(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}

// One converted argument and what has to live as long as the call.
template <typename T>
struct Arg {
  static_assert(std::is_integral<T>::value, "integers here");
  T value;
  bool take(PyObject* o, bool) {
    unsigned long long v;
    if (!to_integer(o, v)) return false;
    value = (T)v;
    return true;
  }
};

template <typename T>
struct Arg<T*> {
  T* value;
  bool take(PyObject* o, bool stream) {
    uintptr_t v;
    if (!(stream ? to_stream(o, v) : to_address(o, v))) return false;
    value = reinterpret_cast<T*>(v);
    return true;
  }
};

template <typename T>
struct Arg<T* const*> {
  T* const* value;
  T* kept[DKV_MAX_SELECT_LAYERS] = {};             // fewer tensors than the call's layers: null pointers
  Py_ssize_t n;                                    // what the sequence held
  bool take(PyObject* o, bool) {
    PyObject* seq = PySequence_Fast(o, "a sequence of tensors is required");
    if (seq == nullptr) return false;
    n = PySequence_Fast_GET_SIZE(seq);
    bool ok = true;
    for (Py_ssize_t i = 0; ok && i < DKV_MAX_SELECT_LAYERS && i < PySequence_Fast_GET_SIZE(seq); ++i) {      // data_ptr() may change a list
      PyObject* item = PySequence_Fast_GET_ITEM(seq, i);
      Py_INCREF(item);
      uintptr_t v = 0;
      ok = tensor_address(item, v);
      Py_DECREF(item);
      kept[i] = reinterpret_cast<T*>(v);
    }
    Py_DECREF(seq);
    value = kept;
    return ok;
  }
};

template <>
struct Arg<const dkv_desc*> {
  const dkv_desc* value;
  Py_buffer view{};
  bool take(PyObject* o, bool) {
    const int is_desc = desc_type == nullptr ? 0 : PyObject_IsInstance(o, desc_type);
    if (is_desc < 0 || (is_desc == 1 && PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0)) return false;
    if (is_desc == 0 || view.len < (Py_ssize_t)sizeof(dkv_desc)) {
      PyErr_SetString(PyExc_TypeError, "a dkv_desc is required");
      return false;
    }
    value = static_cast<const dkv_desc*>(view.buf);
    return true;
  }
  ~Arg() {
    if (view.obj != nullptr) PyBuffer_Release(&view);
  }
};

// Not more tensors than layers (the third argument of the calls that take several).
template <typename A>
bool fits(const A&, long long) {
  return true;
}
template <typename T>
bool fits(const Arg<T* const*>& a, long long layers) {
  if (a.n <= layers) return true;
  PyErr_Format(PyExc_IndexError, "%zd tensors for %lld layers", a.n, layers);
  return false;
}
template <typename T>
struct is_array_of_pointers : std::false_type {};
template <typename T>
struct is_array_of_pointers<T* const*> : std::true_type {};

template <auto Fn, typename Signature>
struct Call;

template <auto Fn, typename... T>
struct Call<Fn, int (*)(T...)> {
  template <size_t... I>
  static PyObject* with(PyObject* const* a, std::index_sequence<I...>) {
    std::tuple<Arg<T>...> args;
    if (!(std::get<I>(args).take(a[I], I + 1 == sizeof...(T)) && ...)) return nullptr;
    if constexpr ((is_array_of_pointers<T>::value || ...))
      if (!(fits(std::get<I>(args), std::get<2>(args).value) && ...)) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = Fn(std::get<I>(args).value...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
  }
  static PyObject* call(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != (Py_ssize_t)sizeof...(T)) {
      PyErr_Format(PyExc_TypeError, "%zd arguments are required, not %zd", (Py_ssize_t)sizeof...(T), n);
      return nullptr;
    }
    return with(a, std::index_sequence_for<T...>{});
  }
};

// address(t): the pointer that a call gets for t (None: a null pointer, as None).
PyObject* address(PyObject*, PyObject* o) {
  if (o == Py_None) Py_RETURN_NONE;
  uintptr_t at;
  if (!to_address(o, at)) return nullptr;
  return PyLong_FromUnsignedLongLong(at);
}

// layer_ptr(t, layer): the address of t[layer], without the tensor.
PyObject* layer_ptr(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 2) {
    PyErr_SetString(PyExc_TypeError, "a tensor and a layer are required");
    return nullptr;
  }
  long long layer, layers, stride, size;
  uintptr_t at;
  PyObject* v = PyNumber_Index(a[1]);
  if (v == nullptr) return nullptr;
  layer = PyLong_AsLongLong(v);
  Py_DECREF(v);
  if (PyErr_Occurred()) return nullptr;
  v = PyObject_GetAttr(a[0], s_shape);
  PyObject* first = v ? PySequence_GetItem(v, 0) : nullptr;
  Py_XDECREF(v);
  if (first == nullptr) return nullptr;
  layers = PyLong_AsLongLong(first);
  Py_DECREF(first);
  if (PyErr_Occurred()) return nullptr;
  if (layer < -layers || layer >= layers)
    return PyErr_Format(PyExc_IndexError, "layer %lld of a tensor of %lld layers", layer, layers);
  v = PyObject_CallMethodOneArg(a[0], s_stride, s_zero);
  if (v == nullptr) return nullptr;
  stride = PyLong_AsLongLong(v);
  Py_DECREF(v);
  if (PyErr_Occurred()) return nullptr;
  v = PyObject_CallMethodNoArgs(a[0], s_element_size);
  if (v == nullptr) return nullptr;
  size = PyLong_AsLongLong(v);
  Py_DECREF(v);
  if (PyErr_Occurred() || !to_address(a[0], at)) return nullptr;
  return PyLong_FromUnsignedLongLong(at + (unsigned long long)((layer >= 0 ? layer : layer + layers) * stride * size));
}

// use_desc(type): the ctypes structure (and its subclasses) that a descriptor has to be.
PyObject* use_desc(PyObject*, PyObject* type) {
  if (!PyType_Check(type)) {
    PyErr_SetString(PyExc_TypeError, "a type is required");
    return nullptr;
  }
  Py_INCREF(type);
  PyObject* before = desc_type;
  desc_type = type;
  Py_XDECREF(before);
  Py_RETURN_NONE;
}

#define DKV_CALL(NAME) \
  { #NAME, (PyCFunction)(void (*)(void))&Call<&NAME, decltype(&NAME)>::call, METH_FASTCALL, nullptr }

PyMethodDef methods[] = {
    DKV_CALL(dkv_score_window), DKV_CALL(dkv_score_window_static), DKV_CALL(dkv_score_window_layers), DKV_CALL(dkv_score_window_stats),
    DKV_CALL(dkv_score_window_emit), DKV_CALL(dkv_score_window_lse), DKV_CALL(dkv_score_window_lse_layers), DKV_CALL(dkv_row_lse),
    DKV_CALL(dkv_select_topk), DKV_CALL(dkv_select_topk_layers), DKV_CALL(dkv_rebalance), DKV_CALL(dkv_rebalance_batch),
    DKV_CALL(dkv_gather_kv), DKV_CALL(dkv_gather_kv_layers), DKV_CALL(dkv_pack_cache), DKV_CALL(dkv_pack_zero_tail),
    DKV_CALL(dkv_decode_attention), DKV_CALL(dkv_decode_attention_layers), DKV_CALL(dkv_apply_budgets), DKV_CALL(dkv_select_recent),
    {"address", address, METH_O, nullptr},
    {"layer_ptr", (PyCFunction)(void (*)(void))&layer_ptr, METH_FASTCALL, nullptr},
    {"use_desc", use_desc, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  s_shape = PyUnicode_InternFromString("shape");
  s_stride = PyUnicode_InternFromString("stride");
  s_element_size = PyUnicode_InternFromString("element_size");
  s_zero = PyLong_FromLong(0);
  return PyModule_Create(&module);
}
