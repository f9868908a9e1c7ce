// Argument marshalling of the library's calls for prompts and decode steps, for binding.py: tensors are checked (on a GPU, dense,
// of the type asked for) and turned into addresses, the current stream is added, and the C function is called with the interpreter's
// lock released.  A small launch is over sooner than the same checks take from Python (one layer of one sequence: 10.6 us a
// step with them in Python, 7 with these; the kernel takes 4.8).
//
// Every function takes the address of the C function, the descriptor and the call's arguments, and returns its status, or
// None when an argument is not what is expected here: binding.py then takes its own way, which accepts it or says what is wrong.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <tuple>

#include "../../include/pe.h"

namespace {

struct Address {  // converts to whatever pointer the C function declares
  void* p = nullptr;
  template <typename T>
  operator T*() const {
    return static_cast<T*>(p);
  }
};

bool address_of(PyObject* o, bool typed, at::ScalarType type, Address* to) {
  if (!THPVariable_Check(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.is_contiguous()) return false;
  if (typed && t.scalar_type() != type) return false;
  to->p = t.data_ptr();
  return true;
}

// What an argument is: get() reads it from the Python object, its C arguments are a tuple.
struct Tensor {
  std::tuple<Address> c;
  bool get(PyObject* o) { return address_of(o, false, at::kInt, &std::get<0>(c)); }
};
struct Ints {
  std::tuple<Address> c;
  bool get(PyObject* o) { return address_of(o, true, at::kInt, &std::get<0>(c)); }
};
struct Floats {
  std::tuple<Address> c;
  bool get(PyObject* o) { return address_of(o, true, at::kFloat, &std::get<0>(c)); }
};
struct IntsOrNone {
  std::tuple<Address> c;
  bool get(PyObject* o) { return o == Py_None || address_of(o, true, at::kInt, &std::get<0>(c)); }
};
struct LastDim {  // the size of a tensor's last dimension
  std::tuple<int32_t> c;
  bool get(PyObject* o) {
    if (!THPVariable_Check(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (t.dim() < 1) return false;
    std::get<0>(c) = (int32_t)t.size(-1);
    return true;
  }
};
template <typename T>
struct Number {
  std::tuple<T> c;
  bool get(PyObject* o) {
    if (!PyLong_CheckExact(o)) return false;
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) {
      PyErr_Clear();
      return false;
    }
    std::get<0>(c) = (T)v;
    return std::get<0>(c) == v;
  }
};
struct Float {
  std::tuple<float> c;
  bool get(PyObject* o) {
    if (!PyFloat_CheckExact(o)) return false;
    std::get<0>(c) = (float)PyFloat_AS_DOUBLE(o);
    return true;
  }
};
struct Workspace {
  std::tuple<Address, size_t> c{Address{}, 0};
  bool get(PyObject* o) {
    if (o == Py_None) return true;
    if (!THPVariable_Check(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    // (its bytes are its own only if nothing else lies between them, whatever the order of its dimensions)
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.is_non_overlapping_and_dense()) return false;
    std::get<0>(c).p = t.data_ptr();
    std::get<1>(c) = t.nbytes();
    return true;
  }
};

// binding.py's ctypes structure (see bind_descriptor); nullptr: not named yet.
PyTypeObject* descriptor_type = nullptr;

// The descriptor: an object of that type and of no other, read through the buffer protocol.
struct Desc {
  pe_cache_desc d;
  bool get(PyObject* o) {
    if (descriptor_type == nullptr || Py_TYPE(o) != descriptor_type) return false;
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
      PyErr_Clear();
      return false;
    }
    const bool fits = b.len == (Py_ssize_t)sizeof(d);
    if (fits) memcpy(&d, b.buf, sizeof(d));
    PyBuffer_Release(&b);
    return fits;
  }
};

template <typename... Args, size_t... I>
bool get_all(std::tuple<Args...>& a, PyObject* const* o, std::index_sequence<I...>) {
  return (std::get<I>(a).get(o[I]) && ...);
}

// args: address of the C function, descriptor, then one object for each of Args
template <typename Fn, typename... Args>
PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != (Py_ssize_t)sizeof...(Args) + 2) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  const auto fn = reinterpret_cast<Fn>(PyLong_AsVoidPtr(args[0]));
  if (fn == nullptr) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no function");
    return nullptr;
  }
  try {
    Desc desc;
    std::tuple<Args...> a;
    if (!desc.get(args[1]) || !get_all(a, args + 2, std::index_sequence_for<Args...>{})) Py_RETURN_NONE;
    const auto stream = c10::hip::getCurrentHIPStream().stream();
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = std::apply([&](auto&... x) {
      return std::apply(fn, std::tuple_cat(std::make_tuple((const pe_cache_desc*)&desc.d), x.c..., std::make_tuple((void*)stream)));
    }, a);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
  } catch (const std::exception&) {  // e.g. a tensor without storage
    Py_RETURN_NONE;
  }
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyMethodDef method(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL, nullptr};
}

// Names the type of the descriptor, once, when the library is loaded.  Returns the C structure's layout for a comparison with
// it: its size, then name, offset and size of each field.
PyObject* bind_descriptor(PyObject*, PyObject* type) {
  if (!PyType_Check(type)) {
    PyErr_SetString(PyExc_TypeError, "the type of the descriptor");
    return nullptr;
  }
#define PE_FIELD(f) #f, (Py_ssize_t)offsetof(pe_cache_desc, f), (Py_ssize_t)sizeof(pe_cache_desc::f)
  PyObject* layout = Py_BuildValue(
      "(n(snn)(snn)(snn)(snn)(snn)(snn)(snn)(snn)(snn)(snn)(snn)(snn))", (Py_ssize_t)sizeof(pe_cache_desc), PE_FIELD(dtype),
      PE_FIELD(num_seqs), PE_FIELD(num_kv_heads), PE_FIELD(num_q_heads), PE_FIELD(head_dim), PE_FIELD(block_size),
      PE_FIELD(max_blocks), PE_FIELD(num_phys_blocks), PE_FIELD(layout), PE_FIELD(decode_splits), PE_FIELD(decode_shape),
      PE_FIELD(decode_flat_order));
#undef PE_FIELD
  if (layout == nullptr) return nullptr;
  Py_INCREF(type);
  Py_XDECREF((PyObject*)descriptor_type);
  descriptor_type = reinterpret_cast<PyTypeObject*>(type);
  return layout;
}

PyMethodDef methods[] = {
    {"bind_descriptor", bind_descriptor, METH_O, nullptr},
    // q, k_pool, v_pool, block_table, seq_lens, softmax_scale, out, workspace
    method<call<decltype(&pe_paged_decode), Tensor, Tensor, Tensor, Ints, Ints, Float, Tensor, Workspace>>("paged_decode"),
    // new_k, new_v, q, k_pool, v_pool, block_table, seq_lens, seq_lens_out, freed_phys, spare, spare_used, spare, softmax_scale,
    // out, workspace
    method<call<decltype(&pe_append_paged_decode), Tensor, Tensor, Tensor, Tensor, Tensor, Ints, Ints, Ints, Ints, Ints, Ints,
                LastDim, Float, Tensor, Workspace>>("append_paged_decode"),
    // num_layers, then as above
    method<call<decltype(&pe_append_paged_decode_layers), Number<int32_t>, Tensor, Tensor, Tensor, Tensor, Tensor, Ints, Ints, Ints,
                Ints, Ints, Ints, LastDim, Float, Tensor, Workspace>>("append_paged_decode_layers"),
    // k_in, v_in, cu_seqlens, total_tokens, max_seqlen, budget_tokens, k_pool, v_pool, block_table, seq_lens_out, kept_idx_out,
    // workspace
    method<call<decltype(&pe_prefill_prune), Tensor, Tensor, Ints, Number<int64_t>, Number<int32_t>, Number<int32_t>, Tensor, Tensor,
                Ints, Ints, IntsOrNone, Workspace>>("prefill_prune"),
    // k_pool, v_pool, block_table, seq_lens, budget_tokens, scores_inout
    method<call<decltype(&pe_score_triggered_blocks), Tensor, Tensor, Ints, Ints, Number<int32_t>, Floats>>(
        "score_triggered_blocks"),
    // the same with `recent`
    method<call<decltype(&pe_score_recent_blocks), Tensor, Tensor, Ints, Ints, Number<int32_t>, Floats>>("score_recent_blocks"),
    // scores, block_table, seq_lens, budget_tokens, evicted_logical_out, freed_phys_out
    method<call<decltype(&pe_evict_blocks), Floats, Ints, Ints, Number<int32_t>, Ints, Ints>>("evict_blocks"),
    method<call<decltype(&pe_evict_blocks_cached), Floats, Ints, Ints, Number<int32_t>, Ints, Ints>>("evict_blocks_cached"),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pe_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pe_host() { return PyModule_Create(&module); }
