// Python module `_marshal`: the arguments of the library's calls, taken from torch tensors (host only).
//
// A call of a few microseconds on the GPU is launched by a few microseconds on the host, and most of those were spent
// in Python on checking tensors, asking for their addresses and converting numbers for ctypes.  Here a call is one native function: what
// each parameter of the C function is made of stands in a string of codes (TABLE), the parameter types come from the
// header's own declarations.  (Host time, launches included: the four calls of a tiny step 31.9 us, now 19.6; the 13 of six
// drafting levels 108 and 69; one attention call of two launches 15.6 and 13.0.  A launch itself is 3.4 us of it.)
//
// The library is not linked: function(name, address) gives a callable for the function at that address, so that the
// module serves the library that binding.py has loaded.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <exception>
#include <string>
#include <type_traits>
#include <utility>
#include <vector>

#include <ATen/core/Tensor.h>
#include <c10/core/impl/DeviceGuardImplInterface.h>
#include <torch/csrc/autograd/python_variable.h>

#include "heterospec.h"

namespace {

// One code to a parameter of the C function.  Tensors: on the GPU and contiguous, of the type that the code says.
//   i l f u   int32, int64, float32, uint8        (I F: may be None)
//   t         float32 or bfloat16, all of a call of one type; D: that type's code (takes no argument)
//   o         an address only, not looked at any further (may be None)
//   h H       on the host, int32 or int64, whatever its layout (converted where needed)
//   w W       a workspace tensor (may be None) and, without an argument of its own, its size
// Numbers: n integer, d float; e: a sequence of floats.  s: a stream object, None for the current one.
struct Entry {
  const char* name;
  const char* codes;
  const char* names;  // of the arguments that are checked (codes i l f u I F t), in order
  PyObject* (*call)(const Entry&, void*, PyObject* const*, Py_ssize_t);
};

struct Failed {};  // a Python error is set

const char* type_name(at::ScalarType t) {
  switch (t) {
    case at::kInt: return "torch.int32";
    case at::kLong: return "torch.int64";
    case at::kFloat: return "torch.float32";
    case at::kByte: return "torch.uint8";
    case at::kBFloat16: return "torch.bfloat16";
    default: return "torch";
  }
}

PyObject* raw_stream_fn = nullptr;  // torch._C._cuda_getCurrentRawStream

struct Call {
  const Entry& e;
  PyObject* const* args;
  Py_ssize_t n_args, at = 0;
  const char* names;
  bool typed = false;
  at::ScalarType type = at::kFloat;
  size_t ws_bytes = 0;
  std::vector<at::Tensor> keep;             // converted host arrays, until the call has returned
  std::vector<std::vector<float>> floats;

  Call(const Entry& entry, PyObject* const* a, Py_ssize_t n) : e(entry), args(a), n_args(n), names(entry.names) { floats.reserve(2); }

  PyObject* next() {
    if (at >= n_args) {
      PyErr_Format(PyExc_TypeError, "%s: too few arguments", e.name);
      throw Failed{};
    }
    return args[at++];
  }
  std::string next_name() {
    const char* end = names;
    while (*end != '\0' && *end != ' ') ++end;
    std::string s(names, end);
    names = *end == ' ' ? end + 1 : end;
    return s;
  }
  const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) {
      PyErr_Format(PyExc_TypeError, "%s: a tensor was expected, not %s", e.name, Py_TYPE(o)->tp_name);
      throw Failed{};
    }
    return THPVariable_Unpack(o);
  }
  void* checked(at::ScalarType want, bool optional) {
    PyObject* o = next();
    if (optional && o == Py_None) {
      next_name();
      return nullptr;
    }
    const at::Tensor& t = tensor(o);
    if (!t.is_cuda() || t.scalar_type() != want || !t.is_contiguous()) {
      PyErr_Format(PyExc_ValueError, "%s must be a contiguous %s tensor on the GPU", next_name().c_str(), type_name(want));
      throw Failed{};
    }
    next_name();
    return t.data_ptr();
  }
  void* host(at::ScalarType want) {
    const at::Tensor& t = tensor(next());
    if (t.scalar_type() == want && t.device().is_cpu() && t.is_contiguous()) return t.data_ptr();
    keep.push_back(t.to(at::Device(at::kCPU), want).contiguous());
    return keep.back().data_ptr();
  }
  void* stream() {
    PyObject* o = next();
    PyObject* v;
    if (o == Py_None) {
      const int dev = c10::impl::getDeviceGuardImpl(c10::DeviceType::CUDA)->getDevice().index();
      PyObject* d = PyLong_FromLong(dev);
      v = d == nullptr ? nullptr : PyObject_CallOneArg(raw_stream_fn, d);
      Py_XDECREF(d);
    } else {
      v = PyObject_GetAttrString(o, "cuda_stream");
    }
    if (v == nullptr) throw Failed{};
    void* p = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (p == nullptr && PyErr_Occurred()) throw Failed{};
    return p;
  }
  void* pointer(char code) {
    switch (code) {
      case 'i': return checked(at::kInt, false);
      case 'I': return checked(at::kInt, true);
      case 'l': return checked(at::kLong, false);
      case 'f': return checked(at::kFloat, false);
      case 'F': return checked(at::kFloat, true);
      case 'u': return checked(at::kByte, false);
      case 't': {
        if (!typed) {
          if (at < n_args) type = tensor(args[at]).scalar_type();
          if (type != at::kFloat && type != at::kBFloat16) {
            PyErr_SetString(PyExc_ValueError, "q/k/v must be float32 or bfloat16");
            throw Failed{};
          }
          typed = true;
        }
        return checked(type, false);
      }
      case 'o': {
        PyObject* o = next();
        return o == Py_None ? nullptr : tensor(o).data_ptr();
      }
      case 'h': return host(at::kInt);
      case 'H': return host(at::kLong);
      case 'w': {
        PyObject* o = next();
        if (o == Py_None) return nullptr;
        const at::Tensor& t = tensor(o);
        ws_bytes = (size_t)t.numel();
        return t.data_ptr();
      }
      case 'e': {
        PyObject* seq = PySequence_Fast(next(), "a sequence of floats was expected");
        if (seq == nullptr) throw Failed{};
        floats.emplace_back();
        std::vector<float>& f = floats.back();
        for (Py_ssize_t k = 0; k < PySequence_Fast_GET_SIZE(seq); ++k) f.push_back((float)PyFloat_AsDouble(PySequence_Fast_GET_ITEM(seq, k)));
        Py_DECREF(seq);
        f.push_back(0.f);  // (an empty sequence has an address as well)
        if (PyErr_Occurred()) throw Failed{};
        return f.data();
      }
      default: return stream();  // 's'
    }
  }
  template <typename P>
  P take(char code) {
    if constexpr (std::is_pointer_v<P>) {
      return static_cast<P>(pointer(code));
    } else if constexpr (std::is_floating_point_v<P>) {
      const double v = PyFloat_AsDouble(next());
      if (v == -1.0 && PyErr_Occurred()) throw Failed{};
      return (P)v;
    } else {
      if (code == 'W') return static_cast<P>(ws_bytes);
      if (code == 'D') return static_cast<P>(type == at::kBFloat16 ? HS_BF16 : HS_F32);
      const long long v = PyLong_AsLongLong(next());
      if (v == -1 && PyErr_Occurred()) throw Failed{};
      if constexpr (!std::is_enum_v<P>) {
        if (v != (long long)(P)v) {
          PyErr_Format(PyExc_OverflowError, "%s: %lld does not fit its parameter", e.name, v);
          throw Failed{};
        }
      }
      return static_cast<P>(v);
    }
  }
};

template <typename... P, size_t... I>
hs_status invoke(hs_status (*fn)(P...), Call& c, std::index_sequence<I...>) {
  std::tuple<P...> p{c.take<P>(c.e.codes[I])...};  // (braces: from left to right)
  if (c.at != c.n_args) {
    PyErr_Format(PyExc_TypeError, "%s: too many arguments", c.e.name);
    throw Failed{};
  }
  hs_status st;
  Py_BEGIN_ALLOW_THREADS;
  st = std::apply(fn, p);
  Py_END_ALLOW_THREADS;
  return st;
}

template <typename F>
struct Wrap;
template <typename... P>
struct Wrap<hs_status(P...)> {
  static PyObject* call(const Entry& e, void* fn, PyObject* const* args, Py_ssize_t n) {
    try {
      Call c(e, args, n);
      return PyLong_FromLong((long)invoke(reinterpret_cast<hs_status (*)(P...)>(fn), c, std::index_sequence_for<P...>{}));
    } catch (const Failed&) {
      return nullptr;
    } catch (const std::exception& x) {
      PyErr_SetString(PyExc_RuntimeError, x.what());
      return nullptr;
    } catch (...) {
      PyErr_Format(PyExc_RuntimeError, "%s: unknown error", e.name);
      return nullptr;
    }
  }
};

template <typename F>
constexpr int n_params = 0;
template <typename... P>
constexpr int n_params<hs_status(P...)> = sizeof...(P);
constexpr int length(const char* s) { return *s == '\0' ? 0 : 1 + length(s + 1); }

#define HS_ENTRY(fn, codes, names)                                                                   \
  (static_cast<void>(std::integral_constant<int, 1 / (n_params<decltype(fn)> == length(codes) ? 1 : 0)>{}), \
   Entry{#fn, codes, names, &Wrap<decltype(fn)>::call})
#define HS_TREE "parent logc node_offsets"
const Entry TABLE[] = {
    HS_ENTRY(hs_draft_entropy_topk, "onnnndooooowWs", ""),
    HS_ENTRY(hs_draft_entropy_topk_rows, "oninnndooooowWs", "row_index"),
    HS_ENTRY(hs_draft_entropy_topk_fused, "onInnndooooowWs", "row_index"),
    HS_ENTRY(hs_tree_prune, "ifinnifioooooowWs", HS_TREE " d_max theta max_nodes"),
    HS_ENTRY(hs_tree_prune_counted, "ifiinnifioooooowWs", HS_TREE " node_counts d_max theta max_nodes"),
    HS_ENTRY(hs_tree_expand, "iiffifiiiiiiffInnnnns",
             "parent token logc cumlogp depth ent n_nodes level frontier n_frontier frontier_rows topk_idx topk_logp ent_topk d_limit"),
    HS_ENTRY(hs_adaptive_control, "iffiInnenennnnnooooos", "parent logc ent node_offsets node_counts"),
    HS_ENTRY(hs_tree_attention, "tttttiilhHnnnnDdoowWs", "q k_prefix v_prefix k_tree v_tree parent node_offsets prefix_offsets"),
    HS_ENTRY(hs_tree_attention_shared_tree, "tttttiilhHnnnnDdoowWs", "q k_prefix v_prefix k_tree v_tree parent node_offsets prefix_offsets"),
    HS_ENTRY(hs_tree_attention_lens, "tttttiilhHlHnnnnDdoowWs",
             "q k_prefix v_prefix k_tree v_tree parent node_offsets prefix_offsets prefix_lens"),
    HS_ENTRY(hs_tree_attention_paged, "tttttiihinnlHnnnnDdoowWs",
             "q k_pages v_pages k_tree v_tree parent node_offsets block_table prefix_lens"),
    HS_ENTRY(hs_verify_accept, "ooniiinnnndFnooowWs", "token parent node_offsets uniforms"),
    HS_ENTRY(hs_kv_commit, "ttiiinttllnnnDs", "k_tree v_tree node_offsets accept_path accept_len k_cache v_cache cache_offsets cache_lens"),
    HS_ENTRY(hs_kv_commit_paged, "ttiiinttinnlnnnDs",
             "k_tree v_tree node_offsets accept_path accept_len k_pages v_pages block_table cache_lens"),
};

// A bound function: self is a tuple (capsule of the entry, capsule of the address).
PyObject* bound_call(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  const Entry* e = static_cast<const Entry*>(PyCapsule_GetPointer(PyTuple_GET_ITEM(self, 0), "entry"));
  void* fn = PyCapsule_GetPointer(PyTuple_GET_ITEM(self, 1), "address");
  if (e == nullptr || fn == nullptr) return nullptr;
  return e->call(*e, fn, args, n);
}
PyMethodDef bound_def = {"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(bound_call)), METH_FASTCALL, nullptr};

PyObject* function(PyObject*, PyObject* args) {
  const char* name;
  unsigned long long address;
  if (!PyArg_ParseTuple(args, "sK", &name, &address)) return nullptr;
  for (const Entry& e : TABLE) {
    if (std::string(name) != e.name) continue;
    PyObject* self = Py_BuildValue("(NN)", PyCapsule_New(const_cast<Entry*>(&e), "entry", nullptr),
                                   PyCapsule_New(reinterpret_cast<void*>(address), "address", nullptr));
    if (self == nullptr) return nullptr;
    PyObject* f = PyCFunction_New(&bound_def, self);
    Py_DECREF(self);
    return f;
  }
  PyErr_Format(PyExc_KeyError, "%s", name);
  return nullptr;
}

PyMethodDef methods[] = {{"function", function, METH_VARARGS, "function(name, address): the call at that address, on torch tensors"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
  PyObject* c = PyImport_ImportModule("torch._C");
  if (c == nullptr) return nullptr;
  raw_stream_fn = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");  // (absent in builds of torch without a GPU)
  Py_DECREF(c);
  if (raw_stream_fn == nullptr) return nullptr;
  return PyModule_Create(&module);
}
