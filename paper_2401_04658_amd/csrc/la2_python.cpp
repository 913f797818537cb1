// CPython module of the binding's per-call work: argument checks, output tensors, descriptors and the call into libla2.so.
//
// A small call costs what the host takes for it: batch 1, 16 heads, a decode step's kernel runs 3 us and a short prefill's 8 to 14, a
// launch takes the host 3.6, and checks, allocations and marshalling in Python and ctypes took 4 to 9 more (decode 7.8 us a call,
// la2_fwd_state 13.1, la2_fwd with la2_bwd 25.6; from here 5.2, 6.8, 14.2).  Every entry point of the library is
// wrapped by its own type: a pointer takes a tensor (its data), None or a handle, a size also a tensor (its bytes), a descriptor a
// [batch, heads, seqlen, head_dim] tensor or a la2_desc in a buffer.  The interpreter lock is released for the call.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_strided.h>

#include <cstring>
#include <exception>
#include <tuple>
#include <utility>

#include "../../include/la2.h"

namespace {

struct Raised {};   // a Python exception has been set

[[noreturn]] void raise(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw Raised{};
}

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "la2: expected a tensor, got %s", Py_TYPE(o)->tp_name);
    throw Raised{};
  }
  return THPVariable_Unpack(o);
}

int32_t dtype_code(const at::Tensor& t) {
  const auto s = t.scalar_type();
  if (s == at::kBFloat16) return LA2_BF16;
  if (s == at::kHalf) return LA2_F16;
  if (s == at::kFloat) return LA2_F32;
  PyErr_Format(PyExc_TypeError, "la2: dtype must be torch.bfloat16, torch.float16 or torch.float32, got %s", c10::toString(s));
  throw Raised{};
}

int32_t extent(int64_t n) {
  if (n > INT32_MAX) raise(PyExc_OverflowError, "la2: an extent of 2^31 or more");
  return (int32_t)n;
}

la2_desc desc_of(const at::Tensor& t) {
  if (t.dim() != 4) raise(PyExc_ValueError, "la2: expected a [batch, heads, seqlen, head_dim] tensor");
  if (t.size(3) > 1 && t.stride(3) != 1) raise(PyExc_ValueError, "la2: the feature dimension must be contiguous");
  la2_desc d{};
  d.batch = extent(t.size(0));
  d.heads = extent(t.size(1));
  d.seqlen = extent(t.size(2));
  d.head_dim = extent(t.size(3));
  d.dtype = dtype_code(t);
  d.stride_b = t.stride(0);
  d.stride_h = t.stride(1);
  d.stride_n = t.stride(2);
  return d;
}

// ---- one argument of an entry point, by its type
template <typename T>
struct Arg;

template <typename T>
struct Arg<T*> {
  T* value;
  explicit Arg(PyObject* o) {
    if (o == Py_None) {
      value = nullptr;
    } else if (PyLong_Check(o)) {
      value = static_cast<T*>(PyLong_AsVoidPtr(o));
      if (PyErr_Occurred()) throw Raised{};
    } else {
      value = static_cast<T*>(tensor(o).data_ptr());
    }
  }
  T* get() const { return value; }
};
template <>
struct Arg<const la2_desc*> {
  la2_desc desc;
  explicit Arg(PyObject* o) {
    if (THPVariable_Check(o)) {
      desc = desc_of(THPVariable_Unpack(o));
      return;
    }
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) throw Raised{};
    const bool fits = b.len == (Py_ssize_t)sizeof(desc);
    if (fits) std::memcpy(&desc, b.buf, sizeof(desc));
    PyBuffer_Release(&b);
    if (!fits) raise(PyExc_ValueError, "la2: not a la2_desc");
  }
  const la2_desc* get() const { return &desc; }
};
template <typename T>
struct Integer {
  T value;
  explicit Integer(PyObject* o) {
    const long long x = PyLong_AsLongLong(o);
    if (x == -1 && PyErr_Occurred()) throw Raised{};
    value = (T)x;
    if ((long long)value != x) raise(PyExc_OverflowError, "la2: an integer argument out of range");
  }
  T get() const { return value; }
};
template <>
struct Arg<int32_t> : Integer<int32_t> { using Integer::Integer; };
template <>
struct Arg<int64_t> : Integer<int64_t> { using Integer::Integer; };
template <>
struct Arg<size_t> {
  size_t value;
  explicit Arg(PyObject* o) {
    if (o == Py_None) {
      value = 0;
    } else if (THPVariable_Check(o)) {
      const at::Tensor& t = THPVariable_Unpack(o);
      value = (size_t)t.numel() * t.element_size();
    } else {
      value = PyLong_AsSize_t(o);
      if (PyErr_Occurred()) throw Raised{};
    }
  }
  size_t get() const { return value; }
};
template <>
struct Arg<float> {
  float value;
  explicit Arg(PyObject* o) {   // what float(o) takes
    PyObject* const f = PyNumber_Float(o);
    if (f == nullptr) throw Raised{};
    value = (float)PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
  }
  float get() const { return value; }
};

template <typename F>
PyObject* guarded(F f) {
  try {
    return f();
  } catch (const Raised&) {
  } catch (const std::exception& e) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
  } catch (...) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "la2: unknown C++ exception");
  }
  return nullptr;
}

template <auto F>
struct Entry;
template <typename... A, la2_status (*F)(A...)>
struct Entry<F> {
  template <size_t... I>
  static PyObject* run(PyObject* const* args, std::index_sequence<I...>) {
    const std::tuple<Arg<A>...> a{Arg<A>(args[I])...};
    la2_status st;
    Py_BEGIN_ALLOW_THREADS
    st = F(std::get<I>(a).get()...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
  }
  static PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
      if (n != (Py_ssize_t)sizeof...(A)) {
        PyErr_Format(PyExc_TypeError, "la2: %zd arguments, not %zd", (Py_ssize_t)sizeof...(A), n);
        throw Raised{};
      }
      return run(args, std::index_sequence_for<A...>{});
    });
  }
};

// ---- checks and tensors
// same_layout(ref, ...): ValueError unless all have ref's shape, strides, dtype and device
PyObject* same_layout(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n < 1) raise(PyExc_TypeError, "la2: no tensor");
    const at::Tensor& ref = tensor(args[0]);
    for (Py_ssize_t i = 1; i < n; i++) {
      const at::Tensor& o = tensor(args[i]);
      if (o.sizes() != ref.sizes() || o.strides() != ref.strides() || o.scalar_type() != ref.scalar_type() || o.device() != ref.device())
        raise(PyExc_ValueError, "la2: all sequence tensors must share shape, strides, dtype and device");
    }
    Py_RETURN_NONE;
  });
}

// The Python functions hand these arguments on as they are, and an entry point also takes a number for a pointer: the caller's own
// number is refused here, before it can become an address on the device.
void tensor_or_none(PyObject* o) {
  if (o != Py_None) tensor(o);
}

// given(lam, ...): TypeError unless lam is a tensor and every other one a tensor or None
PyObject* given(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n < 1) raise(PyExc_TypeError, "la2: no decay");
    tensor(args[0]);
    for (Py_ssize_t i = 1; i < n; i++) tensor_or_none(args[i]);
    Py_RETURN_NONE;
  });
}

// like(t): an uninitialised tensor of t's shape, strides, dtype and device
PyObject* like(PyObject*, PyObject* arg) {
  return guarded([&] {
    const at::Tensor& t = tensor(arg);
    return THPVariable_Wrap(at::empty_strided(t.sizes(), t.strides(), at::TensorOptions().dtype(t.dtype()).device(t.device())));
  });
}

// f32(t, extent, ...): an uninitialised fp32 tensor of these extents on t's device
PyObject* f32(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&] {
    int64_t size[8];
    if (n < 1 || n > 9) raise(PyExc_TypeError, "la2: one to eight extents");
    for (Py_ssize_t i = 1; i < n; i++) size[i - 1] = Integer<int64_t>(args[i]).get();
    return THPVariable_Wrap(at::empty(at::IntArrayRef(size, n - 1), at::TensorOptions().dtype(at::kFloat).device(tensor(args[0]).device())));
  });
}

// workspace(t, op): the workspace that la2_workspace_bytes asks for, or None
PyObject* workspace(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 2) raise(PyExc_TypeError, "la2: a tensor and an operation");
    const at::Tensor& t = tensor(args[0]);
    const la2_desc d = desc_of(t);
    const size_t need = la2_workspace_bytes(&d, Integer<int32_t>(args[1]).get());
    if (need == 0) Py_RETURN_NONE;
    return THPVariable_Wrap(at::empty({(int64_t)need}, at::TensorOptions().dtype(at::kByte).device(t.device())));
  });
}

// state(s, t, name[, sequences]): s where it is a dense fp32 [batch, heads, d, d] state of t [batch, heads, n, d] (or
// [sequences, heads, d, d] of a packed t [positions, heads, d]) on t's device; None for None and for a state of no elements
PyObject* state(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 3 && n != 4) raise(PyExc_TypeError, "la2: a state, a tensor, a name and a number of sequences");
    if (args[0] == Py_None) Py_RETURN_NONE;
    const at::Tensor &s = tensor(args[0]), &t = tensor(args[1]);
    const int64_t d = t.size(-1), rows = n == 4 ? Integer<int64_t>(args[3]).get() : t.size(0), heads = t.size(1);
    if (s.scalar_type() != at::kFloat || s.dim() != 4 || s.size(0) != rows || s.size(1) != heads || s.size(2) != d || s.size(3) != d ||
        !s.is_contiguous() || s.device() != t.device()) {
      PyErr_Format(PyExc_ValueError, "%U must be dense fp32 %s on the tensors' device", args[2],
                   n == 4 ? "[sequences, H, d, d]" : "[b, H, d, d]");
      throw Raised{};
    }
    if (s.numel() == 0) Py_RETURN_NONE;
    Py_INCREF(args[0]);
    return args[0];
  });
}

// decode_shape(name, dims, q, k, v, kv[, lam, ...]): checks a decoding call's tensors (dims 3: [b, H, d], 4: [b, H, T, d]; lam and what
// follows as given() does); q's extents and the dtype's code
PyObject* decode_shape(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n < 6) raise(PyExc_TypeError, "la2: name, dims, q, k, v, kv");
    if (n > 6) tensor(args[6]);
    for (Py_ssize_t i = 7; i < n; i++) tensor_or_none(args[i]);
    const int64_t dims = Integer<int64_t>(args[1]).get();
    const at::Tensor& q = tensor(args[2]);
    if (q.dim() != dims) {
      PyErr_Format(PyExc_ValueError, "%U: q must have %d dimensions", args[0], (int)dims);
      throw Raised{};
    }
    for (int i = 2; i < 5; i++) {
      const at::Tensor& x = tensor(args[i]);
      if (x.sizes() != q.sizes() || x.scalar_type() != q.scalar_type() || !x.is_contiguous()) {
        PyErr_Format(PyExc_ValueError, "%U: q, k, v must be dense %s of one dtype", args[0], dims == 3 ? "[b, H, d]" : "[b, H, T, d]");
        throw Raised{};
      }
    }
    const at::Tensor& kv = tensor(args[5]);
    const int64_t d = q.size(dims - 1);
    if (kv.scalar_type() != at::kFloat || kv.dim() != 4 || kv.size(0) != q.size(0) || kv.size(1) != q.size(1) || kv.size(2) != d ||
        kv.size(3) != d || !kv.is_contiguous()) {
      PyErr_Format(PyExc_ValueError, "%U: kv_state must be dense fp32 [b, H, d, d]", args[0]);
      throw Raised{};
    }
    const int code = dtype_code(q);
    if (dims == 3) return Py_BuildValue("LLLi", (long long)q.size(0), (long long)q.size(1), (long long)d, code);
    return Py_BuildValue("LLLLi", (long long)q.size(0), (long long)q.size(1), (long long)q.size(2), (long long)d, code);
  });
}

#define FAST(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL, nullptr}
#define ENTRY(f) FAST(#f, (&Entry<f>::call))
PyMethodDef methods[] = {
    ENTRY(la2_fwd), ENTRY(la2_fwd_noalloc), ENTRY(la2_bwd), ENTRY(la2_fwd_state), ENTRY(la2_bwd_saved), ENTRY(la2_fwd_norm),
    ENTRY(la2_bwd_norm), ENTRY(la2_fwd_state_norm), ENTRY(la2_bwd_state_norm), ENTRY(la2_fwd_varlen), ENTRY(la2_bwd_varlen),
    ENTRY(la2_fwd_varlen_state), ENTRY(la2_bwd_varlen_state), ENTRY(la2_fwd_varlen_norm), ENTRY(la2_bwd_varlen_norm),
    ENTRY(la2_decode_step), ENTRY(la2_decode_step_norm), ENTRY(la2_decode_multi), ENTRY(la2_decode_multi_norm),
    ENTRY(la2_left_product_fwd), ENTRY(la2_left_product_bwd),
    FAST("same_layout", same_layout), FAST("given", given), FAST("f32", f32), FAST("workspace", workspace), FAST("state", state),
    FAST("decode_shape", decode_shape),
    {"like", like, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
#undef ENTRY
#undef FAST

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_la2_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the Python and the torch whose headers this was compiled with; the binding refuses any other (a tensor's layout in memory
// is what the checks above read)
PyMODINIT_FUNC PyInit__la2_native() {
  PyObject* const m = PyModule_Create(&module);
  if (m == nullptr) return nullptr;
  PyObject* const built = Py_BuildValue("(iis)", PY_MAJOR_VERSION, PY_MINOR_VERSION, LA2_TORCH_VERSION);
  if (built == nullptr || PyModule_AddObject(m, "built_for", built) != 0) {
    Py_XDECREF(built);
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
