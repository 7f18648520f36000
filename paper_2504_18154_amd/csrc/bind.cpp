// The marshalling of the hot calls' arguments (binding.py) in C++: tensors to addresses, sizes and row strides, the current
// stream's handle, and the call of the C ABI without the interpreter's lock.  Every function returns the call's status, or -1 for
// arguments that it does not take (anything but tensors or None, and integers of 32 bits): binding.py then goes the way through ctypes, which
// decides what such arguments mean and raises what is to be raised.
//
// Why: a call on a small batch keeps the GPU busy for 4 to 8 us, and the way through ctypes took the host 5.3 to 5.9 before the
// launch, of which 2 to 3 were a method call into the tensor per address and dimension; here it is 0.8 to 1.  Launches included, the
// host takes 64 us for 16 decode calls on one sequence (111 before; the device 131), 134 us for 16 times append and prefill of one short
// prompt (185 before), about as long as the device (132 replayed from a graph): 188 -> 132 to 147 us back to back.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <limits>

#include "../../include/ecoserve.h"

namespace {

// The entry points, as the library that binding.py has loaded holds them.
struct Entries {
  decltype(&ecoserve_kv_append_strided) append;
  decltype(&ecoserve_attn_prefill_strided) prefill;
  decltype(&ecoserve_attn_decode_strided) decode;
  decltype(&ecoserve_attn_decode_append) decode_append;
  decltype(&ecoserve_attn_decode_noalloc) noalloc;
} entry;

// Reads the arguments of a call.  What is binding.py's business is noted, and not thrown: an exception takes 2.5 us, half of what the
// other way takes for such a call.
struct Arguments {
  PyObject* const* a;
  bool taken = true;

  const at::Tensor* tensor(int i) {
    if (THPVariable_CheckExact(a[i])) return &THPVariable_Unpack(a[i]);
    taken = false;
    return nullptr;
  }
  void* address(int i) {
    if (a[i] == Py_None) return nullptr;
    const at::Tensor* const t = tensor(i);
    return t ? t->data_ptr() : nullptr;
  }
  template <typename T>
  T* as(int i) {
    return static_cast<T*>(address(i));
  }
  int32_t narrow(int64_t n) {
    if (n < std::numeric_limits<int32_t>::min() || n > std::numeric_limits<int32_t>::max()) taken = false;
    return (int32_t)n;
  }
  int64_t integer(int i) {
    if (!PyLong_CheckExact(a[i])) return taken = false;
    int overflow = 0;
    const long long n = PyLong_AsLongLongAndOverflow(a[i], &overflow);
    if (overflow) taken = false;
    return n;
  }
  int32_t narrow_integer(int i) { return narrow(integer(i)); }
  void* handle(int i) { return reinterpret_cast<void*>((uintptr_t)integer(i)); }
  int32_t size(int i, int64_t d) {
    const at::Tensor* const t = tensor(i);
    if (t && t->dim() > d) return narrow(t->size(d));
    return taken = false;
  }
  int32_t numel(int i) {
    const at::Tensor* const t = tensor(i);
    return t ? narrow(t->numel()) : 0;
  }
  // Elements between consecutive tokens of a [tokens, heads, D] tensor or view whose heads are contiguous.
  int64_t row_stride(int i) {
    const at::Tensor* const t = tensor(i);
    if (!t || t->dim() != 3 || t->stride(2) != 1 || t->stride(1) != t->size(2)) return taken = false;
    return t->size(0) > 1 ? t->stride(0) : t->size(1) * t->size(2);
  }
  int32_t or_all(int i, int32_t all) { return a[i] == Py_None ? all : narrow_integer(i); }
};

// Runs f on `want` arguments; -1: not taken.
template <typename F>
PyObject* guarded(PyObject* const* a, Py_ssize_t n, Py_ssize_t want, F f) {
  int status = -1;
  try {
    Arguments in{a};
    if (n == want) status = f(in);
  } catch (...) {  // (what torch throws for a tensor without storage: the other way raises it again, for the caller)
    status = -1;
  }
  return PyLong_FromLong(status);
}
// The call itself on the current stream, without the interpreter's lock, if all its arguments are taken.
template <typename F>
int unlocked(const Arguments& in, F f) {
  if (!in.taken) return -1;
  void* const s = c10::hip::getCurrentHIPStream().stream();
  struct Unlocked {
    PyThreadState* const state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
  } scope;
  return f(s);
}

// (handle, k_cache, v_cache, k_new, v_new, cu_q, ctx_before, block_table, max_new_len, row stride of a packed array or 0: the tensors')
PyObject* kv_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(a, n, 10, [](Arguments& in) {
    auto* const c = static_cast<ecoserve_ctx*>(in.handle(0));
    void *const kc = in.address(1), *const vc = in.address(2), *const kn = in.address(3), *const vn = in.address(4);
    const auto *cu = in.as<const int32_t>(5), *before = in.as<const int32_t>(6), *table = in.as<const int32_t>(7);
    const int32_t B = in.numel(6), T = in.size(3, 0), width = in.size(7, 1), most = in.or_all(8, T);
    int64_t stride = in.integer(9);
    if (stride == 0) {
      stride = in.row_stride(3);
      if (stride != in.row_stride(4)) in.taken = false;
    }
    return unlocked(in, [&](void* s) { return entry.append(c, kc, vc, kn, vn, stride, cu, before, table, width, B, T, most, s); });
  });
}

// (handle, q, k_cache, v_cache, cu_q, ctx_before, block_table, out, lse, max_q_len, row stride of a packed array or 0: the tensor's)
PyObject* attn_prefill(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(a, n, 11, [](Arguments& in) {
    auto* const c = static_cast<ecoserve_ctx*>(in.handle(0));
    void *const q = in.address(1), *const kc = in.address(2), *const vc = in.address(3), *const out = in.address(7);
    const auto *cu = in.as<const int32_t>(4), *before = in.as<const int32_t>(5), *table = in.as<const int32_t>(6);
    auto* const lse = in.as<float>(8);
    const int32_t B = in.numel(5), T = in.size(1, 0), width = in.size(6, 1), most = in.or_all(9, T);
    const int64_t packed = in.integer(10), stride = packed ? packed : in.row_stride(1);
    return unlocked(in, [&](void* s) { return entry.prefill(c, q, stride, kc, vc, cu, before, table, width, out, lse, B, T, most, s); });
  });
}

// (handle, q, k_cache, v_cache, block_table, ctx_len, out, max_ctx_len, lse, row stride of a packed array or 0: the tensor's)
PyObject* attn_decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(a, n, 10, [](Arguments& in) {
    auto* const c = static_cast<ecoserve_ctx*>(in.handle(0));
    void *const q = in.address(1), *const kc = in.address(2), *const vc = in.address(3), *const out = in.address(6);
    const auto *table = in.as<const int32_t>(4), *len = in.as<const int32_t>(5);
    auto* const lse = in.as<float>(8);
    const int32_t B = in.numel(5), width = in.size(4, 1), most = in.narrow_integer(7);
    const int64_t packed = in.integer(9), stride = packed ? packed : in.row_stride(1);
    return unlocked(in, [&](void* s) { return entry.decode(c, q, stride, kc, vc, table, width, len, out, lse, B, most, s); });
  });
}

// (handle, q, k_new, v_new, k_cache, v_cache, block_table, ctx_len, out, max_ctx_len, lse)
PyObject* attn_decode_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(a, n, 11, [](Arguments& in) {
    auto* const c = static_cast<ecoserve_ctx*>(in.handle(0));
    const int64_t stride = in.row_stride(1), fresh = in.row_stride(2);
    if (fresh != in.row_stride(3)) in.taken = false;
    void *const q = in.address(1), *const kn = in.address(2), *const vn = in.address(3), *const kc = in.address(4), *const vc = in.address(5), *const out = in.address(8);
    const auto *table = in.as<const int32_t>(6), *len = in.as<const int32_t>(7);
    auto* const lse = in.as<float>(10);
    const int32_t B = in.numel(7), width = in.size(6, 1), most = in.narrow_integer(9);
    return unlocked(in, [&](void* s) { return entry.decode_append(c, q, stride, kn, vn, fresh, kc, vc, table, width, len, out, lse, B, most, s); });
  });
}

// (device, address of the layout, q, k_cache, v_cache, block_table, ctx_len, out, max_ctx_len, lse)
PyObject* attn_decode_noalloc(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(a, n, 10, [](Arguments& in) {
    const int32_t device = in.narrow_integer(0);
    const auto* const layout = static_cast<const ecoserve_layout*>(in.handle(1));
    void *const q = in.address(2), *const kc = in.address(3), *const vc = in.address(4), *const out = in.address(7);
    const auto *table = in.as<const int32_t>(5), *len = in.as<const int32_t>(6);
    auto* const lse = in.as<float>(9);
    const int32_t B = in.numel(6), width = in.size(5, 1), most = in.narrow_integer(8);
    return unlocked(in, [&](void* s) { return entry.noalloc(device, layout, q, kc, vc, table, width, len, out, lse, B, most, s); });
  });
}

// (addresses of the entry points, in the order of Entries)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* at[5];
  if (n != 5) {
    PyErr_SetString(PyExc_TypeError, "bind() takes five addresses");
    return nullptr;
  }
  for (int i = 0; i < 5; ++i) {
    at[i] = PyLong_AsVoidPtr(a[i]);
    if (!at[i] && PyErr_Occurred()) return nullptr;
  }
  entry.append = reinterpret_cast<decltype(entry.append)>(at[0]);
  entry.prefill = reinterpret_cast<decltype(entry.prefill)>(at[1]);
  entry.decode = reinterpret_cast<decltype(entry.decode)>(at[2]);
  entry.decode_append = reinterpret_cast<decltype(entry.decode_append)>(at[3]);
  entry.noalloc = reinterpret_cast<decltype(entry.noalloc)>(at[4]);
  Py_RETURN_NONE;
}

#define ECO_FAST(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ECO_FAST(bind), ECO_FAST(kv_append), ECO_FAST(attn_prefill), ECO_FAST(attn_decode), ECO_FAST(attn_decode_append),
                         ECO_FAST(attn_decode_noalloc), {nullptr, nullptr, 0, nullptr}};
// (ECO_BIND_FITS: the interpreter and the torch that this is compiled for; build.py looks for it in the built file)
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bind", "Marshalling of the hot calls' arguments, " ECO_BIND_FITS, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bind() { return PyModule_Create(&module); }
