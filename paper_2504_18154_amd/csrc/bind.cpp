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

struct NotTaken {};  // thrown for arguments that are binding.py's business

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw NotTaken();
  return THPVariable_Unpack(o);
}
void* address(PyObject* o) { return o == Py_None ? nullptr : tensor(o).data_ptr(); }
template <typename T>
T* as(PyObject* o) {
  return static_cast<T*>(address(o));
}

int32_t narrow(int64_t n) {
  if (n < std::numeric_limits<int32_t>::min() || n > std::numeric_limits<int32_t>::max()) throw NotTaken();
  return (int32_t)n;
}
int64_t integer(PyObject* o) {
  int overflow = 0;
  if (!PyLong_CheckExact(o)) throw NotTaken();
  const long long n = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow) throw NotTaken();
  return n;
}
void* handle(PyObject* o) { return reinterpret_cast<void*>((uintptr_t)integer(o)); }

int32_t size(PyObject* o, int64_t d) {
  const at::Tensor& t = tensor(o);
  if (t.dim() <= d) throw NotTaken();
  return narrow(t.size(d));
}
int32_t numel(PyObject* o) { return narrow(tensor(o).numel()); }
// Elements between consecutive tokens of a [tokens, heads, D] tensor or view whose heads are contiguous.
int64_t row_stride(PyObject* o) {
  const at::Tensor& t = tensor(o);
  if (t.dim() != 3 || t.stride(2) != 1 || t.stride(1) != t.size(2)) throw NotTaken();
  return t.size(0) > 1 ? t.stride(0) : t.size(1) * t.size(2);
}
int32_t or_all(PyObject* most, int32_t all) { return most == Py_None ? all : narrow(integer(most)); }
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Runs f with `want` arguments at hand; -1: not taken.
template <typename F>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, F f) {
  int status = -1;
  try {
    if (n == want) status = f();
  } catch (...) {  // (NotTaken, and what torch throws for a tensor without storage: the other way raises it again, for the caller)
    status = -1;
  }
  return PyLong_FromLong(status);
}
template <typename F>
int unlocked(F f) {
  struct Unlocked {
    PyThreadState* const state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
  } scope;
  return f();
}

// (handle, k_cache, v_cache, k_new, v_new, cu_q, ctx_before, block_table, max_new_len, row stride of a packed array or 0: the tensors')
PyObject* kv_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 10, [&] {
    auto* const c = static_cast<ecoserve_ctx*>(handle(a[0]));
    void *const kc = address(a[1]), *const vc = address(a[2]), *const kn = address(a[3]), *const vn = address(a[4]);
    const auto *cu = as<const int32_t>(a[5]), *before = as<const int32_t>(a[6]), *table = as<const int32_t>(a[7]);
    const int32_t B = numel(a[6]), T = size(a[3], 0), width = size(a[7], 1), most = or_all(a[8], T);
    int64_t stride = integer(a[9]);
    if (stride == 0) {
      stride = row_stride(a[3]);
      if (stride != row_stride(a[4])) throw NotTaken();
    }
    void* const s = stream();
    return unlocked([&] { return entry.append(c, kc, vc, kn, vn, stride, cu, before, table, width, B, T, most, s); });
  });
}

// (handle, q, k_cache, v_cache, cu_q, ctx_before, block_table, out, lse, max_q_len, row stride of a packed array or 0: the tensor's)
PyObject* attn_prefill(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&] {
    auto* const c = static_cast<ecoserve_ctx*>(handle(a[0]));
    void *const q = address(a[1]), *const kc = address(a[2]), *const vc = address(a[3]), *const out = address(a[7]);
    const auto *cu = as<const int32_t>(a[4]), *before = as<const int32_t>(a[5]), *table = as<const int32_t>(a[6]);
    auto* const lse = as<float>(a[8]);
    const int32_t B = numel(a[5]), T = size(a[1], 0), width = size(a[6], 1), most = or_all(a[9], T);
    const int64_t packed = integer(a[10]), stride = packed ? packed : row_stride(a[1]);
    void* const s = stream();
    return unlocked([&] { return entry.prefill(c, q, stride, kc, vc, cu, before, table, width, out, lse, B, T, most, s); });
  });
}

// (handle, q, k_cache, v_cache, block_table, ctx_len, out, max_ctx_len, lse, row stride of a packed array or 0: the tensor's)
PyObject* attn_decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 10, [&] {
    auto* const c = static_cast<ecoserve_ctx*>(handle(a[0]));
    void *const q = address(a[1]), *const kc = address(a[2]), *const vc = address(a[3]), *const out = address(a[6]);
    const auto *table = as<const int32_t>(a[4]), *len = as<const int32_t>(a[5]);
    auto* const lse = as<float>(a[8]);
    const int32_t B = numel(a[5]), width = size(a[4], 1), most = narrow(integer(a[7]));
    const int64_t packed = integer(a[9]), stride = packed ? packed : row_stride(a[1]);
    void* const s = stream();
    return unlocked([&] { return entry.decode(c, q, stride, kc, vc, table, width, len, out, lse, B, most, s); });
  });
}

// (handle, q, k_new, v_new, k_cache, v_cache, block_table, ctx_len, out, max_ctx_len, lse)
PyObject* attn_decode_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&] {
    auto* const c = static_cast<ecoserve_ctx*>(handle(a[0]));
    const int64_t stride = row_stride(a[1]), fresh = row_stride(a[2]);
    if (fresh != row_stride(a[3])) throw NotTaken();
    void *const q = address(a[1]), *const kn = address(a[2]), *const vn = address(a[3]), *const kc = address(a[4]), *const vc = address(a[5]), *const out = address(a[8]);
    const auto *table = as<const int32_t>(a[6]), *len = as<const int32_t>(a[7]);
    auto* const lse = as<float>(a[10]);
    const int32_t B = numel(a[7]), width = size(a[6], 1), most = narrow(integer(a[9]));
    void* const s = stream();
    return unlocked([&] { return entry.decode_append(c, q, stride, kn, vn, fresh, kc, vc, table, width, len, out, lse, B, most, s); });
  });
}

// (device, address of the layout, q, k_cache, v_cache, block_table, ctx_len, out, max_ctx_len, lse)
PyObject* attn_decode_noalloc(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 10, [&] {
    const int32_t device = narrow(integer(a[0]));
    const auto* const layout = static_cast<const ecoserve_layout*>(handle(a[1]));
    void *const q = address(a[2]), *const kc = address(a[3]), *const vc = address(a[4]), *const out = address(a[7]);
    const auto *table = as<const int32_t>(a[5]), *len = as<const int32_t>(a[6]);
    auto* const lse = as<float>(a[9]);
    const int32_t B = numel(a[6]), width = size(a[5], 1), most = narrow(integer(a[8]));
    void* const s = stream();
    return unlocked([&] { return entry.noalloc(device, layout, q, kc, vc, table, width, len, out, lse, B, most, s); });
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
