// Python module _native: torch tensors -> tr_tensor descriptors -> the C ABI of libtokenring, argument marshalling only.
//
// A call on the smallest sizes is bound by its marshalling: through ctypes, with the descriptors packed by Python, a block step cost
// the host 6.9 us, more than the kernel's own 5.6; here 4.1, of which the launch is most.  What this module does not know (tensor subclasses, tensors without
// strides or storage, wrong types) goes through the Python packer, whose exceptions are the ones callers see.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "tokenring.h"

namespace {

__attribute__((used)) const char source_hash_tag[] = "TR_SOURCE_HASH=" TR_SOURCE_HASH_STR;

// Set once by bind(): packer(tensor) -> bytes, torch.cuda.is_initialized, and torch._C's device and raw stream getters (either
// may be None); stream_of(None) is the way when these do not apply.
PyObject *packer, *is_initialized, *get_device, *raw_stream, *stream_of;

bool pack(PyObject* obj, tr_tensor& d) {
  if (THPVariable_CheckExact(obj)) {
    try {
      const at::Tensor& t = THPVariable_Unpack(obj);
      const auto type = t.scalar_type();
      const int64_t n = t.dim();
      if ((type == at::kBFloat16 || type == at::kFloat) && (n == 3 || n == 4) && t.layout() == at::kStrided) {
        const auto size = t.sizes(), stride = t.strides();
        if (n == 3 || stride[3] == 1 || size[3] <= 1) {
          d.ptr = t.data_ptr();
          d.dtype = type == at::kBFloat16 ? TR_BF16 : TR_F32;
          d.B = size[0]; d.H = size[1]; d.S = size[2]; d.D = n == 4 ? size[3] : 1;
          d.stride_b = stride[0]; d.stride_h = stride[1]; d.stride_s = stride[2];
          return true;
        }
      }
    } catch (...) {   // no storage, symbolic sizes and the like: Python says what is wrong
    }
  }
  PyObject* bytes = PyObject_CallOneArg(packer, obj);
  if (!bytes) return false;
  char* at = nullptr;
  Py_ssize_t n = 0;
  const bool ok = PyBytes_AsStringAndSize(bytes, &at, &n) == 0 && n >= (Py_ssize_t)sizeof(d);
  if (ok) memcpy(&d, at, sizeof(d));
  else if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "a packed descriptor is too short");
  Py_DECREF(bytes);
  return ok;
}

// int(x) as an argument of the C ABI takes it: the low bits.
bool to_int(PyObject* obj, int64_t& x) {
  PyObject* n = PyLong_CheckExact(obj) ? (Py_INCREF(obj), obj) : PyNumber_Long(obj);
  if (!n) return false;
  x = (int64_t)PyLong_AsUnsignedLongLongMask(n);
  Py_DECREF(n);
  return !(x == -1 && PyErr_Occurred());
}
bool to_float(PyObject* obj, float& x) {
  PyObject* f = PyFloat_CheckExact(obj) ? (Py_INCREF(obj), obj) : PyNumber_Float(obj);
  if (!f) return false;
  x = (float)PyFloat_AS_DOUBLE(f);
  Py_DECREF(f);
  return true;
}
bool to_bool(PyObject* obj, int64_t& x) {
  const int b = PyObject_IsTrue(obj);
  x = b;
  return b >= 0;
}

bool to_stream(PyObject* obj, void*& stream) {
  PyObject* handle = nullptr;
  if (obj != Py_None) {
    handle = PyObject_GetAttrString(obj, "cuda_stream");
  } else {
    PyObject* ready = raw_stream == Py_None || get_device == Py_None ? (Py_INCREF(Py_False), Py_False) : PyObject_CallNoArgs(is_initialized);
    if (!ready) return false;
    if (ready == Py_True) {
      PyObject* device = PyObject_CallNoArgs(get_device);
      handle = device ? PyObject_CallOneArg(raw_stream, device) : nullptr;
      Py_XDECREF(device);
    } else {
      handle = PyObject_CallOneArg(stream_of, Py_None);
    }
    Py_DECREF(ready);
  }
  if (!handle) return false;
  int64_t h = 0;
  const bool ok = to_int(handle, h);
  Py_DECREF(handle);
  stream = (void*)(uintptr_t)h;
  return ok;
}

bool argc_is(Py_ssize_t n, Py_ssize_t want) {
  if (n != want) PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
  return n == want;
}
template <typename F>
PyObject* call(F f) {
  tr_status st;
  Py_BEGIN_ALLOW_THREADS
  st = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// q, k, v and, from index `at` on, out and lse
struct Five {
  tr_tensor q, k, v, out, lse;
  bool take(PyObject* const* a, int at) { return pack(a[0], q) && pack(a[1], k) && pack(a[2], v) && pack(a[at], out) && pack(a[at + 1], lse); }
};

PyObject* block_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {   // q, k, v, mask_kind, scale, out, lse, stream
  Five t;
  int64_t mask;
  float scale;
  void* stream;
  if (!argc_is(n, 8) || !t.take(a, 5) || !to_int(a[3], mask) || !to_float(a[4], scale) || !to_stream(a[7], stream)) return nullptr;
  return call([&] { return tr_block_attn(&t.q, &t.k, &t.v, (int)mask, scale, &t.out, &t.lse, stream); });
}
PyObject* block_attn_merge(PyObject*, PyObject* const* a, Py_ssize_t n) {   // the same
  Five t;
  int64_t mask;
  float scale;
  void* stream;
  if (!argc_is(n, 8) || !t.take(a, 5) || !to_int(a[3], mask) || !to_float(a[4], scale) || !to_stream(a[7], stream)) return nullptr;
  return call([&] { return tr_block_attn_merge(&t.q, &t.k, &t.v, (int)mask, scale, &t.out, &t.lse, stream); });
}
PyObject* block_attn_causal_at(PyObject*, PyObject* const* a, Py_ssize_t n) {   // q, k, v, q_pos0, k_pos0, scale, out, lse, stream
  Five t;
  int64_t q0, k0;
  float scale;
  void* stream;
  if (!argc_is(n, 9) || !t.take(a, 6) || !to_int(a[3], q0) || !to_int(a[4], k0) || !to_float(a[5], scale) || !to_stream(a[8], stream)) return nullptr;
  return call([&] { return tr_block_attn_causal_at(&t.q, &t.k, &t.v, q0, k0, scale, &t.out, &t.lse, stream); });
}
PyObject* merge(PyObject*, PyObject* const* a, Py_ssize_t n) {   // out_acc, lse_acc, block_out, block_lse, stream
  tr_tensor t[4];
  void* stream;
  if (!argc_is(n, 5) || !pack(a[0], t[0]) || !pack(a[1], t[1]) || !pack(a[2], t[2]) || !pack(a[3], t[3]) || !to_stream(a[4], stream)) return nullptr;
  return call([&] { return tr_merge(&t[0], &t[1], &t[2], &t[3], stream); });
}
bool pack_all(PyObject* seq, std::vector<tr_tensor>& d, std::vector<const tr_tensor*>& at) {
  PyObject* items = PySequence_Fast(seq, "a sequence of tensors is expected");
  if (!items) return false;
  bool ok = true;
  try {
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(items);
    d.resize(n + 1);
    at.resize(n + 1);
    for (Py_ssize_t i = 0; ok && i < n && i < PySequence_Fast_GET_SIZE(items); i++) {   // (the packer may run Python code)
      ok = pack(PySequence_Fast_GET_ITEM(items, i), d[i]);
      at[i] = &d[i];
    }
  } catch (const std::bad_alloc&) {
    PyErr_NoMemory();
    ok = false;
  }
  Py_DECREF(items);
  return ok;
}
PyObject* merge_n(PyObject*, PyObject* const* a, Py_ssize_t n) {   // out, lse, block_outs, block_lses, accumulate, stream
  tr_tensor out, lse;
  std::vector<tr_tensor> o, l;
  std::vector<const tr_tensor*> po, pl;
  int64_t accumulate;
  void* stream;
  if (!argc_is(n, 6) || !pack_all(a[2], o, po) || !pack_all(a[3], l, pl) || !pack(a[0], out) || !pack(a[1], lse) || !to_bool(a[4], accumulate) ||
      !to_stream(a[5], stream))
    return nullptr;
  if (o.size() != l.size()) {
    PyErr_SetString(PyExc_ValueError, "block_outs and block_lses differ in length");
    return nullptr;
  }
  return call([&] { return tr_merge_n(&out, &lse, po.data(), pl.data(), (int)(o.size() - 1), (int)accumulate, stream); });
}
PyObject* ring_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {   // q, k, v, n_chunks, causal, out, lse, scale, workspace address, bytes, stream
  Five t;
  int64_t chunks, causal, ws, bytes;
  float scale;
  void* stream;
  if (!argc_is(n, 11) || !t.take(a, 5) || !to_int(a[3], chunks) || !to_bool(a[4], causal) || !to_float(a[7], scale) || !to_int(a[8], ws) ||
      !to_int(a[9], bytes) || !to_stream(a[10], stream))
    return nullptr;
  return call([&] {
    return tr_ring_attn(&t.q, &t.k, &t.v, (int)chunks, (int)causal, &t.out, &t.lse, scale, (void*)(uintptr_t)ws, (size_t)bytes, stream);
  });
}
PyObject* ring_attn_noalloc(PyObject*, PyObject* const* a, Py_ssize_t n) {   // q, k, v, n_chunks, causal, out, lse, scale, stream
  Five t;
  int64_t chunks, causal;
  float scale;
  void* stream;
  if (!argc_is(n, 9) || !t.take(a, 5) || !to_int(a[3], chunks) || !to_bool(a[4], causal) || !to_float(a[7], scale) || !to_stream(a[8], stream)) return nullptr;
  return call([&] { return tr_ring_attn_noalloc(&t.q, &t.k, &t.v, (int)chunks, (int)causal, &t.out, &t.lse, scale, stream); });
}
PyObject* ring_attn_sched(PyObject*, PyObject* const* a, Py_ssize_t n) {   // q, k, v, n_devices, causal, schedule, n_inner, out, lse, scale, stream
  Five t;
  int64_t devices, causal, schedule, inner;
  float scale;
  void* stream;
  if (!argc_is(n, 11) || !t.take(a, 7) || !to_int(a[3], devices) || !to_bool(a[4], causal) || !to_int(a[5], schedule) || !to_int(a[6], inner) ||
      !to_float(a[9], scale) || !to_stream(a[10], stream))
    return nullptr;
  return call([&] {
    return tr_ring_attn_sched(&t.q, &t.k, &t.v, (int)devices, (int)causal, (int)schedule, (int)inner, &t.out, &t.lse, scale, stream);
  });
}
PyObject* ring_attn_blocks(PyObject*, PyObject* const* a, Py_ssize_t n) {   // q, k, v, n_chunks, causal, out, lse, scale, block_dtype, ws address, bytes, stream
  Five t;
  int64_t chunks, causal, dtype, ws, bytes;
  float scale;
  void* stream;
  if (!argc_is(n, 12) || !t.take(a, 5) || !to_int(a[3], chunks) || !to_bool(a[4], causal) || !to_float(a[7], scale) || !to_int(a[8], dtype) ||
      !to_int(a[9], ws) || !to_int(a[10], bytes) || !to_stream(a[11], stream))
    return nullptr;
  return call([&] {
    return tr_ring_attn_blocks(&t.q, &t.k, &t.v, (int)chunks, (int)causal, &t.out, &t.lse, scale, (int)dtype, (void*)(uintptr_t)ws, (size_t)bytes, stream);
  });
}
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!argc_is(n, 5)) return nullptr;
  PyObject** const slots[5] = {&packer, &is_initialized, &get_device, &raw_stream, &stream_of};
  for (int i = 0; i < 5; i++) {
    Py_INCREF(a[i]);
    PyObject* old = *slots[i];
    *slots[i] = a[i];
    Py_XDECREF(old);
  }
  Py_RETURN_NONE;
}

#define TR_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {TR_METHOD(bind), TR_METHOD(block_attn), TR_METHOD(block_attn_merge), TR_METHOD(block_attn_causal_at), TR_METHOD(merge),
                         TR_METHOD(merge_n), TR_METHOD(ring_attn), TR_METHOD(ring_attn_noalloc), TR_METHOD(ring_attn_sched),
                         TR_METHOD(ring_attn_blocks), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Calls into libtokenring with torch tensors; status codes come back.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
