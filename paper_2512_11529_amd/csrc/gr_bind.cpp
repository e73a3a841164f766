// Argument marshalling of the Python binding for the calls of the decode loop: tensors are checked, the parameter structs of
// the C ABI are filled and the calls made here.  In Python (per-attribute checks, ctypes structs) this took 8 to 13 us a call, longer
// than the kernels of a small batch; here it is about one.  Host code only; the library is reached through the addresses that
// bind() is given, so whatever libgr.so the package has loaded is the one that runs.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>

#include "gr.h"

namespace {

decltype(&gr_beam_attn) p_attn = nullptr;
decltype(&gr_beam_attn_slots) p_attn_slots = nullptr;
decltype(&gr_beam_attn_fp8kv) p_attn_fp8kv = nullptr;
decltype(&gr_beam_attn_workspace_bytes) p_attn_ws = nullptr;
decltype(&gr_prefill_attn) p_prefill = nullptr;
decltype(&gr_beam_select) p_select = nullptr;
decltype(&gr_beam_select_noalloc) p_select_noalloc = nullptr;
decltype(&gr_beam_select_workspace_bytes) p_select_ws = nullptr;
decltype(&gr_beam_reorder) p_reorder = nullptr;
decltype(&gr_beam_slot_update) p_slot_update = nullptr;

struct Error {};        // a Python exception is set

std::string shape_text(c10::IntArrayRef s) {
  std::string t = "(";
  for (size_t i = 0; i < s.size(); i++) t += (i ? ", " : "") + std::to_string(s[i]);
  return t + (s.size() == 1 ? ",)" : ")");
}
const char* dtype_text(at::ScalarType t) {
  return t == at::kBFloat16 ? "torch.bfloat16" : t == at::kFloat ? "torch.float32" : t == at::kInt ? "torch.int32" : t == at::kByte ? "torch.uint8" : "another type";
}

// A contiguous GPU tensor of the type; of so many dimensions, or of the shape.
const at::Tensor& tensor_nd(PyObject* o, at::ScalarType dt, const char* name, int dims) {
  const at::Tensor* t = THPVariable_Check(o) ? &THPVariable_Unpack(o) : nullptr;
  if (!t || !t->is_cuda() || !t->is_contiguous()) {
    PyErr_Format(PyExc_TypeError, "%s: expected a contiguous CUDA tensor", name);
    throw Error();
  }
  if (t->scalar_type() != dt) {
    PyErr_Format(PyExc_TypeError, "%s: expected %s, got %s", name, dtype_text(dt), dtype_text(t->scalar_type()));
    throw Error();
  }
  if (t->dim() != dims) {
    PyErr_Format(PyExc_ValueError, "%s: expected %d dimensions, got shape %s", name, dims, shape_text(t->sizes()).c_str());
    throw Error();
  }
  return *t;
}
const at::Tensor& tensor(PyObject* o, at::ScalarType dt, const char* name, c10::IntArrayRef shape) {
  const at::Tensor* t = THPVariable_Check(o) ? &THPVariable_Unpack(o) : nullptr;
  if (t && t->is_cuda() && t->is_contiguous() && t->scalar_type() == dt && t->sizes() != shape) {
    PyErr_Format(PyExc_ValueError, "%s: expected shape %s, got %s", name, shape_text(shape).c_str(), shape_text(t->sizes()).c_str());
    throw Error();
  }
  return tensor_nd(o, dt, name, (int)shape.size());
}
const void* any_tensor(PyObject* o, size_t* bytes) {        // None or a tensor of any kind
  if (o == Py_None) { *bytes = 0; return nullptr; }
  if (!THPVariable_Check(o)) { PyErr_SetString(PyExc_TypeError, "expected a tensor or None"); throw Error(); }
  const at::Tensor& t = THPVariable_Unpack(o);
  *bytes = (size_t)t.numel() * t.element_size();
  return t.data_ptr();
}
long long integer(PyObject* o) {                            // int(o)
  if (PyLong_CheckExact(o)) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Error();
    return v;
  }
  PyObject* i = PyNumber_Long(o);
  if (!i) throw Error();
  const long long v = PyLong_AsLongLong(i);
  Py_DECREF(i);
  if (v == -1 && PyErr_Occurred()) throw Error();
  return v;
}
double real(PyObject* o) {                                  // float(o)
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Error();
  return v;
}
PyObject* current_stream = nullptr;                         // callable: the current stream's handle
void* stream_of(PyObject* o) {                              // a torch stream, or None for the current one
  PyObject* h = o == Py_None ? PyObject_CallNoArgs(current_stream) : PyObject_GetAttrString(o, "cuda_stream");
  if (!h) throw Error();
  const unsigned long long v = PyLong_AsUnsignedLongLongMask(h);
  Py_DECREF(h);
  if (PyErr_Occurred()) throw Error();
  return (void*)(uintptr_t)v;
}
void* pointer(PyObject* o) { return (void*)(uintptr_t)(unsigned long long)integer(o); }
void count(Py_ssize_t n, Py_ssize_t want) {
  if (n != want) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); throw Error(); }
}

template <class F>
PyObject* guarded(F&& f) {
  try {
    return f();
  } catch (const Error&) {
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}
// the call itself, without the interpreter lock (a full launch queue makes it wait)
template <class F>
PyObject* status_of(F&& call) {
  gr_status rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}
PyObject* workspace_wanted(size_t need) { return PyLong_FromUnsignedLongLong(need); }

// attn(q, k, v, cu_seqlens, k_own, v_own, slot | None, u, sm_scale, max_L, total_L, out, lse | None, workspace | None, stream, fp8, k_scale, v_scale)
//   -> status (<= 0), or the workspace bytes that the call needs when none was given
PyObject* attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    count(n, 18);
    const bool fp8 = a[15] == Py_True;
    const at::ScalarType kv = fp8 ? at::kByte : at::kBFloat16;
    const at::Tensor& q = tensor_nd(a[0], at::kBFloat16, "q", 4);
    const int64_t B = q.size(0), W = q.size(1), Hq = q.size(2), d = q.size(3);
    const at::Tensor& k = tensor_nd(a[1], kv, fp8 ? "k_shared_fp8" : "k_shared", 3);
    const int64_t rows = k.size(0), Hkv = k.size(1);
    tensor(a[1], kv, fp8 ? "k_shared_fp8" : "k_shared", {rows, Hkv, d});
    const at::Tensor& v = tensor(a[2], kv, fp8 ? "v_shared_fp8" : "v_shared", {rows, Hkv, d});
    const at::Tensor& cu = tensor(a[3], at::kInt, "cu_seqlens", {B + 1});
    const at::Tensor& ku = tensor_nd(a[4], at::kBFloat16, "k_unshared", 5);
    const int64_t ND = ku.size(2);
    tensor(a[4], at::kBFloat16, "k_unshared", {B, W, ND, Hkv, d});
    const at::Tensor& vu = tensor(a[5], at::kBFloat16, "v_unshared", {B, W, ND, Hkv, d});
    const long long total_L = integer(a[10]);
    if (rows < total_L) {
      PyErr_Format(PyExc_ValueError, "%s has fewer rows than total_L", fp8 ? "k_shared_fp8" : "k_shared");
      throw Error();
    }
    const at::Tensor& out = tensor(a[11], at::kBFloat16, "out", {B, W, Hq, d});
    gr_attn_fp8kv_params p;
    p.attn.B = (int32_t)B; p.attn.W = (int32_t)W; p.attn.Hq = (int32_t)Hq; p.attn.Hkv = (int32_t)Hkv; p.attn.d = (int32_t)d;
    p.attn.ND = (int32_t)ND; p.attn.u = (int32_t)integer(a[7]);
    p.attn.max_L = (int32_t)integer(a[9]); p.attn.total_L = total_L; p.attn.sm_scale = (float)real(a[8]);
    p.attn.q = q.data_ptr(); p.attn.k_shared = k.data_ptr(); p.attn.v_shared = v.data_ptr(); p.attn.cu_seqlens = (const int32_t*)cu.data_ptr();
    p.attn.k_unshared = ku.data_ptr(); p.attn.v_unshared = vu.data_ptr(); p.attn.out = out.data_ptr();
    p.attn.lse_out = a[12] == Py_None ? nullptr : (float*)tensor(a[12], at::kFloat, "lse_out", {B, W, Hq}).data_ptr();
    p.k_scale = (float)real(a[16]); p.v_scale = (float)real(a[17]);
    const int32_t* slot = a[6] == Py_None ? nullptr : (const int32_t*)tensor(a[6], at::kInt, "slot", {B, W, ND}).data_ptr();
    size_t ws_bytes;
    void* ws = const_cast<void*>(any_tensor(a[13], &ws_bytes));
    void* stream = stream_of(a[14]);
    if (a[13] == Py_None) {
      const size_t need = p_attn_ws(&p.attn);
      if (need > 0) return workspace_wanted(need);
    }
    return status_of([&] {
      return fp8 ? p_attn_fp8kv(&p, ws, ws_bytes, stream) : slot ? p_attn_slots(&p.attn, slot, ws, ws_bytes, stream) : p_attn(&p.attn, ws, ws_bytes, stream);
    });
  });
}

// prefill(q, k, v, cu_seqlens, sm_scale, max_L, total_L, out, lse | None, stream) -> status
PyObject* prefill(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    count(n, 10);
    const at::Tensor& q = tensor_nd(a[0], at::kBFloat16, "q", 3);
    const int64_t T = q.size(0), Hq = q.size(1), d = q.size(2);
    const at::Tensor& k = tensor_nd(a[1], at::kBFloat16, "k", 3);
    const int64_t Hkv = k.size(1);
    tensor(a[1], at::kBFloat16, "k", {T, Hkv, d});
    const at::Tensor& v = tensor(a[2], at::kBFloat16, "v", {T, Hkv, d});
    const at::Tensor& cu = tensor_nd(a[3], at::kInt, "cu_seqlens", 1);
    const long long total_L = integer(a[6]);
    if (T < total_L) { PyErr_SetString(PyExc_ValueError, "q has fewer rows than total_L"); throw Error(); }
    const at::Tensor& out = tensor(a[7], at::kBFloat16, "out", {T, Hq, d});
    gr_prefill_params p;
    p.B = (int32_t)(cu.size(0) - 1); p.Hq = (int32_t)Hq; p.Hkv = (int32_t)Hkv; p.d = (int32_t)d;
    p.max_L = (int32_t)integer(a[5]); p.total_L = total_L; p.sm_scale = (float)real(a[4]);
    p.q = q.data_ptr(); p.k = k.data_ptr(); p.v = v.data_ptr(); p.cu_seqlens = (const int32_t*)cu.data_ptr(); p.out = out.data_ptr();
    p.lse_out = a[8] == Py_None ? nullptr : (float*)tensor(a[8], at::kFloat, "lse_out", {T, Hq}).data_ptr();
    void* stream = stream_of(a[9]);
    return status_of([&] { return p_prefill(&p, stream); });
  });
}

// select(mask | None, logits, scores_in, prefix_in, range_in, step, flags, parent, token, scores, prefix, range, item_index,
//        workspace | None, noalloc, stream) -> status, or the workspace bytes that the call needs
PyObject* select(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    count(n, 16);
    const at::Tensor& logits = tensor_nd(a[1], at::kFloat, "logits", 3);
    const int64_t B = logits.size(0), W = logits.size(1), V = logits.size(2);
    gr_select_params p;
    p.logits = (const float*)logits.data_ptr();
    p.scores_in = (const float*)tensor(a[2], at::kFloat, "scores_in", {B, W}).data_ptr();
    const at::Tensor& prefix = tensor_nd(a[3], at::kInt, "prefix_in", 3);
    const int64_t depth = prefix.size(2);
    p.prefix_in = (const int32_t*)tensor(a[3], at::kInt, "prefix_in", {B, W, depth}).data_ptr();
    p.range_in = (const int32_t*)tensor(a[4], at::kInt, "range_in", {B, W, 2}).data_ptr();
    p.parent_out = (int32_t*)tensor(a[7], at::kInt, "parent", {B, W}).data_ptr();
    p.token_out = (int32_t*)tensor(a[8], at::kInt, "token", {B, W}).data_ptr();
    p.scores_out = (float*)tensor(a[9], at::kFloat, "scores", {B, W}).data_ptr();
    p.prefix_out = (int32_t*)tensor(a[10], at::kInt, "prefix", {B, W, depth}).data_ptr();
    p.range_out = (int32_t*)tensor(a[11], at::kInt, "range", {B, W, 2}).data_ptr();
    p.item_index_out = (int32_t*)tensor(a[12], at::kInt, "item_index", {B, W}).data_ptr();
    p.B = (int32_t)B; p.W = (int32_t)W; p.V = (int32_t)V; p.depth = (int32_t)depth;
    p.step = (int32_t)integer(a[5]); p.flags = (int32_t)integer(a[6]);
    size_t bytes;
    p.mask = any_tensor(a[0], &bytes);
    void* ws = const_cast<void*>(any_tensor(a[13], &bytes));
    const bool noalloc = a[14] == Py_True;
    void* stream = stream_of(a[15]);
    if (!noalloc && a[13] == Py_None) return workspace_wanted(p_select_ws(p.B, p.W, p.V, p.depth));
    return status_of([&] { return noalloc ? p_select_noalloc(&p, stream) : p_select(&p, ws, bytes, stream); });
  });
}

// reorder(parent, k_own, v_own, u, stream) -> status
PyObject* reorder(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    count(n, 5);
    const at::Tensor& k = tensor_nd(a[1], at::kBFloat16, "k_unshared", 5);
    const at::Tensor& parent = tensor(a[0], at::kInt, "parent", {k.size(0), k.size(1)});
    const at::Tensor& v = tensor(a[2], at::kBFloat16, "v_unshared", k.sizes());
    const int32_t u = (int32_t)integer(a[3]);
    void* stream = stream_of(a[4]);
    return status_of([&] {
      return p_reorder((int32_t)k.size(0), (int32_t)k.size(1), (int32_t)k.size(2), (int32_t)k.size(3), (int32_t)k.size(4), u, (const int32_t*)parent.data_ptr(),
                       k.data_ptr(), v.data_ptr(), stream);
    });
  });
}

// slot_update(parent, slot_in | None, u, ND, out, stream) -> status
PyObject* slot_update(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    count(n, 6);
    const at::Tensor& parent = tensor_nd(a[0], at::kInt, "parent", 2);
    const int64_t B = parent.size(0), W = parent.size(1), ND = integer(a[3]);
    const int32_t* slot_in = a[1] == Py_None ? nullptr : (const int32_t*)tensor(a[1], at::kInt, "slot_in", {B, W, ND}).data_ptr();
    int32_t* out = (int32_t*)tensor(a[4], at::kInt, "out", {B, W, ND}).data_ptr();
    const int32_t u = (int32_t)integer(a[2]);
    void* stream = stream_of(a[5]);
    return status_of([&] { return p_slot_update((int32_t)B, (int32_t)W, (int32_t)ND, u, (const int32_t*)parent.data_ptr(), slot_in, out, stream); });
  });
}

// bind(addresses of the ten entry points in the order of their declaration above, callable that returns the current stream's handle)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    count(n, 11);
    p_attn = (decltype(p_attn))pointer(a[0]);
    p_attn_slots = (decltype(p_attn_slots))pointer(a[1]);
    p_attn_fp8kv = (decltype(p_attn_fp8kv))pointer(a[2]);
    p_attn_ws = (decltype(p_attn_ws))pointer(a[3]);
    p_prefill = (decltype(p_prefill))pointer(a[4]);
    p_select = (decltype(p_select))pointer(a[5]);
    p_select_noalloc = (decltype(p_select_noalloc))pointer(a[6]);
    p_select_ws = (decltype(p_select_ws))pointer(a[7]);
    p_reorder = (decltype(p_reorder))pointer(a[8]);
    p_slot_update = (decltype(p_slot_update))pointer(a[9]);
    Py_INCREF(a[10]);
    Py_XSETREF(current_stream, a[10]);
    Py_RETURN_NONE;
  });
}

PyMethodDef methods[] = {{"attn", (PyCFunction)(void*)attn, METH_FASTCALL, nullptr},
                         {"prefill", (PyCFunction)(void*)prefill, METH_FASTCALL, nullptr},
                         {"select", (PyCFunction)(void*)select, METH_FASTCALL, nullptr},
                         {"reorder", (PyCFunction)(void*)reorder, METH_FASTCALL, nullptr},
                         {"slot_update", (PyCFunction)(void*)slot_update, METH_FASTCALL, nullptr},
                         {"bind", (PyCFunction)(void*)bind, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "gr_bind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_gr_bind(void) { return PyModule_Create(&module); }
