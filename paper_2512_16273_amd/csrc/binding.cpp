// The calls of a serving loop from Python without ctypes: the same checks as in tslt.py, made on the tensors themselves, then
// the library's function (whose address tslt.load() hands over, so that any build of the ABI will do).  Whatever is not the plain case
// (another type, layout, device, a missing tensor) returns None, and tslt.py goes through it step by step and says what is wrong.
//
// A call through ctypes costs the host 7 us beside its launches (twenty arguments converted, four questions to each of eight tensors), more
// than half of what a small call takes on the device; so 1 to 2.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/autograd/python_variable.h>

#include "tslt.h"

namespace {

struct Library {
  decltype(&tslt_workspace_bytes) workspace_bytes;
  decltype(&tslt_truncate_sample) truncate_sample;
  decltype(&tslt_verify) verify, verify_accept, verify_resample;
  decltype(&tslt_verify_tree) verify_tree;
  decltype(&tslt_pack_bound_words) pack_bound_words;
  decltype(&tslt_pack_cleared) pack_cleared;
  decltype(&tslt_unpack) unpack;
} lib;
bool bound = false;

PyObject *k_idx, *k_logit, *k_prob, *k_count, *k_mass, *k_status, *k_token, *k_slot, *k_accept_len, *k_tokens, *k_ratio, *k_beta, *k_seq,
    *k_len, *k_node_token, *k_node_slot, *k_words, *k_row_offset;

// A strided tensor on a GPU that no transform has wrapped, else null.
const at::Tensor* plain(PyObject* o) {
  if (o == nullptr || !THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage()) return nullptr;
  constexpr c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                         c10::DispatchKey::Functionalize, c10::DispatchKey::Batched});
  return t.key_set().has_any(wrapped) ? nullptr : &t;
}
const at::Tensor* dense(PyObject* o, at::ScalarType type) {
  const at::Tensor* t = plain(o);
  return t != nullptr && t->scalar_type() == type && t->is_contiguous() ? t : nullptr;
}
int dtype_code(const at::Tensor& t) {
  switch (t.scalar_type()) {
    case at::kFloat: return TSLT_F32;
    case at::kBFloat16: return TSLT_BF16;
    case at::kHalf: return TSLT_F16;
    default: return -1;
  }
}
// Pointer of an output; `there` is false for what is no plain tensor (None counts as a null pointer where that is allowed).
template <typename T> T* out_ptr(PyObject* dict, PyObject* key, bool optional, bool& there) {
  PyObject* o = PyDict_GetItem(dict, key);
  if (o == nullptr || o == Py_None) {
    there = there && optional;
    return nullptr;
  }
  const at::Tensor* t = plain(o);
  if (t == nullptr) { there = false; return nullptr; }
  return reinterpret_cast<T*>(t->data_ptr());
}
template <typename T> T* ptr(const at::Tensor* t) { return reinterpret_cast<T*>(t->data_ptr()); }
// An argument that is no such number, or too large for its type: ctypes may know what to do with it.
bool unread() {
  if (PyErr_Occurred() == nullptr) return false;
  PyErr_Clear();
  return true;
}
PyObject* result(int code) { return PyLong_FromLong(code); }

PyObject* py_bind(PyObject*, PyObject* args) {
  unsigned long long a[9];
  if (!PyArg_ParseTuple(args, "KKKKKKKKK", &a[0], &a[1], &a[2], &a[3], &a[4], &a[5], &a[6], &a[7], &a[8])) return nullptr;
  lib.workspace_bytes = reinterpret_cast<decltype(lib.workspace_bytes)>(a[0]);
  lib.truncate_sample = reinterpret_cast<decltype(lib.truncate_sample)>(a[1]);
  lib.verify = reinterpret_cast<decltype(lib.verify)>(a[2]);
  lib.verify_accept = reinterpret_cast<decltype(lib.verify)>(a[3]);
  lib.verify_resample = reinterpret_cast<decltype(lib.verify)>(a[4]);
  lib.verify_tree = reinterpret_cast<decltype(lib.verify_tree)>(a[5]);
  lib.pack_bound_words = reinterpret_cast<decltype(lib.pack_bound_words)>(a[6]);
  lib.pack_cleared = reinterpret_cast<decltype(lib.pack_cleared)>(a[7]);
  lib.unpack = reinterpret_cast<decltype(lib.unpack)>(a[8]);
  bound = true;
  Py_RETURN_NONE;
}

// truncate(logits, temperature, top_k, top_p, k_cap, payload, without_replacement, out, u, stream)
PyObject* py_truncate(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 10 || !bound) Py_RETURN_NONE;
  const at::Tensor *z = plain(a[0]), *u = dense(a[8], at::kFloat);
  const double T = PyFloat_AsDouble(a[1]), top_p = PyFloat_AsDouble(a[3]);
  const long long top_k = PyLong_AsLongLong(a[2]), k_cap = PyLong_AsLongLong(a[4]), payload = PyLong_AsLongLong(a[5]);
  const int wor = PyObject_IsTrue(a[6]);
  void* stream = PyLong_AsVoidPtr(a[9]);
  if (unread()) Py_RETURN_NONE;
  if (z == nullptr || u == nullptr || !PyDict_CheckExact(a[7]) || z->dim() < 1) Py_RETURN_NONE;
  const int dt = dtype_code(*z);
  const int64_t V = z->size(-1);
  if (dt < 0 || V <= 0 || z->stride(-1) != 1) Py_RETURN_NONE;
  int64_t rows, stride;
  if (z->is_contiguous()) { rows = z->numel() / V; stride = V; }
  else if (z->dim() == 2) { rows = z->size(0); stride = z->stride(0); }
  else Py_RETURN_NONE;
  if (rows <= 0 || u->numel() == 0 || u->numel() % rows != 0) Py_RETURN_NONE;
  bool there = true;
  int32_t* idx = out_ptr<int32_t>(a[7], k_idx, false, there);
  float* logit = out_ptr<float>(a[7], k_logit, false, there);
  float* prob = out_ptr<float>(a[7], k_prob, true, there);
  int32_t* count = out_ptr<int32_t>(a[7], k_count, false, there);
  float* mass = out_ptr<float>(a[7], k_mass, true, there);
  int32_t* status = out_ptr<int32_t>(a[7], k_status, true, there);
  int32_t* token = out_ptr<int32_t>(a[7], k_token, false, there);
  int32_t* slot = out_ptr<int32_t>(a[7], k_slot, true, there);
  if (!there) Py_RETURN_NONE;
  const int64_t samples = u->numel() / rows;
  // (a few long rows: memory in which the workgroups that share each of them hand over what they have found)
  const size_t ws_bytes = lib.workspace_bytes(TSLT_OP_TRUNCATE_SHARED, rows, 0, V, int32_t(k_cap));
  at::Tensor ws;
  if (ws_bytes > 0) ws = at::empty({int64_t(ws_bytes)}, at::TensorOptions().dtype(at::kByte).device(z->device()));
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = lib.truncate_sample(z->data_ptr(), tslt_dtype(dt), rows, V, stride, float(T), int32_t(top_k), float(top_p), int32_t(k_cap),
                             tslt_dtype(payload), idx, logit, prob, count, mass, status, ptr<float>(u), int32_t(samples), wor, token, slot,
                             ws_bytes > 0 ? ws.data_ptr() : nullptr, ws_bytes, stream);
  Py_END_ALLOW_THREADS
  return result(code);
}

// verify(phase, target, temperature, q_idx, q_logit, q_count, draft_tokens, u_accept, u_resample, out, workspace, stream)
PyObject* py_verify(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 12 || !bound) Py_RETURN_NONE;
  const long phase = PyLong_AsLong(a[0]);
  const double T = PyFloat_AsDouble(a[2]);
  void* stream = PyLong_AsVoidPtr(a[11]);
  if (unread()) Py_RETURN_NONE;
  const at::Tensor *t = plain(a[1]), *qi = dense(a[3], at::kInt), *ql = dense(a[4], at::kFloat), *qc = dense(a[5], at::kInt),
                   *x = dense(a[6], at::kInt), *ua = dense(a[7], at::kFloat), *ur = dense(a[8], at::kFloat), *ws = plain(a[10]);
  if (!t || !qi || !ql || !qc || !x || !ua || !ur || !ws || !PyDict_CheckExact(a[9])) Py_RETURN_NONE;
  const int dt = dtype_code(*t);
  if (dt < 0 || t->dim() != 3 || !t->is_contiguous() || qi->dim() < 1) Py_RETURN_NONE;
  const int64_t B = t->size(0), gamma = t->size(1) - 1, V = t->size(2), k_cap = qi->size(-1);
  if (qi->numel() != B * gamma * k_cap || ur->numel() != B * (gamma + 1) || ua->numel() != B * gamma) Py_RETURN_NONE;
  bool there = true;
  int32_t* accept_len = out_ptr<int32_t>(a[9], k_accept_len, false, there);
  int32_t* tokens = out_ptr<int32_t>(a[9], k_tokens, false, there);
  float* ratio = out_ptr<float>(a[9], k_ratio, true, there);
  float* beta = out_ptr<float>(a[9], k_beta, true, there);
  int32_t* status = out_ptr<int32_t>(a[9], k_status, true, there);
  if (!there) Py_RETURN_NONE;
  const auto fn = phase == 0 ? lib.verify : (phase == 1 ? lib.verify_accept : lib.verify_resample);
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = fn(t->data_ptr(), tslt_dtype(dt), B, int32_t(gamma), V, t->stride(1), float(T), ptr<int32_t>(qi), ptr<float>(ql), ptr<int32_t>(qc),
            int32_t(k_cap), ptr<int32_t>(x), ptr<float>(ua), ptr<float>(ur), accept_len, tokens, ratio, beta, status, ws->data_ptr(),
            size_t(ws->numel()), stream);
  Py_END_ALLOW_THREADS
  return result(code);
}

// verify_tree(target, temperature, expansion, q_idx, q_logit, q_count, cand_tokens, u_accept, u_resample, without_replacement, out,
//             workspace, stream)
PyObject* py_verify_tree(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 13 || !bound) Py_RETURN_NONE;
  const double T = PyFloat_AsDouble(a[1]);
  const int wor = PyObject_IsTrue(a[9]);
  void* stream = PyLong_AsVoidPtr(a[12]);
  if (unread()) Py_RETURN_NONE;
  if (!PyList_CheckExact(a[2]) && !PyTuple_CheckExact(a[2])) Py_RETURN_NONE;
  int32_t expansion[64];
  const Py_ssize_t depth = PySequence_Fast_GET_SIZE(a[2]);
  if (depth > 64) Py_RETURN_NONE;
  for (Py_ssize_t i = 0; i < depth; ++i) {
    PyObject* k = PySequence_Fast_GET_ITEM(a[2], i);
    if (!PyLong_CheckExact(k)) Py_RETURN_NONE;
    const long long v = PyLong_AsLongLong(k);
    if (unread()) Py_RETURN_NONE;
    expansion[i] = int32_t(v);
  }
  const at::Tensor *t = plain(a[0]), *qi = dense(a[3], at::kInt), *ql = dense(a[4], at::kFloat), *qc = dense(a[5], at::kInt),
                   *x = dense(a[6], at::kInt), *ua = dense(a[7], at::kFloat), *ur = dense(a[8], at::kFloat), *ws = plain(a[11]);
  if (!t || !qi || !ql || !qc || !x || !ua || !ur || !ws || !PyDict_CheckExact(a[10])) Py_RETURN_NONE;
  const int dt = dtype_code(*t);
  if (dt < 0 || t->dim() != 3 || !t->is_contiguous() || qi->dim() < 1) Py_RETURN_NONE;
  bool there = true;
  int32_t* node_token = out_ptr<int32_t>(a[10], k_node_token, true, there);
  int32_t* node_slot = out_ptr<int32_t>(a[10], k_node_slot, true, there);
  int32_t* seq = out_ptr<int32_t>(a[10], k_seq, false, there);
  int32_t* len = out_ptr<int32_t>(a[10], k_len, false, there);
  float* ratio = out_ptr<float>(a[10], k_ratio, true, there);
  float* beta = out_ptr<float>(a[10], k_beta, true, there);
  int32_t* status = out_ptr<int32_t>(a[10], k_status, true, there);
  if (!there) Py_RETURN_NONE;
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = lib.verify_tree(t->data_ptr(), tslt_dtype(dt), t->size(0), t->size(2), t->stride(1), float(T), int32_t(depth), expansion,
                         ptr<int32_t>(qi), ptr<float>(ql), ptr<int32_t>(qc), int32_t(qi->size(-1)), ptr<int32_t>(x), ptr<float>(ua),
                         ptr<float>(ur), wor, node_token, node_slot, seq, len, ratio, beta, status, ws->data_ptr(), size_t(ws->numel()), stream);
  Py_END_ALLOW_THREADS
  return result(code);
}

// (code, dict) of tensors that were made here; takes them over
PyObject* with_code(int code, std::initializer_list<std::pair<PyObject*, at::Tensor>> made) {
  PyObject* dict = PyDict_New();
  if (dict == nullptr) return nullptr;
  for (const auto& m : made) {
    PyObject* t = THPVariable_Wrap(m.second);
    if (t == nullptr || PyDict_SetItem(dict, m.first, t) != 0) {
      Py_XDECREF(t);
      Py_DECREF(dict);
      return nullptr;
    }
    Py_DECREF(t);
  }
  return Py_BuildValue("(iN)", code, dict);
}

// pack(idx, logit, count, V, payload, stream)
PyObject* py_pack(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 6 || !bound) Py_RETURN_NONE;
  const long long V = PyLong_AsLongLong(a[3]), payload = PyLong_AsLongLong(a[4]);
  void* stream = PyLong_AsVoidPtr(a[5]);
  if (unread()) Py_RETURN_NONE;
  const at::Tensor *idx = dense(a[0], at::kInt), *logit = dense(a[1], at::kFloat), *count = dense(a[2], at::kInt);
  if (!idx || !logit || !count || idx->dim() != 2) Py_RETURN_NONE;
  const int64_t rows = idx->size(0), k_cap = idx->size(1);
  const int64_t cap = lib.pack_bound_words(rows, int32_t(k_cap), V);
  if (cap <= 0) Py_RETURN_NONE;
  at::Tensor words = at::empty({cap}, at::TensorOptions().dtype(at::kInt).device(idx->device()));
  at::Tensor offs = at::empty({rows + 1}, at::TensorOptions().dtype(at::kLong).device(idx->device()));
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = lib.pack_cleared(ptr<int32_t>(idx), ptr<float>(logit), ptr<int32_t>(count), rows, int32_t(k_cap), V, tslt_dtype(payload),
                          reinterpret_cast<uint32_t*>(words.data_ptr()), cap, reinterpret_cast<int64_t*>(offs.data_ptr()), stream);
  Py_END_ALLOW_THREADS
  return with_code(code, {{k_words, words}, {k_row_offset, offs}});
}

// unpack(words, row_offset, rows, k_cap, V, payload, stream)
PyObject* py_unpack(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 7 || !bound) Py_RETURN_NONE;
  const long long rows = PyLong_AsLongLong(a[2]), k_cap = PyLong_AsLongLong(a[3]), V = PyLong_AsLongLong(a[4]), payload = PyLong_AsLongLong(a[5]);
  void* stream = PyLong_AsVoidPtr(a[6]);
  if (unread()) Py_RETURN_NONE;
  const at::Tensor *words = dense(a[0], at::kInt), *offs = dense(a[1], at::kLong);
  if (!words || !offs || rows <= 0 || k_cap <= 0 || k_cap > TSLT_MAX_K_CAP) Py_RETURN_NONE;
  const auto on = at::TensorOptions().device(words->device());
  at::Tensor idx = at::empty({rows, k_cap}, on.dtype(at::kInt)), logit = at::empty({rows, k_cap}, on.dtype(at::kFloat));
  at::Tensor count = at::empty({rows}, on.dtype(at::kInt));
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = lib.unpack(reinterpret_cast<const uint32_t*>(words->data_ptr()), reinterpret_cast<const int64_t*>(offs->data_ptr()), rows, int32_t(k_cap), V,
                    tslt_dtype(payload), ptr<int32_t>(&idx), ptr<float>(&logit), ptr<int32_t>(&count), stream);
  Py_END_ALLOW_THREADS
  return with_code(code, {{k_idx, idx}, {k_logit, logit}, {k_count, count}});
}

// What a call into torch throws (no memory left, say) becomes a Python exception, as from torch itself.
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)> PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  return F(self, a, n);
  END_HANDLE_TH_ERRORS
}
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)> PyMethodDef fast(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<F>)), METH_FASTCALL, nullptr};
}
PyMethodDef methods[] = {
    {"bind", py_bind, METH_VARARGS, nullptr}, fast<py_truncate>("truncate"), fast<py_verify>("verify"), fast<py_verify_tree>("verify_tree"),
    fast<py_pack>("pack"), fast<py_unpack>("unpack"), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
  const std::pair<PyObject**, const char*> keys[] = {
      {&k_idx, "idx"}, {&k_logit, "logit"}, {&k_prob, "prob"}, {&k_count, "count"}, {&k_mass, "mass"}, {&k_status, "status"},
      {&k_token, "token"}, {&k_slot, "slot"}, {&k_accept_len, "accept_len"}, {&k_tokens, "tokens"}, {&k_ratio, "ratio"}, {&k_beta, "beta"},
      {&k_seq, "seq"}, {&k_len, "len"}, {&k_node_token, "node_token"}, {&k_node_slot, "node_slot"}, {&k_words, "words"}, {&k_row_offset, "row_offset"}};
  for (const auto& k : keys)
    if ((*k.first = PyUnicode_InternFromString(k.second)) == nullptr) return nullptr;
  PyObject* m = PyModule_Create(&module);
  if (m != nullptr && PyModule_AddStringConstant(m, "built_for", TSLT_BUILT_FOR) != 0) Py_CLEAR(m);
  return m;
}
