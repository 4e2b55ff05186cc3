// The binding's usual case in one native call: every tensor argument is checked (exact torch.Tensor, element type, shape,
// contiguous, on the device) and the library called with their addresses.  None is returned, and nothing has happened,
// where an argument is not of that kind: the binding then goes through its checks one by one and says what is wrong.
// Host only.  A verify and a hand-over check 18 tensors; in Python that was two thirds of the 18 us that both calls took,
// whose three kernels take 8: 18.5 -> 11.3 us back to back (32000 logits, 16 candidates of 3), 48 -> 34 for a first call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <initializer_list>

#include "../../include/spec.h"

namespace {

decltype(&spec_verify) f_verify;
decltype(&spec_verify_dynamic) f_verify_dynamic;
decltype(&spec_advance) f_advance;
decltype(&spec_tree_metadata) f_tree_metadata;
decltype(&spec_draft) f_draft;
PyObject* f_stream;   // the binding's _stream_ptr

const at::Tensor* tensor(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

template <typename T>
bool usual(PyObject* o, at::ScalarType dtype, std::initializer_list<int64_t> shape, T** at) {
  const at::Tensor* t = tensor(o);
  if (!t || t->scalar_type() != dtype || t->sizes() != at::IntArrayRef(shape) || !t->is_contiguous() || !t->is_cuda()) return false;
  *at = static_cast<T*>(t->mutable_data_ptr());
  return true;
}
template <typename T>
bool usual_or_none(PyObject* o, at::ScalarType dtype, std::initializer_list<int64_t> shape, T** at) {
  *at = nullptr;
  return o == Py_None || usual(o, dtype, shape, at);
}

// 4-dimensional float32 or bfloat16 input; false: not of that kind
bool floats4(PyObject* o, int64_t (&size)[4], int32_t* code, at::ScalarType* dtype, void** at) {
  const at::Tensor* t = tensor(o);
  if (!t || t->dim() != 4) return false;
  *dtype = t->scalar_type();
  if (*dtype == at::kFloat) *code = SPEC_F32;
  else if (*dtype == at::kBFloat16) *code = SPEC_BF16;
  else return false;
  for (int i = 0; i < 4; ++i) size[i] = t->size(i);
  for (int i = 0; i < 4; ++i)
    if (size[i] > INT32_MAX) return false;
  return usual(o, *dtype, {size[0], size[1], size[2], size[3]}, at);
}

// false with an exception set: the caller returns nullptr
bool stream_of(PyObject* o, void** stream) {
  PyObject* p = PyObject_CallOneArg(f_stream, o);
  if (!p) return false;
  *stream = p == Py_None ? nullptr : PyLong_AsVoidPtr(p);
  Py_DECREF(p);
  return !PyErr_Occurred();
}

template <typename F>
PyObject* status_of(F&& call) {
  spec_status_t s;
  Py_BEGIN_ALLOW_THREADS
  s = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(s);
}

// logits, cand_tokens, n_cand (None: spec_verify), greedy, accept_len, best_cand, out_tokens, n_out, accept_all, stream
PyObject* verify(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 10) Py_RETURN_NONE;
  try {
    int64_t d[4];
    int32_t code;
    at::ScalarType dt;
    void *logits, *stream;
    int32_t *cand, *n_cand, *greedy, *len, *best, *out, *n_out, *all;
    if (!floats4(a[0], d, &code, &dt, &logits)) Py_RETURN_NONE;
    const int64_t b = d[0], B = d[1], n1 = d[2];
    if (!usual(a[1], at::kInt, {b, B, n1 - 1}, &cand) || !usual_or_none(a[2], at::kInt, {b}, &n_cand) ||
        !usual(a[3], at::kInt, {b, B, n1}, &greedy) || !usual(a[4], at::kInt, {b}, &len) || !usual(a[5], at::kInt, {b}, &best) ||
        !usual(a[6], at::kInt, {b, n1}, &out) || !usual(a[7], at::kInt, {b}, &n_out) ||
        !usual_or_none(a[8], at::kInt, {b, B}, &all))
      Py_RETURN_NONE;
    if (!stream_of(a[9], &stream)) return nullptr;
    const int32_t V = (int32_t)d[3], np = (int32_t)n1 - 1;
    return status_of([&] {
      return n_cand ? f_verify_dynamic(logits, code, cand, n_cand, (int32_t)b, (int32_t)B, np, V, greedy, len, best, out, n_out, all, stream)
                    : f_verify(logits, code, cand, (int32_t)b, (int32_t)B, np, V, greedy, len, best, out, n_out, all, stream);
    });
  } catch (...) {   // a tensor without storage, say
    Py_RETURN_NONE;
  }
}

// hidden, best_cand, accept_len, out_tokens, next_state, next_tok, stream
PyObject* advance(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 7) Py_RETURN_NONE;
  try {
    int64_t d[4];
    int32_t code;
    at::ScalarType dt;
    void *hidden, *state, *stream;
    int32_t *best, *len, *out, *tok;
    if (!floats4(a[0], d, &code, &dt, &hidden) || !usual(a[1], at::kInt, {d[0]}, &best) || !usual(a[2], at::kInt, {d[0]}, &len) ||
        !usual(a[3], at::kInt, {d[0], d[2]}, &out) || !usual(a[4], dt, {d[0], d[3]}, &state) || !usual(a[5], at::kInt, {d[0]}, &tok))
      Py_RETURN_NONE;
    if (!stream_of(a[6], &stream)) return nullptr;
    return status_of([&] {
      return f_advance(hidden, code, (int32_t)d[0], (int32_t)d[1], (int32_t)d[2] - 1, (int32_t)d[3], best, len, out, state, tok, stream);
    });
  } catch (...) {
    Py_RETURN_NONE;
  }
}

// cand_tokens, node_tok, node_parent, node_depth, n_nodes, cand_node, mask, stream
PyObject* tree_metadata(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 8) Py_RETURN_NONE;
  try {
    const at::Tensor* t = tensor(a[0]);
    if (!t || t->dim() != 3) Py_RETURN_NONE;
    const int64_t b = t->size(0), B = t->size(1), np = t->size(2);
    if (b > INT32_MAX || B > INT32_MAX || np > INT32_MAX) Py_RETURN_NONE;
    const int64_t M = B * np;
    int32_t *cand, *tok, *parent, *depth, *count, *node;
    uint8_t* mask;
    void* stream;
    if (!usual(a[0], at::kInt, {b, B, np}, &cand) || !usual(a[1], at::kInt, {b, M}, &tok) || !usual(a[2], at::kInt, {b, M}, &parent) ||
        !usual(a[3], at::kInt, {b, M}, &depth) || !usual(a[4], at::kInt, {b}, &count) || !usual(a[5], at::kInt, {b, B, np}, &node) ||
        !usual_or_none(a[6], at::kByte, {b, M, M}, &mask))
      Py_RETURN_NONE;
    if (!stream_of(a[7], &stream)) return nullptr;
    return status_of([&] {
      return f_tree_metadata(cand, (int32_t)b, (int32_t)B, (int32_t)np, tok, parent, depth, count, node, mask, stream);
    });
  } catch (...) {
    Py_RETURN_NONE;
  }
}

// handle (address or None), n_predict, emb_dim, weight_dtype, state, last_tok, top_k, B, cand_tokens, cand_scores, cand_leaf, stream
PyObject* draft(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 12 || !PyLong_CheckExact(a[0]) || !PyLong_CheckExact(a[7])) Py_RETURN_NONE;
  if (!PyTuple_CheckExact(a[6]) && !PyList_CheckExact(a[6])) Py_RETURN_NONE;
  try {
    const long np = PyLong_AsLong(a[1]), E = PyLong_AsLong(a[2]), code = PyLong_AsLong(a[3]);
    int over = 0;
    const long B = PyLong_AsLongAndOverflow(a[7], &over);
    if (over || B < 0 || B > INT32_MAX || np < 1 || np > SPEC_MAX_STAGES || (code != SPEC_F32 && code != SPEC_BF16) ||
        PySequence_Fast_GET_SIZE(a[6]) != np)
      Py_RETURN_NONE;
    int32_t top_k[SPEC_MAX_STAGES];
    for (long i = 0; i < np; ++i) {
      PyObject* k = PySequence_Fast_GET_ITEM(a[6], i);
      if (!PyLong_CheckExact(k)) Py_RETURN_NONE;
      const long v = PyLong_AsLongAndOverflow(k, &over);
      if (over || v < INT32_MIN || v > INT32_MAX) Py_RETURN_NONE;
      top_k[i] = (int32_t)v;
    }
    const at::Tensor* t = tensor(a[4]);
    if (!t || t->dim() != 2 || t->size(0) > INT32_MAX) Py_RETURN_NONE;
    const int64_t b = t->size(0);
    void *state, *stream;
    int32_t *last, *tokens, *leaf;
    float* scores;
    if (!usual(a[4], code == SPEC_BF16 ? at::kBFloat16 : at::kFloat, {b, E}, &state) || !usual(a[5], at::kInt, {b}, &last) ||
        !usual(a[8], at::kInt, {b, B, np}, &tokens) || !usual(a[9], at::kFloat, {b, B}, &scores) || !usual(a[10], at::kInt, {b, B}, &leaf))
      Py_RETURN_NONE;
    spec_model_t* model = static_cast<spec_model_t*>(PyLong_AsVoidPtr(a[0]));
    if (!stream_of(a[11], &stream)) return nullptr;
    return status_of([&] { return f_draft(model, state, last, (int32_t)b, top_k, (int32_t)B, tokens, scores, leaf, nullptr, stream); });
  } catch (...) {
    Py_RETURN_NONE;
  }
}

// addresses of spec_verify, spec_verify_dynamic, spec_advance, spec_tree_metadata, spec_draft; the binding's stream lookup
PyObject* bind(PyObject*, PyObject* args) {
  unsigned long long v, vd, ad, tm, dr;
  PyObject* s;
  if (!PyArg_ParseTuple(args, "KKKKKO", &v, &vd, &ad, &tm, &dr, &s)) return nullptr;
  f_verify = reinterpret_cast<decltype(f_verify)>(v);
  f_verify_dynamic = reinterpret_cast<decltype(f_verify_dynamic)>(vd);
  f_advance = reinterpret_cast<decltype(f_advance)>(ad);
  f_tree_metadata = reinterpret_cast<decltype(f_tree_metadata)>(tm);
  f_draft = reinterpret_cast<decltype(f_draft)>(dr);
  Py_INCREF(s);
  Py_XDECREF(f_stream);
  f_stream = s;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"verify", reinterpret_cast<PyCFunction>(verify), METH_FASTCALL, nullptr},
    {"advance", reinterpret_cast<PyCFunction>(advance), METH_FASTCALL, nullptr},
    {"tree_metadata", reinterpret_cast<PyCFunction>(tree_metadata), METH_FASTCALL, nullptr},
    {"draft", reinterpret_cast<PyCFunction>(draft), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call() { return PyModule_Create(&module); }
