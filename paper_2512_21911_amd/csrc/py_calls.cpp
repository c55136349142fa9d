// The calls of one verification step from Python, without an interpreter-level argument walk.
//
// A launch of this library lasts ten microseconds or less, and a call through ctypes took 7 - 11 us
// of host time (a wrapper object per argument, a stream lookup through two Python layers): a
// program that makes its calls one by one was bound by that, not by the GPU.  Here an argument is a
// pointer read out of the tensor object; a call costs what the launch itself costs.
//
// Every function has the name and the arguments of the C entry point it calls (include/*.h), keyword
// arguments included, and does no arithmetic.  A tensor argument may be None (NULL); a shape is the
// ctypes structure that mirrors the C one; work is enqueued on torch's current stream.
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include <vector>

#include "svf.h"
#include "svf_ffn.h"
#include "svf_rules.h"

namespace {

struct Failed {};                      // a Python error is set

enum Kind : uint8_t { kShape, kTensor, kInt, kNumber };   // kNumber: whatever int() takes

struct Param {
  const char* name;
  Kind kind;
  bool has_default;                    // tensors: None, integers: `value`
  int64_t value;
  PyObject* key = nullptr;             // the interned name
};

// The arguments of one call, in the order of the Python signature.
struct Args {
  static constexpr int kMost = 20;
  void* ptr[kMost] = {};               // tensors and shapes
  int64_t num[kMost] = {};             // integers; for tensors the number of elements (a workspace is bytes)
  PyObject* obj[kMost] = {};
  Py_buffer view[2];
  int views = 0;
  ~Args() {
    for (int i = 0; i < views; ++i) PyBuffer_Release(&view[i]);
  }
};

struct Signature {
  const char* where;
  std::vector<Param> params;
};

void take(const Signature& s, int i, PyObject* o, Args& a) {
  const Param& p = s.params[i];
  a.obj[i] = o;
  switch (p.kind) {
    case kNumber:
    case kInt: {
      PyObject* whole = p.kind == kNumber && !PyLong_Check(o) ? PyNumber_Long(o) : nullptr;
      if (p.kind == kNumber && !PyLong_Check(o) && !whole) throw Failed{};
      const int64_t v = PyLong_AsLongLong(whole ? whole : o);
      Py_XDECREF(whole);
      if (v == -1 && PyErr_Occurred()) throw Failed{};
      if (v != (int32_t)v) {
        PyErr_Format(PyExc_OverflowError, "%s(): %s does not fit a 32-bit integer", s.where, p.name);
        throw Failed{};
      }
      a.num[i] = v;
      return;
    }
    case kShape: {
      if (PyObject_GetBuffer(o, &a.view[a.views], PyBUF_SIMPLE) != 0) throw Failed{};
      a.ptr[i] = a.view[a.views].buf;
      a.num[i] = (int64_t)a.view[a.views].len;
      ++a.views;
      return;
    }
    case kTensor: {
      if (o == Py_None) return;
      if (THPVariable_Check(o)) {
        const at::Tensor& t = THPVariable_Unpack(o);
        a.ptr[i] = t.data_ptr();
        a.num[i] = t.numel();
        return;
      }
      PyErr_Format(PyExc_TypeError, "%s(): %s must be a tensor or None", s.where, p.name);
      throw Failed{};
    }
  }
}

void parse(const Signature& s, PyObject* const* args, Py_ssize_t n, PyObject* kwnames, Args& a) {
  const int np = (int)s.params.size();
  if (n > np) {
    PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", s.where, np, n);
    throw Failed{};
  }
  for (int i = 0; i < (int)n; ++i) take(s, i, args[i], a);
  const Py_ssize_t nk = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
  for (Py_ssize_t k = 0; k < nk; ++k) {
    PyObject* key = PyTuple_GET_ITEM(kwnames, k);
    int i = 0;
    while (i < np && s.params[i].key != key) ++i;                       // keyword names are interned as a rule
    if (i == np)
      for (i = 0; i < np && PyUnicode_Compare(s.params[i].key, key) != 0; ++i) {}
    if (i == np || a.obj[i]) {
      PyErr_Format(PyExc_TypeError, i == np ? "%s() got an unexpected keyword argument '%U'"
                                            : "%s() got multiple values for argument '%U'", s.where, key);
      throw Failed{};
    }
    take(s, i, args[n + k], a);
  }
  for (int i = 0; i < np; ++i) {
    if (a.obj[i]) continue;
    const Param& p = s.params[i];
    if (!p.has_default) {
      PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", s.where, p.name);
      throw Failed{};
    }
    a.num[i] = p.value;
  }
}

// The interpreter is let go for the call itself (a launch waits when the stream's queue is full).
struct NoGil {
  PyThreadState* state = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(state); }
};

void* stream() { return static_cast<void*>(c10::hip::getCurrentHIPStream().stream()); }

PyObject* finish(const Signature& s, int rc) {
  if (rc == SVF_OK) Py_RETURN_NONE;
  PyObject* m = PyImport_ImportModule("paper_2512_21911_amd.binding");
  PyObject* cls = m ? PyObject_GetAttrString(m, "SvfError") : nullptr;
  PyObject* e = cls ? PyObject_CallFunction(cls, "is", rc, s.where) : nullptr;
  if (e) PyErr_SetObject(cls, e);
  Py_XDECREF(e);
  Py_XDECREF(cls);
  Py_XDECREF(m);
  return nullptr;
}

// A tensor's sizes, which must be `dims` many.
const int64_t* sizes_of(const Signature& s, const Args& a, int i, int64_t dims) {
  if (!a.ptr[i] && a.obj[i] == Py_None) {
    PyErr_Format(PyExc_TypeError, "%s(): %s must be a tensor", s.where, s.params[i].name);
    throw Failed{};
  }
  const at::Tensor& t = THPVariable_Unpack(a.obj[i]);
  if (t.dim() != dims) {
    PyErr_Format(PyExc_ValueError, "%s(): %s must have %d dimensions", s.where, s.params[i].name, (int)dims);
    throw Failed{};
  }
  return t.sizes().data();
}

template <typename Shape>
const Shape* shape_of(const Signature& s, const Args& a, int i) {
  if (a.num[i] < (int64_t)sizeof(Shape)) {
    PyErr_Format(PyExc_TypeError, "%s(): %s is not the structure this call takes", s.where, s.params[i].name);
    throw Failed{};
  }
  return static_cast<const Shape*>(a.ptr[i]);
}

Param shape(const char* n) { return {n, kShape, false, 0}; }
Param tensor(const char* n) { return {n, kTensor, false, 0}; }
Param tensor_or_none(const char* n) { return {n, kTensor, true, 0}; }
Param number(const char* n) { return {n, kNumber, false, 0}; }
Param integer(const char* n, int64_t v) { return {n, kInt, true, v}; }

// One function: its signature and the call of the C entry point with the parsed arguments.
#define SVF_CALL(NAME, CALL, ...)                                                                      \
  Signature sig_##NAME{#NAME, {__VA_ARGS__}};                                                          \
  PyObject* NAME##_py(PyObject*, PyObject* const* args, Py_ssize_t n, PyObject* kwnames) {              \
    const Signature& s = sig_##NAME;                                                                   \
    try {                                                                                              \
      Args a;                                                                                          \
      parse(s, args, n, kwnames, a);                                                                   \
      int rc = SVF_OK;                                                                                 \
      { CALL; }                                                                                        \
      return finish(s, rc);                                                                            \
    } catch (const Failed&) {                                                                          \
      return nullptr;                                                                                  \
    } catch (const std::exception& e) {                                                                \
      PyErr_SetString(PyExc_RuntimeError, e.what());                                                   \
      return nullptr;                                                                                  \
    }                                                                                                  \
  }

#define I32(i) static_cast<const int32_t*>(a.ptr[i])
#define F32(i) static_cast<const float*>(a.ptr[i])
#define U64(i) static_cast<const uint64_t*>(a.ptr[i])
#define WS(i) a.ptr[i], (size_t)a.num[i]

SVF_CALL(svf_block_reps,
         const auto* sh = shape_of<svf_shape_t>(s, a, 0); void* st = stream(); NoGil free;
         rc = svf_block_reps(sh, a.ptr[1], I32(2), I32(3), (int32_t)a.num[5], (int32_t)a.num[6],
                             static_cast<float*>(a.ptr[4]), st),
         shape("shape"), tensor("K"), tensor("block_table"), tensor("seq_lens"), tensor("reps"), integer("first_block", 0),
         integer("n_blocks", -1))

SVF_CALL(svf_score_select,
         const auto* sh = shape_of<svf_shape_t>(s, a, 0); void* st = stream(); NoGil free;
         rc = svf_score_select(sh, a.ptr[1], F32(2), I32(3), static_cast<int32_t*>(a.ptr[4]),
                               static_cast<int32_t*>(a.ptr[5]), static_cast<float*>(a.ptr[7]), WS(6), st),
         shape("shape"), tensor("q"), tensor("reps"), tensor("seq_lens"), tensor("sel_idx"), tensor("sel_cnt"), tensor("ws"),
         tensor_or_none("scores"))

SVF_CALL(svf_verify_attn,
         const auto* sh = shape_of<svf_shape_t>(s, a, 0); void* st = stream(); NoGil free;
         rc = svf_verify_attn(sh, a.ptr[1], a.ptr[2], a.ptr[3], I32(4), I32(5), a.ptr[6], a.ptr[7],
                              U64(8), I32(9), I32(10), a.ptr[11], static_cast<float*>(a.ptr[13]), WS(12), st),
         shape("shape"), tensor("q"), tensor("K"), tensor("V"), tensor("block_table"), tensor("seq_lens"), tensor("k_draft"),
         tensor("v_draft"), tensor("draft_mask"), tensor("sel_idx"), tensor("sel_cnt"), tensor("out"), tensor("ws"),
         tensor_or_none("lse"))

SVF_CALL(svf_verify_attn_static_ws,
         const auto* sh = shape_of<svf_shape_t>(s, a, 0); void* st = stream(); NoGil free;
         rc = svf_verify_attn_static_ws(sh, a.ptr[1], a.ptr[2], a.ptr[3], I32(4), I32(5), a.ptr[6],
                                        a.ptr[7], U64(8), I32(9), I32(10), a.ptr[11], static_cast<float*>(a.ptr[12]), st),
         shape("shape"), tensor("q"), tensor("K"), tensor("V"), tensor("block_table"), tensor("seq_lens"), tensor("k_draft"),
         tensor("v_draft"), tensor("draft_mask"), tensor("sel_idx"), tensor("sel_cnt"), tensor("out"), tensor_or_none("lse"))

SVF_CALL(svf_verify_step,
         const auto* sh = shape_of<svf_shape_t>(s, a, 0); void* st = stream(); NoGil free;
         rc = svf_verify_step(sh, (int)a.num[1], a.ptr[2], F32(3), a.ptr[4], a.ptr[5], I32(6), I32(7),
                              a.ptr[8], a.ptr[9], U64(10), static_cast<int32_t*>(a.ptr[11]), static_cast<int32_t*>(a.ptr[12]),
                              a.ptr[13], static_cast<float*>(a.ptr[15]), WS(14), st),
         shape("shape"), number("mode"), tensor("q"), tensor("reps"), tensor("K"), tensor("V"), tensor("block_table"),
         tensor("seq_lens"), tensor("k_draft"), tensor("v_draft"), tensor("draft_mask"), tensor("sel_idx"), tensor("sel_cnt"),
         tensor("out"), tensor("ws"), tensor_or_none("lse"))

SVF_CALL(svf_block_summaries,
         const auto* sh = shape_of<svf_shape_t>(s, a, 0); const auto* rt = shape_of<svf_retrieval_t>(s, a, 1);
         void* st = stream(); NoGil free;
         rc = svf_block_summaries(sh, rt, a.ptr[2], I32(3), I32(4),
                                  (int32_t)a.num[6], (int32_t)a.num[7], a.ptr[5], st),
         shape("shape"), shape("retrieval"), tensor("K"), tensor("block_table"), tensor("seq_lens"), tensor("summaries"),
         integer("first_block", 0), integer("n_blocks", -1))

SVF_CALL(svf_retrieve,
         const auto* sh = shape_of<svf_shape_t>(s, a, 0); const auto* rt = shape_of<svf_retrieval_t>(s, a, 1);
         void* st = stream(); NoGil free;
         rc = svf_retrieve(sh, rt, a.ptr[2], a.ptr[3], I32(4),
                           static_cast<int32_t*>(a.ptr[5]), static_cast<int32_t*>(a.ptr[6]), static_cast<float*>(a.ptr[8]), WS(7),
                           st),
         shape("shape"), shape("retrieval"), tensor("q"), tensor("summaries"), tensor("seq_lens"), tensor("sel_idx"),
         tensor("sel_cnt"), tensor("ws"), tensor_or_none("scores"))

SVF_CALL(svf_sparse_ffn,
         const auto* sh = shape_of<svf_ffn_shape_t>(s, a, 0); void* st = stream(); NoGil free;
         rc = svf_sparse_ffn(sh, a.ptr[1], a.ptr[2], a.ptr[3], a.ptr[4], F32(7), F32(8), F32(9),
                             a.ptr[5], static_cast<uint64_t*>(a.ptr[10]), WS(6), st),
         shape("shape"), tensor("x"), tensor("w_gate"), tensor("w_up"), tensor("w_down_t"), tensor("y"), tensor("ws"),
         tensor_or_none("b_gate"), tensor_or_none("b_up"), tensor_or_none("b_down"), tensor_or_none("active"))

SVF_CALL(svf_moe_skip,
         const int64_t* d = sizes_of(s, a, 0, 2); void* st = stream(); NoGil free;
         rc = svf_moe_skip(F32(0), (int32_t)d[0], (int32_t)d[1], (int32_t)a.num[1], F32(2), static_cast<int32_t*>(a.ptr[3]),
                           static_cast<uint32_t*>(a.ptr[4]), st),
         tensor("w"), number("m"), tensor("beta"), tensor("n_skip"), tensor("keep_mask"))

SVF_CALL(svf_accept_resample,
         const int64_t* d = sizes_of(s, a, 0, 3); void* st = stream(); NoGil free;
         rc = svf_accept_resample(F32(0), F32(1), I32(2), F32(3), F32(4), (int32_t)d[0], (int32_t)d[1], (int32_t)d[2],
                                  static_cast<int32_t*>(a.ptr[5]), static_cast<int32_t*>(a.ptr[6]), st),
         tensor("p_target"), tensor("p_draft"), tensor("draft_tokens"), tensor("u_accept"), tensor("u_resample"),
         tensor("n_accepted"), tensor("resampled"))

#define SVF_METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME##_py, METH_FASTCALL | METH_KEYWORDS, nullptr}
PyMethodDef methods[] = {SVF_METHOD(svf_block_reps), SVF_METHOD(svf_score_select), SVF_METHOD(svf_verify_attn),
                         SVF_METHOD(svf_verify_attn_static_ws), SVF_METHOD(svf_verify_step), SVF_METHOD(svf_block_summaries),
                         SVF_METHOD(svf_retrieve), SVF_METHOD(svf_sparse_ffn), SVF_METHOD(svf_moe_skip),
                         SVF_METHOD(svf_accept_resample), {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_svf_calls", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__svf_calls(void) {
  for (Signature* s : {&sig_svf_block_reps, &sig_svf_score_select, &sig_svf_verify_attn, &sig_svf_verify_attn_static_ws,
                       &sig_svf_verify_step, &sig_svf_block_summaries, &sig_svf_retrieve, &sig_svf_sparse_ffn,
                       &sig_svf_moe_skip, &sig_svf_accept_resample}) {
    static_assert(Args::kMost >= 16, "arguments of svf_verify_step");
    for (Param& p : s->params) p.key = PyUnicode_InternFromString(p.name);
  }
  return PyModule_Create(&module);
}
