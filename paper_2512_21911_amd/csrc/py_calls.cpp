// The calls of one verification step from Python, without an interpreter-level argument walk.
//
// A launch of this library lasts ten microseconds or less, and a call through ctypes took 7 - 11 us
// of host time (a wrapper object per argument, a stream lookup through two Python layers): a
// program that makes its calls one by one was bound by that, not by the GPU.  Here an argument is a
// pointer read out of the tensor object; a call costs what the launch itself costs.
//
// Every function has the name and the arguments of the C entry point it calls (include/*.h), keyword
// arguments included, and does no arithmetic.  A tensor argument may be None (NULL) and is otherwise a
// tensor or any object with its data_ptr() (and numel() or shape where a call needs them); a shape is an
// instance of the ctypes structure that mirrors the C one, and of no other (a buffer of the right size would do
// for the pointer, with its fields read as something else); work is enqueued on torch's current stream.
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include <string>
#include <vector>

#include "svf.h"
#include "svf_ffn.h"
#include "svf_rules.h"

namespace {

struct Failed {};                      // a Python error is set

// kNumber: whatever int() takes; kWorkspace: a tensor whose number of elements is asked for
enum Kind : uint8_t { kShape, kTensor, kWorkspace, kInt, kNumber };

// The ctypes structures (set_structures), in the order of this enumeration.
enum Structure : uint8_t { kSvfShape, kSvfRetrieval, kSvfFfnShape, kStructures };
PyTypeObject* structures[kStructures];

struct Param {
  const char* name;
  Kind kind;
  bool has_default;                    // tensors: None, integers: `value`
  int64_t value;                       // (shapes: which structure)
  PyObject* key = nullptr;             // the interned name
};

// The arguments of one call, in the order of the Python signature.
struct Args {
  static constexpr int kMost = 20;
  void* ptr[kMost] = {};               // tensors and shapes
  int64_t num[kMost] = {};             // integers; for workspaces the number of elements
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

// What a method of `o` without arguments returns, as an integer (None: 0).
int64_t ask(PyObject* o, const char* method) {
  PyObject* r = PyObject_CallMethod(o, method, nullptr);
  if (!r) throw Failed{};
  int64_t v = 0;
  if (r != Py_None) {
    PyObject* whole = PyNumber_Index(r);
    if (whole) v = (int64_t)PyLong_AsUnsignedLongLongMask(whole);
    Py_XDECREF(whole);
  }
  Py_DECREF(r);
  if (PyErr_Occurred()) throw Failed{};
  return v;
}

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
      if (!PyObject_TypeCheck(o, structures[p.value])) {
        PyErr_Format(PyExc_TypeError, "%s(): %s must be a %s, not %s", s.where, p.name, structures[p.value]->tp_name,
                     Py_TYPE(o)->tp_name);
        throw Failed{};
      }
      if (PyObject_GetBuffer(o, &a.view[a.views], PyBUF_SIMPLE) != 0) throw Failed{};
      a.ptr[i] = a.view[a.views].buf;
      ++a.views;
      return;
    }
    case kTensor:
    case kWorkspace: {
      if (o == Py_None) return;
      if (THPVariable_Check(o)) {
        const at::Tensor& t = THPVariable_Unpack(o);
        a.ptr[i] = t.data_ptr();
        a.num[i] = p.kind == kWorkspace ? t.numel() : 0;
        return;
      }
      a.ptr[i] = reinterpret_cast<void*>(ask(o, "data_ptr"));
      if (p.kind == kWorkspace) a.num[i] = ask(o, "numel");
      return;
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

// A tensor's sizes, which must be `dims` many, as the C entry points take them.
struct Sizes {
  int32_t of[4];
  int32_t operator[](int i) const { return of[i]; }
};
Sizes sizes_of(const Signature& s, const Args& a, int i, int dims) {
  Sizes r{};
  if (THPVariable_Check(a.obj[i])) {
    const at::Tensor& t = THPVariable_Unpack(a.obj[i]);
    if (t.dim() == dims) {
      for (int d = 0; d < dims; ++d) r.of[d] = (int32_t)t.size(d);
      return r;
    }
  }
  PyObject* shape = PyObject_GetAttrString(a.obj[i], "shape");
  PyObject* seq = shape ? PySequence_Fast(shape, "a shape is a sequence") : nullptr;
  Py_XDECREF(shape);
  if (!seq) throw Failed{};
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
  for (Py_ssize_t d = 0; n == dims && d < n; ++d)
    r.of[d] = (int32_t)PyLong_AsUnsignedLongMask(PySequence_Fast_GET_ITEM(seq, d));
  Py_DECREF(seq);
  if (n != dims) PyErr_Format(PyExc_ValueError, "%s(): %s must have %d dimensions", s.where, s.params[i].name, dims);
  if (PyErr_Occurred()) throw Failed{};
  return r;
}

template <typename Shape>
const Shape* shape_of(const Args& a, int i) { return static_cast<const Shape*>(a.ptr[i]); }

Param shape(const char* n, Structure which = kSvfShape) { return {n, kShape, false, which}; }
Param tensor(const char* n) { return {n, kTensor, false, 0}; }
Param tensor_or_none(const char* n) { return {n, kTensor, true, 0}; }
Param workspace(const char* n) { return {n, kWorkspace, false, 0}; }
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
         const auto* sh = shape_of<svf_shape_t>(a, 0); void* st = stream(); NoGil free;
         rc = svf_block_reps(sh, a.ptr[1], I32(2), I32(3), (int32_t)a.num[5], (int32_t)a.num[6],
                             static_cast<float*>(a.ptr[4]), st),
         shape("shape"), tensor("K"), tensor("block_table"), tensor("seq_lens"), tensor("reps"), integer("first_block", 0),
         integer("n_blocks", -1))

SVF_CALL(svf_score_select,
         const auto* sh = shape_of<svf_shape_t>(a, 0); void* st = stream(); NoGil free;
         rc = svf_score_select(sh, a.ptr[1], F32(2), I32(3), static_cast<int32_t*>(a.ptr[4]),
                               static_cast<int32_t*>(a.ptr[5]), static_cast<float*>(a.ptr[7]), WS(6), st),
         shape("shape"), tensor("q"), tensor("reps"), tensor("seq_lens"), tensor("sel_idx"), tensor("sel_cnt"), workspace("ws"),
         tensor_or_none("scores"))

SVF_CALL(svf_verify_attn,
         const auto* sh = shape_of<svf_shape_t>(a, 0); void* st = stream(); NoGil free;
         rc = svf_verify_attn(sh, a.ptr[1], a.ptr[2], a.ptr[3], I32(4), I32(5), a.ptr[6], a.ptr[7],
                              U64(8), I32(9), I32(10), a.ptr[11], static_cast<float*>(a.ptr[13]), WS(12), st),
         shape("shape"), tensor("q"), tensor("K"), tensor("V"), tensor("block_table"), tensor("seq_lens"), tensor("k_draft"),
         tensor("v_draft"), tensor("draft_mask"), tensor("sel_idx"), tensor("sel_cnt"), tensor("out"), workspace("ws"),
         tensor_or_none("lse"))

SVF_CALL(svf_verify_attn_static_ws,
         const auto* sh = shape_of<svf_shape_t>(a, 0); void* st = stream(); NoGil free;
         rc = svf_verify_attn_static_ws(sh, a.ptr[1], a.ptr[2], a.ptr[3], I32(4), I32(5), a.ptr[6],
                                        a.ptr[7], U64(8), I32(9), I32(10), a.ptr[11], static_cast<float*>(a.ptr[12]), st),
         shape("shape"), tensor("q"), tensor("K"), tensor("V"), tensor("block_table"), tensor("seq_lens"), tensor("k_draft"),
         tensor("v_draft"), tensor("draft_mask"), tensor("sel_idx"), tensor("sel_cnt"), tensor("out"), tensor_or_none("lse"))

SVF_CALL(svf_verify_step,
         const auto* sh = shape_of<svf_shape_t>(a, 0); void* st = stream(); NoGil free;
         rc = svf_verify_step(sh, (int)a.num[1], a.ptr[2], F32(3), a.ptr[4], a.ptr[5], I32(6), I32(7),
                              a.ptr[8], a.ptr[9], U64(10), static_cast<int32_t*>(a.ptr[11]), static_cast<int32_t*>(a.ptr[12]),
                              a.ptr[13], static_cast<float*>(a.ptr[15]), WS(14), st),
         shape("shape"), number("mode"), tensor("q"), tensor("reps"), tensor("K"), tensor("V"), tensor("block_table"),
         tensor("seq_lens"), tensor("k_draft"), tensor("v_draft"), tensor("draft_mask"), tensor("sel_idx"), tensor("sel_cnt"),
         tensor("out"), workspace("ws"), tensor_or_none("lse"))

SVF_CALL(svf_block_summaries,
         const auto* sh = shape_of<svf_shape_t>(a, 0); const auto* rt = shape_of<svf_retrieval_t>(a, 1);
         void* st = stream(); NoGil free;
         rc = svf_block_summaries(sh, rt, a.ptr[2], I32(3), I32(4),
                                  (int32_t)a.num[6], (int32_t)a.num[7], a.ptr[5], st),
         shape("shape"), shape("retrieval", kSvfRetrieval), tensor("K"), tensor("block_table"), tensor("seq_lens"), tensor("summaries"),
         integer("first_block", 0), integer("n_blocks", -1))

SVF_CALL(svf_retrieve,
         const auto* sh = shape_of<svf_shape_t>(a, 0); const auto* rt = shape_of<svf_retrieval_t>(a, 1);
         void* st = stream(); NoGil free;
         rc = svf_retrieve(sh, rt, a.ptr[2], a.ptr[3], I32(4),
                           static_cast<int32_t*>(a.ptr[5]), static_cast<int32_t*>(a.ptr[6]), static_cast<float*>(a.ptr[8]), WS(7),
                           st),
         shape("shape"), shape("retrieval", kSvfRetrieval), tensor("q"), tensor("summaries"), tensor("seq_lens"), tensor("sel_idx"),
         tensor("sel_cnt"), workspace("ws"), tensor_or_none("scores"))

SVF_CALL(svf_sparse_ffn,
         const auto* sh = shape_of<svf_ffn_shape_t>(a, 0); void* st = stream(); NoGil free;
         rc = svf_sparse_ffn(sh, a.ptr[1], a.ptr[2], a.ptr[3], a.ptr[4], F32(7), F32(8), F32(9),
                             a.ptr[5], static_cast<uint64_t*>(a.ptr[10]), WS(6), st),
         shape("shape", kSvfFfnShape), tensor("x"), tensor("w_gate"), tensor("w_up"), tensor("w_down_t"), tensor("y"), workspace("ws"),
         tensor_or_none("b_gate"), tensor_or_none("b_up"), tensor_or_none("b_down"), tensor_or_none("active"))

SVF_CALL(svf_moe_skip,
         const Sizes d = sizes_of(s, a, 0, 2); void* st = stream(); NoGil free;
         rc = svf_moe_skip(F32(0), d[0], d[1], (int32_t)a.num[1], F32(2), static_cast<int32_t*>(a.ptr[3]),
                           static_cast<uint32_t*>(a.ptr[4]), st),
         tensor("w"), number("m"), tensor("beta"), tensor("n_skip"), tensor("keep_mask"))

SVF_CALL(svf_accept_resample,
         const Sizes d = sizes_of(s, a, 0, 3); void* st = stream(); NoGil free;
         rc = svf_accept_resample(F32(0), F32(1), I32(2), F32(3), F32(4), d[0], d[1], d[2],
                                  static_cast<int32_t*>(a.ptr[5]), static_cast<int32_t*>(a.ptr[6]), st),
         tensor("p_target"), tensor("p_draft"), tensor("draft_tokens"), tensor("u_accept"), tensor("u_resample"),
         tensor("n_accepted"), tensor("resampled"))

// Which classes the shapes are instances of; the binding says so before it makes the first call.
PyObject* set_structures_py(PyObject*, PyObject* args) {
  PyObject* c[kStructures];
  if (!PyArg_ParseTuple(args, "O!O!O!", &PyType_Type, &c[0], &PyType_Type, &c[1], &PyType_Type, &c[2])) return nullptr;
  for (int i = 0; i < kStructures; ++i) {
    Py_INCREF(c[i]);
    Py_XDECREF(reinterpret_cast<PyObject*>(structures[i]));
    structures[i] = reinterpret_cast<PyTypeObject*>(c[i]);
  }
  Py_RETURN_NONE;
}

// The signature as inspect.signature() reads it.
std::string doc_of(const Signature& s) {
  std::string d = std::string(s.where) + "($module";
  for (const Param& p : s.params) {
    d += std::string(", ") + p.name;
    if (p.has_default) d += p.kind == kInt ? "=" + std::to_string(p.value) : "=None";
  }
  return d + ")\n--\n\nThe C entry point of this name (include/*.h), on torch's current stream.";
}

#define SVF_METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME##_py, METH_FASTCALL | METH_KEYWORDS, nullptr}
PyMethodDef methods[] = {SVF_METHOD(svf_block_reps), SVF_METHOD(svf_score_select), SVF_METHOD(svf_verify_attn),
                         SVF_METHOD(svf_verify_attn_static_ws), SVF_METHOD(svf_verify_step), SVF_METHOD(svf_block_summaries),
                         SVF_METHOD(svf_retrieve), SVF_METHOD(svf_sparse_ffn), SVF_METHOD(svf_moe_skip),
                         SVF_METHOD(svf_accept_resample),
                         {"set_structures", set_structures_py, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_svf_calls", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__svf_calls(void) {
  // (in the order of `methods`)
  Signature* const all[] = {&sig_svf_block_reps, &sig_svf_score_select, &sig_svf_verify_attn, &sig_svf_verify_attn_static_ws,
                            &sig_svf_verify_step, &sig_svf_block_summaries, &sig_svf_retrieve, &sig_svf_sparse_ffn,
                            &sig_svf_moe_skip, &sig_svf_accept_resample};
  static std::string docs[sizeof(all) / sizeof(all[0])];
  static_assert(Args::kMost >= 16, "arguments of svf_verify_step");
  for (size_t i = 0; i < sizeof(all) / sizeof(all[0]); ++i) {
    for (Param& p : all[i]->params) p.key = PyUnicode_InternFromString(p.name);
    docs[i] = doc_of(*all[i]);
    methods[i].ml_doc = docs[i].c_str();
  }
  for (PyTypeObject*& t : structures) {      // (no instance fits before set_structures)
    t = Py_TYPE(Py_NotImplemented);
    Py_INCREF(reinterpret_cast<PyObject*>(t));
  }
  return PyModule_Create(&module);
}
