// Argument marshalling of the hot entry points for Python callers: tensors to data pointers, the current stream, and the
// call, without an interpreter frame in between.
//
// A verification step of one layer is five calls of this library behind one another, and on short prefixes the host is
// what bounds it.  Marshalled in Python through ctypes, a call costs 1.5 - 2.2 us beside its launches (10 - 14 method calls
// on tensors, a conversion of every argument); here 0.25 - 0.3.
//
// Only the plain case is taken: exact torch.Tensor, int, float, bool and None arguments and the library's own descriptor.
// Whatever else arrives - subclasses, numpy numbers, stream objects, a wrong or missing argument, a tensor without
// storage, an active torch-function mode - goes to the Python function of the same name, which converts it or raises as it
// always did.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

namespace {

enum Kind : uint8_t {
  kDesc,      // descriptor, by address
  kPtr,       // tensor, address or None
  kI32,       // int, its low 32 bits (as ctypes passes it)
  kI64,
  kF32,
  kBytes,     // bytes of the tensor `workspace`, if None
  kStream,    // address, or None for the current stream
  kCheck      // raise on a status other than zero
};

union Slot {
  void* p;
  int64_t i;
  float f;
};

struct Param {
  const char* name;
  Kind kind;
  bool optional;
  Slot value;      // of an optional parameter that is left out
};

Param need(const char* n, Kind k) { return {n, k, false, {nullptr}}; }
Param opt(const char* n, Kind k, int64_t v = 0) {
  Param p{n, k, true, {nullptr}};
  p.value.i = v;
  return p;
}
Param opt_f(const char* n, float v) {
  Param p{n, kF32, true, {nullptr}};
  p.value.i = 0;
  p.value.f = v;
  return p;
}

constexpr int kMaxParams = 24;

// One function: its parameters in Python's order, and the call with the slots in that order.
struct Function {
  const char* name;      // of the Python function; the C entry point is specext_<name>
  int n;
  Param param[kMaxParams];
  int (*call)(void* fn, const Slot* s);
  void* fn = nullptr;    // address of the entry point
  PyObject* names[kMaxParams] = {};
  int workspace = -1;    // slot of the workspace, whose size a kBytes parameter defaults to
  int check = -1;        // slot of `check`
};

using P = void*;
using I = int32_t;
using L = int64_t;

I i32(const Slot& s) { return static_cast<I>(s.i); }
size_t bytes(const Slot& s) { return static_cast<size_t>(s.i); }

Function functions[] = {
    {"verify_attn", 13,
     {need("desc", kDesc), need("q", kPtr), need("k_prefix", kPtr), need("v_prefix", kPtr), need("k_tree", kPtr),
      need("v_tree", kPtr), need("parent", kPtr), need("out", kPtr), need("lse", kPtr), need("workspace", kPtr),
      opt("workspace_nbytes", kBytes), opt("stream", kStream), opt("check", kCheck, 1)},
     [](void* fn, const Slot* s) {
       return reinterpret_cast<int (*)(P, P, P, P, P, P, P, P, P, P, size_t, P)>(fn)(
           s[0].p, s[1].p, s[2].p, s[3].p, s[4].p, s[5].p, s[6].p, s[7].p, s[8].p, s[9].p, bytes(s[10]), s[11].p);
     }},
    {"verify_attn_static", 12,
     {need("desc", kDesc), need("q", kPtr), need("k_prefix", kPtr), need("v_prefix", kPtr), need("k_tree", kPtr),
      need("v_tree", kPtr), need("parent", kPtr), need("out", kPtr), need("lse", kPtr), opt("status_out", kPtr),
      opt("stream", kStream), opt("check", kCheck, 1)},
     [](void* fn, const Slot* s) {
       return reinterpret_cast<int (*)(P, P, P, P, P, P, P, P, P, P, P)>(fn)(
           s[0].p, s[1].p, s[2].p, s[3].p, s[4].p, s[5].p, s[6].p, s[7].p, s[8].p, s[9].p, s[10].p);
     }},
    {"chunk_scores", 7,
     {need("desc", kDesc), need("workspace", kPtr), need("score_row", kI32), need("scores", kPtr),
      opt("workspace_nbytes", kBytes), opt("stream", kStream), opt("check", kCheck, 1)},
     [](void* fn, const Slot* s) {
       return reinterpret_cast<int (*)(P, P, size_t, I, P, P)>(fn)(s[0].p, s[1].p, bytes(s[4]), i32(s[2]), s[3].p, s[5].p);
     }},
    {"chunk_scores_accepted", 8,
     {need("desc", kDesc), need("workspace", kPtr), need("path", kPtr), need("n_accept", kPtr), need("scores", kPtr),
      opt("workspace_nbytes", kBytes), opt("stream", kStream), opt("check", kCheck, 1)},
     [](void* fn, const Slot* s) {
       return reinterpret_cast<int (*)(P, P, size_t, P, P, P, P)>(fn)(s[0].p, s[1].p, bytes(s[5]), s[2].p, s[3].p, s[4].p,
                                                                      s[6].p);
     }},
    {"chunk_scores_select", 12,
     {need("desc", kDesc), need("workspace", kPtr), need("score_row", kI32), need("k", kI32), need("idx_out", kPtr),
      need("n_out", kPtr), opt("scores", kPtr), opt("path", kPtr), opt("n_accept", kPtr), opt("workspace_nbytes", kBytes),
      opt("stream", kStream), opt("check", kCheck, 1)},
     [](void* fn, const Slot* s) {
       return reinterpret_cast<int (*)(P, P, size_t, I, P, P, I, P, P, P, P)>(fn)(
           s[0].p, s[1].p, bytes(s[9]), i32(s[2]), s[7].p, s[8].p, i32(s[3]), s[6].p, s[4].p, s[5].p, s[10].p);
     }},
    {"select_chunks", 7,
     {need("scores", kPtr), need("n_chunks", kI32), need("k", kI32), need("idx_out", kPtr), need("n_out", kPtr),
      opt("stream", kStream), opt("check", kCheck, 1)},
     [](void* fn, const Slot* s) {
       return reinterpret_cast<int (*)(P, I, I, P, P, P)>(fn)(s[0].p, i32(s[1]), i32(s[2]), s[3].p, s[4].p, s[5].p);
     }},
    {"gather_draft_kv", 19,
     {need("k_src", kPtr), need("v_src", kPtr), need("k_dst", kPtr), need("v_dst", kPtr), need("idx", kPtr),
      need("n_idx", kPtr), need("max_idx", kI32), need("n_layers", kI32), need("n_kv_heads", kI32), need("src_len", kI32),
      need("dst_cap", kI32), need("head_dim", kI32), need("chunk_size", kI32), need("elem_bytes", kI32),
      opt("pos_out", kPtr), opt("len_out", kPtr), opt("stream", kStream), opt("check", kCheck, 1), opt("src_cap", kI32)},
     [](void* fn, const Slot* s) {
       return reinterpret_cast<int (*)(P, P, P, P, P, P, I, I, I, I, I, I, I, I, I, P, P, P)>(fn)(
           s[0].p, s[1].p, s[2].p, s[3].p, s[4].p, s[5].p, i32(s[6]), i32(s[7]), i32(s[8]), i32(s[9]), i32(s[18]), i32(s[10]),
           i32(s[11]), i32(s[12]), i32(s[13]), s[14].p, s[15].p, s[16].p);
     }},
    {"accept_greedy", 10,
     {need("parent", kPtr), need("draft_token", kPtr), need("target_token", kPtr), need("first_target", kPtr),
      need("n_tree", kI32), need("path_out", kPtr), need("n_accept_out", kPtr), need("next_token_out", kPtr),
      opt("stream", kStream), opt("check", kCheck, 1)},
     [](void* fn, const Slot* s) {
       return reinterpret_cast<int (*)(P, P, P, P, I, P, P, P, P)>(fn)(s[0].p, s[1].p, s[2].p, s[3].p, i32(s[4]), s[5].p,
                                                                       s[6].p, s[7].p, s[8].p);
     }},
    {"commit_tree_kv", 22,
     {need("k_tree", kPtr), need("v_tree", kPtr), need("k_cache", kPtr), need("v_cache", kPtr), need("path", kPtr),
      need("n_accept", kPtr), need("max_accept", kI32), need("n_tree", kI32), need("n_layers", kI32),
      need("n_kv_heads", kI32), need("head_dim", kI32), need("elem_bytes", kI32), need("prefix_len", kI32),
      need("cache_capacity", kI32), opt("tree_stride_layer", kI64), opt("tree_stride_h", kI64), opt("tree_stride_t", kI64),
      opt("cache_stride_layer", kI64), opt("cache_stride_h", kI64), opt("cache_stride_l", kI64), opt("stream", kStream),
      opt("check", kCheck, 1)},
     [](void* fn, const Slot* s) {
       return reinterpret_cast<int (*)(P, P, P, P, P, P, I, I, I, I, I, I, I, I, L, L, L, L, L, L, P)>(fn)(
           s[0].p, s[1].p, s[2].p, s[3].p, s[4].p, s[5].p, i32(s[6]), i32(s[7]), i32(s[8]), i32(s[9]), i32(s[10]), i32(s[11]),
           i32(s[12]), i32(s[13]), s[14].i, s[15].i, s[16].i, s[17].i, s[18].i, s[19].i, s[20].p);
     }},
    {"prefill_attn", 21,
     {need("q", kPtr), need("k", kPtr), need("v", kPtr), need("out", kPtr), need("lse", kPtr), need("n_q_heads", kI32),
      need("n_kv_heads", kI32), need("head_dim", kI32), need("q_len", kI32), need("kv_len", kI32), opt("dtype", kI32, 1),
      opt("out_dtype", kI32, 1), opt_f("softmax_scale", 0.f), opt("q_stride_t", kI64), opt("q_stride_h", kI64),
      opt("kv_stride_h", kI64), opt("kv_stride_l", kI64), opt("o_stride_t", kI64), opt("o_stride_h", kI64),
      opt("stream", kStream), opt("check", kCheck, 1)},
     [](void* fn, const Slot* s) {
       return reinterpret_cast<int (*)(P, P, P, P, P, I, I, I, I, I, I, I, float, L, L, L, L, L, L, P)>(fn)(
           s[0].p, s[1].p, s[2].p, s[3].p, s[4].p, i32(s[5]), i32(s[6]), i32(s[7]), i32(s[8]), i32(s[9]), i32(s[10]),
           i32(s[11]), s[12].f, s[13].i, s[14].i, s[15].i, s[16].i, s[17].i, s[18].i, s[19].p);
     }},
};

bool stream_ready = false;      // the GPU runtime is up (Python has read a current stream once)

struct Call {
  PyObject_HEAD
  vectorcallfunc vectorcall;
  Function* function;
  PyObject* slow;        // the Python function
  PyTypeObject* desc;    // type of the descriptor
  PyObject* raise;       // (status, name of the C entry point) -> raises
  PyObject* weak;        // weak references to this
};

// int within 64 bits
bool to_i64(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long long x = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow) return false;
  *v = x;
  return true;
}

bool is_plain_tensor(PyObject* o) { return Py_TYPE(o) == reinterpret_cast<PyTypeObject*>(THPVariableClass); }

// Converts one argument; false = leave the call to the Python function.
bool convert(const Call& c, Kind kind, PyObject* o, Slot* s) {
  switch (kind) {
    case kDesc: {
      if (Py_TYPE(o) != c.desc) return false;
      Py_buffer view;
      if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return false;
      s->p = view.buf;             // the caller's argument keeps the object alive over the call
      PyBuffer_Release(&view);
      return true;
    }
    case kPtr:
      if (is_plain_tensor(o)) {
        s->p = THPVariable_Unpack(o).data_ptr();
        return true;
      }
      [[fallthrough]];
    case kStream:
      if (o == Py_None) {
        s->p = nullptr;
        return true;
      }
      return to_i64(o, &s->i) && s->i >= 0;
    case kBytes:
      return to_i64(o, &s->i) && s->i >= 0;
    case kI32:
    case kI64:
      return to_i64(o, &s->i);
    case kF32:
      if (!PyFloat_CheckExact(o)) return false;
      s->f = static_cast<float>(PyFloat_AS_DOUBLE(o));
      return true;
    case kCheck:
      s->i = o == Py_True;
      return o == Py_True || o == Py_False;
  }
  return false;
}

// Fills the slots; false (with no exception set) = leave the call to the Python function.
bool marshal(const Call& c, PyObject* const* args, Py_ssize_t n_pos, PyObject* kwnames, Slot* slot) {
  const Function& f = *c.function;
  if (!f.fn || n_pos > f.n || at::impl::torch_function_mode_enabled()) return false;
  PyObject* given[kMaxParams] = {};
  for (Py_ssize_t i = 0; i < n_pos; ++i) given[i] = args[i];
  const Py_ssize_t n_kw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
  for (Py_ssize_t k = 0; k < n_kw; ++k) {
    PyObject* name = PyTuple_GET_ITEM(kwnames, k);
    int at = 0;
    while (at < f.n && f.names[at] != name) ++at;          // both interned as a rule
    if (at == f.n || given[at]) return false;
    given[at] = args[n_pos + k];
  }
  for (int i = 0; i < f.n; ++i) {
    const Param& p = f.param[i];
    PyObject* o = given[i];
    if (!o && !p.optional) return false;
    if ((p.kind == kStream || p.kind == kBytes) && (!o || o == Py_None)) {
      if (p.kind == kStream) {
        if (!stream_ready) return false;
        slot[i].p = c10::hip::getCurrentHIPStream().stream();
      } else {
        if (!given[f.workspace] || !is_plain_tensor(given[f.workspace])) return false;
        const at::Tensor& t = THPVariable_Unpack(given[f.workspace]);
        slot[i].i = t.numel() * t.element_size();
      }
    } else if (!o) {
      slot[i] = p.value;
    } else if (!convert(c, p.kind, o, &slot[i])) {
      return false;
    }
  }
  return true;
}

PyObject* call(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* kwnames) {
  const Call& c = *reinterpret_cast<Call*>(self);
  const Function& f = *c.function;
  const Py_ssize_t n_pos = PyVectorcall_NARGS(nargsf);
  Slot slot[kMaxParams];
  bool plain = false;
  try {
    plain = marshal(c, args, n_pos, kwnames, slot);
  } catch (...) {               // what a tensor or the runtime threw, the Python function will report
  }
  if (!plain) {
    PyErr_Clear();
    return PyObject_Vectorcall(c.slow, args, n_pos, kwnames);
  }
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = f.call(f.fn, slot);
  Py_END_ALLOW_THREADS
  if (status != 0 && slot[f.check].i) {
    char name[64];
    PyOS_snprintf(name, sizeof name, "specext_%s", f.name);
    PyObject* r = PyObject_CallFunction(c.raise, "is", status, name);
    if (!r) return nullptr;
    Py_DECREF(r);
  }
  return PyLong_FromLong(status);
}

int call_traverse(PyObject* self, visitproc visit, void* arg) {
  Call* c = reinterpret_cast<Call*>(self);
  Py_VISIT(c->slow);
  Py_VISIT(c->desc);
  Py_VISIT(c->raise);
  return 0;
}

int call_clear(PyObject* self) {
  Call* c = reinterpret_cast<Call*>(self);
  Py_CLEAR(c->slow);
  Py_CLEAR(c->desc);
  Py_CLEAR(c->raise);
  return 0;
}

void call_dealloc(PyObject* self) {
  PyObject_GC_UnTrack(self);
  if (reinterpret_cast<Call*>(self)->weak) PyObject_ClearWeakRefs(self);
  call_clear(self);
  Py_TYPE(self)->tp_free(self);
}

// In everything but the call and its type this is the Python function: its attributes are that one's, to read and to write, as
// a class attribute it binds, and copy and pickle refer to it by its name.
PyObject* call_getattro(PyObject* self, PyObject* name) {
  PyObject* slow = reinterpret_cast<Call*>(self)->slow;
  if (PyUnicode_Check(name)) {
    if (PyUnicode_CompareWithASCIIString(name, "__wrapped__") == 0) {
      Py_INCREF(slow);
      return slow;
    }
    for (const char* of_type : {"__class__", "__call__", "__get__", "__reduce__", "__reduce_ex__"})
      if (PyUnicode_CompareWithASCIIString(name, of_type) == 0) return PyObject_GenericGetAttr(self, name);
  }
  return PyObject_GetAttr(slow, name);
}

int call_setattro(PyObject* self, PyObject* name, PyObject* value) {      // value NULL: deleted
  return PyObject_SetAttr(reinterpret_cast<Call*>(self)->slow, name, value);
}

PyObject* call_repr(PyObject* self) { return PyObject_Repr(reinterpret_cast<Call*>(self)->slow); }

PyObject* call_descr_get(PyObject* self, PyObject* object, PyObject*) {
  if (object && object != Py_None) return PyMethod_New(self, object);
  Py_INCREF(self);
  return self;
}

PyObject* call_reduce(PyObject* self, PyObject*) {
  return PyObject_GetAttrString(reinterpret_cast<Call*>(self)->slow, "__qualname__");
}

PyMethodDef call_methods[] = {{"__reduce__", call_reduce, METH_NOARGS, nullptr},
                              {"__reduce_ex__", call_reduce, METH_O, nullptr},
                              {nullptr, nullptr, 0, nullptr}};

PyTypeObject call_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyObject* py_wrap(PyObject*, PyObject* args) {
  const char* name;
  PyObject *slow, *desc, *raise;
  if (!PyArg_ParseTuple(args, "sOO!O", &name, &slow, &PyType_Type, &desc, &raise)) return nullptr;
  for (Function& f : functions) {
    if (std::strcmp(f.name, name) != 0) continue;
    Call* c = PyObject_GC_New(Call, &call_type);
    if (!c) return nullptr;
    c->vectorcall = call;
    c->function = &f;
    Py_INCREF(slow);
    c->slow = slow;
    Py_INCREF(desc);
    c->desc = reinterpret_cast<PyTypeObject*>(desc);
    Py_INCREF(raise);
    c->raise = raise;
    c->weak = nullptr;
    PyObject_GC_Track(c);
    return reinterpret_cast<PyObject*>(c);
  }
  return PyErr_Format(PyExc_KeyError, "no function %s", name);
}

PyObject* py_bind(PyObject*, PyObject* args) {
  const char* name;
  unsigned long long address;
  if (!PyArg_ParseTuple(args, "sK", &name, &address)) return nullptr;
  for (Function& f : functions)
    if (std::strcmp(f.name, name) == 0) {
      f.fn = reinterpret_cast<void*>(static_cast<uintptr_t>(address));
      Py_RETURN_NONE;
    }
  return PyErr_Format(PyExc_KeyError, "no function %s", name);
}

PyObject* py_set_stream_ready(PyObject*, PyObject*) {
  stream_ready = true;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"wrap", py_wrap, METH_VARARGS, "wrap(name, python_function, descriptor_type, raise_on_status): callable of the same signature"},
    {"bind", py_bind, METH_VARARGS, "bind(name, address of the C entry point); 0: every call goes to the Python function"},
    {"set_stream_ready", py_set_stream_ready, METH_NOARGS, "the GPU runtime is up: current streams may be read"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "argument marshalling of the hot entry points", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
  for (Function& f : functions) {
    for (int i = 0; i < f.n; ++i) {
      f.names[i] = PyUnicode_InternFromString(f.param[i].name);
      if (!f.names[i]) return nullptr;
      if (std::strcmp(f.param[i].name, "workspace") == 0) f.workspace = i;
      if (f.param[i].kind == kCheck) f.check = i;
    }
  }
  call_type.tp_name = "paper_2505_20776_amd._marshal.Call";
  call_type.tp_basicsize = sizeof(Call);
  call_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL;
  call_type.tp_vectorcall_offset = offsetof(Call, vectorcall);
  call_type.tp_call = PyVectorcall_Call;
  call_type.tp_traverse = call_traverse;
  call_type.tp_clear = call_clear;
  call_type.tp_dealloc = call_dealloc;
  call_type.tp_getattro = call_getattro;
  call_type.tp_setattro = call_setattro;
  call_type.tp_repr = call_repr;
  call_type.tp_descr_get = call_descr_get;
  call_type.tp_methods = call_methods;
  call_type.tp_weaklistoffset = offsetof(Call, weak);
  if (PyType_Ready(&call_type) < 0) return nullptr;
  PyObject* m = PyModule_Create(&module);
  if (!m) return nullptr;
  PyObject* names = PyTuple_New(sizeof(functions) / sizeof(functions[0]));
  if (!names) return nullptr;
  for (size_t i = 0; i < sizeof(functions) / sizeof(functions[0]); ++i)
    PyTuple_SET_ITEM(names, i, PyUnicode_FromString(functions[i].name));
  if (PyModule_AddObject(m, "FUNCTIONS", names) < 0) return nullptr;
  return m;
}
