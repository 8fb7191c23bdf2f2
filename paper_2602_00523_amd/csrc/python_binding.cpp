// Python side of the C ABI (include/sage.h): calls that take torch tensors, marshalled in native code.
//
// The calls of a decoding step run for a few microseconds on the GPU each, so what the host spends per call decides how
// fast a program that issues them one by one can go: with the arguments marshalled in Python and passed through ctypes a
// call cost about 9 us of host time before the launch itself (5 us of building the list, 2 us of converting it); here it is
// well under one.  A call is described by two strings (see sage.py): its Python parameters, and one item per C argument
// that says where the argument comes from.  Both are parsed once, into a flat list of operations; calling it fills the C
// arguments from the tensors and numbers and jumps to the library.  `bind` does the same but stops before the jump and
// returns a callable that makes it (sage.prepare).  Nothing here computes anything or knows a device.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>
#include <structmember.h>

#include <cstdint>
#include <cstring>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "sage.h"

namespace {

constexpr int MAX_PARAMS = 48, MAX_ARGS = 56;

// One C argument: integers and pointers as they are, floats in `f`.
union Value { int64_t i; double f; };
template <class T> T as(Value v) {
    if constexpr (std::is_pointer_v<T>) return reinterpret_cast<T>(static_cast<uintptr_t>(v.i));
    else if constexpr (std::is_floating_point_v<T>) return static_cast<T>(v.f);
    else return static_cast<T>(v.i);
}
using Invoke = int (*)(void*, const Value*);
template <class F> struct Caller;
template <class... A> struct Caller<int (*)(A...)> {
    static constexpr int COUNT = sizeof...(A);
    template <size_t... I> static int go(void* fn, const Value* v, std::index_sequence<I...>) {
        return reinterpret_cast<int (*)(A...)>(fn)(as<A>(v[I])...);
    }
    static int invoke(void* fn, const Value* v) { return go(fn, v, std::index_sequence_for<A...>{}); }
};
struct Entry { const char* name; Invoke invoke; int count; };
#define SAGE_ENTRY(f) {#f, &Caller<decltype(&f)>::invoke, Caller<decltype(&f)>::COUNT}
const Entry ENTRIES[] = {
    SAGE_ENTRY(sage_entropy_topk), SAGE_ENTRY(sage_build_tree), SAGE_ENTRY(sage_tree_attention), SAGE_ENTRY(sage_tree_attention_static),
    SAGE_ENTRY(sage_tree_attention_with_plan), SAGE_ENTRY(sage_verify_accept), SAGE_ENTRY(sage_commit_path),
    SAGE_ENTRY(sage_advance_kv_len), SAGE_ENTRY(sage_update_history), SAGE_ENTRY(sage_close_step), SAGE_ENTRY(sage_lm_head_topk),
    SAGE_ENTRY(sage_entropy_topk_slices), SAGE_ENTRY(sage_entropy_topk_slices_pair), SAGE_ENTRY(sage_build_tree_from_slices),
    SAGE_ENTRY(sage_verify_accept_from_slices), SAGE_ENTRY(sage_verify_accept_close_from_slices)};

// What an operation does with its parameter(s); the checks produce no argument.
enum Kind { PTR, INT, FLOAT, SIZE, STRIDE, DTYPE, NBYTES, STRUCT, STREAM, CHECK_DIM, CHECK_UNIT, CHECK_SIZE, CHECK_DTYPE };
struct Op { Kind kind; int n; int a, b; };

struct Program {
    const Entry* entry;
    void* fn;
    std::vector<PyObject*> names;        // parameter names, interned
    std::vector<bool> optional;
    std::vector<PyObject*> defaults;     // for optional parameters
    std::vector<Op> ops;
    PyObject* error;                     // exception class: error(call, status)
    PyObject *module, *doc, *signature;  // what the call shows as __module__, __doc__ and __signature__
};

struct PythonError {};                   // thrown while arguments are read: the Python error is set
struct Reference {                       // owns one
    PyObject* o;
    explicit Reference(PyObject* given) : o(given) { if (!o) throw PythonError{}; }
    ~Reference() { Py_DECREF(o); }
    Reference(const Reference&) = delete;
    Reference& operator=(const Reference&) = delete;
};
int64_t integer(PyObject* o) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw PythonError{};
    return v;
}

// What the operations read of a tensor argument.  A torch.Tensor (or Parameter) is read directly; anything else that has a
// tensor's methods, a subclass that overrides them among it, through these; an object without them is a TypeError.
class TensorArgument {
public:
    TensorArgument(const Program& p, int param, PyObject* o) : program(p), index(param), object(o) {
        if (THPVariable_CheckExact(o)) tensor = &THPVariable_Unpack(o);
    }
    uint64_t address() const {
        if (tensor) return reinterpret_cast<uintptr_t>(tensor->data_ptr());
        const Reference v(PyObject_CallNoArgs(attribute("data_ptr").o));
        const unsigned long long a = PyLong_AsUnsignedLongLongMask(v.o);
        if (PyErr_Occurred()) throw PythonError{};
        return a;
    }
    int64_t nbytes() const {
        if (tensor) return tensor->numel() * static_cast<int64_t>(tensor->element_size());
        const Reference n(PyObject_CallNoArgs(attribute("numel").o)), each(PyObject_CallNoArgs(attribute("element_size").o));
        return integer(n.o) * integer(each.o);
    }
    int64_t dim() const {
        if (tensor) return tensor->dim();
        const Py_ssize_t n = PySequence_Size(attribute("shape").o);
        if (n < 0) throw PythonError{};
        return n;
    }
    int64_t size(int i) const {
        if (tensor) return tensor->size(i);
        const Reference n(PySequence_GetItem(attribute("shape").o, i));
        return integer(n.o);
    }
    int64_t stride(int i) const {
        if (tensor) return tensor->stride(i);
        const Reference n(PyObject_CallFunction(attribute("stride").o, "i", i));
        return integer(n.o);
    }
    at::ScalarType dtype() const {
        if (tensor) return tensor->scalar_type();
        const Reference d = attribute("dtype");
        return THPDtype_Check(d.o) ? reinterpret_cast<THPDtype*>(d.o)->scalar_type : at::ScalarType::Undefined;
    }

private:
    Reference attribute(const char* name) const {
        PyObject* a = PyObject_GetAttrString(object, name);
        if (!a && PyErr_ExceptionMatches(PyExc_AttributeError))
            PyErr_Format(PyExc_TypeError, "%s: %U must be a tensor, not %s", program.entry->name, program.names[index],
                         Py_TYPE(object)->tp_name);
        return Reference(a);
    }
    const Program& program;
    int index;
    PyObject* object;
    const at::Tensor* tensor = nullptr;
};

// The parameters of one call, by position and keyword.  New references are not taken: the caller's objects outlive this.
bool take_parameters(const Program& p, PyObject* const* args, size_t npos, PyObject* kwnames, PyObject** slot) {
    const size_t n = p.names.size();
    if (npos > n) {
        PyErr_Format(PyExc_TypeError, "%s takes at most %zu arguments (%zu given)", p.entry->name, n, npos);
        return false;
    }
    for (size_t i = 0; i < npos; ++i) slot[i] = args[i];
    for (size_t i = npos; i < n; ++i) slot[i] = nullptr;
    const size_t nkw = kwnames ? static_cast<size_t>(PyTuple_GET_SIZE(kwnames)) : 0;
    for (size_t j = 0; j < nkw; ++j) {
        PyObject* key = PyTuple_GET_ITEM(kwnames, j);
        size_t at = n;
        for (size_t i = 0; i < n && at == n; ++i)
            if (p.names[i] == key) at = i;
        for (size_t i = 0; i < n && at == n; ++i)
            if (PyUnicode_Compare(p.names[i], key) == 0) at = i;
        if (at == n || slot[at]) {
            PyErr_Format(PyExc_TypeError, at == n ? "%s got an unexpected argument %R" : "%s got multiple values for argument %R",
                         p.entry->name, key);
            return false;
        }
        slot[at] = args[npos + j];
    }
    for (size_t i = 0; i < n; ++i) {
        if (slot[i]) continue;
        if (!p.optional[i]) {
            PyErr_Format(PyExc_TypeError, "%s is missing the argument %R", p.entry->name, p.names[i]);
            return false;
        }
        slot[i] = p.defaults[i];
    }
    return true;
}

bool fill(const Program& p, PyObject* const* slot, Value* out) {
    for (const Op& op : p.ops) {
        PyObject* o = slot[op.a];
        switch (op.kind) {
            case PTR: {
                if (o == Py_None) { (out++)->i = 0; break; }
                (out++)->i = static_cast<int64_t>(TensorArgument(p, op.a, o).address());
                break;
            }
            case INT: {
                (out++)->i = integer(o);
                break;
            }
            case FLOAT: {
                const double v = PyFloat_AsDouble(o);
                if (v == -1.0 && PyErr_Occurred()) return false;
                (out++)->f = v;
                break;
            }
            case NBYTES: {
                if (o == Py_None) { (out++)->i = 0; break; }
                (out++)->i = TensorArgument(p, op.a, o).nbytes();
                break;
            }
            case STRUCT: {               // a ctypes structure, by address
                Py_buffer view;
                if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return false;
                const bool fits = view.len >= static_cast<Py_ssize_t>(sizeof(sage_tree_params));
                (out++)->i = static_cast<int64_t>(reinterpret_cast<uintptr_t>(view.buf));
                PyBuffer_Release(&view);
                if (!fits) {
                    PyErr_Format(PyExc_TypeError, "%s: %U is too small", p.entry->name, p.names[op.a]);
                    return false;
                }
                break;
            }
            case STREAM: {
                if (o == Py_None) {
                    (out++)->i = static_cast<int64_t>(reinterpret_cast<uintptr_t>(c10::hip::getCurrentHIPStream().stream()));
                    break;
                }
                PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
                if (!h) return false;
                const unsigned long long v = PyLong_AsUnsignedLongLongMask(h);
                Py_DECREF(h);
                if (PyErr_Occurred()) return false;
                (out++)->i = static_cast<int64_t>(v);
                break;
            }
            default: {
                const TensorArgument t(p, op.a, o);
                if (op.kind == CHECK_DIM) {
                    if (t.dim() != op.n) {
                        PyErr_Format(PyExc_ValueError, "%s: %U must have %d dimensions", p.entry->name, p.names[op.a], op.n);
                        return false;
                    }
                } else if (op.kind == DTYPE) {
                    const at::ScalarType type = t.dtype();
                    if (type != at::kFloat && type != at::kBFloat16) {
                        PyErr_SetString(PyExc_TypeError, "float32 or bfloat16 expected");
                        return false;
                    }
                    (out++)->i = type == at::kFloat ? SAGE_F32 : SAGE_BF16;
                } else if (op.kind == CHECK_SIZE || op.kind == CHECK_DTYPE) {
                    const TensorArgument u(p, op.b, slot[op.b]);
                    const bool ok = op.kind == CHECK_DTYPE ? t.dtype() == u.dtype()
                                                           : op.n < t.dim() && op.n < u.dim() && t.size(op.n) == u.size(op.n);
                    if (!ok) {
                        PyErr_Format(PyExc_AssertionError, "%s: %U and %U do not agree", p.entry->name, p.names[op.a], p.names[op.b]);
                        return false;
                    }
                } else {                 // SIZE, STRIDE, CHECK_UNIT: one dimension
                    if (op.n >= t.dim()) {
                        PyErr_Format(PyExc_ValueError, "%s: %U has too few dimensions", p.entry->name, p.names[op.a]);
                        return false;
                    }
                    if (op.kind == SIZE) (out++)->i = t.size(op.n);
                    else if (op.kind == STRIDE) (out++)->i = t.stride(op.n);
                    else if (t.stride(op.n) != 1) {
                        PyErr_Format(PyExc_AssertionError, "%s: %U must be contiguous along its last dimension", p.entry->name, p.names[op.a]);
                        return false;
                    }
                }
            }
        }
    }
    return true;
}

// torch throws for what it cannot give (the address or a stride of a sparse or batched tensor, a stream without a device):
// a Python error, since no C++ exception may leave through the interpreter.
bool marshal(const Program& p, PyObject* const* slot, Value* out) {
    try {
        return fill(p, slot, out);
    } catch (const PythonError&) {
    } catch (const c10::Error& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return false;
}

PyObject* jump(const Program& p, const Value* v) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = p.entry->invoke(p.fn, v);
    Py_END_ALLOW_THREADS
    if (rc == 0) Py_RETURN_NONE;
    PyObject* e = PyObject_CallFunction(p.error, "si", p.entry->name, rc);
    if (e) {
        PyErr_SetObject(p.error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

// ---- the two Python types: a call, and a call with its arguments (both live as long as the process or their last user)
struct CallObject {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    Program* program;
};
struct BoundObject {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    PyObject* call;                      // the CallObject
    PyObject* held;                      // everything the arguments came from
    Value v[MAX_ARGS];
};
PyTypeObject* bound_type = nullptr;

PyObject* call_vectorcall(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* kwnames) {
    const Program& p = *reinterpret_cast<CallObject*>(self)->program;
    PyObject* slot[MAX_PARAMS];
    Value v[MAX_ARGS];
    if (!take_parameters(p, args, PyVectorcall_NARGS(nargsf), kwnames, slot) || !marshal(p, slot, v)) return nullptr;
    return jump(p, v);
}

PyObject* bound_vectorcall(PyObject* self, PyObject* const*, size_t nargsf, PyObject* kwnames) {
    if (PyVectorcall_NARGS(nargsf) != 0 || (kwnames && PyTuple_GET_SIZE(kwnames) != 0)) {
        PyErr_SetString(PyExc_TypeError, "a prepared call takes no arguments");
        return nullptr;
    }
    auto* b = reinterpret_cast<BoundObject*>(self);
    return jump(*reinterpret_cast<CallObject*>(b->call)->program, b->v);
}

PyObject* call_bind(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    const Program& p = *reinterpret_cast<CallObject*>(self)->program;
    PyObject* slot[MAX_PARAMS];
    Value v[MAX_ARGS];
    if (!take_parameters(p, args, static_cast<size_t>(nargs), kwnames, slot) || !marshal(p, slot, v)) return nullptr;
    PyObject* held = PyTuple_New(static_cast<Py_ssize_t>(p.names.size()));
    if (!held) return nullptr;
    for (size_t i = 0; i < p.names.size(); ++i) {
        Py_INCREF(slot[i]);
        PyTuple_SET_ITEM(held, static_cast<Py_ssize_t>(i), slot[i]);
    }
    auto* b = PyObject_New(BoundObject, bound_type);
    if (!b) {
        Py_DECREF(held);
        return nullptr;
    }
    b->vectorcall = bound_vectorcall;
    Py_INCREF(self);
    b->call = self;
    b->held = held;
    std::memcpy(b->v, v, sizeof(v));
    return reinterpret_cast<PyObject*>(b);
}

void call_dealloc(PyObject* self) {
    auto* c = reinterpret_cast<CallObject*>(self);
    if (c->program) {
        for (PyObject* o : c->program->names) Py_DECREF(o);
        for (PyObject* o : c->program->defaults) Py_XDECREF(o);
        Py_XDECREF(c->program->error);
        Py_XDECREF(c->program->module);
        Py_XDECREF(c->program->doc);
        Py_XDECREF(c->program->signature);
        delete c->program;
    }
    PyTypeObject* t = Py_TYPE(self);
    PyObject_Free(self);
    Py_DECREF(t);
}
void bound_dealloc(PyObject* self) {
    auto* b = reinterpret_cast<BoundObject*>(self);
    Py_DECREF(b->held);
    Py_DECREF(b->call);
    PyTypeObject* t = Py_TYPE(self);
    PyObject_Free(self);
    Py_DECREF(t);
}

// A call stands in for a function of its module: it has that one's names, docstring and signature and is pickled by name.
PyObject* call_name(PyObject* self, void*) { return PyUnicode_FromString(reinterpret_cast<CallObject*>(self)->program->entry->name); }
template <PyObject* Program::*WHAT> PyObject* call_get(PyObject* self, void*) {
    PyObject* o = reinterpret_cast<CallObject*>(self)->program->*WHAT;
    Py_INCREF(o);
    return o;
}
PyObject* call_reduce(PyObject* self, PyObject*) { return call_name(self, nullptr); }

PyGetSetDef call_getset[] = {{"__name__", call_name, nullptr, nullptr, nullptr}, {"__qualname__", call_name, nullptr, nullptr, nullptr},
                             {"__module__", call_get<&Program::module>, nullptr, nullptr, nullptr},
                             {"__doc__", call_get<&Program::doc>, nullptr, nullptr, nullptr},
                             {"__signature__", call_get<&Program::signature>, nullptr, nullptr, nullptr},
                             {nullptr, nullptr, nullptr, nullptr, nullptr}};
PyMethodDef call_methods[] = {
    {"__reduce__", call_reduce, METH_NOARGS, nullptr},
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(call_bind)), METH_FASTCALL | METH_KEYWORDS,
     "bind(*args, **kwargs): the call with these arguments, as a callable without any"},
    {nullptr, nullptr, 0, nullptr}};
PyMemberDef call_members[] = {{"__vectorcalloffset__", T_PYSSIZET, offsetof(CallObject, vectorcall), READONLY, nullptr},
                              {nullptr, 0, 0, 0, nullptr}};
PyMemberDef bound_members[] = {{"__vectorcalloffset__", T_PYSSIZET, offsetof(BoundObject, vectorcall), READONLY, nullptr},
                               {nullptr, 0, 0, 0, nullptr}};
PyType_Slot call_slots[] = {{Py_tp_dealloc, reinterpret_cast<void*>(call_dealloc)}, {Py_tp_call, reinterpret_cast<void*>(PyVectorcall_Call)},
                            {Py_tp_methods, call_methods}, {Py_tp_getset, call_getset}, {Py_tp_members, call_members}, {0, nullptr}};
PyType_Slot bound_slots[] = {{Py_tp_dealloc, reinterpret_cast<void*>(bound_dealloc)},
                             {Py_tp_call, reinterpret_cast<void*>(PyVectorcall_Call)}, {Py_tp_members, bound_members}, {0, nullptr}};
PyType_Spec call_spec = {"paper_2602_00523_amd._binding.Call", sizeof(CallObject), 0, Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL,
                         call_slots};
PyType_Spec bound_spec = {"paper_2602_00523_amd._binding.Bound", sizeof(BoundObject), 0,
                          Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL, bound_slots};
PyTypeObject* call_type = nullptr;

std::vector<std::string> words(const char* text) {
    std::vector<std::string> out;
    for (const char* s = text; *s;) {
        while (*s == ' ') ++s;
        const char* e = s;
        while (*e && *e != ' ') ++e;
        if (e != s) out.emplace_back(s, e);
        s = e;
    }
    return out;
}

// make(name, address, params, args, error, module, doc, signature): params = "logits k ... n_valid=None rows=1", args = "ptr:logits dtype:logits ...".
// Raises ValueError when the description does not fit the function's declaration.
PyObject* make(PyObject*, PyObject* args) {
    const char *name, *params, *cargs;
    unsigned long long address;
    PyObject *error, *module, *doc, *signature;
    if (!PyArg_ParseTuple(args, "sKssOUUO", &name, &address, &params, &cargs, &error, &module, &doc, &signature)) return nullptr;
    auto* c = PyObject_New(CallObject, call_type);
    if (!c) return nullptr;
    c->vectorcall = call_vectorcall;
    c->program = new (std::nothrow) Program{};
    auto fail = [&](const std::string& why) -> PyObject* {
        Py_DECREF(c);
        PyErr_Format(PyExc_ValueError, "%s: %s", name, why.c_str());
        return nullptr;
    };
    if (!c->program) return fail("out of memory");
    Program& p = *c->program;
    for (const Entry& e : ENTRIES)
        if (std::strcmp(e.name, name) == 0) p.entry = &e;
    if (!p.entry) return fail("no such call");
    p.fn = reinterpret_cast<void*>(static_cast<uintptr_t>(address));
    Py_INCREF(error);
    p.error = error;
    Py_INCREF(module);
    p.module = module;
    Py_INCREF(doc);
    p.doc = doc;
    Py_INCREF(signature);
    p.signature = signature;
    std::vector<std::string> names;
    for (const std::string& w : words(params)) {
        const size_t eq = w.find('=');
        names.push_back(w.substr(0, eq));
        p.names.push_back(PyUnicode_InternFromString(names.back().c_str()));
        p.optional.push_back(eq != std::string::npos);
        PyObject* d = nullptr;
        if (eq != std::string::npos) {
            if (w.substr(eq + 1) == "None") {
                Py_INCREF(Py_None);
                d = Py_None;
            } else {
                d = PyLong_FromString(w.c_str() + eq + 1, nullptr, 10);
            }
        }
        p.defaults.push_back(d);
    }
    if (names.size() > MAX_PARAMS) return fail("too many parameters");
    auto index = [&](const std::string& s) {
        for (size_t i = 0; i < names.size(); ++i)
            if (names[i] == s) return static_cast<int>(i);
        return -1;
    };
    int count = 0;
    for (const std::string& w : words(cargs)) {
        const size_t colon = w.find(':');
        if (colon == std::string::npos) return fail("bad item " + w);
        std::string what = w.substr(0, colon), first = w.substr(colon + 1), second;
        const size_t comma = first.find(',');
        if (comma != std::string::npos) {
            second = first.substr(comma + 1);
            first.resize(comma);
        }
        int n = 0;
        if (!what.empty() && what.back() >= '0' && what.back() <= '9') {
            n = what.back() - '0';
            what.pop_back();
        }
        static const struct { const char* name; Kind kind; } KINDS[] = {
            {"ptr", PTR}, {"int", INT}, {"float", FLOAT}, {"size", SIZE}, {"stride", STRIDE}, {"dtype", DTYPE}, {"nbytes", NBYTES},
            {"struct", STRUCT}, {"stream", STREAM}, {"dim", CHECK_DIM}, {"unit", CHECK_UNIT}, {"same", CHECK_SIZE}, {"sametype", CHECK_DTYPE}};
        const Kind* kind = nullptr;
        for (const auto& k : KINDS)
            if (what == k.name) kind = &k.kind;
        const int a = index(first), b = second.empty() ? 0 : index(second);
        if (!kind || a < 0 || b < 0) return fail("bad item " + w);
        p.ops.push_back(Op{*kind, n, a, b});
        if (*kind < CHECK_DIM) ++count;
    }
    if (count != p.entry->count || count > MAX_ARGS) return fail("the description has another number of arguments than the declaration");
    return reinterpret_cast<PyObject*>(c);
}

PyMethodDef module_methods[] = {{"make", make, METH_VARARGS, "make(name, address, params, args, error, module, doc, signature): a call"}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_binding", "Calls of libsage_hip.so with torch tensors, marshalled natively.", -1,
                          module_methods};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
    call_type = reinterpret_cast<PyTypeObject*>(PyType_FromSpec(&call_spec));
    bound_type = reinterpret_cast<PyTypeObject*>(PyType_FromSpec(&bound_spec));
    if (!call_type || !bound_type) return nullptr;
    return PyModule_Create(&module_def);
}
