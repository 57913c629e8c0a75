// Argument marshalling of the Python binding (host code).  A hook step issued
// call by call from Python is bound by this work when its kernels are small: a
// toy step of one 3 us kernel took 15 us, 11 of them in attribute lookups and
// ctypes conversions.  A Function holds one C entry point, the checks of its
// Python arguments and the order of its C arguments, parsed once at import from
// two lines of text; a call then checks and converts every tensor directly.
//
// Arguments, one word each, in Python order:
//   name:dtype[dims]  a CUDA, contiguous tensor; dtype i32, f32, bf16, an upper
//                     case letter (any activation type, the same wherever the
//                     letter stands) or * (any); dims: numbers, names (bound
//                     where they stand first, equal elsewhere) or _ (any), after
//                     "..." the last ones only; {dim}: the element count instead;
//                     dim^: a Route is passed on with at most so many slots, so
//                     that a kernel which reads all rows of its slots stays inside
//                     a tensor of fewer rows
//   name?:...         the same, or None (a null pointer)
//   name:struct(S)    an object whose `struct` is of the ctypes class given for S;
//                     that struct is passed
//   name:rt(S)        the same, its T_max bound to T
//   name:bits(n)      a sequence of ints (at most 32 pass); n is bound to its length
//   name:int          an int
//   name:dim          an int that the dim of this name is bound to
//   name:stream       None (the current stream), a torch stream or a handle
//                     (anything that int() takes)
// C arguments: an argument's name, a bound dim, @L (the type code of letter L),
// #name (the element count of a tensor), %name (its bytes, 0 for None).
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cstdint>
#include <map>
#include <string>
#include <vector>

#include "../../include/xmix.h"

namespace {

constexpr int kMaxArgs = 24, kMaxDims = 12, kMaxBits = 32, kMaxBitArgs = 2;

enum Kind { TENSOR, STRUCT, BITS, INT, STREAM };
enum { ANY_TYPE = -1, LETTER = -2 };

struct Arg {
    std::string name;
    Kind kind = TENSOR;
    bool optional = false;
    int dtype = ANY_TYPE;  // at::ScalarType, ANY_TYPE or LETTER
    int letter = 0;
    bool tail = false, count = false, shaped = false;
    int cut = -1;               // the dim with a ^
    std::vector<int64_t> dims;  // >= 0: a number; -1: any; <= -2: name -2 - v
    int bind = -1;              // STRUCT, BITS, INT: the dim that is bound (-1: none)
    PyTypeObject* type = nullptr;  // STRUCT: the class of the struct (a reference)
};
struct Out {
    enum What { ARG, DIM, TYPE, COUNT, BYTES } what;
    int i;
};

struct Function {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    void* addr;
    std::string* name;
    std::vector<Arg>* args;
    std::vector<Out>* outs;
    PyObject* spec;  // the texts and classes it was made of
    int n_dims;
    int route;  // the Route argument where a tensor may cut it, else -1
};

PyObject *s_T_max, *s_struct, *s_cuda_stream, *raw_stream, *get_device;

// References held for the length of a call.
struct Held {
    PyObject* o[kMaxArgs];
    int n = 0;
    ~Held() {
        for (int i = 0; i < n; ++i) Py_DECREF(o[i]);
    }
};

PyObject* fail(const Function* f, const Arg& a, const char* what) {
    return PyErr_Format(PyExc_AssertionError, "%s: %s: %s", f->name->c_str(), a.name.c_str(), what);
}

// A dim is bound by its first use (-1: not yet) and compared after it; a
// negative int is no size.
bool bind(int64_t* dims, int i, int64_t v) {
    if (dims[i] < 0) dims[i] = v;
    return v >= 0 && dims[i] == v;
}
bool dim_ok(int64_t* dims, int64_t want, int64_t v) {
    if (want >= 0) return want == v;
    return want == -1 || bind(dims, static_cast<int>(-2 - want), v);
}

bool attr_u64(PyObject* o, PyObject* name, uint64_t* v) {
    PyObject* x = PyObject_GetAttr(o, name);
    if (!x) return false;
    *v = PyLong_AsUnsignedLongLongMask(x);
    Py_DECREF(x);
    return !PyErr_Occurred();
}

PyObject* call(PyObject* self, PyObject* const* argv, size_t nargsf, PyObject* kwnames) {
    HANDLE_TH_ERRORS  // a tensor without storage throws when asked for its data
    Function* f = reinterpret_cast<Function*>(self);
    const std::vector<Arg>& args = *f->args;
    const size_t n = static_cast<size_t>(PyVectorcall_NARGS(nargsf));
    if (n != args.size() || (kwnames && PyTuple_GET_SIZE(kwnames) > 0))
        return PyErr_Format(PyExc_TypeError, "%s takes %zu positional arguments", f->name->c_str(),
                            args.size());
    uint64_t value[kMaxArgs];
    int64_t count[kMaxArgs], bytes[kMaxArgs], dims[kMaxDims];
    int letters[26];
    int32_t bits[kMaxBitArgs][kMaxBits];
    int n_bits = 0;
    Held held;
    int64_t slots = INT64_MAX;  // most slots of a Route that is passed on
    xmix_route route;
    for (int i = 0; i < f->n_dims; ++i) dims[i] = -1;
    for (int& l : letters) l = -1;
    for (size_t i = 0; i < n; ++i) {
        const Arg& a = args[i];
        PyObject* o = argv[i];
        value[i] = 0;
        count[i] = bytes[i] = 0;
        switch (a.kind) {
            case TENSOR: {
                if (o == Py_None && a.optional) break;
                if (!THPVariable_Check(o)) return fail(f, a, "a tensor is needed");
                const at::Tensor& t = THPVariable_Unpack(o);
                if (!t.is_cuda()) {
                    PyErr_SetString(PyExc_ValueError, "tensor must live on the GPU");
                    return nullptr;
                }
                if (!t.is_contiguous()) {
                    PyErr_SetString(PyExc_ValueError, "tensor must be contiguous");
                    return nullptr;
                }
                const int type = static_cast<int>(t.scalar_type());
                if (a.dtype == LETTER) {
                    int& l = letters[a.letter];
                    if (l < 0) {
                        if (type != static_cast<int>(at::kBFloat16) &&
                            type != static_cast<int>(at::kFloat)) {
                            PyErr_SetString(PyExc_TypeError, "unsupported activation dtype");
                            return nullptr;
                        }
                        l = type;
                    }
                    if (l != type) return fail(f, a, "another dtype is needed");
                } else if (a.dtype != ANY_TYPE && a.dtype != type) {
                    return fail(f, a, "another dtype is needed");
                }
                count[i] = t.numel();
                bytes[i] = count[i] * static_cast<int64_t>(t.element_size());
                if (a.count) {
                    if (!dim_ok(dims, a.dims[0], count[i])) return fail(f, a, "wrong size");
                    if (a.cut == 0) slots = std::min(slots, count[i]);
                } else if (a.shaped) {
                    const int64_t nd = t.dim(), want = static_cast<int64_t>(a.dims.size());
                    if (a.tail ? nd < want : nd != want) return fail(f, a, "wrong shape");
                    for (int64_t k = 0; k < want; ++k)
                        if (!dim_ok(dims, a.dims[k], t.size(nd - want + k)))
                            return fail(f, a, "wrong shape");
                    if (a.cut >= 0) slots = std::min(slots, t.size(nd - want + a.cut));
                }
                value[i] = reinterpret_cast<uint64_t>(t.mutable_data_ptr());
                break;
            }
            case STRUCT: {
                PyObject* st = PyObject_GetAttr(o, s_struct);
                if (!st) return nullptr;
                held.o[held.n++] = st;
                if (!PyObject_TypeCheck(st, a.type))
                    return PyErr_Format(PyExc_TypeError, "%s: %s: a struct of class %s is needed",
                                        f->name->c_str(), a.name.c_str(), a.type->tp_name);
                Py_buffer view;  // a ctypes struct exports its memory, which lives as long as it
                if (PyObject_GetBuffer(st, &view, PyBUF_SIMPLE) < 0) return nullptr;
                value[i] = reinterpret_cast<uint64_t>(view.buf);
                PyBuffer_Release(&view);
                uint64_t T = 0;
                if (a.bind >= 0 && !attr_u64(o, s_T_max, &T)) return nullptr;
                if (a.bind >= 0 && !bind(dims, a.bind, static_cast<int64_t>(T)))
                    return fail(f, a, "made for another number of token slots");
                break;
            }
            case BITS: {
                PyObject* seq = PySequence_Fast(o, "app bits must be a sequence");
                if (!seq) return nullptr;
                const Py_ssize_t nb = PySequence_Fast_GET_SIZE(seq);
                if (!bind(dims, a.bind, nb)) {
                    Py_DECREF(seq);
                    return fail(f, a, "wrong number of app bits");
                }
                // (more than 32 are counted, and refused by the C entry point)
                for (Py_ssize_t k = 0; k < nb && k < kMaxBits; ++k) {
                    const long v = PyLong_AsLong(PySequence_Fast_GET_ITEM(seq, k));
                    if (v == -1 && PyErr_Occurred()) {
                        Py_DECREF(seq);
                        return nullptr;
                    }
                    bits[n_bits][k] = static_cast<int32_t>(v);
                }
                Py_DECREF(seq);
                value[i] = reinterpret_cast<uint64_t>(bits[n_bits++]);
                break;
            }
            case INT: {
                const long long v = PyLong_AsLongLong(o);
                if (v == -1 && PyErr_Occurred()) return nullptr;
                value[i] = static_cast<uint64_t>(v);
                if (a.bind >= 0 && !bind(dims, a.bind, v)) return fail(f, a, "wrong size");
                break;
            }
            case STREAM: {
                PyObject* s = nullptr;
                if (o == Py_None) {
                    PyObject* dev = PyObject_CallNoArgs(get_device);
                    if (!dev) return nullptr;
                    s = PyObject_CallOneArg(raw_stream, dev);
                    Py_DECREF(dev);
                } else if (PyLong_Check(o)) {
                    s = o;
                    Py_INCREF(s);
                } else {
                    s = PyObject_GetAttr(o, s_cuda_stream);
                    if (!s && PyErr_ExceptionMatches(PyExc_AttributeError)) {
                        PyErr_Clear();
                        s = PyNumber_Long(o);
                    }
                }
                if (!s) return nullptr;
                value[i] = PyLong_AsUnsignedLongLongMask(s);
                Py_DECREF(s);
                if (PyErr_Occurred()) return nullptr;
                break;
            }
        }
    }
    if (f->route >= 0) {
        route = *reinterpret_cast<const xmix_route*>(value[f->route]);
        if (route.T_max > slots) {
            route.T_max = static_cast<int32_t>(slots);
            value[f->route] = reinterpret_cast<uint64_t>(&route);
        }
    }
    uint64_t c[kMaxArgs] = {};
    for (size_t i = 0; i < f->outs->size(); ++i) {
        const Out& o = (*f->outs)[i];
        switch (o.what) {
            case Out::ARG: c[i] = value[o.i]; break;
            case Out::DIM: c[i] = static_cast<uint64_t>(dims[o.i] < 0 ? 0 : dims[o.i]); break;
            case Out::TYPE:
                c[i] = letters[o.i] == static_cast<int>(at::kBFloat16) ? 1u : 0u;
                break;
            case Out::COUNT: c[i] = static_cast<uint64_t>(count[o.i]); break;
            case Out::BYTES: c[i] = static_cast<uint64_t>(bytes[o.i]); break;
        }
    }
    // Every C argument is a pointer or an integer of at most 64 bits, so each
    // takes one register or one eight-byte stack slot (System V x86-64), and
    // slots past the callee's own are not looked at.
    using U = uint64_t;
    using Fn = int (*)(U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U);
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = reinterpret_cast<Fn>(f->addr)(
        c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7], c[8], c[9], c[10], c[11], c[12], c[13],
        c[14], c[15], c[16], c[17], c[18], c[19], c[20], c[21], c[22], c[23]);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
    END_HANDLE_TH_ERRORS
}

std::vector<std::string> words(const std::string& s, char sep) {
    std::vector<std::string> w(1);
    for (char ch : s) {
        if (ch == sep) {
            if (!w.back().empty()) w.emplace_back();
        } else {
            w.back() += ch;
        }
    }
    if (w.back().empty()) w.pop_back();
    return w;
}

struct Parser {
    PyObject* structs;  // name -> ctypes class
    std::map<std::string, int> dim_of;
    int dim(const std::string& n) {
        return dim_of.emplace(n, static_cast<int>(dim_of.size())).first->second;
    }
    int64_t dim_word(const std::string& w) {
        if (w == "_") return -1;
        if (w[0] >= '0' && w[0] <= '9') return std::stoll(w);
        return -2 - dim(w);
    }
    bool arg(const std::string& w, Arg* a) {
        const size_t colon = w.find(':');
        if (colon == std::string::npos) return false;
        a->name = w.substr(0, colon);
        if (a->name.back() == '?') {
            a->optional = true;
            a->name.pop_back();
        }
        std::string t = w.substr(colon + 1);
        const bool rt = t.rfind("rt(", 0) == 0;
        if ((rt || t.rfind("struct(", 0) == 0) && t.back() == ')') {
            const size_t open = t.find('(') + 1;
            PyObject* type = PyDict_GetItemString(structs, t.substr(open, t.size() - open - 1).c_str());
            if (!type || !PyType_Check(type)) return false;
            a->kind = STRUCT;
            a->type = reinterpret_cast<PyTypeObject*>(type);
            if (rt) a->bind = dim("T");
        } else if (t == "int" || t == "dim") {
            a->kind = INT;
            if (t == "dim") a->bind = dim(a->name);
        } else if (t == "stream") {
            a->kind = STREAM;
        } else if (t.rfind("bits(", 0) == 0 && t.back() == ')') {
            a->kind = BITS;
            a->bind = dim(t.substr(5, t.size() - 6));
        } else {
            const size_t open = t.find_first_of("[{");
            const std::string type = t.substr(0, open);
            if (type == "i32") a->dtype = static_cast<int>(at::kInt);
            else if (type == "f32") a->dtype = static_cast<int>(at::kFloat);
            else if (type == "bf16") a->dtype = static_cast<int>(at::kBFloat16);
            else if (type == "*") a->dtype = ANY_TYPE;
            else if (type.size() == 1 && type[0] >= 'A' && type[0] <= 'Z') {
                a->dtype = LETTER;
                a->letter = type[0] - 'A';
            } else {
                return false;
            }
            if (open != std::string::npos) {
                a->shaped = true;
                a->count = t[open] == '{';
                std::string in = t.substr(open + 1, t.size() - open - 2);
                if (in.rfind("...,", 0) == 0) {
                    a->tail = true;
                    in = in.substr(4);
                }
                for (std::string d : words(in, ',')) {
                    if (d.back() == '^') {
                        a->cut = static_cast<int>(a->dims.size());
                        d.pop_back();
                    }
                    if (d.empty()) return false;
                    a->dims.push_back(dim_word(d));
                }
                if (a->dims.empty()) return false;
            }
        }
        return true;
    }
};

int init(PyObject* self, PyObject* args, PyObject*) {
    Function* f = reinterpret_cast<Function*>(self);
    const char *name, *in, *out;
    unsigned long long addr;
    PyObject* structs;
    if (!PyArg_ParseTuple(args, "sKssO!", &name, &addr, &in, &out, &PyDict_Type, &structs)) return -1;
    f->spec = PyTuple_GetSlice(args, 2, 5);
    if (!f->spec) return -1;
    f->addr = reinterpret_cast<void*>(addr);
    f->name = new std::string(name);
    f->args = new std::vector<Arg>;
    f->outs = new std::vector<Out>;
    Parser p{structs};
    int bit_args = 0;
    bool cut = false;
    for (const std::string& w : words(in, ' ')) {
        Arg a;
        if (!p.arg(w, &a)) {
            PyErr_Format(PyExc_ValueError, "%s: bad argument '%s'", name, w.c_str());
            return -1;
        }
        bit_args += a.kind == BITS;
        Py_XINCREF(a.type);
        cut = cut || a.cut >= 0;
        f->args->push_back(a);
    }
    auto arg_of = [&](const std::string& n) {
        for (size_t i = 0; i < f->args->size(); ++i)
            if ((*f->args)[i].name == n) return static_cast<int>(i);
        return -1;
    };
    for (const std::string& w : words(out, ' ')) {
        Out o{Out::ARG, arg_of(w)};
        if (w[0] == '@') o = {Out::TYPE, w[1] - 'A'};
        else if (w[0] == '#') o = {Out::COUNT, arg_of(w.substr(1))};
        else if (w[0] == '%') o = {Out::BYTES, arg_of(w.substr(1))};
        else if (o.i < 0 && p.dim_of.count(w)) o = {Out::DIM, p.dim_of[w]};
        if (o.i < 0) {
            PyErr_Format(PyExc_ValueError, "%s: unknown C argument '%s'", name, w.c_str());
            return -1;
        }
        f->outs->push_back(o);
    }
    f->n_dims = static_cast<int>(p.dim_of.size());
    f->route = cut ? arg_of("route") : -1;
    if (cut && (f->route < 0 || (*f->args)[f->route].kind != STRUCT)) {
        PyErr_Format(PyExc_ValueError, "%s: no route to cut", name);
        return -1;
    }
    if (f->args->size() > kMaxArgs || f->outs->size() > kMaxArgs || f->n_dims > kMaxDims ||
        bit_args > kMaxBitArgs) {
        PyErr_Format(PyExc_ValueError, "%s: too many arguments", name);
        return -1;
    }
    f->vectorcall = call;
    return 0;
}

void dealloc(PyObject* self) {
    Function* f = reinterpret_cast<Function*>(self);
    if (f->args)
        for (const Arg& a : *f->args) Py_XDECREF(a.type);
    Py_XDECREF(f->spec);
    delete f->name;
    delete f->args;
    delete f->outs;
    Py_TYPE(self)->tp_free(self);
}

PyMemberDef members[] = {
    {"spec", T_OBJECT_EX, offsetof(Function, spec), READONLY, "(arguments, C arguments, structs)"},
    {nullptr, 0, 0, 0, nullptr}};
PyTypeObject function_type = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) {
    function_type.tp_name = "_call.Function";
    function_type.tp_basicsize = sizeof(Function);
    function_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL;
    function_type.tp_vectorcall_offset = offsetof(Function, vectorcall);
    function_type.tp_members = members;
    function_type.tp_call = PyVectorcall_Call;
    function_type.tp_new = PyType_GenericNew;
    function_type.tp_init = init;
    function_type.tp_dealloc = dealloc;
    if (PyType_Ready(&function_type) < 0) return nullptr;
    PyObject* c = PyImport_ImportModule("torch._C");
    if (!c) return nullptr;
    raw_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
    get_device = PyObject_GetAttrString(c, "_cuda_getDevice");
    Py_DECREF(c);
    if (!raw_stream || !get_device) return nullptr;
    s_T_max = PyUnicode_InternFromString("T_max");
    s_struct = PyUnicode_InternFromString("struct");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    PyObject* m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&function_type);
    if (PyModule_AddObject(m, "Function", reinterpret_cast<PyObject*>(&function_type)) < 0) return nullptr;
    return m;
}
