// Calls of the C entry points from Python with torch tensors: one native object per handle and entry point that checks the
// call's tensors and passes their addresses on.  In Python the checks of a tensor took 0.33 us, half of the host time of a call;
// the forward layer of a tiny model (five calls, 21 tensors) was bound by them.
//
// A Call is made from the entry's address and, for each of its arguments (all of them pointers), what stands there: an int, passed
// on as it is; "int", an int given at the call; or (dtype, numel, name), a tensor given at the call, None for a null pointer.  A
// tensor that is not plainly fine (of the dtype, contiguous, on the device, large enough) goes to the Python check instead, which
// raises the error or returns its address.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/Dtype.h>

#include <cstddef>
#include <utility>

namespace {

constexpr int MAX_ARGS = 16;
struct Arg { enum Kind { FIXED, INT, TENSOR } kind; void* fixed; PyObject *dtype, *numel, *name; at::ScalarType type; int64_t least; };
struct Call {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    void* entry;
    PyObject* check;                                       // the Python check: (tensor, dtype, numel, name) -> address
    int n, n_given;
    Arg args[MAX_ARGS];
};

template <size_t... I> int call_entry(void* f, void** a, std::index_sequence<I...>)
{
    typedef int (*fn)(decltype((void)I, (void*)nullptr)...);
    return reinterpret_cast<fn>(f)(a[I]...);
}
template <size_t N> int call_n(void* f, void** a) { return call_entry(f, a, std::make_index_sequence<N>{}); }
typedef int (*caller)(void*, void**);
template <size_t... I> caller caller_of(int n, std::index_sequence<I...>)
{
    static const caller all[] = {call_n<I>...};
    return all[n];
}

// The address of a tensor that is plainly fine.
bool plain_address(PyObject* o, const Arg& a, void** p)
{
    if (!THPVariable_CheckExact(o)) return false;
    try {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.defined() || !t.is_cuda() || t.scalar_type() != a.type || t.layout() != at::kStrided || !t.is_contiguous() || t.numel() < a.least) return false;
        *p = t.data_ptr();
        return true;
    } catch (...) {
        return false;
    }
}

PyObject* call_vector(PyObject* self, PyObject* const* given, size_t nargsf, PyObject* kwnames)
{
    Call* c = reinterpret_cast<Call*>(self);
    if (PyVectorcall_NARGS(nargsf) != c->n_given || (kwnames && PyTuple_GET_SIZE(kwnames))) {
        PyErr_Format(PyExc_TypeError, "%d positional arguments expected", c->n_given);
        return nullptr;
    }
    void* p[MAX_ARGS];
    for (int i = 0; i < c->n; ++i) {
        const Arg& a = c->args[i];
        if (a.kind == Arg::FIXED) { p[i] = a.fixed; continue; }
        PyObject* o = *given++;
        if (a.kind == Arg::TENSOR) {
            if (o == Py_None) { p[i] = nullptr; continue; }
            if (plain_address(o, a, &p[i])) continue;
            PyObject* r = PyObject_CallFunctionObjArgs(c->check, o, a.dtype, a.numel, a.name, nullptr);
            if (!r) return nullptr;
            p[i] = r == Py_None ? nullptr : PyLong_AsVoidPtr(r);
            Py_DECREF(r);
        } else {
            p[i] = PyLong_AsVoidPtr(o);
        }
        if (!p[i] && PyErr_Occurred()) return nullptr;
    }
    const caller f = caller_of(c->n, std::make_index_sequence<MAX_ARGS + 1>{});
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f(c->entry, p);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

void drop(Call* c)
{
    for (int i = 0; i < c->n; ++i) { Py_XDECREF(c->args[i].dtype); Py_XDECREF(c->args[i].numel); Py_XDECREF(c->args[i].name); }
    Py_XDECREF(c->check);
}
void call_dealloc(PyObject* self)
{
    drop(reinterpret_cast<Call*>(self));
    Py_TYPE(self)->tp_free(self);
}

// Call(entry, args, check)
PyObject* call_new(PyTypeObject* type, PyObject* args, PyObject*)
{
    PyObject *entry, *spec, *check;
    if (!PyArg_ParseTuple(args, "OO!O", &entry, &PyTuple_Type, &spec, &check)) return nullptr;
    if (PyTuple_GET_SIZE(spec) > MAX_ARGS) { PyErr_SetString(PyExc_ValueError, "too many arguments"); return nullptr; }
    Call* c = reinterpret_cast<Call*>(type->tp_alloc(type, 0));        // zeroed
    if (!c) return nullptr;
    c->vectorcall = call_vector;
    c->entry = PyLong_AsVoidPtr(entry);
    Py_INCREF(check);
    c->check = check;
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(spec) && !PyErr_Occurred(); ++i) {
        PyObject* o = PyTuple_GET_ITEM(spec, i);
        Arg& a = c->args[c->n++];
        if (PyLong_Check(o)) { a.kind = Arg::FIXED; a.fixed = PyLong_AsVoidPtr(o); continue; }
        ++c->n_given;
        if (PyUnicode_Check(o)) { a.kind = Arg::INT; continue; }
        a.kind = Arg::TENSOR;
        if (!PyArg_ParseTuple(o, "OOO", &a.dtype, &a.numel, &a.name)) { a.dtype = a.numel = a.name = nullptr; break; }
        Py_INCREF(a.dtype); Py_INCREF(a.numel); Py_INCREF(a.name);
        if (!THPDtype_Check(a.dtype)) { PyErr_SetString(PyExc_TypeError, "a torch.dtype expected"); break; }
        a.type = reinterpret_cast<THPDtype*>(a.dtype)->scalar_type;
        a.least = PyLong_AsLongLong(a.numel);
    }
    if (PyErr_Occurred()) { Py_DECREF(c); return nullptr; }
    return reinterpret_cast<PyObject*>(c);
}

PyTypeObject CallType = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", "Native calls of the entry points", -1, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall()
{
    CallType.tp_name = "_pycall.Call";
    CallType.tp_basicsize = sizeof(Call);
    CallType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL;
    CallType.tp_vectorcall_offset = offsetof(Call, vectorcall);
    CallType.tp_call = PyVectorcall_Call;
    CallType.tp_new = call_new;
    CallType.tp_dealloc = call_dealloc;
    if (PyType_Ready(&CallType) < 0) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&CallType);
    if (PyModule_AddObject(m, "Call", reinterpret_cast<PyObject*>(&CallType)) < 0) { Py_DECREF(m); return nullptr; }
    return m;
}
