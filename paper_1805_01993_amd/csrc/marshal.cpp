// Native argument marshalling for binding.py (the module _marshal): checks the tensors of a call, takes their addresses and
// torch's current stream, and calls the C entry point.  A small pass is bound by what the host does between two launches: a
// one-launch call took 4.8 us through ctypes and tensor attributes read from Python, 1.5 of them before the library was
// entered.  Only the ordinary case is taken: plain torch tensors that fit, and no mode that wants to see what is asked of
// tensors (torch.overrides.TorchFunctionMode).  Everything else is answered with
// None, and binding.py goes its own way, which accepts what it accepted and raises what it raised.
#include <Python.h>

#include <cstddef>
#include <cstdint>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

constexpr int kMaxTensors = 3, kMaxCalls = 16, kBuffers = 5;
using Call2 = int (*)(const void *, void *, void *, void *);
using Call3 = int (*)(const void *, void *, void *, void *, void *);
using NodeCall2 = int (*)(const void *, int, void *, void *, void *);
using NodeCall3 = int (*)(const void *, int, void *, void *, void *, void *);

// The entry points, as calls() has named them once: address, whether a node number comes first, the buffers.
struct Entry {
    uintptr_t fn = 0;
    bool node = false;
    int tensors = 0;
    int buffer[kMaxTensors] = {};
};
Entry table[kMaxCalls];
int entries = 0;

// The calls of one bound plan.
struct Marshal {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    const void *plan;
    PyObject *fail;                   // fail(status, call) raises
    int64_t elem_bytes;
    int64_t numel[kBuffers];          // elements of V, Vbar, X, D, Phi
};

// marshal(call, [node,] tensor, ...) -> 0, or None: not an ordinary call.  Raises what fail() makes of another status.
PyObject *marshal_call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames)
{
    const Marshal *m = reinterpret_cast<const Marshal *>(self);
    const Py_ssize_t n = PyVectorcall_NARGS(nargsf);
    if (kwnames || n < 1 || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    const long id = PyLong_AsLong(args[0]);
    if (id < 0 || id >= entries) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const Entry &e = table[id];
    const Py_ssize_t first = e.node ? 2 : 1;
    if (n != first + e.tensors) Py_RETURN_NONE;
    int node = 0;
    if (e.node) {
        if (!PyLong_CheckExact(args[1])) Py_RETURN_NONE;
        const long v = PyLong_AsLong(args[1]);
        if (v < -1 || v > INT32_MAX || (v == -1 && PyErr_Occurred())) {       // no long either: -1 and an exception
            PyErr_Clear();
            Py_RETURN_NONE;
        }
        node = (int)v;
    }
    void *ptr[kMaxTensors];
    void *stream;
    try {
        for (int i = 0; i < e.tensors; i++) {
            PyObject *o = args[first + i];
            if (!THPVariable_CheckExact(o)) Py_RETURN_NONE;
            const at::Tensor &t = THPVariable_Unpack(o);
            if (t.numel() != m->numel[e.buffer[i]] || !t.is_cuda() || !t.is_contiguous() || (int64_t)t.element_size() != m->elem_bytes)
                Py_RETURN_NONE;
            ptr[i] = t.data_ptr();
        }
        stream = c10::hip::getCurrentHIPStream().stream();
    } catch (...) {
        Py_RETURN_NONE;
    }
    int status;
    Py_BEGIN_ALLOW_THREADS
    const void *plan = m->plan;
    if (e.node)
        status = e.tensors == 2 ? reinterpret_cast<NodeCall2>(e.fn)(plan, node, ptr[0], ptr[1], stream)
                                : reinterpret_cast<NodeCall3>(e.fn)(plan, node, ptr[0], ptr[1], ptr[2], stream);
    else
        status = e.tensors == 2 ? reinterpret_cast<Call2>(e.fn)(plan, ptr[0], ptr[1], stream)
                                : reinterpret_cast<Call3>(e.fn)(plan, ptr[0], ptr[1], ptr[2], stream);
    Py_END_ALLOW_THREADS
    if (status != 0) return PyObject_CallFunction(m->fail, "il", status, id);
    return PyLong_FromLong(0);
}

// Marshal(plan, fail, elem_bytes, elements of V, Vbar, X, D, Phi)
PyObject *marshal_new(PyTypeObject *type, PyObject *args, PyObject *)
{
    unsigned long long plan;
    long long elem_bytes, numel[kBuffers];
    PyObject *fail;
    if (!PyArg_ParseTuple(args, "KOLLLLLL", &plan, &fail, &elem_bytes, &numel[0], &numel[1], &numel[2], &numel[3], &numel[4]))
        return nullptr;
    PyObject *self = type->tp_alloc(type, 0);
    if (!self) return nullptr;
    Marshal *m = reinterpret_cast<Marshal *>(self);
    m->vectorcall = marshal_call;
    m->plan = reinterpret_cast<const void *>((uintptr_t)plan);
    m->fail = Py_NewRef(fail);
    m->elem_bytes = elem_bytes;
    for (int i = 0; i < kBuffers; i++) m->numel[i] = numel[i];
    return self;
}

// calls([(function address, takes a node, (buffer, ...)), ...]): once, when the library is loaded
PyObject *set_calls(PyObject *, PyObject *calls)
{
    if (!PyList_Check(calls) || PyList_GET_SIZE(calls) > kMaxCalls) {
        PyErr_SetString(PyExc_ValueError, "a list of calls");
        return nullptr;
    }
    Entry read[kMaxCalls];
    for (Py_ssize_t i = 0; i < PyList_GET_SIZE(calls); i++) {
        unsigned long long fn;
        int node;
        PyObject *buffers;
        if (!PyArg_ParseTuple(PyList_GET_ITEM(calls, i), "KpO!", &fn, &node, &PyTuple_Type, &buffers)) return nullptr;
        Entry &e = read[i];
        e.fn = (uintptr_t)fn;
        e.node = node != 0;
        e.tensors = (int)PyTuple_GET_SIZE(buffers);
        for (int t = 0; t < e.tensors && t < kMaxTensors; t++) {
            const long b = PyLong_AsLong(PyTuple_GET_ITEM(buffers, t));
            if (b < 0 || b >= kBuffers) e.tensors = -1;
            else e.buffer[t] = (int)b;
        }
        if (PyErr_Occurred()) return nullptr;
        if (e.tensors < 2 || e.tensors > kMaxTensors) {
            PyErr_SetString(PyExc_ValueError, "two or three buffers of five");
            return nullptr;
        }
    }
    entries = (int)PyList_GET_SIZE(calls);
    for (int i = 0; i < entries; i++) table[i] = read[i];
    Py_RETURN_NONE;
}

void marshal_dealloc(PyObject *self)
{
    Py_XDECREF(reinterpret_cast<Marshal *>(self)->fail);
    Py_TYPE(self)->tp_free(self);
}

PyTypeObject marshal_type = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyMethodDef functions[] = {{"calls", set_calls, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, functions, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void)
{
    marshal_type.tp_name = "_marshal.Marshal";
    marshal_type.tp_basicsize = sizeof(Marshal);
    marshal_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL;
    marshal_type.tp_vectorcall_offset = offsetof(Marshal, vectorcall);
    marshal_type.tp_call = PyVectorcall_Call;
    marshal_type.tp_new = marshal_new;
    marshal_type.tp_dealloc = marshal_dealloc;
    if (PyType_Ready(&marshal_type) < 0) return nullptr;
    PyObject *m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&marshal_type);
    if (PyModule_AddObject(m, "Marshal", reinterpret_cast<PyObject *>(&marshal_type)) < 0) {
        Py_DECREF(&marshal_type);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
