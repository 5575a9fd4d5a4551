// Argument marshalling of the Python binding in native code: a call object holds the address of one C entry point and what each
// of its arguments has to be, checks the tensors it is handed (on the GPU, contiguous, of the type wanted) and calls the entry
// point with their addresses.  A call of the library costs the host some 3 us for the launch; the same checks made tensor by
// tensor in Python and passed through ctypes cost as much again (host time of one layer's append and attention, 17 tensors: 18.6 us so, 14.8 here; of an
// early exit's rank check, compaction and restore 30.2 and 17.0).
//
// Argument kinds: 't' any tensor, 'f' 'i' 'b' 'l' tensor of float32 / int32 / uint8 / int64 (all: or None, a null pointer),
// 'S' an object with a buffer (a ctypes structure), 'n' an integer.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <structmember.h>
#include <hip/hip_runtime_api.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/cuda/Event.h>

#include <cstdint>
#include <string>
#include <vector>

namespace {

constexpr int kMaxArgs = 20;

struct Call {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    void* address;
    std::string* kinds;
    std::vector<std::string>* names;
};

// All arguments are pointers or integers, which the System V x86-64 convention passes alike, one register or stack word each.
template <int... I>
long long invoke_n(void* f, const uint64_t* a, std::integer_sequence<int, I...>) {
    return reinterpret_cast<int (*)(decltype((void)I, uint64_t{})...)>(f)(a[I]...);
}
template <int N>
int invoke(void* f, const uint64_t* a) { return (int)invoke_n(f, a, std::make_integer_sequence<int, N>{}); }
typedef int (*Invoke)(void*, const uint64_t*);
template <int... N>
Invoke invoke_of(int n, std::integer_sequence<int, N...>) {
    static const Invoke table[] = {invoke<N>...};
    return table[n];
}

// Address of tensor `o` (None: 0).  False with a Python error set.
bool address_of(PyObject* o, char kind, const std::string& name, uint64_t& out) {
    if (o == Py_None) {
        out = 0;
        return true;
    }
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a tensor", name.c_str());
        return false;
    }
    try {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda()) {
            PyErr_Format(PyExc_ValueError, "%s must live on the GPU", name.c_str());
            return false;
        }
        if (!t.is_contiguous()) {
            PyErr_Format(PyExc_ValueError, "%s must be contiguous", name.c_str());
            return false;
        }
        const at::ScalarType have = t.scalar_type();
        const at::ScalarType want = kind == 'f' ? at::kFloat : kind == 'i' ? at::kInt : kind == 'b' ? at::kByte : kind == 'l' ? at::kLong : have;
        if (have != want) {
            const char* type = kind == 'f' ? "torch.float32" : kind == 'i' ? "torch.int32" : kind == 'b' ? "torch.uint8" : "torch.int64";
            PyObject* dtype = PyObject_GetAttrString(o, "dtype");
            if (dtype) PyErr_Format(PyExc_ValueError, "%s must be %s, got %S", name.c_str(), type, dtype);
            Py_XDECREF(dtype);
            return false;
        }
        out = (uint64_t)t.data_ptr();
        return true;
    } catch (const std::exception& e) {  // (tensors without storage, for one)
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return false;
    }
}

PyObject* call(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* kwnames) {
    const Call* c = reinterpret_cast<Call*>(self);
    const Py_ssize_t n = PyVectorcall_NARGS(nargsf);
    if ((kwnames && PyTuple_GET_SIZE(kwnames) > 0) || n != (Py_ssize_t)c->kinds->size()) {
        PyErr_Format(PyExc_TypeError, "expected %zu positional arguments, got %zd", c->kinds->size(), n);
        return nullptr;
    }
    uint64_t a[kMaxArgs];
    Py_buffer held[2];
    int n_held = 0;
    bool ok = true;
    for (Py_ssize_t k = 0; ok && k < n; ++k) {
        const char kind = (*c->kinds)[k];
        if (kind == 'n') {
            a[k] = PyLong_AsUnsignedLongLongMask(args[k]);
            ok = !(a[k] == (uint64_t)-1 && PyErr_Occurred());
        } else if (kind == 'S') {
            ok = PyObject_GetBuffer(args[k], &held[n_held], PyBUF_SIMPLE) == 0;
            if (ok) a[k] = (uint64_t)held[n_held++].buf;
        } else {
            ok = address_of(args[k], kind, (*c->names)[k], a[k]);
        }
    }
    int rc = 0;
    if (ok) {
        const Invoke f = invoke_of((int)n, std::make_integer_sequence<int, kMaxArgs + 1>{});
        Py_BEGIN_ALLOW_THREADS
        rc = f(c->address, a);
        Py_END_ALLOW_THREADS
    }
    while (n_held > 0) PyBuffer_Release(&held[--n_held]);
    return ok ? PyLong_FromLong(rc) : nullptr;
}

void dealloc(PyObject* self) {
    Call* c = reinterpret_cast<Call*>(self);
    delete c->kinds;
    delete c->names;
    PyTypeObject* type = Py_TYPE(self);
    type->tp_free(self);
    Py_DECREF(type);
}

PyMemberDef members[] = {{"__vectorcalloffset__", T_PYSSIZET, offsetof(Call, vectorcall), READONLY, nullptr},
                         {nullptr, 0, 0, 0, nullptr}};
PyType_Slot slots[] = {{Py_tp_dealloc, (void*)dealloc}, {Py_tp_call, (void*)PyVectorcall_Call}, {Py_tp_members, members}, {0, nullptr}};
PyType_Spec spec = {"_marshal.Call", sizeof(Call), 0, Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL | Py_TPFLAGS_DISALLOW_INSTANTIATION, slots};
PyObject* call_type = nullptr;

// make(address, kinds, names) -> call object
PyObject* make(PyObject*, PyObject* args) {
    unsigned long long address;
    const char* kinds;
    PyObject* names;
    if (!PyArg_ParseTuple(args, "KsO!", &address, &kinds, &PyTuple_Type, &names)) return nullptr;
    const std::string k(kinds);
    size_t buffers = 0;
    for (char x : k) buffers += x == 'S';
    if ((Py_ssize_t)k.size() != PyTuple_GET_SIZE(names) || k.size() > kMaxArgs || buffers > 2 || k.find_first_not_of("tfiblSn") != std::string::npos) {
        PyErr_SetString(PyExc_ValueError, "one name for each of at most 20 kinds out of t f i b l S n, at most two of them S");
        return nullptr;
    }
    std::vector<std::string> list;
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(names); ++i) {
        const char* s = PyUnicode_AsUTF8(PyTuple_GET_ITEM(names, i));
        if (!s) return nullptr;
        list.push_back(s);
    }
    PyTypeObject* type = reinterpret_cast<PyTypeObject*>(call_type);
    Call* c = reinterpret_cast<Call*>(type->tp_alloc(type, 0));
    if (!c) return nullptr;
    c->vectorcall = call;
    c->address = (void*)(uintptr_t)address;
    c->kinds = new std::string(k);
    c->names = new std::vector<std::string>(std::move(list));
    return reinterpret_cast<PyObject*>(c);
}

// without_system_fence(event): the unrecorded torch.cuda.Event gets a HIP event that releases nothing to the host when it is
// recorded; it can still be asked whether the work before it is done.  Between two launches the ordinary one costs the GPU
// 2.9 us, this one 1.1: 32 layers of attention 1431 -> 1370 us, one of a few short requests 12.1 -> 10.4.
PyObject* event_base = nullptr;  // torch._C._CudaEventBase
PyObject* without_system_fence(PyObject*, PyObject* event) {
    const int is = PyObject_IsInstance(event, event_base);
    if (is != 1) {
        if (is == 0) PyErr_SetString(PyExc_TypeError, "a torch.cuda.Event is wanted");
        return nullptr;
    }
    reinterpret_cast<THCPEvent*>(event)->cuda_event = at::cuda::CUDAEvent(hipEventDisableTiming | hipEventDisableSystemFence);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"without_system_fence", without_system_fence, METH_O, "make an unrecorded torch.cuda.Event a light one"},
                         {"make", make, METH_VARARGS, "make(address, kinds, names): a callable for the C entry point"}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
    call_type = PyType_FromSpec(&spec);
    PyObject* torch_c = call_type ? PyImport_ImportModule("torch._C") : nullptr;
    event_base = torch_c ? PyObject_GetAttrString(torch_c, "_CudaEventBase") : nullptr;
    Py_XDECREF(torch_c);
    return event_base ? PyModule_Create(&module) : nullptr;
}
