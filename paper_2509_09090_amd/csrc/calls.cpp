// Argument marshalling of the entry points that a program calls once per layer or per token: torch tensors in, the C ABI's pointers,
// sizes and pitches out.  A call through ctypes spends 1.3 us on them (a conversion object per argument, a Python call per pointer, size
// and pitch), as much again as half of the launch itself (2.1 us), and the small launches of this library are over in 2 to 4 us; here it
// takes 0.2 us.  Nothing is computed or kept: what a function is told is read from the tensors on every call.
//
// A `Calls` object is made from the addresses of the loaded library's functions and has a method per function; a status that is not zero
// goes to the Python function that raises.
// Arguments that are not plain tensors (subclasses, which may answer for themselves) are asked the way Python would ask them.
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>

#include "sqap.h"

namespace {

struct PyFailed {};                       // a Python exception has been set

void check(bool ok)
{
    if (!ok) throw PyFailed{};
}

struct Ref {
    PyObject *p;
    explicit Ref(PyObject *owned) : p(owned) { check(p != nullptr); }
    ~Ref() { Py_XDECREF(p); }
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
};

// integers as ctypes takes them: whatever has an index, the low bits
int64_t as_i64(PyObject *o)
{
    if (PyFloat_Check(o)) {
        PyErr_SetString(PyExc_TypeError, "int expected instead of float instance");
        throw PyFailed{};
    }
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    check(v != (unsigned long long)-1 || !PyErr_Occurred());
    return (int64_t)v;
}
int32_t as_i32(PyObject *o) { return (int32_t)as_i64(o); }
double as_double(PyObject *o)
{
    const double v = PyFloat_AsDouble(o);
    check(v != -1.0 || !PyErr_Occurred());
    return v;
}

bool plain(PyObject *o) { return THPVariable_CheckExact(o); }

void *ptr(PyObject *o)
{
    if (o == Py_None) return nullptr;
    if (plain(o)) return THPVariable_Unpack(o).data_ptr();
    const Ref v(PyObject_CallMethod(o, "data_ptr", nullptr));
    return reinterpret_cast<void *>(as_i64(v.p));
}
template <class T>
T *ptr(PyObject *o) { return static_cast<T *>(ptr(o)); }

int64_t size(PyObject *o, int dim)
{
    if (plain(o)) {
        const auto sizes = THPVariable_Unpack(o).sizes();
        if (dim < (int)sizes.size()) return sizes[dim];
        PyErr_SetString(PyExc_IndexError, "tuple index out of range");
        throw PyFailed{};
    }
    const Ref shape(PyObject_GetAttrString(o, "shape"));
    const Ref v(PySequence_GetItem(shape.p, dim));
    return as_i64(v.p);
}

// the size of `dim`, of a tensor that has to have `dims` of them
int64_t size_of(PyObject *o, int dims, int dim)
{
    int64_t have;
    if (plain(o)) {
        have = THPVariable_Unpack(o).dim();
    } else {
        const Ref shape(PyObject_GetAttrString(o, "shape"));
        have = PySequence_Size(shape.p);
        check(have >= 0);
    }
    if (have != dims) {
        PyErr_Format(PyExc_ValueError, "%s values to unpack (expected %d)", have < dims ? "not enough" : "too many", dims);
        throw PyFailed{};
    }
    return size(o, dim);
}

int64_t pitch(PyObject *o)
{
    if (plain(o)) return THPVariable_Unpack(o).stride(0);
    const Ref v(PyObject_CallMethod(o, "stride", "i", 0));
    return as_i64(v.p);
}

int64_t count(PyObject *o)
{
    if (plain(o)) return THPVariable_Unpack(o).numel();
    const Ref v(PyObject_CallMethod(o, "numel", nullptr));
    return as_i64(v.p);
}

size_t bytes(PyObject *o)
{
    if (o == Py_None) return 0;
    if (plain(o)) {
        const at::Tensor &t = THPVariable_Unpack(o);
        return (size_t)t.numel() * t.element_size();
    }
    const Ref v(PyObject_CallMethod(o, "element_size", nullptr));
    return (size_t)count(o) * (size_t)as_i64(v.p);
}

// a handle as ctypes keeps it (c_void_p, None once it has been freed)
template <class T>
T *handle(PyObject *o)
{
    if (o == Py_None) return nullptr;
    const Ref v(PyObject_GetAttrString(o, "value"));
    return v.p == Py_None ? nullptr : reinterpret_cast<T *>(as_i64(v.p));
}

int64_t rows_of(PyObject *X, PyObject *rows) { return rows == Py_None ? size(X, 0) : count(rows); }

struct Calls {
    PyObject_HEAD
    decltype(&sqap_attn_scores_batch) attn_scores_batch;
    decltype(&sqap_prune_topk) prune_topk;
    decltype(&sqap_kept_rows) kept_rows;
    decltype(&sqap_prune_rows) prune_rows;
    decltype(&sqap_prune_select) prune_select;
    decltype(&sqap_quantize_act) quantize_act;
    decltype(&sqap_rmsnorm_quantize_act) rmsnorm_quantize_act;
    decltype(&sqap_swiglu_quantize_act) swiglu_quantize_act;
    decltype(&sqap_rope) rope;
    decltype(&sqap_rope_append) rope_append;
    decltype(&sqap_attention) attention;
    decltype(&sqap_decode_attention) decode_attention;
    decltype(&sqap_w4a4_linear) w4a4_linear;
    decltype(&sqap_group_run) group_run;
    decltype(&sqap_decoder_step) decoder_step;
    PyObject *failed;                     // called with a status that is not zero: raises
    PyObject *current_stream;             // asked for the stream of a call that names none ...
    char one_device;                      // ... unless it has found torch initialised with one device only: then torch's own table is
};

void *stream(const Calls *c, PyObject *o)
{
    if (o != Py_None) {
        const Ref v(PyNumber_Long(o));
        return reinterpret_cast<void *>(as_i64(v.p));
    }
    if (c->one_device) return c10::hip::getCurrentHIPStream(0).stream();
    const Ref v(PyObject_CallNoArgs(c->current_stream));
    return reinterpret_cast<void *>(as_i64(v.p));
}

// One call: `args` has to have as many elements as the method names; the library is called without the interpreter's lock, as ctypes does.
template <class Body>
PyObject *call(const Calls *c, Py_ssize_t n, Py_ssize_t want, Body body)
{
    if (n != want) {
        PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
        return nullptr;
    }
    try {
        const long status = body();
        if (status != 0) Ref(PyObject_CallFunction(c->failed, "l", status));
        Py_RETURN_NONE;
    } catch (const PyFailed &) {
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

// (The arguments are evaluated before the lock is given up.  It is taken again outside of any destructor: where the interpreter has ended
// meanwhile, as for a daemon thread, that ends the thread by unwinding its stack, which a destructor would turn into an abort.)
template <class F, class... A>
long run(F f, A... a)
{
    PyThreadState *const state = PyEval_SaveThread();
    const long status = f(a...);
    PyEval_RestoreThread(state);
    return status;
}

#define SQAP_METHOD(NAME, N, BODY)                                                       \
    PyObject *m_##NAME(PyObject *self, PyObject *const *a, Py_ssize_t n)                 \
    {                                                                                    \
        const Calls *c = reinterpret_cast<const Calls *>(self);                          \
        return call(c, n, N, [&]() -> long { return BODY; });                               \
    }

SQAP_METHOD(attn_scores_batch, 7,
            run(c->attn_scores_batch, ptr<sqap_f16>(a[0]), ptr<sqap_f16>(a[1]), (int32_t)size_of(a[1], 4, 0), (int32_t)size_of(a[1], 4, 1),
                (int32_t)size_of(a[1], 4, 2), (int32_t)size_of(a[1], 4, 3), as_i32(a[2]), as_i32(a[3]), ptr<float>(a[4]), ptr(a[5]),
                bytes(a[5]), stream(c, a[6])))
SQAP_METHOD(prune_topk, 4,
            run(c->prune_topk, ptr<float>(a[0]), (int32_t)size_of(a[0], 2, 0), (int32_t)size_of(a[0], 2, 1), as_i32(a[1]), ptr<int32_t>(a[2]),
                stream(c, a[3])))
SQAP_METHOD(kept_rows, 6,
            run(c->kept_rows, ptr<int32_t>(a[0]), (int32_t)size_of(a[0], 2, 0), (int32_t)size_of(a[0], 2, 1), as_i32(a[1]), as_i32(a[2]),
                as_i32(a[3]), ptr<int32_t>(a[4]), stream(c, a[5])))
SQAP_METHOD(prune_rows, 7,
            run(c->prune_rows, ptr<float>(a[0]), (int32_t)size_of(a[0], 2, 0), (int32_t)size_of(a[0], 2, 1), as_i32(a[1]), as_i32(a[2]),
                as_i32(a[3]), ptr<int32_t>(a[4]), ptr<int32_t>(a[5]), stream(c, a[6])))
SQAP_METHOD(prune_select, 10,
            run(c->prune_select, ptr<float>(a[0]), (int32_t)size(a[0], 0), as_i32(a[1]), as_i32(a[2]), as_i32(a[3]), as_i32(a[4]),
                ptr<double>(a[5]), as_i32(a[6]), ptr<int32_t>(a[7]), (int32_t)size(a[7], 1), ptr<int32_t>(a[8]), stream(c, a[9])))
SQAP_METHOD(quantize_act, 6,
            run(c->quantize_act, ptr<sqap_f16>(a[0]), pitch(a[0]), ptr<int32_t>(a[1]), (int32_t)rows_of(a[0], a[1]), (int32_t)size(a[0], 1),
                (uint32_t)as_i64(a[4]), ptr<uint8_t>(a[2]), ptr<sqap_f16>(a[3]), stream(c, a[5])))
SQAP_METHOD(rmsnorm_quantize_act, 12,
            run(c->rmsnorm_quantize_act, ptr<sqap_f16>(a[0]), pitch(a[0]), ptr<int32_t>(a[1]), (int32_t)rows_of(a[0], a[1]),
                (int32_t)size(a[0], 1), ptr<sqap_f16>(a[6]), ptr<sqap_f16>(a[2]), (float)as_double(a[3]), (uint32_t)as_i64(a[7]),
                ptr<sqap_f16>(a[8]), ptr<sqap_f16>(a[9]), ptr<sqap_f16>(a[10]), ptr<uint8_t>(a[4]), ptr<sqap_f16>(a[5]), stream(c, a[11])))
SQAP_METHOD(swiglu_quantize_act, 7,
            run(c->swiglu_quantize_act, ptr<sqap_f16>(a[0]), pitch(a[0]), ptr<sqap_f16>(a[1]), pitch(a[1]), (int32_t)size_of(a[0], 2, 0),
                (int32_t)size_of(a[0], 2, 1), ptr<sqap_f16>(a[4]), ptr<sqap_f16>(a[5]), ptr<uint8_t>(a[2]), ptr<sqap_f16>(a[3]),
                stream(c, a[6])))
SQAP_METHOD(rope, 6,
            run(c->rope, ptr<sqap_f16>(a[0]), pitch(a[0]), ptr<int32_t>(a[1]), (int32_t)size(a[0], 0), as_i32(a[2]), as_i32(a[3]),
                as_double(a[4]), stream(c, a[5])))
SQAP_METHOD(rope_append, 7,
            run(c->rope_append, ptr<sqap_f16>(a[0]), pitch(a[0]), ptr<int32_t>(a[1]), (int32_t)size(a[0], 0), as_i32(a[2]), as_i32(a[3]),
                as_double(a[5]), ptr<sqap_f16>(a[4]), pitch(a[4]), stream(c, a[6])))
SQAP_METHOD(decode_attention, 12,
            run(c->decode_attention, ptr<sqap_f16>(a[0]), ptr<int32_t>(a[1]), as_i32(a[2]), as_i32(a[3]), as_double(a[10]),
                ptr<sqap_f16>(a[4]), pitch(a[4]), as_i32(a[5]), ptr<sqap_f16>(a[6]), ptr<uint8_t>(a[7]), ptr<sqap_f16>(a[8]),
                ptr<uint32_t>(a[9]), stream(c, a[11])))
SQAP_METHOD(w4a4_linear, 7,
            run(c->w4a4_linear, ptr<uint8_t>(a[0]), ptr<sqap_f16>(a[1]), (int32_t)size(a[0], 0), handle<sqap_weight>(a[2]), ptr<sqap_f16>(a[3]),
                pitch(a[3]), ptr<int32_t>(a[4]), ptr(a[5]), bytes(a[5]), stream(c, a[6])))
SQAP_METHOD(group_run, 2, run(c->group_run, handle<sqap_group>(a[0]), stream(c, a[1])))
SQAP_METHOD(decoder_step, 7,
            run(c->decoder_step, handle<sqap_decoder>(a[0]), ptr<sqap_f16>(a[1]), ptr<int32_t>(a[2]), as_i32(a[3]), ptr<sqap_f16>(a[4]),
                ptr<sqap_f16>(a[5]), stream(c, a[6])))

long attention_call(const Calls *c, PyObject *const *a)
{
    const int64_t batch = as_i64(a[6]);
    if (batch == 0) {
        PyErr_SetString(PyExc_ZeroDivisionError, "integer division or modulo by zero");
        throw PyFailed{};
    }
    auto per_sequence = [&](PyObject *o) {                     // rounded down, as Python divides
        const int64_t n = size(o, 0), q = n / batch;
        return (int32_t)(n % batch != 0 && (n < 0) != (batch < 0) ? q - 1 : q);
    };
    return run(c->attention, ptr<sqap_f16>(a[0]), pitch(a[0]), ptr<sqap_f16>(a[1]), pitch(a[1]), ptr<sqap_f16>(a[2]), pitch(a[2]),
               (int32_t)batch, per_sequence(a[0]), per_sequence(a[1]), as_i32(a[3]), as_i32(a[4]), ptr<sqap_f16>(a[5]), pitch(a[5]),
               stream(c, a[7]));
}
SQAP_METHOD(attention, 8, attention_call(c, a))
#undef SQAP_METHOD

#define SQAP_CALLS(X)                                                                                                                   \
    X(attn_scores_batch) X(prune_topk) X(kept_rows) X(prune_rows) X(prune_select) X(quantize_act) X(rmsnorm_quantize_act)              \
    X(swiglu_quantize_act) X(rope) X(rope_append) X(attention) X(decode_attention) X(w4a4_linear) X(group_run) X(decoder_step)

PyMethodDef methods[] = {
#define SQAP_ENTRY(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(m_##NAME)), METH_FASTCALL, nullptr},
    SQAP_CALLS(SQAP_ENTRY)
#undef SQAP_ENTRY
    {nullptr, nullptr, 0, nullptr}};

// Calls(address, current_stream, failed): address(name) -> int, the library's function of that name.  (All of it in the constructor: an
// object without addresses must not come into being.)
PyObject *calls_new(PyTypeObject *type, PyObject *args, PyObject *)
{
    PyObject *address, *current_stream, *failed;
    if (!PyArg_ParseTuple(args, "OOO", &address, &current_stream, &failed)) return nullptr;
    PyObject *self = type->tp_alloc(type, 0);
    if (!self) return nullptr;
    Calls *c = reinterpret_cast<Calls *>(self);
    auto find = [&](const char *name, auto &slot) {
        const Ref v(PyObject_CallFunction(address, "s", name));
        slot = reinterpret_cast<std::decay_t<decltype(slot)>>(as_i64(v.p));
    };
    try {
#define SQAP_FIND(NAME) find("sqap_" #NAME, c->NAME);
        SQAP_CALLS(SQAP_FIND)
#undef SQAP_FIND
    } catch (const PyFailed &) {
        Py_DECREF(self);
        return nullptr;
    }
    Py_INCREF(current_stream);
    c->current_stream = current_stream;
    Py_INCREF(failed);
    c->failed = failed;
    return self;
}

void calls_dealloc(PyObject *self)
{
    Py_XDECREF(reinterpret_cast<Calls *>(self)->current_stream);
    Py_XDECREF(reinterpret_cast<Calls *>(self)->failed);
    Py_TYPE(self)->tp_free(self);
}

PyObject *get_one_device(PyObject *self, void *) { return PyBool_FromLong(reinterpret_cast<Calls *>(self)->one_device); }
int set_one_device(PyObject *self, PyObject *v, void *)
{
    const int truth = v ? PyObject_IsTrue(v) : 0;
    if (truth < 0) return -1;
    reinterpret_cast<Calls *>(self)->one_device = (char)truth;
    return 0;
}
PyGetSetDef getset[] = {{"one_device", get_one_device, set_one_device, nullptr, nullptr}, {nullptr, nullptr, nullptr, nullptr, nullptr}};

PyTypeObject calls_type = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls()
{
    static const char *const volatile mark = SQAP_TORCH_MARK;       // (which torch's headers these were: build.py looks for it)
    (void)mark;
    calls_type.tp_name = "_calls.Calls";
    calls_type.tp_basicsize = sizeof(Calls);
    calls_type.tp_flags = Py_TPFLAGS_DEFAULT;
    calls_type.tp_new = calls_new;
    calls_type.tp_dealloc = calls_dealloc;
    calls_type.tp_methods = methods;
    calls_type.tp_getset = getset;
    if (PyType_Ready(&calls_type) < 0) return nullptr;
    PyObject *m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&calls_type);
    if (PyModule_AddObject(m, "Calls", reinterpret_cast<PyObject *>(&calls_type)) < 0) return nullptr;
    return m;
}
