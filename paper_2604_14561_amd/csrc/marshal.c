/* Marshalling of the binding's calls in native code: tensors, shapes and numbers to the C ABI's arguments.
 *
 * A Calls object holds the addresses of one loaded libcocodiff.so.  calls(which, *arguments) converts the arguments and makes the call
 * with the interpreter's lock released; it returns the call's code, or None if an argument is not of the kinds handled here -- raw
 * pointers, streams given by the caller, subclasses, tensors that are refused: the binding then takes its general way, which also words
 * the errors.  Handled are contiguous GPU tensors (torch.Tensor and torch.nn.Parameter themselves), None, Shape and Rope, plain int and
 * float, and the current stream.
 *
 * What this is for: a call of one launch took the host 5 to 6 us, two thirds of it in Python and ctypes; calls on a few MB take
 * the GPU 3. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "../../include/cocodiff.h"

/* which, the function, its arguments as the binding passes them: S shape, r rope, R rope or None, t tensor or None, w tensor passed with its size in
 * bytes, i int32, f float; the stream follows the last one.  The binding holds NAMES, KINDS and SIZES (of the structures) against its own
 * when it loads. */
#define FUNCTIONS(F)                                                                                                         \
    F(qkv_proj, "Sttttttt") F(qk_norm_rope, "Sttttfr") F(qkv_proj_pack, "Sttttttti") F(qkv_proj_hs, "Sttttttt")           \
    F(qk_norm_rope_pack, "Sttttfrtti") F(a2a_unpack_norm_rope, "Sttttttfri") F(a2a_unpack_select, "Stittifttttiw")           \
    F(a2a_pack, "Stti") F(a2a_unpack, "Stti") F(vmajor_select, "iiiittfttttiw") F(vmajor_gather, "iiiitttti")                \
    F(vmajor_scatter, "iiiitttti") F(vmajor_token_metric, "iiittt") F(vmajor_topk, "iitiitt") F(a2a_pack_hs, "Stti")         \
    F(a2a_unpack_seq, "Stti") F(qkv_proj_fused, "SttttttfRtttittt") F(qkv_proj_fused_select, "SttttttfRtttittttiftttt" "iw")

enum {
#define F(name, kinds) CALL_##name,
    FUNCTIONS(F)
#undef F
    N_CALLS
};
static const char* const kKinds[N_CALLS] = {
#define F(name, kinds) kinds,
    FUNCTIONS(F)
#undef F
};
static const char* const kNames[N_CALLS] = {
#define F(name, kinds) #name,
    FUNCTIONS(F)
#undef F
};

typedef struct {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    void* address[N_CALLS];
    PyObject *tensor, *parameter, *shape, *rope; /* types */
    PyObject *device, *stream;                   /* () -> index of the current device; (index) -> its current stream */
} Calls;

static PyObject *s_is_cuda, *s_is_contiguous, *s_data_ptr, *s_numel, *s_element_size;

typedef union {
    void* p;
    int32_t i;
    float f;
} Argument;

static int as_number(PyObject* from, unsigned long long* to) {
    if (!from) return 0;
    *to = PyLong_AsUnsignedLongLong(from);
    Py_DECREF(from);
    return !(*to == (unsigned long long)-1 && PyErr_Occurred());
}

static int as_tensor(const Calls* c, PyObject* t, void** to) {
    unsigned long long at;
    PyObject* yes;
    int ok;
    if ((PyObject*)Py_TYPE(t) != c->tensor && (PyObject*)Py_TYPE(t) != c->parameter) return 0;
    yes = PyObject_GetAttr(t, s_is_cuda);
    ok = yes == Py_True;
    Py_XDECREF(yes);
    if (!ok) return 0;
    yes = PyObject_CallMethodNoArgs(t, s_is_contiguous);
    ok = yes == Py_True;
    Py_XDECREF(yes);
    if (!ok || !as_number(PyObject_CallMethodNoArgs(t, s_data_ptr), &at)) return 0;
    *to = (void*)(uintptr_t)at;
    return 1;
}

/* The structure's own memory: the argument keeps it alive through the call. */
static int as_structure(PyObject* from, PyObject* type, size_t bytes, void** to) {
    Py_buffer view;
    if ((PyObject*)Py_TYPE(from) != type || PyObject_GetBuffer(from, &view, PyBUF_SIMPLE) != 0) return 0;
    *to = view.buf;
    const int ok = (size_t)view.len == bytes;
    PyBuffer_Release(&view);
    return ok;
}

static int as_int32(PyObject* from, int32_t* to) {
    int overflow = 0;
    if (!PyLong_CheckExact(from)) return 0;
    const long x = PyLong_AsLongAndOverflow(from, &overflow);
    *to = (int32_t)x;
    return !overflow && x >= INT32_MIN && x <= INT32_MAX;
}

static PyObject* calls_call(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* keywords) {
    const Calls* c = (const Calls*)self;
    const Py_ssize_t n = PyVectorcall_NARGS(nargsf);
    Argument a[32];
    int32_t which = -1, tensors = 0, rc = 0;
    size_t bytes = 0;
    unsigned long long raw = 0;
    void* stream;
    if (keywords || n < 1 || !as_int32(args[0], &which) || which < 0 || which >= N_CALLS || (size_t)(n - 1) != strlen(kKinds[which])) {
        PyErr_SetString(PyExc_TypeError, "calls(which, arguments): no such call, or another number of arguments");
        return NULL;
    }
    for (Py_ssize_t k = 0; k + 1 < n; ++k) {
        PyObject* x = args[k + 1];
        int ok = 1;
        switch (kKinds[which][k]) {
            case 'S': ok = as_structure(x, c->shape, sizeof(cocodiff_shape), &a[k].p); break;
            case 'r':
            case 'R':
                a[k].p = NULL;
                if (x != Py_None || kKinds[which][k] == 'r') ok = as_structure(x, c->rope, sizeof(cocodiff_rope), &a[k].p);
                break;
            case 't':
                a[k].p = NULL;
                if (x != Py_None) ok = as_tensor(c, x, &a[k].p), tensors += ok;
                break;
            case 'w': {
                unsigned long long count = 0, size = 0;
                ok = as_tensor(c, x, &a[k].p) && as_number(PyObject_CallMethodNoArgs(x, s_numel), &count) &&
                     as_number(PyObject_CallMethodNoArgs(x, s_element_size), &size);
                bytes = (size_t)count * (size_t)size;
                break;
            }
            case 'i': ok = as_int32(x, &a[k].i); break;
            default:
                if (PyFloat_CheckExact(x)) a[k].f = (float)PyFloat_AS_DOUBLE(x);
                else if ((ok = PyLong_CheckExact(x))) {
                    const double d = PyLong_AsDouble(x);
                    ok = !(d == -1.0 && PyErr_Occurred());
                    a[k].f = (float)d;
                }
        }
        if (!ok) {
            PyErr_Clear();
            Py_RETURN_NONE;
        }
    }
    if (tensors == 0) Py_RETURN_NONE; /* (a GPU tensor: the device is initialised) */
    {
        PyObject* device = PyObject_CallNoArgs(c->device);
        const int ok = device && as_number(PyObject_CallOneArg(c->stream, device), &raw);
        Py_XDECREF(device);
        if (!ok) {
            PyErr_Clear();
            Py_RETURN_NONE;
        }
    }
    stream = (void*)(uintptr_t)raw;

#define FN(name) ((__typeof__(&cocodiff_##name))c->address[CALL_##name])
#define P(k) a[k].p
#define I(k) a[k].i
#define X(k) a[k].f
    Py_BEGIN_ALLOW_THREADS
    switch (which) {
        case CALL_qkv_proj: rc = FN(qkv_proj)(P(0), P(1), P(2), P(3), P(4), P(5), P(6), P(7), stream); break;
        case CALL_qk_norm_rope: rc = FN(qk_norm_rope)(P(0), P(1), P(2), P(3), P(4), X(5), P(6), stream); break;
        case CALL_qkv_proj_pack: rc = FN(qkv_proj_pack)(P(0), P(1), P(2), P(3), P(4), P(5), P(6), P(7), I(8), stream); break;
        case CALL_qkv_proj_hs: rc = FN(qkv_proj_hs)(P(0), P(1), P(2), P(3), P(4), P(5), P(6), P(7), stream); break;
        case CALL_qk_norm_rope_pack:
            rc = FN(qk_norm_rope_pack)(P(0), P(1), P(2), P(3), P(4), X(5), P(6), P(7), P(8), I(9), stream);
            break;
        case CALL_a2a_unpack_norm_rope:
            rc = FN(a2a_unpack_norm_rope)(P(0), P(1), P(2), P(3), P(4), P(5), P(6), X(7), P(8), I(9), stream);
            break;
        case CALL_a2a_unpack_select:
            rc = FN(a2a_unpack_select)(P(0), P(1), I(2), P(3), P(4), I(5), X(6), P(7), P(8), P(9), P(10), I(11), P(12), bytes, stream);
            break;
        case CALL_a2a_pack: rc = FN(a2a_pack)(P(0), P(1), P(2), I(3), stream); break;
        case CALL_a2a_unpack: rc = FN(a2a_unpack)(P(0), P(1), P(2), I(3), stream); break;
        case CALL_vmajor_select:
            rc = FN(vmajor_select)(I(0), I(1), I(2), I(3), P(4), P(5), X(6), P(7), P(8), P(9), P(10), I(11), P(12), bytes, stream);
            break;
        case CALL_vmajor_gather: rc = FN(vmajor_gather)(I(0), I(1), I(2), I(3), P(4), P(5), P(6), P(7), I(8), stream); break;
        case CALL_vmajor_scatter: rc = FN(vmajor_scatter)(I(0), I(1), I(2), I(3), P(4), P(5), P(6), P(7), I(8), stream); break;
        case CALL_vmajor_token_metric: rc = FN(vmajor_token_metric)(I(0), I(1), I(2), P(3), P(4), P(5), stream); break;
        case CALL_vmajor_topk: rc = FN(vmajor_topk)(I(0), I(1), P(2), I(3), I(4), P(5), P(6), stream); break;
        case CALL_a2a_pack_hs: rc = FN(a2a_pack_hs)(P(0), P(1), P(2), I(3), stream); break;
        case CALL_a2a_unpack_seq: rc = FN(a2a_unpack_seq)(P(0), P(1), P(2), I(3), stream); break;
        case CALL_qkv_proj_fused:
            rc = FN(qkv_proj_fused)(P(0), P(1), P(2), P(3), P(4), P(5), P(6), X(7), P(8), P(9), P(10), P(11), I(12), P(13), P(14), P(15), stream);
            break;
        case CALL_qkv_proj_fused_select:
            rc = FN(qkv_proj_fused_select)(P(0), P(1), P(2), P(3), P(4), P(5), P(6), X(7), P(8), P(9), P(10), P(11), I(12), P(13), P(14), P(15),
                                           P(16), I(17), X(18), P(19), P(20), P(21), P(22), I(23), P(24), bytes, stream);
            break;
    }
    Py_END_ALLOW_THREADS
#undef X
#undef I
#undef P
#undef FN
    return PyLong_FromLong(rc);
}

/* Calls(addresses in the order of NAMES, torch.Tensor, torch.nn.Parameter, Shape, Rope, device, stream) */
static PyObject* calls_new(PyTypeObject* type, PyObject* args, PyObject* keywords) {
    PyObject *addresses, *object[6];
    if (keywords && PyDict_GET_SIZE(keywords)) return PyErr_Format(PyExc_TypeError, "Calls takes no keywords");
    if (!PyArg_ParseTuple(args, "O!OOOOOO", &PyTuple_Type, &addresses, &object[0], &object[1], &object[2], &object[3], &object[4], &object[5])) return NULL;
    if (PyTuple_GET_SIZE(addresses) != N_CALLS) return PyErr_Format(PyExc_ValueError, "Calls takes %d addresses", (int)N_CALLS);
    Calls* c = (Calls*)type->tp_alloc(type, 0);
    if (!c) return NULL;
    PyObject** to[6] = {&c->tensor, &c->parameter, &c->shape, &c->rope, &c->device, &c->stream};
    for (int k = 0; k < 6; ++k) {
        Py_INCREF(object[k]);
        *to[k] = object[k];
    }
    c->vectorcall = calls_call;
    for (int k = 0; k < N_CALLS; ++k) {
        c->address[k] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, k));
        if (!c->address[k]) {
            if (!PyErr_Occurred()) PyErr_Format(PyExc_ValueError, "Calls: no address of %s", kNames[k]);
            Py_DECREF(c);
            return NULL;
        }
    }
    return (PyObject*)c;
}

static void calls_dealloc(PyObject* self) {
    Calls* c = (Calls*)self;
    Py_XDECREF(c->tensor);
    Py_XDECREF(c->parameter);
    Py_XDECREF(c->shape);
    Py_XDECREF(c->rope);
    Py_XDECREF(c->device);
    Py_XDECREF(c->stream);
    Py_TYPE(self)->tp_free(self);
}

static PyTypeObject CallsType = {
    PyVarObject_HEAD_INIT(NULL, 0).tp_name = "_marshal.Calls",
    .tp_basicsize = sizeof(Calls),
    .tp_dealloc = calls_dealloc,
    .tp_vectorcall_offset = offsetof(Calls, vectorcall),
    .tp_call = PyVectorcall_Call,
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_new = calls_new,
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", NULL, -1, NULL, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__marshal(void) {
    PyObject *m, *names, *kinds, *sizes;
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_numel = PyUnicode_InternFromString("numel");
    s_element_size = PyUnicode_InternFromString("element_size");
    if (PyType_Ready(&CallsType) < 0 || !(m = PyModule_Create(&module)) || !(names = PyTuple_New(N_CALLS)) || !(kinds = PyTuple_New(N_CALLS)) ||
        !(sizes = Py_BuildValue("(nn)", (Py_ssize_t)sizeof(cocodiff_shape), (Py_ssize_t)sizeof(cocodiff_rope))))
        return NULL;
    for (int k = 0; k < N_CALLS; ++k) {
        PyTuple_SET_ITEM(names, k, PyUnicode_FromFormat("cocodiff_%s", kNames[k]));
        PyTuple_SET_ITEM(kinds, k, PyUnicode_FromString(kKinds[k]));
    }
    Py_INCREF(&CallsType);
    if (PyModule_AddObject(m, "NAMES", names) < 0 || PyModule_AddObject(m, "KINDS", kinds) < 0 || PyModule_AddObject(m, "SIZES", sizes) < 0 ||
        PyModule_AddObject(m, "Calls", (PyObject*)&CallsType) < 0)
        return NULL;
    return m;
}
