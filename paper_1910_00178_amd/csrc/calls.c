/* The binding's calls that a program makes per product, without ctypes on the way: the arguments of a call are converted here and
 * the C function is called through its address.  Through ctypes a call of the smallest product spends 2.1 of its 5.2 us on that, here
 * 1.0 of 4.2 (1 x 4096 x 1024, pass after pass).
 *
 * A Call wraps one Python function of the binding (its `slow` one) and takes over only where every argument has the type that programs
 * pass: exact ints in range, None, floats, objects with data_ptr(), c_void_p handles, streams.  Whatever else it meets, keywords among
 * it, it hands the call on to the Python function before anything is launched, which converts or refuses it as ever.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>
#include <structmember.h>

enum { KIND_RUN, KIND_STATIC, KIND_REQUANT, KIND_CHANNEL, KIND_UNPACKED, KIND_BATCHED, KIND_PACK, KIND_FREE, KIND_COUNT };

/* One letter per Python argument: h handle, l int64, i int32, z size_t, f float, b truth, d device pointer, s stream, p problems.
 * `need` of them have to be there; the rest are pointers, sizes and streams that default to nothing. */
static const struct { const char *name, *spec; int need; } kinds[KIND_COUNT] = {
    {"run", "hldlihidldzs", 9},           {"static", "hldlihidls", 9},
    {"requant", "hldlihifidldzs", 11},    {"channel", "hldlihidddbidldzs", 14},
    {"unpacked", "hllldlidlidldzs", 14},  {"batched", "hpdzs", 2},
    {"pack", "hlldldzs", 7},              {"free", "h", 1},
};
#define MAX_ARGS 17

typedef union { int64_t l; int32_t i; size_t z; float f; void *p; } Value;

typedef struct {
    PyObject_HEAD
    PyObject *dict, *slow, *name;
    void *fn;
    int kind, nargs;
    vectorcallfunc vectorcall;
} Call;

/* set once by the binding: ctypes.c_void_p, the problem structure, the function that raises for a status */
static PyObject *handle_type, *problem_type, *check;
static Py_ssize_t problem_bytes;
/* torch's: the raw handle of a device's current stream, the current device, whether the runtime is up (and not a forked child's) */
static PyObject *raw_stream, *current_device, *ready;
static PyObject *s_data_ptr, *s_cuda_stream, *s_type;

/* a failed attempt: the Python function will meet (and raise) the same, but an interrupt goes through */
static int give_up(void)
{
    if (PyErr_Occurred() && PyErr_ExceptionMatches(PyExc_Exception)) PyErr_Clear();
    return 0;
}

static int int_of(PyObject *o, int64_t *v)
{
    int over;
    if (!PyLong_CheckExact(o)) return 0;
    *v = PyLong_AsLongLongAndOverflow(o, &over);
    return over == 0;
}

/* an address: of an exact int, 0 for None (a NULL pointer either way) */
static int address_of(PyObject *o, void **p)
{
    int64_t v;
    if (o == Py_None) {
        *p = NULL;
        return 1;
    }
    if (!int_of(o, &v) || v < 0) return 0;
    *p = (void *)(uintptr_t)v;
    return 1;
}

/* the address that o.<method>() or o.<attribute> gives; consumes `got` */
static int address_in(PyObject *got, void **p)
{
    if (!got) return give_up();
    const int ok = got != Py_None && address_of(got, p);
    Py_DECREF(got);
    return ok;
}

static int handle_of(PyObject *o, void **p)
{
    if (Py_TYPE(o) != (PyTypeObject *)handle_type) return address_of(o, p);
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return give_up();
    const int ok = b.len == sizeof(void *);
    if (ok) *p = *(void **)b.buf;
    PyBuffer_Release(&b);
    return ok;
}

/* a ctypes array of problems: its address; the caller's reference to it keeps it alive over the call */
static int problems_of(PyObject *o, void **p, int64_t *count)
{
    PyObject *element = PyObject_GetAttr((PyObject *)Py_TYPE(o), s_type);
    const int same = element == problem_type;
    Py_XDECREF(element);
    const Py_ssize_t n = same ? PyObject_Length(o) : -1;         /* (a pointer to problems has none) */
    Py_buffer b;
    if (n < 0 || n > INT32_MAX || PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return give_up();
    const int ok = b.len == n * problem_bytes;
    *p = b.buf;
    *count = n;
    PyBuffer_Release(&b);
    return ok;
}

static int stream_of(PyObject *o, void **p)
{
    if (o && o != Py_None) return PyLong_CheckExact(o) ? address_of(o, p) : address_in(PyObject_GetAttr(o, s_cuda_stream), p);
    if (!raw_stream) return 0;                                   /* (the first call finds them) */
    PyObject *up = PyObject_CallNoArgs(ready);
    const int is_up = up == Py_True;
    Py_XDECREF(up);
    PyObject *device = is_up ? PyObject_CallNoArgs(current_device) : NULL;
    if (!device) return give_up();
    PyObject *handle = PyObject_CallOneArg(raw_stream, device);
    Py_DECREF(device);
    return address_in(handle, p);
}

static int convert(char what, PyObject *o, Value *v, int64_t *count)
{
    int64_t n;
    switch (what) {
    case 'h': return handle_of(o, &v->p);
    case 'l': return int_of(o, &v->l);
    case 'i':
        if (!int_of(o, &n) || n < INT32_MIN || n > INT32_MAX) return 0;
        v->i = (int32_t)n;
        return 1;
    case 'z':
        if (!o) {
            v->z = 0;
            return 1;
        }
        if (!int_of(o, &n) || n < 0) return 0;
        v->z = (size_t)n;
        return 1;
    case 'f':
        if (!PyFloat_CheckExact(o)) return 0;
        v->f = (float)PyFloat_AS_DOUBLE(o);
        return 1;
    case 'b':
        if (!PyBool_Check(o) && !PyLong_CheckExact(o)) return 0;
        v->i = PyObject_IsTrue(o);
        return 1;
    case 'd':
        if (!o) {
            v->p = NULL;
            return 1;
        }
        if (o == Py_None || PyLong_CheckExact(o)) return address_of(o, &v->p);
        return address_in(PyObject_CallMethodNoArgs(o, s_data_ptr), &v->p);
    case 'p': return problems_of(o, &v->p, count);
    default: return stream_of(o, &v->p);
    }
}

typedef void *P;
typedef int64_t L;
typedef int32_t I;

static PyObject *call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames)
{
    Call *c = (Call *)self;
    const Py_ssize_t n = PyVectorcall_NARGS(nargsf);
    const char *spec = kinds[c->kind].spec;
    Value v[MAX_ARGS];
    int64_t count = 0;
    if ((kwnames && PyTuple_GET_SIZE(kwnames) != 0) || n < kinds[c->kind].need || n > c->nargs) goto slow;
    for (int k = 0; k < c->nargs; ++k)
        if (!convert(spec[k], k < n ? args[k] : NULL, &v[k], &count)) goto slow;
    {
        int status = 0;
        P handle = NULL;
        Py_BEGIN_ALLOW_THREADS
        switch (c->kind) {
        case KIND_RUN:
            status = ((int (*)(P, L, P, L, I, P, I, P, L, P, size_t, P))c->fn)(v[0].p, v[1].l, v[2].p, v[3].l, v[4].i, v[5].p, v[6].i, v[7].p, v[8].l,
                                                                              v[9].p, v[10].z, v[11].p);
            break;
        case KIND_STATIC:
            status = ((int (*)(P, L, P, L, I, P, I, P, L, P))c->fn)(v[0].p, v[1].l, v[2].p, v[3].l, v[4].i, v[5].p, v[6].i, v[7].p, v[8].l, v[9].p);
            break;
        case KIND_REQUANT:
            status = ((int (*)(P, L, P, L, I, P, I, float, I, P, L, P, size_t, P))c->fn)(v[0].p, v[1].l, v[2].p, v[3].l, v[4].i, v[5].p, v[6].i, v[7].f,
                                                                                        v[8].i, v[9].p, v[10].l, v[11].p, v[12].z, v[13].p);
            break;
        case KIND_CHANNEL:
            status = ((int (*)(P, L, P, L, I, P, I, P, P, P, I, I, P, L, P, size_t, P))c->fn)(v[0].p, v[1].l, v[2].p, v[3].l, v[4].i, v[5].p, v[6].i,
                                                                                             v[7].p, v[8].p, v[9].p, v[10].i, v[11].i, v[12].p, v[13].l,
                                                                                             v[14].p, v[15].z, v[16].p);
            break;
        case KIND_UNPACKED:
            status = ((int (*)(P, L, L, L, P, L, I, P, L, I, P, L, P, size_t, P))c->fn)(v[0].p, v[1].l, v[2].l, v[3].l, v[4].p, v[5].l, v[6].i, v[7].p,
                                                                                       v[8].l, v[9].i, v[10].p, v[11].l, v[12].p, v[13].z, v[14].p);
            break;
        case KIND_BATCHED:
            status = ((int (*)(P, int, P, P, size_t, P))c->fn)(v[0].p, (int)count, v[1].p, v[2].p, v[3].z, v[4].p);
            break;
        case KIND_PACK:
            status = ((int (*)(P, L, L, P, L, P, size_t, P, P *))c->fn)(v[0].p, v[1].l, v[2].l, v[3].p, v[4].l, v[5].p, v[6].z, v[7].p, &handle);
            break;
        default:
            status = ((int (*)(P))c->fn)(v[0].p);
            break;
        }
        Py_END_ALLOW_THREADS
        if (status != 0) return PyObject_CallFunction(check, "iO", status, c->name);
        if (c->kind == KIND_PACK) return PyObject_CallFunction(handle_type, "N", PyLong_FromVoidPtr(handle));
        Py_RETURN_NONE;
    }
slow:
    if (PyErr_Occurred()) return NULL;
    return PyObject_Vectorcall(c->slow, args, nargsf, kwnames);
}

static PyObject *new_call(PyTypeObject *type, PyObject *args, PyObject *kw)
{
    PyObject *slow;
    const char *kind;
    unsigned long long fn;
    if (kw && PyDict_GET_SIZE(kw) != 0) return PyErr_Format(PyExc_TypeError, "Call takes no keywords");
    if (!PyArg_ParseTuple(args, "OsK", &slow, &kind, &fn)) return NULL;
    int k = 0;
    while (k < KIND_COUNT && strcmp(kinds[k].name, kind) != 0) ++k;
    if (k == KIND_COUNT || fn == 0 || !handle_type) return PyErr_Format(PyExc_ValueError, "Call: kind '%s'", kind);
    Call *c = (Call *)type->tp_alloc(type, 0);
    if (!c) return NULL;
    c->name = PyObject_GetAttrString(slow, "__name__");
    if (!c->name) {
        Py_DECREF(c);
        return NULL;
    }
    Py_INCREF(slow);
    c->slow = slow;
    c->fn = (void *)(uintptr_t)fn;
    c->kind = k;
    c->nargs = (int)strlen(kinds[k].spec);
    c->vectorcall = call;
    return (PyObject *)c;
}

static int traverse(PyObject *self, visitproc visit, void *arg)
{
    Call *c = (Call *)self;
    Py_VISIT(c->dict);
    Py_VISIT(c->slow);
    Py_VISIT(c->name);
    return 0;
}

static int clear(PyObject *self)
{
    Call *c = (Call *)self;
    Py_CLEAR(c->dict);
    return 0;                                                    /* (the rest stays: a call may still come) */
}

static void dealloc(PyObject *self)
{
    PyObject_GC_UnTrack(self);
    clear(self);
    Py_CLEAR(((Call *)self)->slow);
    Py_CLEAR(((Call *)self)->name);
    Py_TYPE(self)->tp_free(self);
}

static PyObject *reduce(PyObject *self, PyObject *unused)       /* pickled by name, as the function is */
{
    (void)unused;
    Py_INCREF(((Call *)self)->name);
    return ((Call *)self)->name;
}

static PyMethodDef call_methods[] = {{"__reduce__", reduce, METH_NOARGS, NULL}, {NULL, NULL, 0, NULL}};

static PyMemberDef members[] = {
    {"__wrapped__", T_OBJECT, offsetof(Call, slow), READONLY, "the Python function that takes what this one hands on"},
    {"__name__", T_OBJECT, offsetof(Call, name), READONLY, NULL},
    {NULL, 0, 0, 0, NULL},
};

static PyGetSetDef getset[] = {
    {"__dict__", PyObject_GenericGetDict, PyObject_GenericSetDict, NULL, NULL},
    {NULL, NULL, NULL, NULL, NULL},
};

static PyTypeObject CallType = {
    PyVarObject_HEAD_INIT(NULL, 0)
    .tp_name = "paper_1910_00178_amd._calls.Call",
    .tp_basicsize = sizeof(Call),
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_vectorcall_offset = offsetof(Call, vectorcall),
    .tp_call = PyVectorcall_Call,
    .tp_new = new_call,
    .tp_dealloc = dealloc,
    .tp_traverse = traverse,
    .tp_clear = clear,
    .tp_dictoffset = offsetof(Call, dict),
    .tp_methods = call_methods,
    .tp_members = members,
    .tp_getset = getset,
};

static void keep(PyObject **where, PyObject *o)
{
    if (o == Py_None) o = NULL;
    Py_XINCREF(o);
    Py_XSETREF(*where, o);
}

static PyObject *setup(PyObject *m, PyObject *args)
{
    PyObject *h, *p, *c;
    (void)m;
    if (!PyArg_ParseTuple(args, "OOnO", &h, &p, &problem_bytes, &c)) return NULL;
    keep(&handle_type, h);
    keep(&problem_type, p);
    keep(&check, c);
    keep(&raw_stream, NULL);
    Py_RETURN_NONE;
}

static PyObject *streams(PyObject *m, PyObject *args)
{
    PyObject *r, *d, *u;
    (void)m;
    if (!PyArg_ParseTuple(args, "OOO", &r, &d, &u)) return NULL;
    keep(&current_device, d);
    keep(&ready, u);
    keep(&raw_stream, r);
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"setup", setup, METH_VARARGS, "setup(c_void_p, problem structure, its size, check(status, name))"},
    {"streams", streams, METH_VARARGS, "streams(raw handle of a device's stream, current device, runtime is up)"},
    {NULL, NULL, 0, NULL},
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__calls(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    s_type = PyUnicode_InternFromString("_type_");
    if (!s_data_ptr || !s_cuda_stream || !s_type || PyType_Ready(&CallType) < 0) return NULL;
    PyObject *m = PyModule_Create(&module);
    if (!m) return NULL;
    Py_INCREF(&CallType);
    if (PyModule_AddObject(m, "Call", (PyObject *)&CallType) < 0) {
        Py_DECREF(&CallType);
        Py_DECREF(m);
        return NULL;
    }
    return m;
}
