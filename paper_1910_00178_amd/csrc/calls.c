/* The binding's calls that a program makes per product, without ctypes on the way: the arguments of a call are converted here and
 * the C function is called through its address.  The smallest product in a loop (1 x 4096 x 1024, arguments at hand) takes 4.2 us a call
 * through ctypes, 3.2 here.
 *
 * A Call is one Python function of the binding over again: a function object in all but its vectorcall, so that what programs do with
 * functions (weak references, binding in a class, inspection, mocks) stays.  The vectorcall takes over only where every argument has the
 * type that programs pass: exact ints in range, None, floats, objects with data_ptr(), c_void_p handles, streams.  Whatever else it meets,
 * keywords among it, it runs the function's own code before anything is launched, which converts or refuses it as ever; so it
 * does under a tracer or profiler and while any name that this code looks up, or the code itself, is not the binding's own.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>

#if PY_VERSION_HEX >= 0x030A0000 && PY_VERSION_HEX < 0x030B0000      /* (other versions' functions are laid out otherwise: all calls by ctypes there) */

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
    PyFunctionObject f;
    PyObject *code, *defaults;                                   /* as they were */
    void *fn;
    int kind, nargs;
} Call;

/* set once by the binding: ctypes.c_void_p, the problem structure, the function that raises for a status */
static PyObject *handle_type, *problem_type, *check;
static Py_ssize_t problem_bytes;
/* torch's: the raw handle of a device's current stream, the current device, whether the runtime is up (and not a forked child's) */
static PyObject *raw_stream, *current_device, *ready;
static PyObject *s_data_ptr, *s_cuda_stream, *s_type, *s_current_stream;
/* What the Python functions look up: (dict, names, values) for the binding's names and for the library's.  A dict's version tells whether it was
 * written to since `intact` was found, so that a call costs two comparisons.  bound_stream: the binding's _current_stream that calls
 * raw_stream; another one is asked itself. */
enum { WATCHED = 2 };
static PyObject *watched[WATCHED][3], *bound_stream;
static uint64_t version[WATCHED];
static int intact, stream_intact;

static int look_again(void)
{
    intact = stream_intact = 1;
    for (int w = 0; w < WATCHED; ++w) {
        PyObject *dict = watched[w][0];
        if (!dict) return intact = 0;
        version[w] = ((PyDictObject *)dict)->ma_version_tag;
        for (Py_ssize_t k = 0; k < PyTuple_GET_SIZE(watched[w][1]); ++k)
            if (PyDict_GetItem(dict, PyTuple_GET_ITEM(watched[w][1], k)) != PyTuple_GET_ITEM(watched[w][2], k)) intact = 0;
    }
    if (bound_stream && PyDict_GetItem(watched[0][0], s_current_stream) != bound_stream) stream_intact = 0;
    return intact;
}

static int as_it_was(const Call *c)
{
    if (c->f.func_code != c->code || c->f.func_defaults != c->defaults || PyThreadState_Get()->cframe->use_tracing) return 0;
    for (int w = 0; w < WATCHED; ++w)
        if (!watched[w][0] || ((PyDictObject *)watched[w][0])->ma_version_tag != version[w]) return look_again();
    return intact;
}

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
    if (!raw_stream || !stream_intact) return 0;                 /* (the first call finds them) */
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
    if ((kwnames && PyTuple_GET_SIZE(kwnames) != 0) || n < kinds[c->kind].need || n > c->nargs || !as_it_was(c)) goto slow;
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
        if (status != 0) return PyObject_CallFunction(check, "iO", status, c->f.func_name);
        if (c->kind == KIND_PACK) return PyObject_CallFunction(handle_type, "N", PyLong_FromVoidPtr(handle));
        Py_RETURN_NONE;
    }
slow:
    if (PyErr_Occurred()) return NULL;
    return _PyFunction_Vectorcall(self, args, nargsf, kwnames);
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
    if (!PyFunction_Check(slow)) return PyErr_Format(PyExc_TypeError, "Call: a Python function");
    PyObject *dict = PyDict_New();
    if (!dict || PyDict_SetItemString(dict, "__wrapped__", slow) != 0) {
        Py_XDECREF(dict);
        return NULL;
    }
    Call *c = PyObject_GC_New(Call, type);
    if (!c) {
        Py_DECREF(dict);
        return NULL;
    }
    const PyFunctionObject *s = (PyFunctionObject *)slow;
    PyFunctionObject *f = &c->f;
    memcpy((char *)f + sizeof(PyObject), (const char *)s + sizeof(PyObject), sizeof(*f) - sizeof(PyObject));
    PyObject *shared[] = {f->func_globals, f->func_builtins, f->func_name, f->func_qualname, f->func_code, f->func_defaults, f->func_kwdefaults,
                          f->func_closure, f->func_doc, f->func_module, f->func_annotations, f->func_code, f->func_defaults};
    for (size_t k = 0; k < sizeof(shared) / sizeof(shared[0]); ++k) Py_XINCREF(shared[k]);
    f->func_dict = dict;
    f->func_weakreflist = NULL;
    f->vectorcall = call;
    c->code = f->func_code;
    c->defaults = f->func_defaults;
    c->fn = (void *)(uintptr_t)fn;
    c->kind = k;
    c->nargs = (int)strlen(kinds[k].spec);
    PyObject_GC_Track(c);
    return (PyObject *)c;
}

static void dealloc(PyObject *self)
{
    PyObject *code = ((Call *)self)->code, *defaults = ((Call *)self)->defaults;
    PyFunction_Type.tp_dealloc(self);
    Py_DECREF(code);
    Py_XDECREF(defaults);
}

static PyObject *reduce(PyObject *self, PyObject *unused)       /* pickled by name, as the function is */
{
    (void)unused;
    Py_INCREF(((Call *)self)->f.func_name);
    return ((Call *)self)->f.func_name;
}

static PyMethodDef call_methods[] = {{"__reduce__", reduce, METH_NOARGS, NULL}, {NULL, NULL, 0, NULL}};

static PyTypeObject CallType = {                                 /* (what is not here is the function type's, its collector's entries among it) */
    PyVarObject_HEAD_INIT(NULL, 0)
    .tp_name = "paper_1910_00178_amd._calls.Call",
    .tp_basicsize = sizeof(Call),
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_vectorcall_offset = offsetof(PyFunctionObject, vectorcall),
    .tp_call = PyVectorcall_Call,
    .tp_new = new_call,
    .tp_dealloc = dealloc,
    .tp_methods = call_methods,
};

static void keep(PyObject **where, PyObject *o)
{
    if (o == Py_None) o = NULL;
    Py_XINCREF(o);
    Py_XSETREF(*where, o);
}

static PyObject *setup(PyObject *m, PyObject *args)
{
    PyObject *h, *p, *c, *of[WATCHED], *names[WATCHED];
    (void)m;
    if (!PyArg_ParseTuple(args, "OOnOO!O!O!O!", &h, &p, &problem_bytes, &c, &PyDict_Type, &of[0], &PyTuple_Type, &names[0], &PyDict_Type, &of[1],
                          &PyTuple_Type, &names[1])) return NULL;
    for (int w = 0; w < WATCHED; ++w) {
        const Py_ssize_t n = PyTuple_GET_SIZE(names[w]);
        PyObject *values = PyTuple_New(n);
        if (!values) return NULL;
        for (Py_ssize_t k = 0; k < n; ++k) {
            PyObject *v = PyDict_GetItemWithError(of[w], PyTuple_GET_ITEM(names[w], k));
            if (!v) {
                Py_DECREF(values);
                return PyErr_Format(PyExc_KeyError, "setup: %R", PyTuple_GET_ITEM(names[w], k));
            }
            Py_INCREF(v);
            PyTuple_SET_ITEM(values, k, v);
        }
        keep(&watched[w][0], of[w]);
        keep(&watched[w][1], names[w]);
        keep(&watched[w][2], values);
        Py_DECREF(values);
        version[w] = 0;
    }
    keep(&handle_type, h);
    keep(&problem_type, p);
    keep(&check, c);
    keep(&raw_stream, NULL);
    keep(&bound_stream, NULL);
    Py_RETURN_NONE;
}

static PyObject *streams(PyObject *m, PyObject *args)
{
    PyObject *r, *d, *u, *b = NULL;
    (void)m;
    if (!PyArg_ParseTuple(args, "OOO|O", &r, &d, &u, &b)) return NULL;
    keep(&current_device, d);
    keep(&ready, u);
    keep(&raw_stream, r);
    keep(&bound_stream, b);
    version[0] = 0;                                              /* (no dict has it) */
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"setup", setup, METH_VARARGS, "setup(c_void_p, problem structure, its size, check(status, name), the binding's names, those to watch, the library's, those to watch)"},
    {"streams", streams, METH_VARARGS, "streams(raw handle of a device's stream, current device, runtime is up[, the binding's _current_stream that asks them])"},
    {NULL, NULL, 0, NULL},
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__calls(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    s_type = PyUnicode_InternFromString("_type_");
    s_current_stream = PyUnicode_InternFromString("_current_stream");
    CallType.tp_base = &PyFunction_Type;
    if (!s_data_ptr || !s_cuda_stream || !s_type || !s_current_stream || PyType_Ready(&CallType) < 0) return NULL;
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

#else

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, NULL, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__calls(void) { return PyModule_Create(&module); }

#endif
