// The calls of a serving loop (exe_encode, exe_decode_step, exe_seq_release) for Python, as the extension module _call.
//
// A decode iteration of a small model keeps the GPU for 40 us; marshalled by ctypes, of which every pointer into a numpy array is
// several objects, its call took 10 us on top, 6 of them between Model.decode_step and the library.  Here the arrays' addresses
// come through the buffer protocol: 17 calls of two float layers of 256, 4 rows 1037 -> 933 us, 97 of six bf16 layers of 1024, 48
// rows 36.2 -> 35.3 ms.
//
// Each function takes the address of the library's function and the model handle as integers, then that function's arguments in
// their order without the count, which is the length of the first array: int32 arrays as C-contiguous buffers, device pointers as
// integers, either of them None for a null pointer (the first array excepted: without it there is no count).  It returns the
// library's status.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

// the arguments' buffers and addresses; released together
#define MAX_ARGS 8
typedef struct { Py_buffer view[MAX_ARGS]; int n; } Held;

static void release(Held* h)
{
    while (h->n > 0) PyBuffer_Release(&h->view[--h->n]);
}

static int array(PyObject* o, int flags, Held* h, int32_t** p)
{
    *p = NULL;
    if (o == Py_None) return 1;
    if (PyObject_GetBuffer(o, &h->view[h->n], PyBUF_C_CONTIGUOUS | PyBUF_FORMAT | flags) < 0) return 0;
    Py_buffer* v = &h->view[h->n++];
    // "i" of 4 bytes in the machine's order, which may be said
    const char* f = v->format ? v->format : "B";
    if (*f == '@' || *f == '=' || *f == '<') ++f;
    if (v->itemsize != 4 || v->ndim < 1 || (*f != 'i' && *f != 'l') || f[1]) {
        PyErr_SetString(PyExc_TypeError, "expected an int32 array");
        return 0;
    }
    *p = (int32_t*)v->buf;
    return 1;
}

// the first array, whose length is the count
static int first(PyObject* o, Held* h, int32_t** p, int* count)
{
    if (o == Py_None) PyErr_SetString(PyExc_TypeError, "expected an int32 array of sequence ids, got None");
    if (o == Py_None || !array(o, PyBUF_ND, h, p)) return 0;
    *count = (int)h->view[h->n - 1].shape[0];
    return 1;
}

static int address(PyObject* o, void** p)
{
    *p = o == Py_None ? NULL : PyLong_AsVoidPtr(o);
    return !PyErr_Occurred();
}

static int function(PyObject* o, void** p)
{
    if (!address(o, p)) return 0;
    if (!*p) PyErr_SetString(PyExc_ValueError, "null function");
    return *p != NULL;
}

static int takes(Py_ssize_t got, Py_ssize_t want)
{
    if (got != want) PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, got);
    return got == want;
}

static PyObject* py_encode(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    typedef int (*Fn)(void*, int32_t, const int32_t*, const int32_t*, const int32_t*, const int32_t*, const void*, int32_t*, void*);
    void *fn, *model, *hidden, *out;
    int32_t *ids, *lens, *toks, *reserve, *next;
    int count;
    Held h = {.n = 0};
    PyObject* r = NULL;
    if (!takes(n, 9)) return NULL;
    if (function(a[0], &fn) && address(a[1], &model) && first(a[2], &h, &ids, &count) && array(a[3], PyBUF_ND, &h, &lens) &&
        array(a[4], PyBUF_ND, &h, &toks) && array(a[5], PyBUF_ND, &h, &reserve) && address(a[6], &hidden) &&
        array(a[7], PyBUF_ND | PyBUF_WRITABLE, &h, &next) && address(a[8], &out)) {
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = ((Fn)fn)(model, count, ids, lens, toks, reserve, hidden, next, out);
        Py_END_ALLOW_THREADS
        r = PyLong_FromLong(rc);
    }
    release(&h);
    return r;
}

static PyObject* py_decode_step(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    typedef int (*Fn)(void*, int32_t, const int32_t*, const int32_t*, const int32_t*, const void*, int32_t*, void*);
    void *fn, *model, *hidden, *out;
    int32_t *ids, *toks, *lens, *next;
    int count;
    Held h = {.n = 0};
    PyObject* r = NULL;
    if (!takes(n, 8)) return NULL;
    if (function(a[0], &fn) && address(a[1], &model) && first(a[2], &h, &ids, &count) && array(a[3], PyBUF_ND, &h, &toks) &&
        array(a[4], PyBUF_ND, &h, &lens) && address(a[5], &hidden) && array(a[6], PyBUF_ND | PyBUF_WRITABLE, &h, &next) &&
        address(a[7], &out)) {
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = ((Fn)fn)(model, count, ids, toks, lens, hidden, next, out);
        Py_END_ALLOW_THREADS
        r = PyLong_FromLong(rc);
    }
    release(&h);
    return r;
}

static PyObject* py_seq_release(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    typedef int (*Fn)(void*, int32_t, const int32_t*);
    void *fn, *model;
    int32_t* ids;
    int count;
    Held h = {.n = 0};
    PyObject* r = NULL;
    if (!takes(n, 3)) return NULL;
    if (function(a[0], &fn) && address(a[1], &model) && first(a[2], &h, &ids, &count)) {
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = ((Fn)fn)(model, count, ids);
        Py_END_ALLOW_THREADS
        r = PyLong_FromLong(rc);
    }
    release(&h);
    return r;
}

static PyMethodDef methods[] = {
    {"encode", (PyCFunction)(void (*)(void))py_encode, METH_FASTCALL, "exe_encode"},
    {"decode_step", (PyCFunction)(void (*)(void))py_decode_step, METH_FASTCALL, "exe_decode_step"},
    {"seq_release", (PyCFunction)(void (*)(void))py_seq_release, METH_FASTCALL, "exe_seq_release"},
    {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", NULL, -1, methods, NULL, NULL, NULL, NULL};
PyMODINIT_FUNC PyInit__call(void) { return PyModule_Create(&module); }
