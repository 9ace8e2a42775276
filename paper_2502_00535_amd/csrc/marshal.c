/* Native marshalling of the whole-path calls: the checks of binding.py's _ptr on tensors that are in order, and
 * the call itself, without a ctypes conversion per argument.  A call on a small frame is as long as its
 * marshalling (5.7 us through ctypes at 360 boxes, of which the launch is 2.7).
 * Whatever is not in order is left to the Python path, which says what is wrong: the function returns None then. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include "../../include/nms.h"

typedef int (*run_batched_fn)(const float *, const float *, const int32_t *, int, int, float, uint8_t *, void *, size_t, void *);

static PyObject *tensor_type, *dtype_f32, *dtype_i32, *dtype_u8, *current_device, *raw_stream;
static PyObject *n_is_cuda, *n_is_contiguous, *n_numel, *n_dtype, *n_data_ptr, *n_nbytes, *n_cuda_stream;

static int as_i64(PyObject *o, long long *out)
{
    if (o == NULL) return 0;
    *out = PyLong_AsLongLong(o);
    Py_DECREF(o);
    return !(*out == -1 && PyErr_Occurred());
}

/* Address of a contiguous GPU tensor of the given dtype (NULL: any) with at least `need` elements; 0 when it is not that. */
static int address(PyObject *t, PyObject *dtype, long long need, void **out)
{
    long long v;
    PyObject *o;
    int is;
    if (!PyObject_TypeCheck(t, (PyTypeObject *)tensor_type)) return 0;
    o = PyObject_GetAttr(t, n_is_cuda);
    is = o == Py_True;
    Py_XDECREF(o);
    if (!is) return 0;
    if (dtype != NULL) {
        o = PyObject_GetAttr(t, n_dtype);
        is = o == dtype;
        Py_XDECREF(o);
        if (!is) return 0;
    }
    o = PyObject_CallMethodNoArgs(t, n_is_contiguous);
    is = o == Py_True;
    Py_XDECREF(o);
    if (!is) return 0;
    if (need > 0 && (!as_i64(PyObject_CallMethodNoArgs(t, n_numel), &v) || v < need)) return 0;
    o = PyObject_CallMethodNoArgs(t, n_data_ptr);
    if (o == NULL) return 0;
    *out = PyLong_AsVoidPtr(o);
    Py_DECREF(o);
    return !PyErr_Occurred();
}

/* Handle of a torch stream, of the current one for None. */
static int stream_handle(PyObject *stream, void **out)
{
    PyObject *h, *device;
    if (stream != Py_None) {
        h = PyObject_GetAttr(stream, n_cuda_stream);
    } else {
        device = PyObject_CallNoArgs(current_device);
        if (device == NULL) return 0;
        h = PyObject_CallOneArg(raw_stream, device);
        Py_DECREF(device);
    }
    if (h == NULL) return 0;
    *out = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    return !PyErr_Occurred();
}

/* run(fn, boxes, scores, counts or None, n_max, frames, threshold, keep_out, workspace, stream) -> status, or None */
static PyObject *run(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    void *fn, *boxes, *scores, *counts = NULL, *keep, *ws, *stream;
    long long n_max, frames, bytes;
    double threshold;
    int status;
    (void)self;
    if (n != 10) {
        PyErr_SetString(PyExc_TypeError, "run takes ten arguments");
        return NULL;
    }
    /* whole numbers and a float, as they are; sizes that the library would refuse are left to the other path, so that no product overflows */
    if (!PyLong_CheckExact(a[4]) || !PyLong_CheckExact(a[5]) || !PyFloat_CheckExact(a[6]) || raw_stream == NULL) Py_RETURN_NONE;
    n_max = PyLong_AsLongLong(a[4]);
    frames = PyLong_AsLongLong(a[5]);
    threshold = PyFloat_AS_DOUBLE(a[6]);
    if (PyErr_Occurred() || n_max < 0 || frames < 0 || n_max > NMS_MAX_N || frames > NMS_MAX_FRAMES) goto other;
    if (!address(a[1], dtype_f32, 4 * n_max * frames, &boxes) || !address(a[2], dtype_f32, n_max * frames, &scores) ||
        (a[3] != Py_None && !address(a[3], dtype_i32, frames, &counts)) || !address(a[7], dtype_u8, n_max * frames, &keep) ||
        !address(a[8], NULL, 0, &ws) || !as_i64(PyObject_GetAttr(a[8], n_nbytes), &bytes) || !stream_handle(a[9], &stream))
        goto other;
    fn = PyLong_AsVoidPtr(a[0]);
    if (PyErr_Occurred()) goto other;
    Py_BEGIN_ALLOW_THREADS
    status = ((run_batched_fn)fn)(boxes, scores, counts, (int)n_max, (int)frames, (float)threshold, keep, ws, (size_t)bytes, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
other:
    PyErr_Clear();
    Py_RETURN_NONE;
}

/* setup(Tensor, float32, int32, uint8, current device function, raw stream function or None) */
static PyObject *setup(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    (void)self;
    if (n != 6 || !PyType_Check(a[0])) {
        PyErr_SetString(PyExc_TypeError, "setup takes the tensor type, three dtypes and two functions");
        return NULL;
    }
    if (tensor_type != NULL) Py_RETURN_NONE;  /* once per process */
    for (n = 0; n < 6; ++n) Py_INCREF(a[n]);
    current_device = a[4], raw_stream = a[4] == Py_None || a[5] == Py_None ? NULL : a[5];
    tensor_type = a[0], dtype_f32 = a[1], dtype_i32 = a[2], dtype_u8 = a[3];
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"run", (PyCFunction)(void (*)(void))run, METH_FASTCALL, "A whole-path call; None when an argument is not in order."},
    {"setup", (PyCFunction)(void (*)(void))setup, METH_FASTCALL, "The types to compare with."},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__marshal(void)
{
    n_is_cuda = PyUnicode_InternFromString("is_cuda");
    n_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    n_numel = PyUnicode_InternFromString("numel");
    n_dtype = PyUnicode_InternFromString("dtype");
    n_data_ptr = PyUnicode_InternFromString("data_ptr");
    n_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    n_nbytes = PyUnicode_InternFromString("nbytes");
    return PyModule_Create(&module);
}
