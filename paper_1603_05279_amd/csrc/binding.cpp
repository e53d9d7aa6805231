// Argument marshalling of the enqueuing entry points (include/xnor.h) for Python: device tensors to addresses, one C call
// each.  A layer's launch takes the GPU 2 to 5 us at the smallest sizes, less than the same checks and conversions
// cost through ctypes (5.3 us of host time per call, HIP's launch of about 2 us included; 3.5 us here): one 64 x 14 x 14
// block, two calls, 11.6 -> 8.5 us; one row of a 9216 -> 4096 layer 11.2 -> 7.6 us.
//
// Checks of a tensor argument: NULL or a dense device tensor of the stated type, as the callers of xnor.py have always
// been told; sizes are the caller's, as in the C ABI.  The library's entry points are looked up in the file that xnor.py
// names (bind), so that another build of it can be called.
#include <torch/csrc/autograd/python_variable.h>

#include <dlfcn.h>

#include "xnor.h"

namespace {

// The Python error that is already set (thrown so that every exit path of a call is the same).
struct PythonError {};

PyObject *g_raise = nullptr;            // xnor.py's error for a non-zero status: raise(name, status)
PyObject *g_desc = nullptr;             // xnor.py's descriptor class
PyObject *g_current_device = nullptr, *g_raw_stream = nullptr;      // torch's, for calls without a stream

[[noreturn]] void fail(PyObject *type, const char *message)
{
    PyErr_SetString(type, message);
    throw PythonError{};
}

void *tensor(PyObject *o, c10::ScalarType type)
{
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a tensor or None");
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda()) fail(PyExc_ValueError, "libxnor takes device tensors");
    if (!t.is_contiguous()) fail(PyExc_ValueError, "libxnor takes densely packed tensors");
    if (t.scalar_type() != type) {
        PyErr_Format(PyExc_ValueError, "expected %s, got %s", c10::toString(type), c10::toString(t.scalar_type()));
        throw PythonError{};
    }
    return t.data_ptr();
}
float *f32(PyObject *o) { return static_cast<float *>(tensor(o, c10::ScalarType::Float)); }
uint32_t *u32(PyObject *o) { return static_cast<uint32_t *>(tensor(o, c10::ScalarType::Int)); }
int32_t *i32(PyObject *o) { return static_cast<int32_t *>(tensor(o, c10::ScalarType::Int)); }
void *u8(PyObject *o) { return tensor(o, c10::ScalarType::Byte); }

int num(PyObject *o)
{
    const unsigned long v = PyLong_AsUnsignedLongMask(o);           // (C's conversion to int, as ctypes has it)
    if (v == (unsigned long)-1 && PyErr_Occurred()) throw PythonError{};
    return (int)v;
}

// A descriptor (xnor.py's ctypes structure, nothing else that holds as many bytes) through the buffer protocol; held for the
// duration of the call.
struct Desc {
    Py_buffer view{};
    explicit Desc(PyObject *o)
    {
        const int is = PyObject_IsInstance(o, g_desc);
        if (is < 0) throw PythonError{};
        if (!is) fail(PyExc_TypeError, "expected a convolution descriptor");
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw PythonError{};
        if (view.len != (Py_ssize_t)sizeof(xnor_conv_desc)) {
            PyBuffer_Release(&view);
            fail(PyExc_TypeError, "expected a convolution descriptor");
        }
    }
    ~Desc() { PyBuffer_Release(&view); }
    Desc(const Desc &) = delete;
    operator const xnor_conv_desc *() const { return static_cast<const xnor_conv_desc *>(view.buf); }
};

void *stream(PyObject *o)
{
    PyObject *handle;
    if (o != Py_None) {
        handle = PyObject_GetAttrString(o, "cuda_stream");
    } else {
        PyObject *device = PyObject_CallNoArgs(g_current_device);
        if (!device) throw PythonError{};
        handle = PyObject_CallOneArg(g_raw_stream, device);
        Py_DECREF(device);
    }
    if (!handle) throw PythonError{};
    void *s = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    if (!s && PyErr_Occurred()) throw PythonError{};
    return s;
}

// Every entry point: its address in the bound library and the conversion of its arguments, in the C order with the stream
// last.
#define XNOR_CALLS(X)                                                                                                     \
    X(xnor_binarize_pack, 9, f32(a[0]), f32(a[1]), f32(a[2]), u32(a[3]), num(a[4]), num(a[5]), num(a[6]), num(a[7]))      \
    X(xnor_compute_K, 7, f32(a[0]), f32(a[1]), f32(a[2]), f32(a[3]), f32(a[4]), Desc(a[5]))                               \
    X(xnor_binactiv, 8, f32(a[0]), f32(a[1]), f32(a[2]), u32(a[3]), f32(a[4]), f32(a[5]), Desc(a[6]))                     \
    X(xnor_binactiv_streamed, 8, f32(a[0]), f32(a[1]), f32(a[2]), u32(a[3]), f32(a[4]), f32(a[5]), Desc(a[6]))            \
    X(xnor_pool_binactiv, 17, f32(a[0]), f32(a[1]), f32(a[2]), u32(a[3]), f32(a[4]), num(a[5]), num(a[6]), num(a[7]),     \
      num(a[8]), num(a[9]), num(a[10]), num(a[11]), num(a[12]), num(a[13]), num(a[14]), num(a[15]))                       \
    X(xnor_bwn_split, 7, f32(a[0]), u8(a[1]), num(a[2]), num(a[3]), num(a[4]), num(a[5]))                                 \
    X(xnor_bwn_pack_weights, 8, f32(a[0]), f32(a[1]), u8(a[2]), num(a[3]), num(a[4]), num(a[5]), num(a[6]))               \
    X(xnor_bwn_conv2d, 6, u8(a[0]), u8(a[1]), f32(a[2]), f32(a[3]), Desc(a[4]))                                           \
    X(xnor_bingrad_pack_weights, 9, f32(a[0]), u32(a[1]), f32(a[2]), u8(a[3]), num(a[4]), num(a[5]), num(a[6]), num(a[7]))\
    X(xnor_bingrad_binarize, 7, f32(a[0]), f32(a[1]), f32(a[2]), u32(a[3]), f32(a[4]), Desc(a[5]))                        \
    X(xnor_bingrad_conv2d, 11, u32(a[0]), u32(a[1]), u8(a[2]), f32(a[3]), f32(a[4]), f32(a[5]), f32(a[6]), i32(a[7]),     \
      Desc(a[8]), num(a[9]))                                                                                              \
    X(xnor_kbit_pack_input, 8, f32(a[0]), u8(a[1]), num(a[2]), num(a[3]), num(a[4]), num(a[5]), num(a[6]))                \
    X(xnor_kbit_pack_weights, 10, f32(a[0]), f32(a[1]), u8(a[2]), num(a[3]), num(a[4]), num(a[5]), num(a[6]), num(a[7]),  \
      num(a[8]))                                                                                                          \
    X(xnor_kbit_conv2d, 9, u8(a[0]), u8(a[1]), f32(a[2]), f32(a[3]), i32(a[4]), Desc(a[5]), num(a[6]), num(a[7]))         \
    X(xnor_pack_weights, 9, f32(a[0]), u32(a[1]), f32(a[2]), u8(a[3]), num(a[4]), num(a[5]), num(a[6]), num(a[7]))        \
    X(xnor_conv2d, 11, u32(a[0]), u32(a[1]), u8(a[2]), f32(a[3]), f32(a[4]), f32(a[5]), f32(a[6]), i32(a[7]), Desc(a[8]), \
      num(a[9]))                                                                                                          \
    X(xnor_conv2d_pool, 13, u32(a[0]), u8(a[1]), f32(a[2]), f32(a[3]), f32(a[4]), f32(a[5]), Desc(a[6]), num(a[7]),       \
      num(a[8]), num(a[9]), num(a[10]), num(a[11]))                                                                       \
    X(xnor_linear, 12, u32(a[0]), u32(a[1]), u8(a[2]), f32(a[3]), f32(a[4]), f32(a[5]), i32(a[6]), num(a[7]), num(a[8]),  \
      num(a[9]), num(a[10]))                                                                                              \
    X(xnor_conv2d_binactiv, 15, u32(a[0]), u32(a[1]), u8(a[2]), f32(a[3]), f32(a[4]), f32(a[5]), f32(a[6]), f32(a[7]),    \
      u32(a[8]), f32(a[9]), f32(a[10]), u8(a[11]), Desc(a[12]), num(a[13]))                                               \
    X(xnor_conv2d_binactiv_noalloc, 14, u32(a[0]), u32(a[1]), u8(a[2]), f32(a[3]), f32(a[4]), f32(a[5]), f32(a[6]),       \
      f32(a[7]), u32(a[8]), f32(a[9]), f32(a[10]), Desc(a[11]), num(a[12]))

#define XNOR_POINTER(NAME, N, ...) decltype(&::NAME) p_##NAME = nullptr;
XNOR_CALLS(XNOR_POINTER)

// The C call itself runs without the interpreter's lock, as under ctypes: a launch can wait for room in its queue, and what
// empties the queue may be a host function that needs the lock.  A constructor, so that its braces convert the arguments in
// order; they come by reference, and descriptors live in the caller's full expression.
struct Enqueue {
    int status;
    template <class P, class... A> explicit Enqueue(P entry, A &&...args)
    {
        PyThreadState *state = PyEval_SaveThread();
        status = entry(args...);
        PyEval_RestoreThread(state);
    }
};

template <class F> PyObject *guarded(const char *name, F call)
{
    int status;
    try {
        status = call();
    } catch (const PythonError &) {
        return nullptr;
    } catch (const std::exception &e) {                  // (torch refuses the address of a tensor without storage)
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    if (status == XNOR_OK) Py_RETURN_NONE;
    PyObject *r = PyObject_CallFunction(g_raise, "si", name, status);
    Py_XDECREF(r);
    if (r) PyErr_SetString(PyExc_RuntimeError, name);
    return nullptr;
}

#define XNOR_WRAPPER(NAME, N, ...)                                                                       \
    PyObject *call_##NAME(PyObject *, PyObject *const *a, Py_ssize_t n)                                  \
    {                                                                                                    \
        if (n != N || !p_##NAME) {                                                                       \
            PyErr_SetString(PyExc_TypeError, #NAME ": wrong number of arguments, or no library bound");  \
            return nullptr;                                                                              \
        }                                                                                                \
        return guarded(#NAME, [&] { return Enqueue{p_##NAME, __VA_ARGS__, stream(a[N - 1])}.status; });  \
    }
XNOR_CALLS(XNOR_WRAPPER)

// bind(path of the library, raise(name, status), current_device(), raw_stream(device), descriptor class)
PyObject *bind(PyObject *, PyObject *args)
{
    const char *path;
    PyObject *raise, *device, *raw, *desc;
    if (!PyArg_ParseTuple(args, "sOOOO", &path, &raise, &device, &raw, &desc)) return nullptr;
    void *lib = dlopen(path, RTLD_NOW | RTLD_LOCAL);
    if (!lib) {
        PyErr_SetString(PyExc_ImportError, dlerror());
        return nullptr;
    }
#define XNOR_LOOKUP(NAME, N, ...)                                                       \
    if (void *f = dlsym(lib, #NAME)) p_##NAME = reinterpret_cast<decltype(p_##NAME)>(f); \
    else {                                                                              \
        PyErr_SetString(PyExc_ImportError, #NAME " is not in the library");             \
        return nullptr;                                                                 \
    }
    XNOR_CALLS(XNOR_LOOKUP)
    Py_INCREF(raise); Py_INCREF(device); Py_INCREF(raw); Py_INCREF(desc);
    Py_XDECREF(g_raise); Py_XDECREF(g_current_device); Py_XDECREF(g_raw_stream); Py_XDECREF(g_desc);
    g_raise = raise; g_current_device = device; g_raw_stream = raw; g_desc = desc;
    Py_RETURN_NONE;
}

#define XNOR_METHOD(NAME, N, ...) \
    {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call_##NAME)), METH_FASTCALL, nullptr},
PyMethodDef g_methods[] = {XNOR_CALLS(XNOR_METHOD){"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&g_module); }
