// Argument marshalling of binding.py in C++: tensors, descriptors and the current stream to the plain arguments of the C ABI.
//
// A call that enqueues a kernel of a few microseconds is bound by the host.  Enqueueing a plain convolution call took 5.1 us
// from Python, a module call 6.4, of which 3.1 to 3.7 are the HIP runtime's launch; the rest were one Python call per tensor,
// two for the stream and ctypes' conversions.  With these functions it is 3.1 and 4.1: one 14 x 14 image, 64 channels, 5.3 -> 3.3 to 4.2 us
// a pass (3.2 in a graph), one 7 x 7 image, 1024 channels, 5.6 -> 4.7 (5.1 in a graph), a level of six small calls 32 -> 24.
//
// The rules are binding.py's, which stay the fallback for whatever is not the common case (its _ptr, _desc and _stream are
// called for tensor subclasses, descriptors that are no bcnn_conv_desc, stream objects, and before torch has initialised the
// device) and for a Python or torch that this is not built for, where it refuses to load: tensors are read by the layout
// that torch's headers had.  Nothing is kept between calls but the library's entry points, those Python objects and
// whether torch has initialised the device, which a forked child asks again.
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>

#include "bcnn.h"

#include <pthread.h>

#include <cstdio>
#include <cstring>
#include <exception>

namespace {

struct Api {
    decltype(&bcnn_pack) pack;
    decltype(&bcnn_pack_bias) pack_bias;
    decltype(&bcnn_pack_bias_replicated) pack_bias_replicated;
    decltype(&bcnn_conv2d_binary) conv2d_binary;
    decltype(&bcnn_conv2d_binary_sign_pack) conv2d_binary_sign_pack;
    decltype(&bcnn_conv2d_binary_variant) conv2d_binary_variant;
    decltype(&bcnn_conv2d_binary_module) conv2d_binary_module;
    decltype(&bcnn_conv2d_binary_branches) conv2d_binary_branches;
    decltype(&bcnn_conv2d_binary_branches_sign_pack) conv2d_binary_branches_sign_pack;
    decltype(&bcnn_conv2d_binary_branches_module) conv2d_binary_branches_module;
    decltype(&bcnn_avgpool_bias_sign_pack) avgpool_bias_sign_pack;
    decltype(&bcnn_threshold_sign_pack) threshold_sign_pack;
};

Api api;
PyObject *py_ptr, *py_desc, *py_stream, *py_initialized, *desc_type, *argument_error;
// torch has initialised the device in this process (a forked child has not)
bool device_ready = false;

// thrown with a Python error set
struct PythonError {};

void* address(PyObject* o)
{
    if (!PyLong_Check(o)) {
        PyErr_Format(argument_error, "expected an address, not %.100s", Py_TYPE(o)->tp_name);
        throw PythonError{};
    }
    return reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(o)));
}

// what a Python fallback says for an object
void* ask(PyObject* function, PyObject* o)
{
    PyObject* got = PyObject_CallFunctionObjArgs(function, o, nullptr);
    if (!got) throw PythonError{};
    void* p = nullptr;
    try {
        p = got == Py_None ? nullptr : address(got);
    } catch (const PythonError&) {
        Py_DECREF(got);
        throw;
    }
    Py_DECREF(got);
    return p;
}

// Device address of a tensor, a raw address, or null for None.
template <class T>
struct Pointer {
    T* p;
    explicit Pointer(PyObject* o)
    {
        if (o == Py_None) p = nullptr;
        else if (THPVariable_CheckExact(o)) {
            const at::Tensor& t = THPVariable_Unpack(o);
            if (!t.is_contiguous()) {
                PyErr_SetString(PyExc_ValueError, "tensor must be contiguous");
                throw PythonError{};
            }
            p = static_cast<T*>(t.data_ptr());
        } else if (PyLong_Check(o)) p = static_cast<T*>(address(o));
        else p = static_cast<T*>(ask(py_ptr, o));
    }
    operator T*() const { return p; }
};
using Void = Pointer<void>;
using Words = Pointer<uint32_t>;
using Ints = Pointer<int32_t>;
using Floats = Pointer<float>;

// An integer as ctypes takes it: an int or what has an index, cut to the argument's width.
int64_t whole(PyObject* o)
{
    if (PyLong_Check(o)) return static_cast<int64_t>(PyLong_AsUnsignedLongLongMask(o));
    PyObject* n = PyIndex_Check(o) ? PyNumber_Index(o) : nullptr;
    if (!n) {
        if (!PyErr_Occurred()) PyErr_Format(argument_error, "expected an integer, not %.100s", Py_TYPE(o)->tp_name);
        throw PythonError{};
    }
    const int64_t v = static_cast<int64_t>(PyLong_AsUnsignedLongLongMask(n));
    Py_DECREF(n);
    return v;
}
int32_t small(PyObject* o) { return static_cast<int32_t>(whole(o)); }
// an integer that binding.py converts with int() first
int64_t converted(PyObject* o)
{
    if (PyLong_Check(o)) return whole(o);
    PyObject* n = PyNumber_Long(o);
    if (!n) throw PythonError{};
    const int64_t v = static_cast<int64_t>(PyLong_AsUnsignedLongLongMask(n));
    Py_DECREF(n);
    return v;
}

bcnn_conv_desc descriptor(PyObject* o)
{
    PyObject* made = nullptr;
    const int is = PyObject_IsInstance(o, desc_type);
    if (is < 0) throw PythonError{};
    if (!is) {
        made = PyObject_CallFunctionObjArgs(py_desc, o, nullptr);
        if (!made) throw PythonError{};
        o = made;
    }
    bcnn_conv_desc d{};
    Py_buffer view;
    const bool ok = PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) == 0;
    if (ok) {
        std::memcpy(&d, view.buf, view.len < (Py_ssize_t)sizeof d ? view.len : sizeof d);
        PyBuffer_Release(&view);
    }
    Py_XDECREF(made);
    if (!ok) throw PythonError{};
    return d;
}

void* stream(PyObject* o)
{
    if (o == Py_None && !device_ready) {
        PyObject* yes = PyObject_CallFunctionObjArgs(py_initialized, nullptr);
        if (!yes) throw PythonError{};
        device_ready = yes == Py_True;
        Py_DECREF(yes);
    }
    if (o == Py_None && device_ready) return c10::hip::getCurrentHIPStream().stream();
    if (PyLong_Check(o)) return address(o);
    return ask(py_stream, o);
}

// The call itself without the interpreter's lock, as ctypes does it: an enqueue can wait for room in the queue.
template <class F>
PyObject* enqueue(F&& call)
{
    int status;
    PyThreadState* state = PyEval_SaveThread();
    status = call();
    PyEval_RestoreThread(state);
    return PyLong_FromLong(status);
}

// Every method: a fixed number of positional arguments, no C++ exception past it.
template <int N, PyObject* (*BODY)(PyObject* const*)>
PyObject* method(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, %zd given", N, n);
        return nullptr;
    }
    try {
        return BODY(args);
    } catch (const PythonError&) {
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception");
    }
    return nullptr;
}

PyObject* pack(PyObject* const* a)
{
    const Void src(a[0]);
    const int dtype = small(a[1]);
    const int64_t outer = whole(a[2]), channels = whole(a[3]), inner = whole(a[4]);
    const Words dst(a[5]);
    void* st = stream(a[6]);
    return enqueue([&] { return api.pack(src, (bcnn_dtype)dtype, outer, channels, inner, dst, st); });
}

PyObject* pack_bias(PyObject* const* a)
{
    const Void src(a[0]);
    const int dtype = small(a[1]);
    const int64_t outer = whole(a[2]), channels = whole(a[3]), inner = whole(a[4]);
    const Floats bias(a[5]);
    const Words dst(a[6]);
    void* st = stream(a[7]);
    return enqueue([&] { return api.pack_bias(src, (bcnn_dtype)dtype, outer, channels, inner, bias, dst, st); });
}

PyObject* pack_bias_replicated(PyObject* const* a)
{
    const Void src(a[0]);
    const int dtype = small(a[1]);
    const int64_t outer = whole(a[2]), channels = whole(a[3]), inner = whole(a[4]);
    const int32_t replication = (int32_t)converted(a[5]);
    const Floats bias(a[6]);
    const Words dst(a[7]);
    void* st = stream(a[8]);
    return enqueue([&] { return api.pack_bias_replicated(src, (bcnn_dtype)dtype, outer, channels, inner, replication, bias, dst, st); });
}

PyObject* avgpool_bias_sign_pack(PyObject* const* a)
{
    const Void src(a[0]);
    const int dtype = (int)converted(a[1]);
    const int32_t n = small(a[2]), h = small(a[3]), w = small(a[4]), channels = small(a[5]), s = small(a[6]);
    const Floats bias(a[7]);
    const Void pooled(a[8]);
    const Words packed(a[9]);
    void* st = stream(a[10]);
    return enqueue([&] { return api.avgpool_bias_sign_pack(src, (bcnn_dtype)dtype, n, h, w, channels, s, bias, pooled, packed, st); });
}

PyObject* threshold_sign_pack(PyObject* const* a)
{
    const Ints y(a[0]), thr(a[1]);
    const int64_t rows = whole(a[2]), c_out = whole(a[3]);
    const Words packed(a[4]);
    void* st = stream(a[5]);
    return enqueue([&] { return api.threshold_sign_pack(y, thr, rows, c_out, packed, st); });
}

PyObject* conv2d_binary(PyObject* const* a)
{
    const bcnn_conv_desc d = descriptor(a[0]);
    const Words x(a[1]), w(a[2]);
    const Ints y(a[3]);
    void* st = stream(a[4]);
    return enqueue([&] { return api.conv2d_binary(&d, x, w, y, st); });
}

PyObject* conv2d_binary_sign_pack(PyObject* const* a)
{
    const bcnn_conv_desc d = descriptor(a[0]);
    const Words x(a[1]), w(a[2]);
    const Ints thr(a[3]);
    const Words y(a[4]);
    void* st = stream(a[5]);
    return enqueue([&] { return api.conv2d_binary_sign_pack(&d, x, w, thr, y, st); });
}

PyObject* conv2d_binary_variant(PyObject* const* a)
{
    const bcnn_conv_desc d = descriptor(a[0]);
    const Words x(a[1]), w(a[2]);
    const Ints thr(a[3]);
    const Void out(a[4]);
    const int variant = (int)converted(a[5]);
    void* st = stream(a[6]);
    return enqueue([&] { return api.conv2d_binary_variant(&d, x, w, thr, out, variant, st); });
}

PyObject* conv2d_binary_module(PyObject* const* a)
{
    const bcnn_conv_desc d = descriptor(a[0]);
    const Words x(a[1]), w(a[2]);
    bcnn_module_epilogue ep{};
    ep.bn_scale = Floats(a[3]);
    ep.bn_bias = Floats(a[4]);
    ep.identity = Void(a[5]);
    ep.prelu_slope = Floats(a[6]);
    ep.next_bias = Floats(a[7]);
    ep.real_dtype = (int32_t)converted(a[8]);
    const Void r(a[9]);
    const Words next(a[10]);
    const int variant = (int)converted(a[11]);
    void* st = stream(a[12]);
    ep.identity_channels = (int32_t)converted(a[13]);
    return enqueue([&] { return api.conv2d_binary_module(&d, x, w, &ep, r, next, variant, st); });
}

PyObject* conv2d_binary_branches(PyObject* const* a)
{
    const bcnn_conv_desc d = descriptor(a[0]);
    const int32_t branches = (int32_t)converted(a[1]);
    const Words x(a[2]);
    const int64_t step = converted(a[3]);
    const Words w(a[4]), pad(a[5]);
    const int pad_mode = (int)converted(a[6]);
    const Floats scale(a[7]), bias(a[8]), z(a[9]);
    const int variant = (int)converted(a[10]);
    void* st = stream(a[11]);
    return enqueue([&] { return api.conv2d_binary_branches(&d, branches, x, step, w, pad, pad_mode, scale, bias, z, variant, st); });
}

PyObject* conv2d_binary_branches_sign_pack(PyObject* const* a)
{
    const bcnn_conv_desc d = descriptor(a[0]);
    const int32_t branches = (int32_t)converted(a[1]);
    const Words x(a[2]);
    const int64_t step = converted(a[3]);
    const Words w(a[4]), pad(a[5]);
    const int pad_mode = (int)converted(a[6]);
    const Floats scale(a[7]), bias(a[8]);
    const Words z(a[9]);
    const int variant = (int)converted(a[10]);
    void* st = stream(a[11]);
    return enqueue([&] { return api.conv2d_binary_branches_sign_pack(&d, branches, x, step, w, pad, pad_mode, scale, bias, z, variant, st); });
}

PyObject* conv2d_binary_branches_module(PyObject* const* a)
{
    const bcnn_conv_desc d = descriptor(a[0]);
    const int32_t branches = (int32_t)converted(a[1]);
    const Words x(a[2]);
    const int64_t step = converted(a[3]);
    const Words w(a[4]), pad(a[5]);
    const int pad_mode = (int)converted(a[6]);
    const Floats scale(a[7]), bias(a[8]);
    bcnn_module_epilogue ep{};
    ep.identity = Void(a[9]);
    ep.prelu_slope = Floats(a[10]);
    ep.next_bias = Floats(a[11]);
    ep.real_dtype = (int32_t)converted(a[12]);
    const Void r(a[13]);
    const Words next(a[14]);
    const int variant = (int)converted(a[15]);
    void* st = stream(a[16]);
    ep.identity_channels = (int32_t)converted(a[17]);
    return enqueue([&] { return api.conv2d_binary_branches_module(&d, branches, x, step, w, pad, pad_mode, scale, bias, &ep, r, next, variant, st); });
}

// bind(entry points by name, _ptr, _desc, _stream, torch.cuda.is_initialized, bcnn_conv_desc, ctypes.ArgumentError): the library that later calls go to.
PyObject* bind(PyObject* const* a)
{
    auto entry = [&](const char* name) -> void* {
        PyObject* o = PyMapping_GetItemString(a[0], name);
        if (!o) throw PythonError{};
        void* p = PyLong_Check(o) ? reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(o))) : nullptr;
        Py_DECREF(o);
        if (!p) {
            PyErr_Format(PyExc_ValueError, "no address for %s", name);
            throw PythonError{};
        }
        return p;
    };
    Api got;
#define BIND(name) got.name = reinterpret_cast<decltype(got.name)>(entry("bcnn_" #name))
    BIND(pack); BIND(pack_bias); BIND(pack_bias_replicated); BIND(conv2d_binary); BIND(conv2d_binary_sign_pack);
    BIND(conv2d_binary_variant); BIND(conv2d_binary_module); BIND(conv2d_binary_branches); BIND(conv2d_binary_branches_sign_pack);
    BIND(conv2d_binary_branches_module); BIND(avgpool_bias_sign_pack); BIND(threshold_sign_pack);
#undef BIND
    PyObject** const kept[] = {&py_ptr, &py_desc, &py_stream, &py_initialized, &desc_type, &argument_error};
    for (int i = 0; i < 6; ++i) {
        Py_INCREF(a[1 + i]);
        PyObject* old = *kept[i];
        *kept[i] = a[1 + i];
        Py_XDECREF(old);
    }
    api = got;
    Py_RETURN_NONE;
}

#define METHOD(name, n) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&method<n, name>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    METHOD(bind, 7), METHOD(pack, 7), METHOD(pack_bias, 8), METHOD(pack_bias_replicated, 9), METHOD(avgpool_bias_sign_pack, 11),
    METHOD(threshold_sign_pack, 6), METHOD(conv2d_binary, 5), METHOD(conv2d_binary_sign_pack, 6), METHOD(conv2d_binary_variant, 7),
    METHOD(conv2d_binary_module, 14), METHOD(conv2d_binary_branches, 12), METHOD(conv2d_binary_branches_sign_pack, 12),
    METHOD(conv2d_binary_branches_module, 18), {nullptr, nullptr, 0, nullptr}};
#undef METHOD
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void)
{
    int major = 0, minor = 0;
    if (std::sscanf(Py_GetVersion(), "%d.%d", &major, &minor) != 2 || major != PY_MAJOR_VERSION || minor != PY_MINOR_VERSION) {
        PyErr_Format(PyExc_ImportError, "built for Python %d.%d", PY_MAJOR_VERSION, PY_MINOR_VERSION);
        return nullptr;
    }
    PyObject* version = PyImport_ImportModule("torch.version");
    PyObject* text = version ? PyObject_GetAttrString(version, "__version__") : nullptr;
    const char* torch = text ? PyUnicode_AsUTF8(text) : nullptr;
    const bool same = torch && !std::strcmp(torch, BCNN_TORCH_VERSION);
    if (torch && !same) PyErr_Format(PyExc_ImportError, "built for torch %s, not %s", BCNN_TORCH_VERSION, torch);
    Py_XDECREF(text);
    Py_XDECREF(version);
    if (!same) return nullptr;
    pthread_atfork(nullptr, nullptr, [] { device_ready = false; });
    return PyModule_Create(&module);
}
