// Native call path of the Python binding for the calls of a serving loop: hac_dot, shac_dot, im_dot, hac_dot_noalloc and
// hac_forward on torch tensors.  Same checks, exceptions and results as the Python text they replace; nothing is kept
// between calls but the addresses of the library's functions.
//
// Why native: on small products the host, not the GPU, sets the time of a call.  A call through ctypes took 9 us of the
// host's time with buffers the caller keeps (one launch, of which the launch itself is 3) and 11.5 us with buffers made
// here, against 5 to 6 us of the kernel; see the figures at dot().
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <memory>
#include <optional>
#include <vector>

#include "../../include/hac.h"

namespace {

struct Api {
    decltype(&::hac_dot) hac_dot, shac_dot, im_dot;
    decltype(&::hac_dot_noalloc) noalloc;
    decltype(&::hac_workspace_bytes_for) ws_bytes;
    decltype(&::hac_forward) forward;
    decltype(&::hac_forward_workspace_bytes) forward_ws;
} g_api;
PyObject* g_error = nullptr;             // called with (status, function name): raises HacError
PyObject *g_desc, *g_tensor, *g_stream;  // attribute names
PyObject *g_Desc = nullptr, *g_Launch = nullptr;             // the ctypes structures of the header and of a launch

struct Raised {};                        // a Python exception is set

[[noreturn]] void raise(PyObject* type, const char* text)
{
    PyErr_SetString(type, text);
    throw Raised{};
}

struct Ref {                             // owned reference
    PyObject* p;
    explicit Ref(PyObject* q) : p(q) { if (!p) throw Raised{}; }
    ~Ref() { Py_XDECREF(p); }
    Ref(const Ref&) = delete;
    Ref& operator=(const Ref&) = delete;
};

// The bytes of a ctypes structure, looked up anew in every call.
template <class T> struct Struct {
    Py_buffer view;
    Struct(PyObject* o, PyObject* type)
    {
        if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(type))) {
            PyErr_Format(PyExc_TypeError, "expected %s, not %s", reinterpret_cast<PyTypeObject*>(type)->tp_name, Py_TYPE(o)->tp_name);
            throw Raised{};
        }
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE)) throw Raised{};
        if (view.len < (Py_ssize_t)sizeof(T)) { PyBuffer_Release(&view); raise(PyExc_TypeError, "not the expected ctypes structure"); }
    }
    ~Struct() { PyBuffer_Release(&view); }
    Struct(const Struct&) = delete;
    Struct& operator=(const Struct&) = delete;
    const T* get() const { return static_cast<const T*>(view.buf); }
};

struct Blob {                            // a DeviceBlob: .desc and .tensor
    Ref desc_obj, tensor_obj;
    Struct<hac_desc_t> desc;
    void* data;
    explicit Blob(PyObject* o)
        : desc_obj(PyObject_GetAttr(o, g_desc)), tensor_obj(PyObject_GetAttr(o, g_tensor)), desc(desc_obj.p, g_Desc)
    {
        if (!THPVariable_Check(tensor_obj.p)) raise(PyExc_TypeError, "the blob's bytes must be a tensor");
        data = THPVariable_Unpack(tensor_obj.p).data_ptr();
    }
};

const at::Tensor& tensor_of(PyObject* o, const char* otherwise)
{
    if (!THPVariable_Check(o)) raise(PyExc_TypeError, otherwise);
    return THPVariable_Unpack(o);
}

// Other Python threads run while the allocator may free and retry, as with the tensor calls of Python.
struct GilReleased {
    PyThreadState* state = PyEval_SaveThread();
    ~GilReleased() { PyEval_RestoreThread(state); }
};

at::Tensor empty(at::IntArrayRef sizes, at::ScalarType type, const at::Tensor& like)
{
    const GilReleased released;
    return at::empty(sizes, at::TensorOptions().dtype(type).device(like.device()));
}

at::Tensor with_rows(const at::Tensor& X)                    // rows of X contiguous: X, or a copy
{
    if (X.stride(1) == 1) return X;
    const GilReleased released;
    return X.contiguous();
}

// The stream of a call.  Where the caller names another one than X's device is on, it is that device's current one while the
// call's buffers are made: a copy of X is queued, and everything made here is used, freed and made anew, in the order of the
// stream that the product runs on.
struct OnStream {
    hac_stream_t handle;
    std::optional<c10::hip::HIPStream> before;
    OnStream(PyObject* stream, const at::Tensor& X)
    {
        if (stream == Py_None) { handle = (hac_stream_t)c10::hip::getCurrentHIPStream().stream(); return; }
        Ref h(PyObject_GetAttr(stream, g_stream));
        Ref i(PyNumber_Long(h.p));
        handle = (hac_stream_t)PyLong_AsVoidPtr(i.p);
        if (!handle && PyErr_Occurred()) throw Raised{};
        const c10::hip::HIPStream current = c10::hip::getCurrentHIPStream(X.device().index());
        if ((hac_stream_t)current.stream() == handle) return;
        c10::hip::setCurrentHIPStream(c10::hip::getStreamFromExternal((hipStream_t)handle, X.device().index()));
        before = current;
    }
    ~OnStream() { if (before) c10::hip::setCurrentHIPStream(*before); }
    OnStream(const OnStream&) = delete;
    OnStream& operator=(const OnStream&) = delete;
    // a result made here is the caller's to use on the stream it was on: not made anew before that is done
    void hand_over(const at::Tensor& Y) const
    {
        if (before) Y.record_stream(c10::Stream(c10::Stream::UNSAFE, c10::Device(c10::DeviceType::CUDA, before->device_index()), before->id()));
    }
};

bool float_cuda(const at::Tensor& t) { return t.scalar_type() == at::kFloat && t.is_cuda(); }

// Y: given and fit to take the result, or made here.
at::Tensor result(PyObject* y, const at::Tensor& X, int64_t B, int64_t m, const OnStream& on)
{
    if (y == Py_None) {
        at::Tensor Y = empty({B, m}, at::kFloat, X);
        on.hand_over(Y);
        return Y;
    }
    const char* what = "Y must be a B x m float32 CUDA tensor with unit column stride";
    const at::Tensor& Y = tensor_of(y, what);
    if (Y.scalar_type() != at::kFloat || Y.dim() != 2 || Y.size(0) != B || Y.size(1) != m || Y.stride(1) != 1 || !Y.is_cuda()) raise(PyExc_TypeError, what);
    return Y;
}

struct Scratch { at::Tensor keep; void* ptr; size_t bytes; };

Scratch scratch(PyObject* workspace, const at::Tensor& X, size_t need)
{
    Scratch s{ {}, nullptr, 0 };
    if (workspace != Py_None) s.keep = tensor_of(workspace, "workspace must be a tensor");
    else if (need) s.keep = empty({(int64_t)need}, at::kByte, X);
    else return s;
    s.ptr = s.keep.data_ptr();
    s.bytes = (size_t)s.keep.numel() * s.keep.element_size();
    return s;
}

void check(int rc, const char* where)
{
    if (!rc) return;
    Ref r(PyObject_CallFunction(g_error, "is", rc, where));
    raise(PyExc_RuntimeError, where);                        // (not reached: the call above raises)
}

// The arguments of a call by position or name; missing ones are None.
void arguments(PyObject* const* args, Py_ssize_t n, PyObject* kwnames, const char* const* names, int required, int total, PyObject** out)
{
    if (n > total) raise(PyExc_TypeError, "too many arguments");
    for (int i = 0; i < total; ++i) out[i] = i < n ? args[i] : nullptr;
    const Py_ssize_t nk = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < nk; ++k) {
        PyObject* key = PyTuple_GET_ITEM(kwnames, k);
        int i = 0;
        while (i < total && PyUnicode_CompareWithASCIIString(key, names[i])) ++i;
        if (i == total) { PyErr_Format(PyExc_TypeError, "unexpected keyword argument '%U'", key); throw Raised{}; }
        if (out[i]) { PyErr_Format(PyExc_TypeError, "multiple values for argument '%U'", key); throw Raised{}; }
        out[i] = args[n + k];
    }
    for (int i = 0; i < total; ++i) {
        if (out[i]) continue;
        if (i < required) { PyErr_Format(PyExc_TypeError, "missing argument '%s'", names[i]); throw Raised{}; }
        out[i] = Py_None;
    }
}

template <class F> PyObject* guarded(F&& f)
{
    try {
        return f();
    } catch (const Raised&) {
        return nullptr;
    } catch (const std::bad_alloc&) {
        return PyErr_NoMemory();
    } catch (const std::exception&) {                        // torch's as Python sees them: torch.OutOfMemoryError among them
        torch::translate_exception_to_python(std::current_exception());
        return nullptr;
    }
}

const hac_launch_t* launch_of(PyObject* launch, std::unique_ptr<Struct<hac_launch_t>>& keep)
{
    if (launch == Py_None) return nullptr;
    keep.reset(new Struct<hac_launch_t>(launch, g_Launch));
    return keep->get();
}

// dot(name's function)(dblob, X, Y, workspace, launch, stream).  Host time of a call, ctypes -> here: 9.2 -> 4.3 us with the
// caller's buffers and one launch, 14.7 -> 9.3 us with two buffers made here and two launches.
enum Which { HAC, SHAC, IM };
PyObject* dot(Which which, PyObject* const* args, Py_ssize_t n, PyObject* kwnames)
{
    static const char* const names[] = { "dblob", "X", "Y", "workspace", "launch", "stream" };
    static const char* const im_names[] = { "dblob", "X", "Y", "workspace", "stream" };
    static const char* const where[] = { "hac_dot", "shac_dot", "im_dot" };
    return guarded([&]() -> PyObject* {
        PyObject* a[6];
        if (which == IM) {
            arguments(args, n, kwnames, im_names, 2, 5, a);
            a[5] = a[4]; a[4] = Py_None;
        } else {
            arguments(args, n, kwnames, names, 2, 6, a);
        }
        at::Tensor X = tensor_of(a[1], "X must be a 2-D float32 CUDA tensor");
        if (!float_cuda(X) || X.dim() != 2) raise(PyExc_TypeError, "X must be a 2-D float32 CUDA tensor");
        const OnStream on(a[5], X);
        X = with_rows(X);
        const Blob blob(a[0]);
        const hac_desc_t* d = blob.desc.get();
        const int64_t B = X.size(0), rows = (int64_t)d->n, m = (int64_t)d->m;
        if (X.size(1) != rows) raise(PyExc_ValueError, "X has the wrong width");
        at::Tensor Y = result(a[2], X, B, m, on);
        std::unique_ptr<Struct<hac_launch_t>> keep;
        const hac_launch_t* launch = launch_of(a[4], keep);
        const Scratch ws = scratch(a[3], X, a[3] == Py_None ? g_api.ws_bytes(d, B, launch) : 0);
        const int64_t ldx = B > 1 ? X.stride(0) : std::max<int64_t>(rows, 1), ldy = B > 1 ? Y.stride(0) : std::max<int64_t>(m, 1);
        const float* x = static_cast<const float*>(X.data_ptr());
        float* y = static_cast<float*>(Y.data_ptr());
        const auto f = which == HAC ? g_api.hac_dot : which == SHAC ? g_api.shac_dot : g_api.im_dot;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = f(d, blob.data, x, B, ldx, y, ldy, ws.ptr, ws.bytes, launch, on.handle);
        Py_END_ALLOW_THREADS
        check(rc, where[which]);
        if (a[2] != Py_None) { Py_INCREF(a[2]); return a[2]; }
        return THPVariable_Wrap(std::move(Y));
    });
}

PyObject* py_hac_dot(PyObject*, PyObject* const* args, Py_ssize_t n, PyObject* kw) { return dot(HAC, args, n, kw); }
PyObject* py_shac_dot(PyObject*, PyObject* const* args, Py_ssize_t n, PyObject* kw) { return dot(SHAC, args, n, kw); }
PyObject* py_im_dot(PyObject*, PyObject* const* args, Py_ssize_t n, PyObject* kw) { return dot(IM, args, n, kw); }

PyObject* py_noalloc(PyObject*, PyObject* const* args, Py_ssize_t n, PyObject* kwnames)
{
    static const char* const names[] = { "dblob", "X", "Y", "launch", "stream" };
    return guarded([&]() -> PyObject* {
        PyObject* a[5];
        arguments(args, n, kwnames, names, 3, 5, a);
        const char* what = "X must be a 2-D float32 CUDA tensor with unit column stride";
        const at::Tensor& X = tensor_of(a[1], what);
        if (!float_cuda(X) || X.dim() != 2 || X.stride(1) != 1) raise(PyExc_TypeError, what);
        const Blob blob(a[0]);
        const hac_desc_t* d = blob.desc.get();
        const int64_t B = X.size(0), rows = (int64_t)d->n, m = (int64_t)d->m;
        if (X.size(1) != rows) raise(PyExc_ValueError, "X has the wrong width");
        if (a[2] == Py_None) raise(PyExc_TypeError, "Y must be a B x m float32 CUDA tensor with unit column stride");
        const OnStream on(a[4], X);
        const at::Tensor Y = result(a[2], X, B, m, on);
        std::unique_ptr<Struct<hac_launch_t>> keep;
        const hac_launch_t* launch = launch_of(a[3], keep);
        const int64_t ldx = B > 1 ? X.stride(0) : std::max<int64_t>(rows, 1), ldy = B > 1 ? Y.stride(0) : std::max<int64_t>(m, 1);
        const float* x = static_cast<const float*>(X.data_ptr());
        float* y = static_cast<float*>(Y.data_ptr());
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_api.noalloc(d, blob.data, x, B, ldx, y, ldy, launch, on.handle);
        Py_END_ALLOW_THREADS
        check(rc, "hac_dot_noalloc");
        Py_INCREF(a[2]);
        return a[2];
    });
}

PyObject* py_forward(PyObject*, PyObject* const* args, Py_ssize_t n, PyObject* kwnames)
{
    static const char* const names[] = { "layers", "X", "Y", "workspace", "stream" };
    return guarded([&]() -> PyObject* {
        PyObject* a[5];
        arguments(args, n, kwnames, names, 2, 5, a);
        at::Tensor X = tensor_of(a[1], "X must be a 2-D float32 CUDA tensor");
        if (!float_cuda(X) || X.dim() != 2) raise(PyExc_TypeError, "X must be a 2-D float32 CUDA tensor");
        const OnStream on(a[4], X);
        X = with_rows(X);
        const int64_t B = X.size(0);
        Ref seq(PySequence_Fast(a[0], "layers must be a sequence"));
        const Py_ssize_t L = PySequence_Fast_GET_SIZE(seq.p);
        if (L == 0) raise(PyExc_IndexError, "list index out of range");
        std::vector<std::unique_ptr<Blob>> blobs(L);
        std::vector<std::unique_ptr<Ref>> items(L);          // a layer's own references, whatever kind of sequence it is
        std::vector<hac_layer_t> arr(L);
        for (Py_ssize_t i = 0; i < L; ++i) {
            items[i].reset(new Ref(PySequence_Tuple(PySequence_Fast_GET_ITEM(seq.p, i))));
            PyObject* t = items[i]->p;
            if (PyTuple_GET_SIZE(t) != 3) raise(PyExc_ValueError, "a layer is (DeviceBlob, bias or None, relu)");
            blobs[i].reset(new Blob(PyTuple_GET_ITEM(t, 0)));
            PyObject* bias = PyTuple_GET_ITEM(t, 1);
            arr[i] = hac_layer_t{};
            arr[i].desc = blobs[i]->desc.get();
            arr[i].d_blob = blobs[i]->data;
            if (bias != Py_None) {
                const char* what = "bias must be a contiguous float32 CUDA tensor of m elements";
                const at::Tensor& b = tensor_of(bias, what);
                if (!float_cuda(b) || (uint64_t)b.numel() != arr[i].desc->m || !b.is_contiguous()) raise(PyExc_TypeError, what);
                arr[i].d_bias = static_cast<const float*>(b.data_ptr());
            }
            const int relu = PyObject_IsTrue(PyTuple_GET_ITEM(t, 2));
            if (relu < 0) throw Raised{};
            arr[i].activation = relu ? HAC_ACT_RELU : HAC_ACT_NONE;
        }
        const int64_t m = (int64_t)arr[L - 1].desc->m;
        at::Tensor Y = result(a[2], X, B, m, on);
        const Scratch ws = scratch(a[3], X, a[3] == Py_None ? g_api.forward_ws(arr.data(), (uint32_t)L, B) : 0);
        const int64_t ldx = B > 1 ? X.stride(0) : std::max<int64_t>(X.size(1), 1), ldy = B > 1 ? Y.stride(0) : std::max<int64_t>(m, 1);
        const float* x = static_cast<const float*>(X.data_ptr());
        float* y = static_cast<float*>(Y.data_ptr());
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_api.forward(arr.data(), (uint32_t)L, x, B, ldx, y, ldy, ws.ptr, ws.bytes, on.handle);
        Py_END_ALLOW_THREADS
        check(rc, "hac_forward");
        if (a[2] != Py_None) { Py_INCREF(a[2]); return a[2]; }
        return THPVariable_Wrap(std::move(Y));
    });
}

// bind(error, Desc, Launch, hac_dot, shac_dot, im_dot, hac_dot_noalloc, hac_workspace_bytes_for, hac_forward, hac_forward_workspace_bytes): addresses
PyObject* py_bind(PyObject*, PyObject* args)
{
    PyObject *error, *desc, *launch;
    unsigned long long p[7];
    if (!PyArg_ParseTuple(args, "OO!O!KKKKKKK", &error, &PyType_Type, &desc, &PyType_Type, &launch, p, p + 1, p + 2, p + 3, p + 4, p + 5, p + 6)) return nullptr;
    Py_INCREF(error); Py_INCREF(desc); Py_INCREF(launch);
    Py_XDECREF(g_error); Py_XDECREF(g_Desc); Py_XDECREF(g_Launch);
    g_error = error; g_Desc = desc; g_Launch = launch;
    g_api.hac_dot = reinterpret_cast<decltype(g_api.hac_dot)>(p[0]);
    g_api.shac_dot = reinterpret_cast<decltype(g_api.shac_dot)>(p[1]);
    g_api.im_dot = reinterpret_cast<decltype(g_api.im_dot)>(p[2]);
    g_api.noalloc = reinterpret_cast<decltype(g_api.noalloc)>(p[3]);
    g_api.ws_bytes = reinterpret_cast<decltype(g_api.ws_bytes)>(p[4]);
    g_api.forward = reinterpret_cast<decltype(g_api.forward)>(p[5]);
    g_api.forward_ws = reinterpret_cast<decltype(g_api.forward_ws)>(p[6]);
    Py_RETURN_NONE;
}

#define HAC_FAST(name, f) { name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL | METH_KEYWORDS, nullptr }
PyMethodDef methods[] = {
    HAC_FAST("hac_dot", py_hac_dot), HAC_FAST("shac_dot", py_shac_dot), HAC_FAST("im_dot", py_im_dot),
    HAC_FAST("hac_dot_noalloc", py_noalloc), HAC_FAST("hac_forward", py_forward),
    { "bind", py_bind, METH_VARARGS, nullptr }, { nullptr, nullptr, 0, nullptr } };
PyModuleDef module = { PyModuleDef_HEAD_INIT, "_hacbind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr };

} // namespace

PyMODINIT_FUNC PyInit__hacbind()
{
    g_desc = PyUnicode_InternFromString("desc");
    g_tensor = PyUnicode_InternFromString("tensor");
    g_stream = PyUnicode_InternFromString("cuda_stream");
    if (!g_desc || !g_tensor || !g_stream) return nullptr;
    return PyModule_Create(&module);
}
