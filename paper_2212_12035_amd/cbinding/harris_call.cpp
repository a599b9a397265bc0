// The marshalling of binding.py's fused entry points in native code: the checks of torch tensors, the layout structure
// and the call of the library, for calls that need nothing else.  A small image's launch takes the runtime some 3.2 us;
// in Python the checks and the call through ctypes added 2.2 us to it and more (480x640 uint8 with a result
// buffer 6.0 us a call, here 4.0; 64x96 float32 with a new result 7.4 and 4.8).
//
// Every function returns None, with nothing enqueued, for a call that is not plain: an argument of another type, a
// check that fails, tensor subclasses, wrapped tensors and modes that watch torch functions, a device that is not the
// current one.  The caller then goes through the Python code, which handles or refuses it.  Once the library has been
// called the call is not made again: a status other than success, which may come from a launch that was enqueued all
// the same, is raised as the Python code raises it.  No other errors are raised here.
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>

#include <climits>
#include <utility>

#include "harris.h"

namespace {

typedef int (*typed_fn)(const void*, int, int, int, int, const harris_layout*, float, float, int, void*, int, const harris_tuning*, void*);
typedef int (*quantized_fn)(const void*, int, int, int, int, const harris_layout*, float, float, int, float, float, uint8_t*, const harris_tuning*, void*);

// Set by bind(): the library's functions, torch's for the current device and its current stream's handle, and the
// Python code's that raises the error of a status.
typed_fn call_typed = nullptr;
quantized_fn call_quantized = nullptr;
PyObject *get_device = nullptr, *get_stream = nullptr, *raise_status = nullptr;

struct Call {
    const at::Tensor *rgb, *out;
    int dtype, out_dtype, batch, H, W;
    harris_layout layout;
    bool dense;                             // no layout: images and results without gaps
    float k, scale, q_scale, q_offset;
    int window;
};

// A torch tensor with memory of its own on a GPU, or null.
const at::Tensor* plain_tensor(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.is_cuda() && t.layout() == at::kStrided && t.has_storage() ? &t : nullptr;
}
bool number(PyObject* o, float& v) {
    if (!PyFloat_CheckExact(o)) return false;
    v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}
bool whole(PyObject* o, int& v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long x = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow != 0 || x < INT_MIN || x > INT_MAX) return false;
    v = (int)x;
    return true;
}
long long index_from(PyObject* o) {
    if (o == nullptr) { PyErr_Clear(); return -1; }
    const long long v = PyLong_AsLongLong(o);
    Py_DECREF(o);
    if (v == -1 && PyErr_Occurred()) { PyErr_Clear(); return -1; }
    return v;
}

bool image(Call& c) {
    const at::Tensor& t = *c.rgb;
    if (t.dim() != 4 || t.size(1) != 3) return false;
    const int64_t B = t.size(0), H = t.size(2), W = t.size(3);
    if (H < 4 || W < 4 || B > INT_MAX || H > INT_MAX || W > INT_MAX) return false;
    c.batch = (int)B; c.H = (int)H; c.W = (int)W;
    const auto type = t.scalar_type();
    if (type != at::kFloat && type != at::kByte) return false;
    c.dtype = type == at::kByte ? HARRIS_U8 : HARRIS_F32;
    return true;
}
bool result(const Call& c) {
    const at::Tensor &t = *c.out, &rgb = *c.rgb;
    return t.device() == rgb.device() && t.dim() == 3 && t.size(0) == c.batch && t.size(1) == c.H - 4 && t.size(2) == c.W - 4;
}
// The strides as pitches, for views whose last dimension has stride 1.
bool strided(Call& c) {
    const at::Tensor &t = *c.rgb, &o = *c.out;
    const long long n = c.H - 4, m = c.W - 4;
    if (t.stride(3) != 1 || (m > 1 && o.stride(2) != 1)) return false;
    c.layout.rgb_row_pitch = t.stride(2);
    c.layout.rgb_plane_pitch = t.stride(1);
    c.layout.rgb_image_pitch = c.batch > 1 ? t.stride(0) : 3 * t.stride(1);
    c.layout.out_row_pitch = n > 1 ? (long long)o.stride(1) : (m > 1 ? m : 1);
    const long long rows = n * o.stride(1);
    c.layout.out_image_pitch = c.batch > 1 ? (long long)o.stride(0) : (rows > 1 ? rows : 1);
    c.dense = false;
    return true;
}

// Enqueues the call on the current stream of the tensors' device, which has to be the current one.  kDeclined: it has
// not been made.  kRaised: it has, and failed; the error is set.
enum Outcome { kDeclined, kDone, kRaised };
Outcome enqueue(const Call& c) {
    const int index = c.rgb->device().index();
    if (index_from(PyObject_CallNoArgs(get_device)) != index) return kDeclined;
    PyObject* device = PyLong_FromLong(index);
    if (device == nullptr) { PyErr_Clear(); return kDeclined; }
    PyObject* stream = PyObject_CallOneArg(get_stream, device);
    Py_DECREF(device);
    if (stream == nullptr) { PyErr_Clear(); return kDeclined; }
    void* handle = PyLong_AsVoidPtr(stream);
    Py_DECREF(stream);
    if (handle == nullptr && PyErr_Occurred()) { PyErr_Clear(); return kDeclined; }
    const void* in = c.rgb->data_ptr();
    void* out = c.out->data_ptr();
    const harris_layout* layout = c.dense ? nullptr : &c.layout;
    int status;
    Py_BEGIN_ALLOW_THREADS
    if (c.out_dtype == HARRIS_OUT_U8)
        status = call_quantized(in, c.dtype, c.batch, c.H, c.W, layout, c.k, c.scale, c.window, c.q_scale, c.q_offset, static_cast<uint8_t*>(out), nullptr, handle);
    else
        status = call_typed(in, c.dtype, c.batch, c.H, c.W, layout, c.k, c.scale, c.window, out, c.out_dtype, nullptr, handle);
    Py_END_ALLOW_THREADS
    if (status == HARRIS_OK) return kDone;
    PyObject* code = PyLong_FromLong(status);
    if (code == nullptr) return kRaised;
    Py_XDECREF(PyObject_CallOneArg(raise_status, code));
    Py_DECREF(code);
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "the library's status was not raised");
    return kRaised;
}

bool ready() { return call_typed != nullptr && !at::impl::torch_function_mode_enabled() && !c10::impl::TorchDispatchModeTLS::any_modes_set(); }

// A new result for a call.  The interpreter's lock is let go of meanwhile, as torch.empty does: the allocator may have to
// ask the runtime for memory, or to wait for the GPU.
at::Tensor new_result(const Call& c) {
    struct Unlocked {
        PyThreadState* state = PyEval_SaveThread();
        ~Unlocked() { PyEval_RestoreThread(state); }
    };
    const auto options = c.rgb->options().dtype(at::kFloat).requires_grad(false);
    const Unlocked unlocked;
    return at::empty({c.batch, c.H - 4, c.W - 4}, options);
}

// dense(rgb, out or None, k, sobel_scale, window, dtype of rgb or -1 for either) -> out or None
PyObject* dense(PyObject*, PyObject* const* a, Py_ssize_t n) {
    try {
        Call c{};
        int dtype = 0;
        if (n != 6 || !ready() || !number(a[2], c.k) || !number(a[3], c.scale) || !whole(a[4], c.window) || !whole(a[5], dtype)) Py_RETURN_NONE;
        c.rgb = plain_tensor(a[0]);
        if (c.rgb == nullptr || !image(c) || (dtype >= 0 && dtype != c.dtype) || !c.rgb->is_contiguous()) Py_RETURN_NONE;
        c.dense = true;
        c.out_dtype = HARRIS_OUT_F32;
        at::Tensor made;
        struct Owned {
            PyObject* object = nullptr;
            ~Owned() { Py_XDECREF(object); }
        } returned;                             // made before the call: nothing that could fail comes after it
        if (a[1] == Py_None) {
            made = new_result(c);
            c.out = &made;
            if (!made.has_storage()) Py_RETURN_NONE;
            returned.object = THPVariable_Wrap(made);
            if (returned.object == nullptr) { PyErr_Clear(); Py_RETURN_NONE; }
        } else {
            c.out = plain_tensor(a[1]);
            if (c.out == nullptr || c.out->scalar_type() != at::kFloat || !result(c) || !c.out->is_contiguous()) Py_RETURN_NONE;
            returned.object = Py_NewRef(a[1]);
        }
        const Outcome outcome = enqueue(c);
        if (outcome == kRaised) return nullptr;
        if (outcome == kDeclined) Py_RETURN_NONE;
        return std::exchange(returned.object, nullptr);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// views(rgb, out, k, sobel_scale, window, kinds, q_scale, q_offset) -> out or None.  kinds: 0 float32 results, 1 float32
// and 16-bit, 2 8-bit codes.
PyObject* views(PyObject*, PyObject* const* a, Py_ssize_t n) {
    try {
        Call c{};
        int kinds = 0;
        if (n != 8 || !ready() || !number(a[2], c.k) || !number(a[3], c.scale) || !whole(a[4], c.window) || !whole(a[5], kinds) || !number(a[6], c.q_scale) || !number(a[7], c.q_offset)) Py_RETURN_NONE;
        c.rgb = plain_tensor(a[0]);
        c.out = plain_tensor(a[1]);
        if (c.rgb == nullptr || c.out == nullptr || !image(c) || !result(c)) Py_RETURN_NONE;
        const auto type = c.out->scalar_type();
        if (kinds == 2 && type == at::kByte) c.out_dtype = HARRIS_OUT_U8;
        else if (kinds <= 1 && type == at::kFloat) c.out_dtype = HARRIS_OUT_F32;
        else if (kinds == 1 && type == at::kHalf) c.out_dtype = HARRIS_OUT_F16;
        else if (kinds == 1 && type == at::kBFloat16) c.out_dtype = HARRIS_OUT_BF16;
        else Py_RETURN_NONE;
        if (!strided(c)) Py_RETURN_NONE;
        const Outcome outcome = enqueue(c);
        if (outcome == kRaised) return nullptr;
        if (outcome == kDeclined) Py_RETURN_NONE;
        Py_INCREF(a[1]);
        return a[1];
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// bind(address of harris_coarsity_typed, of harris_coarsity_quantized, current-device function, current-stream function,
// function that raises the error of a status)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 5) { PyErr_SetString(PyExc_TypeError, "bind takes five arguments"); return nullptr; }
    void *typed = PyLong_AsVoidPtr(a[0]), *quantized = PyLong_AsVoidPtr(a[1]);
    if (PyErr_Occurred()) return nullptr;
    Py_INCREF(a[2]);
    Py_INCREF(a[3]);
    Py_INCREF(a[4]);
    Py_XDECREF(get_device);
    Py_XDECREF(get_stream);
    Py_XDECREF(raise_status);
    get_device = a[2];
    get_stream = a[3];
    raise_status = a[4];
    call_quantized = reinterpret_cast<quantized_fn>(quantized);
    call_typed = reinterpret_cast<typed_fn>(typed);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"dense", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(dense)), METH_FASTCALL, nullptr},
                         {"views", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(views)), METH_FASTCALL, nullptr},
                         {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(bind)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_harris_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// torch_version: the torch whose headers are compiled in; the binding uses the module with no other.
PyMODINIT_FUNC PyInit__harris_call() {
    PyObject* m = PyModule_Create(&module);
    if (m != nullptr && PyModule_AddStringConstant(m, "torch_version", HARRIS_TORCH_VERSION) != 0) { Py_DECREF(m); return nullptr; }
    return m;
}
