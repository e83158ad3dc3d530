/*
 * paper_2110_15362_amd/_call.so: the calls of libbittrain on torch tensors, for bittrain.py.
 *
 * What a small call costs is the host's work, not the GPU's: the three calls of a training step on one image's
 * layer (fp32, 200,704 elements) keep the GPU busy for 10 us, and checking the tensors and marshalling the arguments with
 * ctypes took 5 to 6 us a call on top of the launch's 2.4.  There are two ways in here, with the same checks in the same order:
 *   plain   all tensors are torch.Tensor or Parameter themselves, dense on a device, and no torch function mode is on: what
 *           the checks need is read from the tensor object through torch's C++ interface (0.2 us a call);
 *   any     else: the attributes of the tensors are read as any Python caller would read them (1.1 to 1.5 us a call), so
 *           subclasses, wrappers and modes see what they have always seen.  Whatever is wrong with a tensor is
 *           reported from here.
 * The library itself is loaded by bittrain.py, which hands over the addresses of the calls (bind), once it has compared the torch
 * that this file was compiled with (torch_version) to the one that is there.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include <chrono>

#include <ATen/Functions.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "bittrain.h"

static struct {
    bt_status (*compress)(const void *, uint64_t, bt_dtype, uint32_t *, void *, uint64_t, uint64_t *, void *, size_t, bt_stream);
    bt_status (*compress_static)(const void *, uint64_t, bt_dtype, uint32_t *, void *, uint64_t, uint64_t *, bt_stream);
    bt_status (*compress_pruned)(const void *, uint64_t, bt_dtype, double, uint32_t *, void *, uint64_t, uint64_t *, void *, size_t,
                                 bt_stream);
    bt_status (*activation_compress)(const void *, uint64_t, bt_dtype, double, void *, uint32_t *, void *, uint64_t, uint64_t *, void *,
                                     size_t, bt_stream);
    bt_status (*compress_indexed)(const void *, uint64_t, bt_dtype, uint32_t *, void *, uint64_t, uint64_t *, uint64_t *, void *, size_t,
                                  bt_stream);
    bt_status (*decompress)(const uint32_t *, const void *, uint64_t, bt_dtype, void *, void *, size_t, bt_stream);
    bt_status (*decompress_indexed)(const uint32_t *, const void *, uint64_t, const uint64_t *, uint64_t, bt_dtype, void *, bt_stream);
    bt_status (*relu_backward)(const uint32_t *, const void *, uint64_t, bt_dtype, void *, bt_stream);
    bt_status (*mask_apply)(const uint32_t *, const void *, uint64_t, bt_dtype, void *, bt_stream);
    bt_status (*relu_forward)(const void *, uint64_t, bt_dtype, void *, uint32_t *, bt_stream);
    size_t (*index_bytes)(uint64_t, bt_dtype);
    size_t (*compressed_size)(uint64_t, uint64_t, bt_dtype);
} lib;

/* Python objects handed over by bind: {dtype: code}, the function that refuses other dtypes, the error class, the
 * function that turns a stream argument into a handle; and whether this torch has devices. */
static PyObject *dtypes, *dtype_code, *error_class, *stream_handle;
static bool has_device;
static PyObject *s_is_cuda, *s_is_contiguous, *s_dtype, *s_numel, *s_element_size, *s_data_ptr;

/* A device pointer, of whatever type a call takes. */
struct address {
    void *p;
    template <class T> operator T *() const { return static_cast<T *>(p); }
};

typedef struct {
    PyObject *t;        /* borrowed */
    const void *dtype;  /* which object it is, to compare: dtypes are singletons */
    int code;           /* bt_dtype, or -1 */
    uint64_t numel, width;
    address ptr;
} tensor;

static int is_true(PyObject *o) {      /* takes the reference; -1: an error is set */
    if (o == NULL) return -1;
    const int r = PyObject_IsTrue(o);
    Py_DECREF(o);
    return r;
}

static int to_u64(PyObject *o, uint64_t *v) {
    if (o == NULL) return -1;
    *v = PyLong_AsUnsignedLongLong(o);
    Py_DECREF(o);
    return *v == (uint64_t)-1 && PyErr_Occurred() ? -1 : 0;
}

/* The tensor lives in device memory and is contiguous: the first thing that is checked of every argument. */
static int on_device(tensor *a, PyObject *t, const char *name) {
    a->t = t;
    int ok = is_true(PyObject_GetAttr(t, s_is_cuda));
    if (ok < 0) return -1;
    if (!ok) {
        PyErr_Format(PyExc_ValueError, "%s must live in device memory", name);
        return -1;
    }
    ok = is_true(PyObject_CallMethodNoArgs(t, s_is_contiguous));
    if (ok < 0) return -1;
    if (!ok) {
        PyErr_Format(PyExc_ValueError, "%s must be contiguous", name);
        return -1;
    }
    return 0;
}

/* What the checks and the call need of it. */
static int describe(tensor *a) {
    PyObject *const dtype = PyObject_GetAttr(a->t, s_dtype);
    if (dtype == NULL) return -1;
    PyObject *const code = PyDict_GetItemWithError(dtypes, dtype);      /* borrowed */
    a->dtype = dtype;
    a->code = code != NULL ? (int)PyLong_AsLong(code) : -1;
    Py_DECREF(dtype);
    if (PyErr_Occurred()) return -1;
    uint64_t p;
    if (to_u64(PyObject_CallMethodNoArgs(a->t, s_numel), &a->numel) != 0 ||
        to_u64(PyObject_CallMethodNoArgs(a->t, s_element_size), &a->width) != 0 ||
        to_u64(PyObject_CallMethodNoArgs(a->t, s_data_ptr), &p) != 0)
        return -1;
    a->ptr.p = (void *)(uintptr_t)p;
    return 0;
}

/* The plain way: what `describe` reads, without Python; false if there is anything about the tensor that the other way has to
 * look at.  (The dispatch keys of an ordinary dense tensor on a device, and nothing else: no subclass, wrapper, lazy or
 * conjugate view.) */
static bool plain(tensor *a, PyObject *o) {
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined()) return false;
    static const c10::DispatchKeySet ordinary = c10::DispatchKeySet(c10::DispatchKey::CUDA) | c10::DispatchKeySet(c10::DispatchKey::AutogradCUDA) |
                                                c10::DispatchKeySet(c10::DispatchKey::AutocastCUDA) | c10::DispatchKeySet(c10::DispatchKey::ADInplaceOrView);
    if ((t.key_set() | ordinary) != ordinary || !t.is_cuda() || !t.is_contiguous()) return false;
    const at::ScalarType type = t.scalar_type();
    a->t = o;
    a->dtype = reinterpret_cast<const void *>(static_cast<uintptr_t>(type) + 1);      /* compared among plain tensors only */
    a->code = type == at::kFloat ? BT_F32 : type == at::kHalf ? BT_F16 : type == at::kBFloat16 ? BT_BF16 : type == at::kDouble ? BT_F64 : -1;
    a->numel = static_cast<uint64_t>(t.numel());
    a->width = t.element_size();
    a->ptr.p = t.data_ptr();
    return true;
}

static bool all_plain(tensor *a, PyObject *const *args, const int count) {
    try {
        if (at::impl::torch_function_mode_enabled()) return false;
        for (int i = 0; i < count; ++i)
            if (!plain(&a[i], args[i])) return false;
        return true;
    } catch (...) {
        return false;      /* the other way reports it */
    }
}

static int take(tensor *a, PyObject *const *args, const char *const *names, const int count) {
    if (all_plain(a, args, count)) return 0;
    for (int i = 0; i < count; ++i)
        if (on_device(&a[i], args[i], names[i]) != 0) return -1;
    for (int i = 0; i < count; ++i)
        if (describe(&a[i]) != 0) return -1;
    return 0;
}

static int fail(PyObject *type, const char *text) {
    PyErr_SetString(type, text);
    return -1;
}

static int check_bitmap(const tensor *bitmap, const uint64_t n) {
    if (bitmap->width != 4 || bitmap->numel * 4 < 4 * ((n + 31) / 32)) return fail(PyExc_ValueError, "bitmap must hold ceil(n/32) 32-bit words");
    return 0;
}

static int check_nnz(const tensor *nnz) {
    if (nnz->width != 8 || nnz->numel < 1) return fail(PyExc_ValueError, "nnz must be one 64-bit integer");
    return 0;
}

static int code_of(const tensor *a, bt_dtype *code) {
    if (a->code < 0) {
        PyObject *const dtype = PyObject_GetAttr(a->t, s_dtype);
        if (dtype != NULL) {
            Py_XDECREF(PyObject_CallOneArg(dtype_code, dtype));      /* raises */
            Py_DECREF(dtype);
        }
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "dtype");
        return -1;
    }
    *code = (bt_dtype)a->code;
    return 0;
}

static int check_index(const tensor *index, const tensor *x) {
    bt_dtype code = BT_F32;
    if (index->width == 8 && code_of(x, &code) != 0) return -1;
    if (index->width != 8 || index->numel * 8 < lib.index_bytes(x->numel, code))
        return fail(PyExc_ValueError, "index must hold one 64-bit integer per tile");
    return 0;
}

/* The stream argument as a handle; None: the current stream of the current device. */
static int stream_of(PyObject *o, bt_stream *stream) {
    uint64_t v;
    if (o == Py_None && has_device) {
        try {
            *stream = (bt_stream)c10::hip::getCurrentHIPStream().stream();
            return 0;
        } catch (const std::exception &e) {
            PyErr_SetString(PyExc_RuntimeError, e.what());
            return -1;
        }
    }
    if (to_u64(PyObject_CallOneArg(stream_handle, o), &v) != 0) return -1;
    *stream = (bt_stream)(uintptr_t)v;
    return 0;
}

static PyObject *done(const char *call, const bt_status st) {
    if (st == BT_OK) Py_RETURN_NONE;
    PyObject *e = PyObject_CallFunction(error_class, "si", call, (int)st);
    if (e != NULL) {
        PyErr_SetObject(error_class, e);
        Py_DECREF(e);
    }
    return NULL;
}

static int expect(const Py_ssize_t got, const Py_ssize_t want) {
    if (lib.compress == NULL) return fail(PyExc_RuntimeError, "the library is not loaded");
    return got == want ? 0 : fail(PyExc_TypeError, "wrong number of arguments");
}

#define CALL(name, expression)              \
    do {                                    \
        bt_status st;                       \
        Py_BEGIN_ALLOW_THREADS              \
        st = (expression);                  \
        Py_END_ALLOW_THREADS                \
        return done(name, st);              \
    } while (0)

/* (x, bitmap, values, nnz, workspace, stream) */
static PyObject *py_compress(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    (void)self;
    static const char *const names[] = {"x", "bitmap", "values", "nnz", "workspace"};
    tensor a[5];
    bt_dtype code = BT_F32;
    bt_stream stream = NULL;
    if (expect(nargs, 6) != 0 || take(a, args, names, 5) != 0) return NULL;
    if (a[2].dtype != a[0].dtype) return fail(PyExc_TypeError, "values must have the dtype of x"), nullptr;
    if (check_bitmap(&a[1], a[0].numel) != 0 || check_nnz(&a[3]) != 0 || code_of(&a[0], &code) != 0 || stream_of(args[5], &stream) != 0)
        return NULL;
    CALL("bt_compress", lib.compress(a[0].ptr, a[0].numel, code, a[1].ptr, a[2].ptr, a[2].numel, a[3].ptr, a[4].ptr,
                                     a[4].numel * a[4].width, stream));
}

/* (x, bitmap, values, nnz, stream) */
static PyObject *py_compress_static(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    (void)self;
    static const char *const names[] = {"x", "bitmap", "values", "nnz"};
    tensor a[4];
    bt_dtype code = BT_F32;
    bt_stream stream = NULL;
    if (expect(nargs, 5) != 0 || take(a, args, names, 4) != 0) return NULL;
    if (a[2].dtype != a[0].dtype) return fail(PyExc_TypeError, "values must have the dtype of x"), nullptr;
    if (check_bitmap(&a[1], a[0].numel) != 0 || check_nnz(&a[3]) != 0 || code_of(&a[0], &code) != 0 || stream_of(args[4], &stream) != 0)
        return NULL;
    CALL("bt_compress_static", lib.compress_static(a[0].ptr, a[0].numel, code, a[1].ptr, a[2].ptr, a[2].numel, a[3].ptr, stream));
}

/* (x, bitmap, values, nnz, workspace, threshold, stream) */
static PyObject *py_compress_pruned(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    (void)self;
    static const char *const names[] = {"x", "bitmap", "values", "nnz", "workspace"};
    tensor a[5];
    bt_dtype code = BT_F32;
    bt_stream stream = NULL;
    if (expect(nargs, 7) != 0 || take(a, args, names, 5) != 0) return NULL;
    if (a[2].dtype != a[0].dtype) return fail(PyExc_TypeError, "values must have the dtype of x"), nullptr;
    if (check_bitmap(&a[1], a[0].numel) != 0 || check_nnz(&a[3]) != 0 || code_of(&a[0], &code) != 0) return NULL;
    const double threshold = PyFloat_AsDouble(args[5]);
    if ((threshold == -1.0 && PyErr_Occurred()) || stream_of(args[6], &stream) != 0) return NULL;
    CALL("bt_compress_pruned", lib.compress_pruned(a[0].ptr, a[0].numel, code, threshold, a[1].ptr, a[2].ptr, a[2].numel, a[3].ptr,
                                                   a[4].ptr, a[4].numel * a[4].width, stream));
}

/* (x, dense_out, bitmap, values, nnz, workspace, threshold, stream) */
static PyObject *py_activation_compress(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    (void)self;
    static const char *const names[] = {"x", "dense_out", "bitmap", "values", "nnz", "workspace"};
    tensor a[6];
    bt_dtype code = BT_F32;
    bt_stream stream = NULL;
    if (expect(nargs, 8) != 0 || take(a, args, names, 6) != 0) return NULL;
    if (a[3].dtype != a[0].dtype || a[1].dtype != a[0].dtype || a[1].numel != a[0].numel)
        return fail(PyExc_TypeError, "values and dense_out must match x"), nullptr;
    if (check_bitmap(&a[2], a[0].numel) != 0 || check_nnz(&a[4]) != 0 || code_of(&a[0], &code) != 0) return NULL;
    const double threshold = PyFloat_AsDouble(args[6]);
    if ((threshold == -1.0 && PyErr_Occurred()) || stream_of(args[7], &stream) != 0) return NULL;
    CALL("bt_activation_compress", lib.activation_compress(a[0].ptr, a[0].numel, code, threshold, a[1].ptr, a[2].ptr, a[3].ptr, a[3].numel,
                                                           a[4].ptr, a[5].ptr, a[5].numel * a[5].width, stream));
}

/* (x, bitmap, values, nnz, index, workspace, stream) */
static PyObject *py_compress_indexed(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    (void)self;
    static const char *const names[] = {"x", "bitmap", "values", "nnz", "index", "workspace"};
    tensor a[6];
    bt_dtype code = BT_F32;
    bt_stream stream = NULL;
    if (expect(nargs, 7) != 0 || take(a, args, names, 6) != 0) return NULL;
    if (a[2].dtype != a[0].dtype) return fail(PyExc_TypeError, "values must have the dtype of x"), nullptr;
    if (check_bitmap(&a[1], a[0].numel) != 0 || check_nnz(&a[3]) != 0 || check_index(&a[4], &a[0]) != 0 ||
        code_of(&a[0], &code) != 0 || stream_of(args[6], &stream) != 0)
        return NULL;
    CALL("bt_compress_indexed", lib.compress_indexed(a[0].ptr, a[0].numel, code, a[1].ptr, a[2].ptr, a[2].numel, a[3].ptr, a[4].ptr,
                                                     a[5].ptr, a[5].numel * a[5].width, stream));
}

/* (bitmap, values, out, workspace, stream) */
static PyObject *py_decompress(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    (void)self;
    static const char *const names[] = {"bitmap", "values", "out", "workspace"};
    tensor a[4];
    bt_dtype code = BT_F32;
    bt_stream stream = NULL;
    if (expect(nargs, 5) != 0 || take(a, args, names, 4) != 0) return NULL;
    if (a[1].dtype != a[2].dtype) return fail(PyExc_TypeError, "values must have the dtype of out"), nullptr;
    if (check_bitmap(&a[0], a[2].numel) != 0 || code_of(&a[2], &code) != 0 || stream_of(args[4], &stream) != 0) return NULL;
    CALL("bt_decompress", lib.decompress(a[0].ptr, a[1].ptr, a[2].numel, code, a[2].ptr, a[3].ptr, a[3].numel * a[3].width, stream));
}

/* (bitmap, values, index, out, stream) */
static PyObject *py_decompress_indexed(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    (void)self;
    static const char *const names[] = {"bitmap", "values", "index", "out"};
    tensor a[4];
    bt_dtype code = BT_F32;
    bt_stream stream = NULL;
    if (expect(nargs, 5) != 0 || take(a, args, names, 4) != 0) return NULL;
    if (a[1].dtype != a[3].dtype) return fail(PyExc_TypeError, "values must have the dtype of out"), nullptr;
    if (check_bitmap(&a[0], a[3].numel) != 0 || check_index(&a[2], &a[3]) != 0 || code_of(&a[3], &code) != 0 ||
        stream_of(args[4], &stream) != 0)
        return NULL;
    CALL("bt_decompress_indexed", lib.decompress_indexed(a[0].ptr, a[1].ptr, a[1].numel, a[2].ptr, a[3].numel, code, a[3].ptr, stream));
}

/* (bitmap, grad_out, grad_in, stream) */
static PyObject *py_relu_backward(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    (void)self;
    static const char *const names[] = {"bitmap", "grad_out", "grad_in"};
    tensor a[3];
    bt_dtype code = BT_F32;
    bt_stream stream = NULL;
    if (expect(nargs, 4) != 0 || take(a, args, names, 3) != 0) return NULL;
    if (a[2].dtype != a[1].dtype || a[2].numel != a[1].numel) return fail(PyExc_TypeError, "grad_in must match grad_out"), nullptr;
    if (check_bitmap(&a[0], a[1].numel) != 0 || code_of(&a[1], &code) != 0 || stream_of(args[3], &stream) != 0) return NULL;
    CALL("bt_relu_backward_from_bitmap", lib.relu_backward(a[0].ptr, a[1].ptr, a[1].numel, code, a[2].ptr, stream));
}

/* (bitmap, x, out, stream) */
static PyObject *py_mask_apply(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    (void)self;
    static const char *const names[] = {"bitmap", "x", "out"};
    tensor a[3];
    bt_dtype code = BT_F32;
    bt_stream stream = NULL;
    if (expect(nargs, 4) != 0 || take(a, args, names, 3) != 0) return NULL;
    if (a[2].dtype != a[1].dtype || a[2].numel != a[1].numel) return fail(PyExc_TypeError, "out must match x"), nullptr;
    if (check_bitmap(&a[0], a[1].numel) != 0 || code_of(&a[1], &code) != 0 || stream_of(args[3], &stream) != 0) return NULL;
    CALL("bt_mask_apply", lib.mask_apply(a[0].ptr, a[1].ptr, a[1].numel, code, a[2].ptr, stream));
}

/* (x, out, bitmap, stream) */
static PyObject *py_relu_forward(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    (void)self;
    static const char *const names[] = {"x", "out", "bitmap"};
    tensor a[3];
    bt_dtype code = BT_F32;
    bt_stream stream = NULL;
    if (expect(nargs, 4) != 0 || take(a, args, names, 3) != 0) return NULL;
    if (a[1].dtype != a[0].dtype || a[1].numel != a[0].numel) return fail(PyExc_TypeError, "out must match x"), nullptr;
    if (check_bitmap(&a[2], a[0].numel) != 0 || code_of(&a[0], &code) != 0 || stream_of(args[3], &stream) != 0) return NULL;
    CALL("bt_relu_forward", lib.relu_forward(a[0].ptr, a[0].numel, code, a[1].ptr, a[2].ptr, stream));
}

/* ---- steps of autograd.py on plain tensors --------------------------------------------------------
 *
 * What autograd.py does around a call, allocations included, in one go: written in Python, packing took the host 35 us beside the
 * compression, and while it waits for nnz all of that is time in which the GPU has nothing to do.  Each returns None for tensors that are not
 * plain or not on the current device, whose stream the calls go to and the copies must be behind them on; autograd.py then takes the
 * general way, or makes their device the current one.  The GIL is released from the first allocation on. */

static at::TensorOptions like(const at::Tensor &t, const at::ScalarType type) { return at::TensorOptions().dtype(type).device(t.device()); }

static bool all_here(tensor *a, PyObject *const *args, const int count) {
    if (!has_device || !all_plain(a, args, count)) return false;
    const c10::DeviceIndex current = c10::hip::current_device();
    for (int i = 0; i < count; ++i)
        if (THPVariable_Unpack(args[i]).device().index() != current) return false;
    return true;
}

static bool aligned(const tensor *a) { return (reinterpret_cast<uintptr_t>(a->ptr.p) & 15) == 0; }

static PyObject *wrap(const at::Tensor &t) {
    if (t.defined()) return THPVariable_Wrap(t);
    Py_RETURN_NONE;
}

/* What a place holds while nothing is queued that could write to it. */
static const int64_t kNotQueued = -2;

/* The nnz of a compression on `stream`, which replaces the -1 at `word` in pinned memory as soon as it is known, a little before the last
 * values are written.  One that failed leaves the -1 there, which is known when the stream has come past it. */
static int64_t wait_for_nnz(const volatile int64_t *word, const c10::hip::HIPStream &stream) {
    using clock = std::chrono::steady_clock;
    const clock::time_point end = clock::now() + std::chrono::milliseconds(2);      /* a host that waits longer sleeps */
    do {
        for (int i = 0; i < 64; ++i) {
            const int64_t nnz = *word;
            if (nnz != -1) return nnz;
            __builtin_ia32_pause();
        }
    } while (clock::now() < end);
    stream.synchronize();
    return *word;
}

/* (x, scratch, workspace, address of the place, wait?) -> None, or (bitmap, index) of the compression that has been started;
 * or, having waited for it, (bitmap, index, nnz, values cut to size): nnz -1 if it failed, values None if it is not worth keeping.
 * The place holds -1 from when the compression may have been queued: whoever catches an error can tell whether it may still be written to. */
static PyObject *py_pack(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    (void)self;
    tensor a[3];
    uint64_t place;
    if (expect(nargs, 5) != 0) return NULL;
    if (!all_here(a, args, 3) || a[0].code < 0 || !aligned(&a[0])) Py_RETURN_NONE;
    if (a[1].dtype != a[0].dtype || a[1].numel < a[0].numel) return fail(PyExc_TypeError, "scratch must have the dtype of x and room for it"), nullptr;
    Py_INCREF(args[3]);
    if (to_u64(args[3], &place) != 0) return NULL;
    const int wait = PyObject_IsTrue(args[4]);
    if (wait < 0) return NULL;
    const at::Tensor x = THPVariable_Unpack(args[0]), scratch = THPVariable_Unpack(args[1]);
    const bt_dtype code = (bt_dtype)a[0].code;
    at::Tensor bitmap, index, values;
    int64_t nnz = -1;
    bt_status st;
    {
        pybind11::gil_scoped_release no_gil;
        const uint64_t n = a[0].numel;
        bitmap = at::empty({(int64_t)((n + 31) / 32)}, like(x, at::kInt));
        index = at::empty({(int64_t)(lib.index_bytes(n, code) / 8)}, like(x, at::kLong));
        const c10::hip::HIPStream stream = c10::hip::getCurrentHIPStream();
        volatile int64_t *const word = (volatile int64_t *)(uintptr_t)place;
        *word = -1;
        st = lib.compress_indexed(a[0].ptr, n, code, (uint32_t *)bitmap.data_ptr(), a[1].ptr, a[1].numel, (uint64_t *)(uintptr_t)place,
                                  (uint64_t *)index.data_ptr(), a[2].ptr, a[2].numel * a[2].width, (bt_stream)stream.stream());
        if (st != BT_OK && st != BT_ERR_HIP) *word = kNotQueued;      /* refused */
        if (st == BT_OK && wait) {
            nnz = wait_for_nnz(word, stream);
            if (nnz >= 0 && lib.compressed_size(n, (uint64_t)nnz, code) + 8 * (uint64_t)index.numel() < n * a[0].width) values = scratch.narrow(0, 0, nnz).clone();
        }
    }
    if (st != BT_OK) return done("bt_compress_indexed", st);
    if (!wait) return Py_BuildValue("(NN)", wrap(bitmap), wrap(index));
    return Py_BuildValue("(NNLN)", wrap(bitmap), wrap(index), (long long)nnz, wrap(values));
    END_HANDLE_TH_ERRORS
}

/* (bitmap, values, index, shape) -> None or the dense tensor */
static PyObject *py_unpack(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    (void)self;
    tensor a[3];
    if (expect(nargs, 4) != 0) return NULL;
    if (!PyTuple_Check(args[3]) || !all_here(a, args, 3) || a[1].code < 0) Py_RETURN_NONE;
    std::vector<int64_t> shape;
    uint64_t n = 1;
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(args[3]); ++i) {
        shape.push_back(PyLong_AsLongLong(PyTuple_GET_ITEM(args[3], i)));
        if (shape.back() == -1 && PyErr_Occurred()) return NULL;
        n *= (uint64_t)shape.back();
    }
    if (a[0].width != 4 || a[0].numel < (n + 31) / 32 || a[2].width != 8 || a[2].numel * 8 < lib.index_bytes(n, (bt_dtype)a[1].code))
        return fail(PyExc_ValueError, "bitmap and index must be those of a tensor of this shape"), nullptr;
    const at::Tensor values = THPVariable_Unpack(args[1]);
    at::Tensor out;
    bt_status st;
    {
        pybind11::gil_scoped_release no_gil;
        out = at::empty(shape, like(values, values.scalar_type()));
        st = lib.decompress_indexed(a[0].ptr, a[1].ptr, a[1].numel, a[2].ptr, n, (bt_dtype)a[1].code, out.data_ptr(),
                                    (bt_stream)c10::hip::getCurrentHIPStream().stream());
    }
    if (st != BT_OK) return done("bt_decompress_indexed", st);
    return wrap(out);
    END_HANDLE_TH_ERRORS
}

/* (x) -> None or (ReLU(x), its bitmap) */
static PyObject *py_relu(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    (void)self;
    tensor a[1];
    if (expect(nargs, 1) != 0) return NULL;
    if (!all_here(a, args, 1) || a[0].code < 0 || !aligned(&a[0])) Py_RETURN_NONE;
    const at::Tensor x = THPVariable_Unpack(args[0]);
    at::Tensor y, bitmap;
    bt_status st;
    {
        pybind11::gil_scoped_release no_gil;
        bitmap = at::empty({(int64_t)((a[0].numel + 31) / 32)}, like(x, at::kInt));
        y = at::empty_like(x);
        st = lib.relu_forward(a[0].ptr, a[0].numel, (bt_dtype)a[0].code, y.data_ptr(), (uint32_t *)bitmap.data_ptr(),
                              (bt_stream)c10::hip::getCurrentHIPStream().stream());
    }
    if (st != BT_OK) return done("bt_relu_forward", st);
    return Py_BuildValue("(NN)", wrap(y), wrap(bitmap));
    END_HANDLE_TH_ERRORS
}

/* (bitmap, gradient) -> None or the gradient behind the ReLU */
static PyObject *py_relu_gradient(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    (void)self;
    tensor a[2];
    if (expect(nargs, 2) != 0) return NULL;
    if (!all_here(a, args, 2) || a[1].code < 0 || !aligned(&a[1])) Py_RETURN_NONE;
    if (check_bitmap(&a[0], a[1].numel) != 0) return NULL;
    const at::Tensor grad = THPVariable_Unpack(args[1]);
    at::Tensor out;
    bt_status st;
    {
        pybind11::gil_scoped_release no_gil;
        out = at::empty_like(grad);
        st = lib.relu_backward(a[0].ptr, a[1].ptr, a[1].numel, (bt_dtype)a[1].code, out.data_ptr(), (bt_stream)c10::hip::getCurrentHIPStream().stream());
    }
    if (st != BT_OK) return done("bt_relu_backward_from_bitmap", st);
    return wrap(out);
    END_HANDLE_TH_ERRORS
}

/* (addresses of the calls in the order of `lib`, the objects above in their order) */
static PyObject *py_bind(PyObject *self, PyObject *args) {
    (void)self;
    PyObject *addresses, *o[4];
    int devices;
    if (!PyArg_ParseTuple(args, "O!O!OOOp", &PyTuple_Type, &addresses, &PyDict_Type, &o[0], &o[1], &o[2], &o[3], &devices)) return NULL;
    void **const slots = (void **)(void *)&lib;
    enum { kSlots = sizeof(lib) / sizeof(void *) };
    uint64_t at[kSlots];
    if (PyTuple_GET_SIZE(addresses) != kSlots) return fail(PyExc_TypeError, "one address per call"), nullptr;
    for (int i = 0; i < kSlots; ++i) {
        at[i] = PyLong_AsUnsignedLongLong(PyTuple_GET_ITEM(addresses, i));
        if (at[i] == (uint64_t)-1 && PyErr_Occurred()) return NULL;
    }
    for (int i = 0; i < kSlots; ++i) slots[i] = (void *)(uintptr_t)at[i];
    PyObject **const keep[4] = {&dtypes, &dtype_code, &error_class, &stream_handle};
    for (int i = 0; i < 4; ++i) {
        Py_INCREF(o[i]);
        Py_XSETREF(*keep[i], o[i]);
    }
    has_device = devices != 0;
    Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {
    FAST(compress), FAST(compress_static), FAST(compress_pruned), FAST(activation_compress), FAST(compress_indexed),
    FAST(decompress), FAST(decompress_indexed), FAST(relu_backward), FAST(mask_apply), FAST(relu_forward),
    FAST(pack), FAST(unpack), FAST(relu), FAST(relu_gradient),
    {"bind", py_bind, METH_VARARGS, NULL}, {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__call(void) {
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_dtype = PyUnicode_InternFromString("dtype");
    s_numel = PyUnicode_InternFromString("numel");
    s_element_size = PyUnicode_InternFromString("element_size");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    if (!s_is_cuda || !s_is_contiguous || !s_dtype || !s_numel || !s_element_size || !s_data_ptr) return NULL;
    PyObject *const m = PyModule_Create(&module);
    if (m != NULL && PyModule_AddStringConstant(m, "torch_version", BT_TORCH_VERSION) != 0) {
        Py_DECREF(m);
        return NULL;
    }
    return m;
}
