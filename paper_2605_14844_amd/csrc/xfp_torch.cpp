// The decode calls of the Python binding: tensors and a descriptor in, one call of the C ABI, the output tensor back.
//
// Why this is native: a decode step is hundreds of calls of a few microseconds each, and a call marshalled in Python
// (ctypes, torch.empty, torch.cuda.current_stream: 8.1 us with an output given, 9.9 us without) takes longer on the
// host than most of these kernels run (512 x 1024: 2.5 us, 8192 x 4096: 6.2 us), so the GPU waits for the host.  What
// is left here is the launch itself (about 2.4 us in the HIP runtime) and the allocation of the output.
//
// Marshalling only: no arithmetic, no state beyond the addresses of the loaded library's entry points.  The rules
// (which stride is passed when, what is shared between slots) are those of the binding's documentation.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/xfp.h"

namespace {

decltype(&xfp_gemv) g_gemv;
decltype(&xfp_gemv_noalloc) g_gemv_noalloc;
decltype(&xfp_gemv_moe) g_moe;
decltype(&xfp_gemv_moe_silu_mul) g_silu;
decltype(&xfp_gemv_moe_combine) g_combine;
PyObject *g_descriptor; // the ctypes structure of the descriptor
PyObject *g_error;      // callable(status[, text]) that raises XfpError

struct Failed {};       // a Python exception is set

// An XfpError for a status of the library, or for an argument this file refuses (then with a text of its own).
[[noreturn]] void fail(int status, const char *text = nullptr)
{
    PyObject *r = text ? PyObject_CallFunction(g_error, "is", status, text) : PyObject_CallFunction(g_error, "i", status);
    Py_XDECREF(r);      // the callable raises
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "xfp call failed");
    throw Failed{};
}

// The host descriptor inside a ctypes structure; valid while the view is held.
struct Descriptor {
    Py_buffer view{};
    explicit Descriptor(PyObject *o)
    {
        const int is = PyObject_IsInstance(o, g_descriptor);       // any other buffer of this length holds no addresses
        if (is == 0) PyErr_Format(PyExc_TypeError, "expected an xfp_weights descriptor, got %s", Py_TYPE(o)->tp_name);
        if (is != 1 || PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Failed{};
    }
    ~Descriptor() { PyBuffer_Release(&view); }
    Descriptor(const Descriptor &) = delete;
    Descriptor &operator=(const Descriptor &) = delete;
    const xfp_weights *operator->() const { return static_cast<const xfp_weights *>(view.buf); }
    const xfp_weights *get() const { return static_cast<const xfp_weights *>(view.buf); }
};

const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "expected a torch.Tensor, got %s", Py_TYPE(o)->tp_name);
        throw Failed{};
    }
    return THPVariable_Unpack(o);
}

// A device pointer; NULL for a tensor without elements (data_ptr of a view of nothing may be anything).
void *ptr(const at::Tensor &t) { return t.numel() ? t.data_ptr() : nullptr; }

int y_code(at::ScalarType y, at::ScalarType x)
{
    int flag = 0;
    if (x == at::kBFloat16) flag = XFP_X_BF16;
    else if (x != at::kHalf) fail(XFP_ERR_UNSUPPORTED, "x dtype must be torch.float16 or torch.bfloat16");
    switch (y) {
    case at::kHalf: return XFP_F16 | flag;
    case at::kFloat: return XFP_F32 | flag;
    case at::kBFloat16: return XFP_BF16 | flag;
    default: fail(XFP_ERR_UNSUPPORTED, "y dtype must be torch.float16, torch.bfloat16 or torch.float32");
    }
}

void *stream_of(PyObject *o)
{
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    PyObject *v = PyObject_GetAttrString(o, "cuda_stream");        // a torch.cuda.Stream
    if (!v) {
        PyErr_Clear();
        v = PyNumber_Long(o);                                      // a raw hipStream_t
        if (!v) throw Failed{};
    }
    void *p = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (!p && PyErr_Occurred()) throw Failed{};
    return p;
}

// The output: the caller's tensor, or a new one (dtype None: torch's default dtype).
at::Tensor output(PyObject *y, PyObject *dtype, at::IntArrayRef shape, const at::Tensor &x)
{
    if (y != Py_None) return tensor(y);
    at::TensorOptions options = at::TensorOptions().device(x.device());
    if (dtype != Py_None) {
        if (!THPDtype_Check(dtype)) {
            PyErr_SetString(PyExc_TypeError, "the output dtype must be a torch.dtype");
            throw Failed{};
        }
        options = options.dtype(reinterpret_cast<THPDtype *>(dtype)->scalar_type);
    }
    return at::empty(shape, options);
}

// what goes back: the caller's own object where there was one
PyObject *result(PyObject *y, at::Tensor &&t)
{
    if (y != Py_None) return Py_NewRef(y);
    return THPVariable_Wrap(std::move(t));
}

template <typename F>
void call(F &&f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    if (rc != XFP_OK) fail(rc);
}

bool arity(Py_ssize_t got, Py_ssize_t want)
{
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, got);
    return false;
}

// gemv(desc, x, y, y_dtype, stream), noalloc(desc, x, y, y_dtype, stream)
template <bool NOALLOC>
PyObject *py_gemv(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (!arity(n, 5)) return nullptr;
    try {
        Descriptor W(a[0]);
        const at::Tensor &x = tensor(a[1]);
        // what is not a matrix is the one row of a matrix: [K] is [1, K] (more dimensions: a row the library refuses as too short)
        const bool flat = x.dim() != 2;
        const int64_t M = flat ? 1 : x.size(0), cols = flat ? x.size(0) : x.size(1);
        at::Tensor y = NOALLOC ? tensor(a[2]) : output(a[2], a[3], {M, (int64_t)W->N}, x);
        const bool yflat = y.dim() != 2;
        const int64_t ldx = M > 1 ? x.stride(0) : std::max<int64_t>(cols, 1);
        const int64_t ycols = yflat ? y.size(0) : y.size(1);
        const int64_t ldy = M <= 1 ? std::max<int64_t>(ycols, 1) : yflat ? y.size(0) * y.stride(0) : y.stride(0);
        const int code = y_code(y.scalar_type(), x.scalar_type());
        void *s = stream_of(a[4]), *xp = ptr(x), *yp = ptr(y);
        call([&] { return (NOALLOC ? g_gemv_noalloc : g_gemv)(W.get(), xp, (int)M, ldx, yp, code, ldy, s); });
        return result(a[2], std::move(y));
    } catch (const Failed &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// x of the slot forms: [K] or [1, K] is shared by all slots (stride 0), else a row per slot
int64_t slot_stride(const at::Tensor &x, int64_t T) { return x.dim() == 1 || (x.size(0) == 1 && T != 1) ? 0 : x.stride(0); }

// moe(desc, expert_ids, x, y, y_dtype, stream)
PyObject *py_moe(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (!arity(n, 6)) return nullptr;
    try {
        Descriptor W(a[0]);
        const at::Tensor &ids = tensor(a[1]), &x = tensor(a[2]);
        const int64_t T = ids.numel(), xs = slot_stride(x, T);
        at::Tensor y = output(a[3], a[4], {T, (int64_t)W->N}, x);
        const int64_t ldy = y.dim() == 2 && T > 1 ? y.stride(0) : (int64_t)W->N;
        const int code = y_code(y.scalar_type(), x.scalar_type());
        void *s = stream_of(a[5]), *ip = ptr(ids), *xp = ptr(x), *yp = T ? ptr(y) : y.data_ptr();
        call([&] { return g_moe(W.get(), static_cast<const int32_t *>(ip), (int)T, xp, xs, yp, code, ldy, s); });
        return result(a[3], std::move(y));
    } catch (const Failed &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// silu(desc, expert_ids or None, x, h, h_dtype, stream)
PyObject *py_silu(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (!arity(n, 6)) return nullptr;
    try {
        Descriptor W(a[0]);
        const at::Tensor &x = tensor(a[2]);
        const at::Tensor *ids = a[1] == Py_None ? nullptr : &tensor(a[1]);
        const int64_t T = ids ? ids->numel() : x.dim() == 1 ? 1 : x.size(0), xs = slot_stride(x, T);
        const int64_t half = (int64_t)(W->N / 2);
        at::Tensor h = output(a[3], a[4], {T, half}, x);
        const int64_t ldh = h.dim() == 2 && T > 1 ? h.stride(0) : half;
        const int code = y_code(h.scalar_type(), x.scalar_type());
        void *s = stream_of(a[5]), *ip = ids ? ptr(*ids) : nullptr, *xp = ptr(x), *hp = T ? ptr(h) : h.data_ptr();
        call([&] { return g_silu(W.get(), static_cast<const int32_t *>(ip), (int)T, xp, xs, hp, code, ldh, s); });
        return result(a[3], std::move(h));
    } catch (const Failed &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// combine(desc, expert_ids, x, slot_weights, y, y_dtype, stream)
PyObject *py_combine(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (!arity(n, 7)) return nullptr;
    try {
        Descriptor W(a[0]);
        const at::Tensor &ids = tensor(a[1]), &x = tensor(a[2]), &w = tensor(a[3]);
        const int64_t T = ids.numel(), xs = slot_stride(x, T);
        if (w.scalar_type() != at::kFloat || w.numel() != T) {
            PyErr_SetString(PyExc_AssertionError, "slot_weights: fp32, one per slot");
            return nullptr;
        }
        at::Tensor y = output(a[4], a[5], {(int64_t)W->N}, x);
        const int code = y_code(y.scalar_type(), x.scalar_type());
        void *s = stream_of(a[6]), *ip = ptr(ids), *xp = ptr(x), *wp = ptr(w), *yp = ptr(y);
        call([&] {
            return g_combine(W.get(), static_cast<const int32_t *>(ip), (int)T, xp, xs, static_cast<const float *>(wp), yp, code, s);
        });
        return result(a[4], std::move(y));
    } catch (const Failed &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// y_code(dtype, x or None): the dtype argument a call would pass
PyObject *py_y_code(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (!arity(n, 2)) return nullptr;
    try {
        if (!THPDtype_Check(a[0])) {
            PyErr_SetString(PyExc_TypeError, "the output dtype must be a torch.dtype");
            return nullptr;
        }
        const at::ScalarType x = a[1] == Py_None ? at::kHalf : tensor(a[1]).scalar_type();
        return PyLong_FromLong(y_code(reinterpret_cast<THPDtype *>(a[0])->scalar_type, x));
    } catch (const Failed &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// bind(addresses of gemv, noalloc, moe, silu_mul, combine; the descriptor's type; callable that raises)
PyObject *py_bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (!arity(n, 7)) return nullptr;
    void *p[5];
    for (int i = 0; i < 5; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a null entry point");
            return nullptr;
        }
    }
    g_gemv = reinterpret_cast<decltype(g_gemv)>(p[0]);
    g_gemv_noalloc = reinterpret_cast<decltype(g_gemv_noalloc)>(p[1]);
    g_moe = reinterpret_cast<decltype(g_moe)>(p[2]);
    g_silu = reinterpret_cast<decltype(g_silu)>(p[3]);
    g_combine = reinterpret_cast<decltype(g_combine)>(p[4]);
    Py_XSETREF(g_descriptor, Py_NewRef(a[5]));
    Py_XSETREF(g_error, Py_NewRef(a[6]));
    Py_RETURN_NONE;
}

#define XFP_FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL
PyMethodDef methods[] = {
    {"bind", XFP_FAST(py_bind), "addresses of the library's entry points, the descriptor's type and the callable that raises"},
    {"gemv", XFP_FAST(py_gemv<false>), "(desc, x, y, y_dtype, stream)"},
    {"noalloc", XFP_FAST(py_gemv<true>), "(desc, x, y, y_dtype, stream)"},
    {"moe", XFP_FAST(py_moe), "(desc, expert_ids, x, y, y_dtype, stream)"},
    {"silu", XFP_FAST(py_silu), "(desc, expert_ids, x, h, h_dtype, stream)"},
    {"combine", XFP_FAST(py_combine), "(desc, expert_ids, x, slot_weights, y, y_dtype, stream)"},
    {"y_code", XFP_FAST(py_y_code), "(dtype, x or None)"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_xfp_torch", "native marshalling of the decode calls", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__xfp_torch(void) { return PyModule_Create(&module); }
