// Argument marshalling of the layer's online calls in native code.  A decode step of a small layer runs for
// 5 to 7 us on the GPU; marshalling it in Python (attribute look-ups, two torch.empty, twenty ctypes conversions)
// took the host about 11 us per call, so that a loop of eager calls was bound by it: 1 x 4096 x 4096 13.9 us a
// call with it, 5.9 us with this.
//
// Every function takes the address of the C entry point (the library is loaded by Python) and returns
//   a tensor or a tuple of tensors   on success,
//   an int                           the entry point's status when it is not W4A8_OK,
//   NotImplemented                   for operands that are not plain torch tensors of the expected kind, and sizes
//                                    that are not 64-bit ints: the caller's Python form decides what to do with them.
// Nothing is cached between calls.  The GIL is released around the entry points, as ctypes does.
#include <torch/extension.h>

#include "../../include/w4a8.h"

namespace {

constexpr int LAYOUT_TILED = W4A8_LAYOUT_TILED;

// an int that fits 64 bits; anything else (floats, strings, array scalars) is the Python form's to convert or refuse
bool to_i64(PyObject *o, int64_t &v)
{
    if (!PyLong_Check(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}
template <typename F>
bool to_fn(PyObject *o, F &f)
{
    f = reinterpret_cast<F>(PyLong_AsVoidPtr(o));
    return !PyErr_Occurred();
}

// plain tensors only (no subclass may observe or replace these calls)
bool plain(PyObject *o) { return THPVariable_CheckExact(o); }
bool plain_or_none(PyObject *o) { return o == Py_None || THPVariable_CheckExact(o); }
void *ptr(PyObject *o) { return o == Py_None ? nullptr : THPVariable_Unpack(o).data_ptr(); }

// element type of activations / outputs: its id, or -1
int dtype_id(at::ScalarType t)
{
    switch (t) {
        case at::kFloat: return W4A8_F32;
        case at::kHalf: return W4A8_F16;
        case at::kBFloat16: return W4A8_BF16;
        default: return -1;
    }
}
at::ScalarType y_type(int64_t id)
{
    return id == W4A8_F16 ? at::kHalf : id == W4A8_BF16 ? at::kBFloat16 : at::kFloat;
}

struct Rows {   // a 2-D activation tensor with contiguous rows
    int64_t M, K, ld;
    int dtype;
    bool ok;
};
Rows rows_of(const at::Tensor &X)
{
    Rows r{0, 0, 0, -1, false};
    if (X.dim() != 2 || X.stride(1) != 1) return r;
    r.M = X.size(0);
    r.K = X.size(1);
    r.ld = r.M > 1 ? X.stride(0) : std::max(X.stride(0), r.K);
    r.dtype = dtype_id(X.scalar_type());
    r.ok = r.dtype >= 0;
    return r;
}

at::Tensor make(const at::Tensor &like, at::IntArrayRef size, at::ScalarType t)
{
    return at::empty(size, like.options().dtype(t));
}

// Scratch of the size that a call would like, or of the size that it has to have where the allocator does not give so much
// (undefined for none).
at::Tensor scratch(const at::Tensor &like, size_t preferred, size_t least)
{
    if (preferred > least) {
        try {
            return make(like, {(int64_t)preferred}, at::kByte);
        } catch (const c10::OutOfMemoryError &) {
        }
    }
    return least > 0 ? make(like, {(int64_t)least}, at::kByte) : at::Tensor();
}
void *data(const at::Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; }
size_t size(const at::Tensor &t) { return t.defined() ? (size_t)t.numel() : 0; }

PyObject *not_implemented() { Py_RETURN_NOTIMPLEMENTED; }
PyObject *status(int rc) { return PyLong_FromLong(rc); }

// act_quant(entry, X, s, stream) -> (Xq, sx)
PyObject *act_quant(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS   // (torch's own translation: an allocation that fails stays torch.OutOfMemoryError)
    if (n != 4 || !plain(a[1]) || !plain_or_none(a[2])) return not_implemented();
    decltype(&quantize_act_int8) entry;
    int64_t stream;
    if (!to_fn(a[0], entry)) return nullptr;
    if (!to_i64(a[3], stream)) return not_implemented();
    const at::Tensor &X = THPVariable_Unpack(a[1]);
    const Rows r = rows_of(X);
    if (!r.ok) return not_implemented();
    at::Tensor Xq = make(X, {r.M, r.K}, at::kChar), sx = make(X, {r.M}, at::kFloat);
    const void *x = X.data_ptr();
    const float *s = (const float *)ptr(a[2]);
    int8_t *q = (int8_t *)Xq.data_ptr();
    float *sxp = (float *)sx.data_ptr();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = entry(x, r.dtype, r.M, r.K, r.ld, s, q, sxp, (void *)stream);
    Py_END_ALLOW_THREADS
    if (rc != W4A8_OK) return status(rc);
    return PyTuple_Pack(2, py::reinterpret_steal<py::object>(THPVariable_Wrap(Xq)).ptr(),
                        py::reinterpret_steal<py::object>(THPVariable_Wrap(sx)).ptr());
    END_HANDLE_TH_ERRORS
}

// act_quant_asym(entry, X, s, stream) -> (Xq, sx, zx)
PyObject *act_quant_asym(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 4 || !plain(a[1]) || !plain_or_none(a[2])) return not_implemented();
    decltype(&quantize_act_int8_asym) entry;
    int64_t stream;
    if (!to_fn(a[0], entry)) return nullptr;
    if (!to_i64(a[3], stream)) return not_implemented();
    const at::Tensor &X = THPVariable_Unpack(a[1]);
    const Rows r = rows_of(X);
    if (!r.ok) return not_implemented();
    at::Tensor Xq = make(X, {r.M, r.K}, at::kChar), sx = make(X, {r.M}, at::kFloat), zx = make(X, {r.M}, at::kInt);
    const void *x = X.data_ptr();
    const float *s = (const float *)ptr(a[2]);
    int8_t *q = (int8_t *)Xq.data_ptr();
    float *sxp = (float *)sx.data_ptr();
    int32_t *zxp = (int32_t *)zx.data_ptr();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = entry(x, r.dtype, r.M, r.K, r.ld, s, q, sxp, zxp, (void *)stream);
    Py_END_ALLOW_THREADS
    if (rc != W4A8_OK) return status(rc);
    return PyTuple_Pack(3, py::reinterpret_steal<py::object>(THPVariable_Wrap(Xq)).ptr(),
                        py::reinterpret_steal<py::object>(THPVariable_Wrap(sx)).ptr(),
                        py::reinterpret_steal<py::object>(THPVariable_Wrap(zx)).ptr());
    END_HANDLE_TH_ERRORS
}

// gemm(entry, preferred_workspace_entry, workspace_entry, Xq, sx, Wp, step, zero, N, K, group_size, layout, y_dtype, stream) -> Y
PyObject *gemm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 14) return not_implemented();
    for (int i = 3; i < 8; ++i)
        if (!plain(a[i])) return not_implemented();
    decltype(&w4a8_gemm) entry;
    decltype(&w4a8_gemm_workspace_bytes) wish, need;
    int64_t N, K, G, layout, yd, stream;
    if (!to_fn(a[0], entry) || !to_fn(a[1], wish) || !to_fn(a[2], need)) return nullptr;
    if (!to_i64(a[8], N) || !to_i64(a[9], K) || !to_i64(a[10], G) ||
        !to_i64(a[11], layout) || !to_i64(a[12], yd) || !to_i64(a[13], stream))
        return not_implemented();
    const at::Tensor &Xq = THPVariable_Unpack(a[3]);
    if (Xq.dim() < 1 || N < 0) return not_implemented();
    const int64_t M = Xq.size(0);
    at::Tensor Y = make(Xq, {M, N}, y_type(yd));
    const at::Tensor ws = scratch(Xq, wish(M, N, K, G, (int)layout), need(M, N, K, G, (int)layout));
    const size_t bytes = size(ws);
    const int8_t *q = (const int8_t *)ptr(a[3]);
    const float *sx = (const float *)ptr(a[4]), *step = (const float *)ptr(a[6]);
    const uint8_t *Wp = (const uint8_t *)ptr(a[5]), *zero = (const uint8_t *)ptr(a[7]);
    void *y = Y.data_ptr(), *w = data(ws);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = entry(q, sx, M, Wp, (int)layout, step, zero, N, K, G, y, (int)yd, N, nullptr, w, bytes, (void *)stream);
    Py_END_ALLOW_THREADS
    return rc != W4A8_OK ? status(rc) : THPVariable_Wrap(Y);
    END_HANDLE_TH_ERRORS
}

// gemm_asym(entry, workspace_entry, Xq, sx, zx, Wp, step, zero, wsum, tsum, N, K, group_size, layout, y_dtype,
//           stream) -> Y
PyObject *gemm_asym(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 16) return not_implemented();
    for (int i = 2; i < 10; ++i)
        if (!plain(a[i])) return not_implemented();
    decltype(&w4a8_gemm_asym) entry;
    decltype(&w4a8_gemm_workspace_bytes) need;
    int64_t N, K, G, layout, yd, stream;
    if (!to_fn(a[0], entry) || !to_fn(a[1], need)) return nullptr;
    if (!to_i64(a[10], N) || !to_i64(a[11], K) || !to_i64(a[12], G) ||
        !to_i64(a[13], layout) || !to_i64(a[14], yd) || !to_i64(a[15], stream))
        return not_implemented();
    const at::Tensor &Xq = THPVariable_Unpack(a[2]);
    if (Xq.dim() < 1 || N < 0) return not_implemented();
    const int64_t M = Xq.size(0);
    at::Tensor Y = make(Xq, {M, N}, y_type(yd));
    const size_t bytes = need(M, N, K, G, (int)layout);
    at::Tensor ws;
    if (bytes > 0) ws = make(Xq, {(int64_t)bytes}, at::kByte);
    const int8_t *q = (const int8_t *)ptr(a[2]);
    const float *sx = (const float *)ptr(a[3]), *step = (const float *)ptr(a[6]);
    const int32_t *zx = (const int32_t *)ptr(a[4]), *wsum = (const int32_t *)ptr(a[8]), *tsum = (const int32_t *)ptr(a[9]);
    const uint8_t *Wp = (const uint8_t *)ptr(a[5]), *zero = (const uint8_t *)ptr(a[7]);
    void *y = Y.data_ptr(), *w = bytes > 0 ? ws.data_ptr() : nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = entry(q, sx, zx, M, Wp, (int)layout, step, zero, wsum, tsum, N, K, G, y, (int)yd, N, nullptr, w, bytes,
               (void *)stream);
    Py_END_ALLOW_THREADS
    return rc != W4A8_OK ? status(rc) : THPVariable_Wrap(Y);
    END_HANDLE_TH_ERRORS
}

// linear(entry, preferred_workspace_entry, workspace_entry, act_quant_entry, gemm_entry, gemm_workspace_entry, X, s, Wp, step,
//        zero, N, group_size, layout, y_dtype, stream) -> Y
PyObject *linear(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 16 || !plain(a[6]) || !plain_or_none(a[7]) || !plain(a[8]) || !plain(a[9]) || !plain(a[10]))
        return not_implemented();
    decltype(&w4a8_linear) entry;
    decltype(&w4a8_linear_workspace_bytes) wish, need;
    decltype(&quantize_act_int8) quantize;
    decltype(&w4a8_gemm) product;
    decltype(&w4a8_gemm_workspace_bytes) product_need;
    int64_t N, G, layout, yd, stream;
    if (!to_fn(a[0], entry) || !to_fn(a[1], wish) || !to_fn(a[2], need) || !to_fn(a[3], quantize) ||
        !to_fn(a[4], product) || !to_fn(a[5], product_need))
        return nullptr;
    if (!to_i64(a[11], N) || !to_i64(a[12], G) ||
        !to_i64(a[13], layout) || !to_i64(a[14], yd) || !to_i64(a[15], stream))
        return not_implemented();
    const at::Tensor &X = THPVariable_Unpack(a[6]);
    const Rows r = rows_of(X);
    if (!r.ok || N < 0) return not_implemented();
    at::Tensor Y = make(X, {r.M, N}, y_type(yd));
    const void *x = X.data_ptr();
    const float *s = (const float *)ptr(a[7]), *step = (const float *)ptr(a[9]);
    const uint8_t *Wp = (const uint8_t *)ptr(a[8]), *zero = (const uint8_t *)ptr(a[10]);
    void *y = Y.data_ptr();
    int rc = W4A8_ERR_WORKSPACE;
    if (r.M > 4 && r.M <= 16 && r.K >= 5120 && r.dtype == W4A8_F16 && layout == LAYOUT_TILED) {
        // the two steps by themselves, faster here than in one launch (the times stand beside w4a8_linear's rule)
        const size_t bytes = product_need(r.M, N, r.K, G, (int)layout);
        const auto up = [](int64_t n) { return (n + 255) / 256 * 256; };   // (one allocation: three cost the host 0.3 us more)
        const int64_t sx_at = up(r.M * r.K), ws_at = sx_at + up(4 * r.M);
        const at::Tensor room = make(X, {ws_at + (int64_t)bytes}, at::kByte);
        uint8_t *p = (uint8_t *)room.data_ptr();
        int8_t *q = (int8_t *)p;
        float *sxp = (float *)(p + sx_at);
        void *w = bytes > 0 ? p + ws_at : nullptr;
        Py_BEGIN_ALLOW_THREADS
        rc = quantize(x, r.dtype, r.M, r.K, r.ld, s, q, sxp, (void *)stream);
        if (rc == W4A8_OK)
            rc = product(q, sxp, r.M, Wp, (int)layout, step, zero, N, r.K, G, y, (int)yd, N, nullptr, w, bytes, (void *)stream);
        Py_END_ALLOW_THREADS
        return rc != W4A8_OK ? status(rc) : THPVariable_Wrap(Y);
    }
    auto call = [&](void *w, size_t bytes) {
        Py_BEGIN_ALLOW_THREADS
        rc = entry(x, r.dtype, r.M, r.K, r.ld, s, Wp, (int)layout, step, zero, N, G, y, (int)yd, N, nullptr, nullptr,
                   nullptr, w, bytes, (void *)stream);
        Py_END_ALLOW_THREADS
    };
    // The one-launch decode step needs no workspace: try without (a call that needs one is turned down
    // before anything is launched).
    if (r.M <= 16 && r.dtype == W4A8_F16 && layout == LAYOUT_TILED) call(nullptr, 0);
    if (rc == W4A8_ERR_WORKSPACE) {
        const at::Tensor ws = scratch(X, wish(r.M, N, r.K, G, (int)layout), need(r.M, N, r.K, G, (int)layout));
        call(data(ws), size(ws));
    }
    return rc != W4A8_OK ? status(rc) : THPVariable_Wrap(Y);
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"act_quant", (PyCFunction)(void (*)(void))act_quant, METH_FASTCALL, nullptr},
    {"act_quant_asym", (PyCFunction)(void (*)(void))act_quant_asym, METH_FASTCALL, nullptr},
    {"gemm", (PyCFunction)(void (*)(void))gemm, METH_FASTCALL, nullptr},
    {"gemm_asym", (PyCFunction)(void (*)(void))gemm_asym, METH_FASTCALL, nullptr},
    {"linear", (PyCFunction)(void (*)(void))linear, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
