// Native marshalling of the eager calls that one small launch follows: a Python extension module (_mqhost) that checks the
// tensors, allocates what the call returns, reads the current stream and calls the C entry point, whose address the
// binding hands over once.  In Python two dozen argument conversions, the allocations and the stream lookup cost 10 us a
// call, more than the kernels of a small layer run: 4 x 1280 x 1280 weight-only 12.9 -> 7.6 us, 256 x 320 x 320 with run-time
// ranges 20.0 -> 12.1, quantising and packing the eight linears of a 1280-channel block 190 -> 89.
//
// Every function takes the ordinary case only, plain tensors on the GPU with the expected sizes and no mode or transform
// that intercepts operations, and returns None for anything else: the binding then goes its general way, which also
// raises the errors.
#include <ATen/ops/empty.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <optional>

namespace {

typedef int (*w_only_fn)(const void*, int, int, int, const void*, int, int, int, const float*, const int32_t*, const void*, void*,
                         int, int, const void*, int, void*, size_t, void*);
typedef int (*w8a8_fn)(const void*, int, int, int, const void*, int, int, int, const float*, const int32_t*, const int32_t*,
                       const float*, const int32_t*, const void*, void*, int, int32_t*, const void*, int, float*, int32_t*, void*,
                       size_t, void*);
typedef int (*wxa8_fn)(const void*, int, int, int, const void*, int, int, const float*, const int32_t*, const int32_t*, const float*,
                       const int32_t*, const void*, void*, int, int32_t*, const void*, int, float*, int32_t*, void*, size_t, void*);
typedef int (*quantize_fn)(const void*, int, int, int, int, int, uint8_t*, float*, int32_t*, void*);
typedef int (*pack_fn)(const uint8_t*, int, int, int, int, int, void*, int32_t*, void*);
typedef size_t (*split_bytes_fn)(int, int, int);
typedef size_t (*a8_bytes_fn)(int, int);
typedef size_t (*packed_bytes_fn)(int, int, int, int);

struct Entry {
    w_only_fn w_only;
    w8a8_fn w8a8;
    wxa8_fn w4a8, w2a8;
    quantize_fn quantize;
    pack_fn pack;
    split_bytes_fn split_bytes;
    a8_bytes_fn a8_bytes;
    packed_bytes_fn packed_bytes;
} entry;

// An ordinary tensor on the GPU (torch.Tensor or Parameter itself), or nullptr.
const at::Tensor* gpu_tensor(PyObject* o) {
    if (!THPVariable_CheckTypeExact(Py_TYPE(o))) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.is_cuda() && t.has_storage() ? &t : nullptr;
}

// An optional operand: its address (null for None), or false for what is no ordinary tensor.
bool optional_ptr(PyObject* o, void*& p, const at::Tensor** t = nullptr) {
    p = nullptr;
    if (o == Py_None) return true;
    const at::Tensor* v = gpu_tensor(o);
    if (!v) return false;
    p = v->data_ptr();
    if (t) *t = v;
    return true;
}

bool small_int(PyObject* o, int& v) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long l = PyLong_AsLongAndOverflow(o, &over);
    if (over || l < INT32_MIN || l > INT32_MAX) return false;
    v = (int)l;
    return true;
}

bool fits(int64_t v) { return v >= 0 && v <= INT32_MAX; }

// Nothing between the caller and the operators that would want to see the allocations.
bool plain_calls() { return !at::impl::torch_function_mode_enabled() && !c10::impl::TorchDispatchModeTLS::any_modes_set(); }

// Gives the interpreter lock up for as long as it lives: for allocations, which wait for the device when the pool has to
// grow, and for the launch.
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked&) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};

void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

at::Tensor empty(at::IntArrayRef size, at::ScalarType type, at::Device device) {
    return at::empty(size, at::TensorOptions().dtype(type).device(device));
}

// [M, N] residual of x's type: its address and row stride.
bool residual_of(PyObject* o, int64_t M, int64_t N, at::ScalarType type, void*& p, int& ld) {
    const at::Tensor* r = nullptr;
    ld = 0;
    if (!optional_ptr(o, p, &r)) return false;
    if (!r) return true;
    if (r->dim() != 2 || r->size(0) != M || r->size(1) != N || r->stride(1) != 1 || r->scalar_type() != type || !fits(r->stride(0)))
        return false;
    ld = (int)r->stride(0);
    return true;
}

// [M, K] activations with contiguous rows.
bool activations(const at::Tensor* x, int K) {
    return x && x->dim() == 2 && x->stride(1) == 1 && x->size(1) == K && fits(x->size(0)) && fits(x->stride(0));
}

PyObject* general() { Py_RETURN_NONE; }

// (x, packed, N, K, bits, layout, scale, zp, bias, out, residual, ws) -> tensor, error code or None
PyObject* qlinear_w_only(PyObject*, PyObject* const* a, Py_ssize_t n) {
    try {
        int N, K, bits, layout, ldr;
        void *packed, *scale, *zp, *bias, *res, *ws;
        const at::Tensor *x, *out = nullptr, *wst = nullptr;
        if (n != 12 || !plain_calls() || !(x = gpu_tensor(a[0])) || !small_int(a[2], N) || !small_int(a[3], K) || N < 0 ||
            !small_int(a[4], bits) || !small_int(a[5], layout) || !activations(x, K) || !optional_ptr(a[1], packed) ||
            !optional_ptr(a[6], scale) || !optional_ptr(a[7], zp) || !optional_ptr(a[8], bias))
            return general();
        const at::ScalarType type = x->scalar_type();
        if (type != at::kHalf && type != at::kBFloat16) return general();
        const int64_t M = x->size(0);
        if (!residual_of(a[10], M, N, type, res, ldr)) return general();
        if (a[9] != Py_None && (!(out = gpu_tensor(a[9])) || out->dim() < 1 || !fits(out->stride(0)))) return general();
        if (!optional_ptr(a[11], ws, &wst)) return general();
        size_t ws_bytes = wst ? wst->nbytes() : 0;
        const void* xp = x->data_ptr();
        void* yp = out ? out->data_ptr() : nullptr;
        const int ldx = (int)x->stride(0), ldy = out ? (int)out->stride(0) : N, dt = type == at::kHalf ? 0 : 1;
        const at::Device device = x->device();
        at::Tensor y, own_ws;
        int rc;
        {
            Unlocked unlocked;
            if (!out) {
                y = empty({M, N}, type, device);
                yp = y.data_ptr();
            }
            if (!wst && (ws_bytes = entry.split_bytes((int)M, N, K)) != 0) {
                own_ws = empty({(int64_t)ws_bytes}, at::kByte, device);
                ws = own_ws.data_ptr();
            }
            rc = entry.w_only(xp, (int)M, K, ldx, packed, N, bits, layout, (const float*)scale, (const int32_t*)zp, bias, yp, ldy, dt, res,
                              ldr, ws, ws_bytes, stream());
        }
        if (rc) return PyLong_FromLong(rc);
        if (a[9] != Py_None) return Py_NewRef(a[9]);
        return THPVariable_Wrap(std::move(y));
    } catch (const std::exception&) {
        PyErr_Clear();
        return general();
    }
}

// (x, packed, N, K, bits, layout, signed, scale, zp, colsum, act_scale, act_zp, bias, out, residual, ws) -> tensor, code or None
PyObject* qlinear_a8(PyObject*, PyObject* const* a, Py_ssize_t n) {
    try {
        int N, K, bits, layout, sgn, ldr;
        void *packed, *scale, *zp, *colsum, *act_s, *act_z, *bias, *res, *ws;
        const at::Tensor *x, *out = nullptr, *wst = nullptr;
        if (n != 16 || !plain_calls() || !(x = gpu_tensor(a[0])) || !small_int(a[2], N) || !small_int(a[3], K) || N < 0 ||
            !small_int(a[4], bits) || !small_int(a[5], layout) || !small_int(a[6], sgn) || !activations(x, K) ||
            x->scalar_type() != at::kHalf || !optional_ptr(a[1], packed) || !optional_ptr(a[7], scale) || !optional_ptr(a[8], zp) ||
            !optional_ptr(a[9], colsum) || !optional_ptr(a[10], act_s) || !optional_ptr(a[11], act_z) || !optional_ptr(a[12], bias))
            return general();
        const int64_t M = x->size(0);
        if (!residual_of(a[14], M, N, at::kHalf, res, ldr)) return general();
        if (a[13] != Py_None && (!(out = gpu_tensor(a[13])) || out->dim() < 1 || !fits(out->stride(0)))) return general();
        if (!optional_ptr(a[15], ws, &wst)) return general();
        size_t ws_bytes = wst ? (size_t)wst->numel() : 0;
        const void* xp = x->data_ptr();
        void* yp = out ? out->data_ptr() : nullptr;
        const int ldx = (int)x->stride(0), ldy = out ? (int)out->stride(0) : N;
        const at::Device device = x->device();
        at::Tensor y, own_ws;
        int rc;
        {
            Unlocked unlocked;
            if (!out) {
                y = empty({M, N}, at::kHalf, device);
                yp = y.data_ptr();
            }
            if (!wst) {
                ws_bytes = entry.a8_bytes((int)M, K) + entry.split_bytes((int)M, N, K);
                own_ws = empty({(int64_t)ws_bytes}, at::kByte, device);
                ws = own_ws.data_ptr();
            }
            void* st = stream();
            if (bits == 8)
                rc = entry.w8a8(xp, (int)M, K, ldx, packed, N, layout, sgn, (const float*)scale, (const int32_t*)zp, (const int32_t*)colsum,
                                (const float*)act_s, (const int32_t*)act_z, bias, yp, ldy, nullptr, res, ldr, nullptr, nullptr, ws,
                                ws_bytes, st);
            else
                rc = (bits == 4 ? entry.w4a8 : entry.w2a8)(xp, (int)M, K, ldx, packed, N, layout, (const float*)scale, (const int32_t*)zp,
                                                           (const int32_t*)colsum, (const float*)act_s, (const int32_t*)act_z, bias, yp,
                                                           ldy, nullptr, res, ldr, nullptr, nullptr, ws, ws_bytes, st);
        }
        if (rc) return PyLong_FromLong(rc);
        if (a[13] != Py_None) return Py_NewRef(a[13]);
        return THPVariable_Wrap(std::move(y));
    } catch (const std::exception&) {
        PyErr_Clear();
        return general();
    }
}

// (w, bits, symmetric) -> (codes, scale, zp), code or None
PyObject* quantize_weights(PyObject*, PyObject* const* a, Py_ssize_t n) {
    try {
        int bits, sym;
        const at::Tensor* w;
        if (n != 3 || !plain_calls() || !(w = gpu_tensor(a[0])) || !small_int(a[1], bits) || !small_int(a[2], sym) || w->dim() != 2 ||
            !w->is_contiguous() || !fits(w->size(0)) || !fits(w->size(1)))
            return general();
        const at::ScalarType type = w->scalar_type();
        if (type != at::kHalf && type != at::kBFloat16) return general();
        const int64_t N = w->size(0), K = w->size(1);
        const void* wp = w->data_ptr();
        const at::Device device = w->device();
        at::Tensor codes, scale, zp;
        int rc;
        {
            Unlocked unlocked;
            codes = empty({N, K}, at::kByte, device), scale = empty({N}, at::kFloat, device), zp = empty({N}, at::kInt, device);
            rc = entry.quantize(wp, (int)N, (int)K, bits, sym, type == at::kHalf ? 0 : 1, (uint8_t*)codes.data_ptr(), (float*)scale.data_ptr(),
                                (int32_t*)zp.data_ptr(), stream());
        }
        if (rc) return PyLong_FromLong(rc);
        PyObject *c = THPVariable_Wrap(std::move(codes)), *s = THPVariable_Wrap(std::move(scale)), *z = THPVariable_Wrap(std::move(zp));
        PyObject* t = c && s && z ? PyTuple_Pack(3, c, s, z) : nullptr;
        Py_XDECREF(c);
        Py_XDECREF(s);
        Py_XDECREF(z);
        return t;
    } catch (const std::exception&) {
        PyErr_Clear();
        return general();
    }
}

// (codes, bits, layout, signed, want_colsum) -> (packed, colsum or None), code or None
PyObject* pack_weights(PyObject*, PyObject* const* a, Py_ssize_t n) {
    try {
        int bits, layout, sgn, want;
        const at::Tensor* codes;
        if (n != 5 || !plain_calls() || !(codes = gpu_tensor(a[0])) || !small_int(a[1], bits) || !small_int(a[2], layout) ||
            !small_int(a[3], sgn) || !small_int(a[4], want) || bits == 16 || codes->scalar_type() != at::kByte || codes->dim() != 2 ||
            !codes->is_contiguous() || !fits(codes->size(0)) || !fits(codes->size(1)))
            return general();
        const int64_t N = codes->size(0), K = codes->size(1);
        const size_t nbytes = entry.packed_bytes((int)N, (int)K, bits, layout);
        const void* cp = codes->data_ptr();
        const at::Device device = codes->device();
        at::Tensor packed, colsum;
        int rc;
        {
            Unlocked unlocked;
            packed = empty({(int64_t)(nbytes ? nbytes : 1)}, at::kByte, device);
            if (want) colsum = empty({N}, at::kInt, device);
            rc = entry.pack((const uint8_t*)cp, (int)N, (int)K, bits, layout, sgn, packed.data_ptr(),
                            want ? (int32_t*)colsum.data_ptr() : nullptr, stream());
        }
        if (rc) return PyLong_FromLong(rc);
        PyObject *p = THPVariable_Wrap(std::move(packed)), *s = want ? THPVariable_Wrap(std::move(colsum)) : Py_NewRef(Py_None);
        PyObject* t = p && s ? PyTuple_Pack(2, p, s) : nullptr;
        Py_XDECREF(p);
        Py_XDECREF(s);
        return t;
    } catch (const std::exception&) {
        PyErr_Clear();
        return general();
    }
}

// Addresses of the C entry points, in the order of Entry.
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    void* p[9];
    if (n != 9) {
        PyErr_SetString(PyExc_TypeError, "bind takes nine addresses");
        return nullptr;
    }
    for (int i = 0; i < 9; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
            return nullptr;
        }
    }
    entry = Entry{(w_only_fn)p[0], (w8a8_fn)p[1], (wxa8_fn)p[2], (wxa8_fn)p[3], (quantize_fn)p[4], (pack_fn)p[5], (split_bytes_fn)p[6],
                  (a8_bytes_fn)p[7], (packed_bytes_fn)p[8]};
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {"qlinear_w_only", (PyCFunction)(void (*)(void))qlinear_w_only, METH_FASTCALL, nullptr},
    {"qlinear_a8", (PyCFunction)(void (*)(void))qlinear_a8, METH_FASTCALL, nullptr},
    {"quantize_weights", (PyCFunction)(void (*)(void))quantize_weights, METH_FASTCALL, nullptr},
    {"pack_weights", (PyCFunction)(void (*)(void))pack_weights, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_mqhost", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__mqhost(void) {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "made_for", MQ_MADE_FOR) < 0) Py_CLEAR(m);
    return m;
}
