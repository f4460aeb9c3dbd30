// The way from a Python call of a product to its launch, for the call as programs make it: plain tensors on the current
// device that pass every check of binding.py.  Anything else (another device, a subclass, an active mode, a shape or a type that does
// not fit) returns None, and the binding's own checks and messages take the call.
//
// What bounds it: products of one to eight rows of a matrix of 2 to 30 MB run 3.5 to 11 us on the device, and the checks, the
// allocation and the marshalling of the Python form took longer than the launch (2.4 us of a call's host time here).  us of host
// time per call, Python form -> here: one row 6.9 -> 3.5, fused 7.7 -> 3.8, BF16 weights 7.0 -> 3.7, tile-major 6.9 -> 3.6,
// verification (two launches) 14.2 -> 7.6, a cast (two outputs) 7.5 -> 4.4.
#include <ATen/ATen.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mxfp4.h"

namespace {

PyObject* g_failed = nullptr;                       // raises the error of a status code

// The kinds of binding.py: 0 MXFP4, 1 E4M3, 2 E2M3, 3 BF16, 4 the tile-major copy, 16 + id the formats chosen by id.
enum { kMx = 0, kE4m3 = 1, kE2m3 = 2, kBf16 = 3, kTiled = 4, kFmt = 16 };

// A tensor whose memory and sizes are what they say: exactly torch.Tensor (or Parameter) and no transform, mode or lazy bit.
const at::Tensor* plain(PyObject* o, at::ScalarType type, c10::Device device)
{
    static const uint64_t allowed =
        c10::DispatchKeySet({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::ADInplaceOrView,
                             c10::DispatchKey::AutocastCUDA}).raw_repr();
    if (!THPVariable_CheckExact(o))
        return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || (t.key_set().raw_repr() & ~allowed) != 0 || t.scalar_type() != type || t.device() != device ||
        !t.has_storage())
        return nullptr;
    return &t;
}

const at::Tensor* rows_of(PyObject* o, c10::Device device)       // [rows, columns] BF16, columns side by side
{
    const at::Tensor* t = plain(o, at::kBFloat16, device);
    return t && t->dim() == 2 && t->stride(1) == 1 ? t : nullptr;
}

const at::Tensor* bytes_of(PyObject* o, c10::Device device)
{
    const at::Tensor* t = plain(o, at::kByte, device);
    return t && t->is_contiguous() ? t : nullptr;
}

// The operands of a product.
struct Operands {
    const void *x, *q, *s = nullptr;
    int64_t m, n, k, ldx, ldw = 0;
    c10::Device device = c10::Device(c10::kCUDA, 0);
    void* stream;
};

// args: kind, x, q (or w), s (or None), n, k (of the tile-major copy).
bool operands(PyObject* const* args, int* kind, Operands* o)
{
    if (at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set())
        return false;
    if (!THPVariable_CheckExact(args[1]) || !THPVariable_Unpack(args[1]).is_cuda())
        return false;                               // (without a device there is no current one to ask for)
    *kind = (int)PyLong_AsLong(args[0]);
    const c10::DeviceIndex at = c10::hip::current_device();
    o->device = c10::Device(c10::kCUDA, at);
    const at::Tensor* x = rows_of(args[1], o->device);
    if (!x)
        return false;
    o->m = x->size(0);
    o->k = x->size(1);
    o->ldx = o->m > 1 ? x->stride(0) : o->k;
    if (*kind == kBf16) {
        const at::Tensor* w = rows_of(args[2], o->device);
        if (!w || w->size(1) != o->k)
            return false;
        o->n = w->size(0);
        o->ldw = o->n > 1 ? w->stride(0) : o->k;
        o->q = w->data_ptr();
    } else {
        const at::Tensor *q = bytes_of(args[2], o->device), *s = bytes_of(args[3], o->device);
        if (!q || !s)
            return false;
        if (*kind == kTiled) {
            if (!PyLong_Check(args[4]) || !PyLong_Check(args[5]) || PyLong_AsLongLong(args[5]) != o->k)
                return false;
            o->n = PyLong_AsLongLong(args[4]);
        } else {
            if (q->dim() != 2 || s->dim() != 2)
                return false;
            o->n = q->size(0);
            const int64_t block = *kind == kMx ? 16 : *kind == kE4m3 ? 32 : *kind == kE2m3 ? 24 : mxfp4_fmt_block_bytes(*kind - kFmt);
            if (block == 0 || o->k % 32 != 0 || q->size(1) != o->k / 32 * block || s->size(0) != o->n || s->size(1) != o->k / 32)
                return false;
        }
        o->q = q->data_ptr();
        o->s = s->data_ptr();
    }
    o->x = x->data_ptr();
    o->stream = c10::hip::getCurrentHIPStream(at).stream();
    return true;
}

// A new tensor on the device: from the allocator behind torch.empty, without the way through the dispatcher, unless something on this
// thread wants to see it there (a transform; autocast and the keys that every thread has do not).  One row of
// 4096 x 4096, which the host bounds: 4.35 -> 4.17 us from call to call.
at::Tensor fresh(at::IntArrayRef size, at::ScalarType type, c10::Device device)
{
    static const uint64_t usual = (c10::default_included_set | c10::autocast_dispatch_keyset).raw_repr();
    if ((c10::impl::tls_local_dispatch_key_set().included_.raw_repr() & ~usual) != 0)
        return at::empty(size, at::TensorOptions().dtype(type).device(device));
    return at::Tensor(at::detail::empty_cuda(size, type, device, std::nullopt));
}

// What the binding's own checks take over: also a number that is none or too large, whose error they raise in their words.
PyObject* left()
{
    PyErr_Clear();
    Py_RETURN_NONE;
}

bool small(PyObject* o, int* v)                     // an int of the C interface as it stands
{
    int over = 0;
    const long long wide = PyLong_Check(o) ? PyLong_AsLongLongAndOverflow(o, &over) : 0;
    *v = (int)wide;
    return PyLong_Check(o) && over == 0 && wide == *v;
}

struct Scratch {
    void* at = nullptr;
    size_t bytes = 0;
};

bool scratch(PyObject* o, c10::Device device, Scratch* s)
{
    if (o == Py_None)
        return true;
    const at::Tensor* t = plain(o, at::kByte, device);
    if (!t)
        return false;
    s->at = t->data_ptr();
    s->bytes = (size_t)t->numel();
    return true;
}

PyObject* finish(int rc, PyObject* (*wrap)(const at::Tensor*), const at::Tensor* out)
{
    if (rc == 0)
        return wrap(out);
    PyObject* raised = PyObject_CallFunction(g_failed, "i", rc);
    Py_XDECREF(raised);
    if (!PyErr_Occurred())
        PyErr_SetString(PyExc_RuntimeError, "mxfp4: status without an error");
    return nullptr;
}

PyObject* wrap_one(const at::Tensor* t) { return THPVariable_Wrap(t[0]); }

PyObject* wrap_list(const at::Tensor* t, int count)
{
    PyObject* tuple = PyTuple_New(count);
    for (int i = 0; tuple && i < count; ++i) {
        PyObject* item = THPVariable_Wrap(t[i]);
        if (!item) {
            Py_DECREF(tuple);
            return nullptr;
        }
        PyTuple_SET_ITEM(tuple, i, item);
    }
    return tuple;
}

PyObject* wrap_three(const at::Tensor* t) { return wrap_list(t, 3); }
PyObject* wrap_two(const at::Tensor* t) { return wrap_list(t, 2); }

// product(kind, x, q, s, n, k, fused, bias, act, residual, path, workspace) -> y, or None
PyObject* product(PyObject*, PyObject* const* args, Py_ssize_t count)
{
    HANDLE_TH_ERRORS
    if (count != 12) {
        PyErr_SetString(PyExc_TypeError, "product: twelve arguments");
        return nullptr;
    }
    int kind;
    Operands o;
    Scratch ws;
    int act, path;
    if (!small(args[8], &act) || !small(args[10], &path) || !operands(args, &kind, &o) || !scratch(args[11], o.device, &ws))
        return left();
    const bool fused = args[6] == Py_True, spare = args[11] != Py_None;
    const int64_t c = act == 1 ? o.n / 2 : o.n;
    const void *bias = nullptr, *residual = nullptr;
    int64_t ldr = 0;
    if (args[7] != Py_None) {
        const at::Tensor* b = plain(args[7], at::kBFloat16, o.device);
        if (!b || b->dim() != 1 || b->size(0) != o.n || !b->is_contiguous())
            return left();
        bias = b->data_ptr();
    }
    if (args[9] != Py_None) {
        const at::Tensor* r = rows_of(args[9], o.device);
        if (!r || r->size(0) != o.m || r->size(1) != c)
            return left();
        residual = r->data_ptr();
        ldr = o.m > 1 ? r->stride(0) : c;
    }
    if (PyErr_Occurred())
        return left();
    at::Tensor y;
    int rc;
    {
        pybind11::gil_scoped_release no_gil;
        y = fresh({o.m, c}, at::kBFloat16, o.device);
        void* out = y.data_ptr();
        if (kind == kTiled)
            rc = fused ? mxfp4_woq_gemm_tiled_fused(o.x, o.m, o.ldx, o.q, o.s, o.n, o.k, bias, act, residual, ldr, out, c, o.stream)
                 : spare ? mxfp4_woq_gemm_tiled_ws(o.x, o.m, o.ldx, o.q, o.s, o.n, o.k, out, c, ws.at, ws.bytes, o.stream)
                         : mxfp4_woq_gemm_tiled(o.x, o.m, o.ldx, o.q, o.s, o.n, o.k, out, c, o.stream);
        else if (kind == kBf16)
            rc = mxfp4_bf16_gemm(o.x, o.m, o.ldx, o.q, o.n, o.k, o.ldw, out, c, o.stream);
        else if (kind == kE4m3)
            rc = mxfp4_e4m3_woq_gemm(o.x, o.m, o.ldx, o.q, o.s, o.n, o.k, out, c, o.stream);
        else if (kind == kE2m3)
            rc = mxfp4_e2m3_woq_gemm(o.x, o.m, o.ldx, o.q, o.s, o.n, o.k, out, c, o.stream);
        else if (kind >= kFmt)
            rc = mxfp4_fmt_woq_gemm(kind - kFmt, o.x, o.m, o.ldx, o.q, o.s, o.n, o.k, out, c, o.stream);
        else
            rc = fused ? mxfp4_woq_gemm_fused(o.x, o.m, o.ldx, o.q, o.s, o.n, o.k, bias, act, residual, ldr, out, c, ws.at,
                                              ws.bytes, path, o.stream)
                 : spare ? mxfp4_woq_gemm_ws(o.x, o.m, o.ldx, o.q, o.s, o.n, o.k, out, c, ws.at, ws.bytes, path, o.stream)
                         : mxfp4_woq_gemm_path(o.x, o.m, o.ldx, o.q, o.s, o.n, o.k, out, c, path, o.stream);
    }
    return finish(rc, wrap_one, &y);
    END_HANDLE_TH_ERRORS
}

// verify(kind, x, q, s, n, k, draft, workspace) -> (accept, index, value), or None: MXFP4, BF16 and the tile-major copy
PyObject* verify(PyObject*, PyObject* const* args, Py_ssize_t count)
{
    HANDLE_TH_ERRORS
    if (count != 8) {
        PyErr_SetString(PyExc_TypeError, "verify: eight arguments");
        return nullptr;
    }
    int kind;
    Operands o;
    Scratch ws;
    if (args[7] == Py_None || !operands(args, &kind, &o) || !scratch(args[7], o.device, &ws) ||
        (kind != kMx && kind != kBf16 && kind != kTiled))
        return left();
    const void* draft = nullptr;
    if (args[6] != Py_None) {
        const at::Tensor* d = plain(args[6], at::kInt, o.device);
        if (!d || d->numel() != o.m - 1 || !d->is_contiguous())
            return left();
        draft = d->data_ptr();
    }
    if (PyErr_Occurred())
        return left();
    at::Tensor out[3];
    int rc;
    {
        pybind11::gil_scoped_release no_gil;
        out[0] = fresh({2}, at::kInt, o.device);
        out[1] = fresh({o.m}, at::kInt, o.device);
        out[2] = fresh({o.m}, at::kFloat, o.device);
        void *accept = out[0].data_ptr(), *index = out[1].data_ptr(), *value = out[2].data_ptr();
        if (kind == kBf16)
            rc = mxfp4_bf16_gemm_verify(o.x, o.m, o.ldx, o.q, o.n, o.k, o.ldw, (const int32_t*)draft, (int32_t*)accept,
                                        (int32_t*)index, (float*)value, ws.at, ws.bytes, o.stream);
        else
            rc = (kind == kTiled ? mxfp4_woq_gemm_tiled_verify : mxfp4_woq_gemm_verify)(
                o.x, o.m, o.ldx, o.q, o.s, o.n, o.k, (const int32_t*)draft, (int32_t*)accept, (int32_t*)index, (float*)value,
                ws.at, ws.bytes, o.stream);
    }
    return finish(rc, wrap_three, out);
    END_HANDLE_TH_ERRORS
}

// cast(w) -> (q, s), or None: BF16 weights to MXFP4
PyObject* cast(PyObject*, PyObject* w_object)
{
    HANDLE_TH_ERRORS
    if (at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set() ||
        !THPVariable_CheckExact(w_object) || !THPVariable_Unpack(w_object).is_cuda())
        return left();
    const c10::DeviceIndex at = c10::hip::current_device();
    const c10::Device device(c10::kCUDA, at);
    const at::Tensor* w = rows_of(w_object, device);
    if (!w || w->size(0) < 1 || w->size(1) < 32 || w->size(1) % 32 != 0)
        return left();
    const int64_t n = w->size(0), k = w->size(1);
    at::Tensor out[2];
    int rc;
    {
        pybind11::gil_scoped_release no_gil;
        out[0] = fresh({n, k / 2}, at::kByte, device);
        out[1] = fresh({n, k / 32}, at::kByte, device);
        rc = mxfp4_direct_cast(w->data_ptr(), n, k, n > 1 ? w->stride(0) : k, out[0].data_ptr(), out[1].data_ptr(),
                               c10::hip::getCurrentHIPStream(at).stream());
    }
    return finish(rc, wrap_two, out);
    END_HANDLE_TH_ERRORS
}

// on_failure(callable): what raises the error of a status code
PyObject* on_failure(PyObject*, PyObject* f)
{
    Py_INCREF(f);
    Py_XSETREF(g_failed, f);
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"product", (PyCFunction)(void (*)(void))product, METH_FASTCALL, nullptr},
    {"verify", (PyCFunction)(void (*)(void))verify, METH_FASTCALL, nullptr},
    {"cast", cast, METH_O, nullptr},
    {"on_failure", on_failure, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host()
{
    PyObject* module = PyModule_Create(&kModule);
    if (module && PyModule_AddStringConstant(module, "torch_version", MXFP4_TORCH_VERSION) < 0) {
        Py_DECREF(module);
        return nullptr;
    }
    return module;
}
