// The binding's per-call work for the plain case of the calls that a decoder makes for every token -- quantize, product, the
// one-launch linears -- in compiled code: a launch of theirs takes 3 us on the GPU, and checks, output tensors and argument
// marshalling in Python took as long as the launch itself (one token against one projection: 6.8 us a call, now 4.7; sixteen tokens through a layer, eight launches: 64, now 44).
//
// Every function returns None for what is not the plain case (a Tensor subclass, a caller's own output or workspace, anything
// that Python code under a mode should see, an argument of another type) and for a call that the library refuses before it launches
// anything: the Python path behind it then takes the call from the start, and raises what it always raised.  An error of the device
// is raised here: the launch has reported it and forgotten it, so that a second try would succeed.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

#include "fp4mr.h"

namespace {

// the library's entry points, handed over by the binding that has loaded it (so that there is one copy of it)
struct Entry {
    decltype(&fp4_rotate_quantize) rotate_quantize;
    decltype(&fp4_quantize_weights) quantize_weights;
    decltype(&fp4_rotate_quantize_dense) rotate_quantize_dense;
    decltype(&fp4_gemm) gemm;
    decltype(&fp4_fused_linear) fused_linear;
    decltype(&fp4_w4a16_linear) w4a16_linear;
    decltype(&fp4_workspace_bytes) workspace_bytes;
    decltype(&fp4_packed_bytes) packed_bytes;
} entry;
PyObject* error;   // the binding's exception, called with a status

// an argument that is a plain Python int in range
bool integer(PyObject* o, int64_t& v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}

// a plain tensor (not a subclass), or with `none` None
bool tensor(PyObject* o, const at::Tensor*& t, bool none = false)
{
    t = nullptr;
    if (none && o == Py_None) return true;
    if (!THPVariable_CheckExact(o)) return false;
    t = &THPVariable_Unpack(o);
    return t->is_cuda();
}

bool bf16_rows(const at::Tensor& x) { return x.scalar_type() == at::kBFloat16 && x.dim() == 2 && x.is_contiguous(); }

void* pointer(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }

at::Tensor empty(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like)
{
    return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}

void* stream() { return c10::hip::getCurrentHIPStream(c10::hip::current_device()).stream(); }

bool plain() { return !at::impl::torch_function_mode_enabled(); }

// what a call returns whose status is not FP4MR_OK
PyObject* refused(fp4mr_status_t status)
{
    if (status != FP4MR_ERR_DEVICE) Py_RETURN_NONE;
    if (PyObject* const e = PyObject_CallFunction(error, "i", (int)status)) {
        PyErr_SetObject(reinterpret_cast<PyObject*>(Py_TYPE(e)), e);
        Py_DECREF(e);
    }
    return nullptr;
}

// quantize(x, had_block, fmt, flags, kind, rot): kind 0 rotate_quantize, 1 quantize_weights, 2 rotate_quantize_dense
PyObject* quantize(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor *x, *rot;
    int64_t b, fmt, flags, kind;
    if (n != 6 || !plain() || !tensor(args[0], x) || !integer(args[1], b) || !integer(args[2], fmt) || !integer(args[3], flags) || !integer(args[4], kind) ||
        !tensor(args[5], rot, true) || !bf16_rows(*x) || (fmt != FP4MR_MXFP4 && fmt != FP4MR_NVFP4) || b < 0 || b > 4096 || flags < 0 || flags > 0xffffffffll ||
        (flags & (FP4MR_SCALE_FIT_RANGE | FP4MR_INPUT_F32 | FP4MR_STATIC_TENSOR_SCALE)) || (kind == 2) != (rot != nullptr) || (rot && (!bf16_rows(*rot) || rot->size(0) != b || rot->size(1) != b)))
        Py_RETURN_NONE;
    const int64_t rows = x->size(0), K = x->size(1);
    size_t code_bytes = 0, scale_bytes = 0;
    if (entry.packed_bytes(rows, K, (fp4mr_fmt_t)fmt, (uint32_t)flags & FP4MR_LAYOUT_GEMM, &code_bytes, &scale_bytes) != FP4MR_OK) Py_RETURN_NONE;
    const at::Tensor codes = empty({(int64_t)code_bytes}, at::kByte, *x), scales = empty({(int64_t)scale_bytes}, at::kByte, *x);
    at::Tensor tensor_scale, workspace;
    if (fmt == FP4MR_NVFP4) tensor_scale = empty({1}, at::kFloat, *x);
    const size_t need = entry.workspace_bytes(kind == 1 ? FP4MR_OP_QUANTIZE_WEIGHTS : FP4MR_OP_ROTATE_QUANTIZE, rows, 0, K, (fp4mr_fmt_t)fmt, (uint32_t)flags);
    if (need) workspace = empty({(int64_t)need}, at::kByte, *x);
    float* const ts = tensor_scale.defined() ? static_cast<float*>(tensor_scale.data_ptr()) : nullptr;
    void* const ws = need ? workspace.data_ptr() : nullptr;
    const void* const px = x->data_ptr();
    void *const pc = codes.data_ptr(), *const ps = scales.data_ptr(), *const pr = pointer(rot), *const st = stream();
    fp4mr_status_t status;
    Py_BEGIN_ALLOW_THREADS;
    if (kind == 2) status = entry.rotate_quantize_dense(px, rows, K, (int)b, pr, (fp4mr_fmt_t)fmt, pc, ps, ts, ws, need, (uint32_t)flags, st);
    else status = (kind == 1 ? entry.quantize_weights : entry.rotate_quantize)(px, rows, K, (int)b, (fp4mr_fmt_t)fmt, pc, ps, ts, ws, need, (uint32_t)flags, st);
    Py_END_ALLOW_THREADS;
    if (status != FP4MR_OK) return refused(status);
    PyObject* const out = PyTuple_New(3);
    if (!out) return nullptr;
    PyTuple_SET_ITEM(out, 0, THPVariable_Wrap(codes));
    PyTuple_SET_ITEM(out, 1, THPVariable_Wrap(scales));
    PyTuple_SET_ITEM(out, 2, THPVariable_Wrap(tensor_scale));   // (an undefined tensor is None)
    for (int i = 0; i < 3; ++i)
        if (!PyTuple_GET_ITEM(out, i)) {
            Py_DECREF(out);
            return nullptr;
        }
    return out;
    END_HANDLE_TH_ERRORS
}

// gemm(a_codes, a_scales, a_tensor_scale, w_codes, w_scales, w_tensor_scale, M, N, K, fmt, flags)
PyObject* gemm(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor *ac, *as, *at_, *wc, *ws, *wt;
    int64_t M, N, K, fmt, flags;
    if (n != 11 || !plain() || !tensor(args[0], ac) || !tensor(args[1], as) || !tensor(args[2], at_, true) || !tensor(args[3], wc) || !tensor(args[4], ws) ||
        !tensor(args[5], wt, true) || !integer(args[6], M) || !integer(args[7], N) || !integer(args[8], K) || !integer(args[9], fmt) || !integer(args[10], flags) ||
        M <= 0 || N <= 0 || K <= 0 || (fmt != FP4MR_MXFP4 && fmt != FP4MR_NVFP4) || flags < 0 || flags > 0xffffffffll)
        Py_RETURN_NONE;
    const at::Tensor out = empty({M, N}, flags & FP4MR_OUT_F32 ? at::kFloat : at::kBFloat16, *ac);
    at::Tensor workspace;
    const size_t need = entry.workspace_bytes(FP4MR_OP_GEMM_FASTEST, M, N, K, (fp4mr_fmt_t)fmt, (uint32_t)flags);
    if (need) workspace = empty({(int64_t)need}, at::kByte, *ac);
    void *const pac = pointer(ac), *const pas = pointer(as), *const pwc = pointer(wc), *const pws = pointer(ws), *const po = out.data_ptr();
    float *const pat = static_cast<float*>(pointer(at_)), *const pwt = static_cast<float*>(pointer(wt));
    void *const pw = need ? workspace.data_ptr() : nullptr, *const st = stream();
    fp4mr_status_t status;
    Py_BEGIN_ALLOW_THREADS;
    status = entry.gemm(pac, pas, pat, pwc, pws, pwt, M, N, K, (fp4mr_fmt_t)fmt, po, pw, need, (uint32_t)flags, st);
    Py_END_ALLOW_THREADS;
    if (status != FP4MR_OK) return refused(status);
    return THPVariable_Wrap(out);
    END_HANDLE_TH_ERRORS
}

// linear(x, had_block, w_codes, w_scales, N, fmt, flags, weight_only)
PyObject* linear(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor *x, *wc, *ws;
    int64_t b, N, fmt, flags, weight_only;
    if (n != 8 || !plain() || !tensor(args[0], x) || !integer(args[1], b) || !tensor(args[2], wc) || !tensor(args[3], ws) || !integer(args[4], N) || !integer(args[5], fmt) ||
        !integer(args[6], flags) || !integer(args[7], weight_only) || !bf16_rows(*x) || b < 0 || b > 4096 || N <= 0 || x->size(0) <= 0 ||
        (fmt != FP4MR_MXFP4 && fmt != FP4MR_NVFP4) || flags < 0 || flags > 0xffffffffll)
        Py_RETURN_NONE;
    const int64_t M = x->size(0), K = x->size(1);
    const at::Tensor out = empty({M, N}, flags & FP4MR_OUT_F32 ? at::kFloat : at::kBFloat16, *x);
    const void* const px = x->data_ptr();
    void *const pwc = pointer(wc), *const pws = pointer(ws), *const po = out.data_ptr(), *const st = stream();
    fp4mr_status_t status;
    Py_BEGIN_ALLOW_THREADS;
    status = (weight_only ? entry.w4a16_linear : entry.fused_linear)(px, M, K, (int)b, pwc, pws, N, (fp4mr_fmt_t)fmt, po, (uint32_t)flags | FP4MR_W_LAYOUT_GEMM, st);
    Py_END_ALLOW_THREADS;
    if (status != FP4MR_OK) return refused(status);
    return THPVariable_Wrap(out);
    END_HANDLE_TH_ERRORS
}

// bind(addresses of the eight entry points, in the order of Entry, and the exception)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    constexpr Py_ssize_t count = sizeof(Entry) / sizeof(void*);
    if (n != count + 1 || !PyCallable_Check(args[count])) {
        PyErr_SetString(PyExc_TypeError, "bind() takes eight addresses and an exception");
        return nullptr;
    }
    void* p[count];
    for (Py_ssize_t i = 0; i < count; ++i) {
        p[i] = PyLong_AsVoidPtr(args[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a null entry point");
            return nullptr;
        }
    }
    static_assert(sizeof(p) == sizeof(entry), "one address per entry point");
    std::memcpy(&entry, p, sizeof(entry));
    Py_INCREF(args[count]);
    Py_XSETREF(error, args[count]);
    Py_RETURN_NONE;
}

template <typename F>
PyCFunction method(F f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }

PyMethodDef methods[] = {{"bind", method(bind), METH_FASTCALL, nullptr},
                         {"quantize", method(quantize), METH_FASTCALL, nullptr},
                         {"gemm", method(gemm), METH_FASTCALL, nullptr},
                         {"linear", method(linear), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
