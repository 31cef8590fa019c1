// The calls of the Python binding that a model makes per layer or per step, without the interpreter between the tensors and the C ABI:
// checks, output allocation and the call itself.  What a call costs the host besides its launches decides the time of a small
// layer.  (Per call, checks in Python and ctypes -> here, on the host of an MI355X: w4ax_gemm 9.4 -> 4.7 us, with its output given 7.9 ->
// 3.8; rotate_quant with code sums 10.5 -> 6.3; of these a launch is 3.6, an allocation 1.  Passes of small layers: 128 x 256 x 256
// 9.0 -> 6.2, the quantizer and three GEMMs of 9 x 384 x 808 38 -> 21.)
//
// Only the plain case is handled: every tensor a torch.Tensor of the expected type, shape and layout on the GPU, no modes
// active.  Anything else returns None, and the Python function goes through its own checks, which raise what there is to
// raise.  A status other than 0 is returned as an int.
#include <Python.h>
#include <stdint.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>

#include "../../include/dvdq.h"

namespace {

decltype(&dvdq_rotate_quant) p_rotate_quant;
decltype(&dvdq_rotate_quant_blockwise) p_rotate_quant_blockwise;
decltype(&dvdq_w4ax_gemm) p_w4ax_gemm;
decltype(&dvdq_qlinear) p_qlinear;
decltype(&dvdq_gbs_reset) p_gbs_reset;
decltype(&dvdq_gbs_step) p_gbs_step;
decltype(&dvdq_codes_bytes) p_codes_bytes;
decltype(&dvdq_qlinear_workspace_bytes) p_qlinear_workspace_bytes;
decltype(&dvdq_w4_native_bytes) p_w4_native_bytes;
decltype(&dvdq_w4_native_fp6_bytes) p_w4_native_fp6_bytes;

PyObject *get_device, *get_raw_stream;   // torch._C's: number of the current device; its current stream's handle

// Arguments of a call.  `ok` turns false at the first that is not the plain case.
struct Args {
    PyObject *const *a;
    bool ok;

    Args(PyObject *const *args, Py_ssize_t n, Py_ssize_t wanted)
        : a(args), ok(n == wanted && at::impl::PythonTorchFunctionTLS::stack_len() == 0 &&
                      c10::impl::TorchDispatchModeTLS::stack_len() == 0) {}

    bool none(int i) const { return a[i] == Py_None; }
    // a contiguous GPU tensor of this type, else nullptr; None only if `optional`, and then nullptr too
    const at::Tensor *tensor(int i, at::ScalarType type, bool optional = false) {
        if (!ok || (optional && none(i))) return nullptr;
        if (THPVariable_CheckExact(a[i])) {
            const at::Tensor &t = THPVariable_Unpack(a[i]);
            static const c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                                      c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                                      c10::DispatchKey::Conjugate, c10::DispatchKey::Negative,
                                                      c10::DispatchKey::ZeroTensor});
            if (t.is_cuda() && t.scalar_type() == type && t.layout() == at::kStrided && t.is_contiguous() &&
                !t.key_set().has_any(wrapped) && t.has_storage())
                return &t;
        }
        ok = false;
        return nullptr;
    }
    void require(bool c) { ok = ok && c; }
    int64_t integer(int i) {
        if (!ok) return 0;
        int overflow = 0;
        const int64_t v = PyLong_Check(a[i]) ? PyLong_AsLongLongAndOverflow(a[i], &overflow) : (ok = false, 0);
        if (overflow) ok = false;
        return v;
    }
    int small(int i) {
        const int64_t v = integer(i);
        if (v != (int)v) ok = false;
        return (int)v;
    }
    // the handle of a torch.cuda.Stream, or of the current one for None; asked for last, when the tensors are known to be on a GPU
    void *stream(int i) {
        if (!ok) return nullptr;
        PyObject *handle = nullptr;
        if (none(i)) {
            if (PyObject *device = PyObject_CallNoArgs(get_device)) {
                handle = PyObject_CallOneArg(get_raw_stream, device);
                Py_DECREF(device);
            }
        } else {
            handle = PyObject_GetAttrString(a[i], "cuda_stream");
        }
        void *p = handle && PyLong_Check(handle) ? PyLong_AsVoidPtr(handle) : (ok = false, nullptr);
        Py_XDECREF(handle);
        if (PyErr_Occurred()) {   // (the Python function will meet it again)
            PyErr_Clear();
            ok = false;
        }
        return p;
    }
    // the given output, or a new one on the device of `like`
    at::Tensor output(int i, at::ScalarType type, at::IntArrayRef shape, const at::Tensor &like) {
        if (none(i)) return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
        const at::Tensor *t = tensor(i, type);
        if (!t || t->sizes() != shape) {
            ok = false;
            return at::Tensor();
        }
        return *t;
    }
};

inline void *ptr(const at::Tensor *t) { return t ? t->data_ptr() : nullptr; }
inline bool vector_of(const at::Tensor *t, int64_t n) { return t->dim() == 1 && t->size(0) == n; }

template <class F>
int unlocked(F f) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

// the caller's own object where it gave one
PyObject *object(PyObject *given, const at::Tensor &t) {
    if (given == Py_None) return THPVariable_Wrap(t);
    Py_INCREF(given);
    return given;
}

// whether the weight buffer holds what the kernels read
bool weights_fit(const at::Tensor &w, int layout, int64_t N, int64_t K) {
    if (layout == DVDQ_W_CANONICAL) return w.dim() == 2 && w.size(0) == N && w.size(1) == K / 2;
    if (layout != DVDQ_W_NATIVE && layout != DVDQ_W_NATIVE_FP6) return false;
    const size_t need = layout == DVDQ_W_NATIVE ? p_w4_native_bytes(N, K) : p_w4_native_fp6_bytes(N, K);
    return need != 0 && (size_t)w.numel() >= need;
}

struct CodesSpec { at::ScalarType type; int64_t shape[2]; int dim; };
// (M, K: the token and channel counts)
CodesSpec codes_spec(int64_t M, int64_t K, int format) {
    if (format == DVDQ_CODES_PACKED4) return {at::kByte, {M, K / 2}, 2};
    if (format == DVDQ_CODES_FP6) return {at::kByte, {(int64_t)p_codes_bytes(M, K, DVDQ_CODES_FP6), 0}, 1};
    return {at::kChar, {M, K}, 2};
}

// x, w, w_scale, had_block, act_bits, w_layout, bias, y, workspace, codes_format, w_zero, stream -> (y, workspace)
PyObject *qlinear(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Args a(args, n, 12);
    const at::Tensor *x = a.tensor(0, at::kBFloat16), *w = a.tensor(1, at::kByte), *ws = a.tensor(2, at::kFloat);
    const int had = a.small(3), bits = a.small(4), layout = a.small(5), format = a.small(9);
    const at::Tensor *bias = a.tensor(6, at::kBFloat16, true), *zero = a.tensor(10, at::kChar, true);
    if (!a.ok || x->dim() != 2 || ws->dim() < 1 || format < 0 || format > 2) Py_RETURN_NONE;
    const int64_t M = x->size(0), K = x->size(1), N = ws->size(0);
    if (!weights_fit(*w, layout, N, K) || (bias && !vector_of(bias, N)) || (zero && !vector_of(zero, N))) Py_RETURN_NONE;
    at::Tensor workspace;
    if (a.none(8)) {
        workspace = at::empty({(int64_t)p_qlinear_workspace_bytes(M, K, format)}, at::TensorOptions().dtype(at::kByte).device(x->device()));
    } else {
        const at::Tensor *t = a.tensor(8, at::kByte);
        if (!t) Py_RETURN_NONE;
        workspace = *t;
    }
    const at::Tensor y = a.output(7, at::kBFloat16, {M, N}, *x);
    void *stream = a.stream(11);
    if (!a.ok) Py_RETURN_NONE;
    const int rc = unlocked([&] {
        return p_qlinear(x->data_ptr(), (const uint8_t *)ptr(w), (const float *)ptr(ws), (const int8_t *)ptr(zero), ptr(bias), M, N, K, had,
                         bits, format, layout, y.data_ptr(), workspace.data_ptr(), (size_t)workspace.numel(), stream);
    });
    if (rc != 0) return PyLong_FromLong(rc);
    return Py_BuildValue("(NN)", object(args[7], y), object(args[8], workspace));
    END_HANDLE_TH_ERRORS
}

// x, had_block, act_bits, codes, x_scale, stream, codes_format, code_rowsum, want_rowsum -> (codes, x_scale[, code_rowsum])
PyObject *rotate_quant(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Args a(args, n, 9);
    const at::Tensor *x = a.tensor(0, at::kBFloat16);
    const int had = a.small(1), bits = a.small(2), format = a.small(6);
    if (!a.ok || x->dim() != 2 || format < 0 || format > 2) Py_RETURN_NONE;
    const int64_t M = x->size(0), K = x->size(1);
    const bool sums = args[8] == Py_True || !a.none(7);
    if (args[8] != Py_True && args[8] != Py_False) Py_RETURN_NONE;
    const CodesSpec spec = codes_spec(M, K, format);
    const at::Tensor codes = a.output(3, spec.type, at::IntArrayRef(spec.shape, spec.dim), *x), scale = a.output(4, at::kFloat, {M}, *x);
    at::Tensor rowsum;
    if (sums && a.ok) rowsum = a.output(7, at::kInt, {M}, *x);
    void *stream = a.stream(5);
    if (!a.ok) Py_RETURN_NONE;
    const int rc = unlocked([&] {
        return p_rotate_quant(x->data_ptr(), M, K, had, bits, format, (int8_t *)codes.data_ptr(), (float *)scale.data_ptr(),
                              sums ? (int32_t *)rowsum.data_ptr() : nullptr, stream);
    });
    if (rc != 0) return PyLong_FromLong(rc);
    if (sums) return Py_BuildValue("(NNN)", object(args[3], codes), object(args[4], scale), object(args[7], rowsum));
    return Py_BuildValue("(NN)", object(args[3], codes), object(args[4], scale));
    END_HANDLE_TH_ERRORS
}

// x, had_block, act_bits, group, values, x_scale, want_rowsum, stream -> (values, x_scale[, rowsum])
PyObject *rotate_quant_blockwise(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Args a(args, n, 8);
    const at::Tensor *x = a.tensor(0, at::kBFloat16);
    const int had = a.small(1), bits = a.small(2), group = a.small(3);
    if (!a.ok || x->dim() != 2 || (args[6] != Py_True && args[6] != Py_False)) Py_RETURN_NONE;
    const int64_t M = x->size(0), K = x->size(1);
    const bool sums = args[6] == Py_True;
    const at::Tensor values = a.output(4, at::kChar, {M, K}, *x), scale = a.output(5, at::kFloat, {M}, *x);
    at::Tensor rowsum;
    void *stream = a.stream(7);
    if (!a.ok) Py_RETURN_NONE;
    if (sums) rowsum = at::empty({M}, at::TensorOptions().dtype(at::kInt).device(x->device()));
    const int rc = unlocked([&] {
        return p_rotate_quant_blockwise(x->data_ptr(), M, K, had, bits, group, (int8_t *)values.data_ptr(), (float *)scale.data_ptr(),
                                        sums ? (int32_t *)rowsum.data_ptr() : nullptr, stream);
    });
    if (rc != 0) return PyLong_FromLong(rc);
    if (sums) return Py_BuildValue("(NNN)", object(args[4], values), object(args[5], scale), THPVariable_Wrap(rowsum));
    return Py_BuildValue("(NN)", object(args[4], values), object(args[5], scale));
    END_HANDLE_TH_ERRORS
}

// codes, x_scale, w, w_scale, act_bits, w_layout, bias, y, stream, codes_format, w_zero, code_rowsum, K -> y
PyObject *w4ax_gemm(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Args a(args, n, 13);
    const int bits = a.small(4), layout = a.small(5), format = a.small(9);
    a.require(format >= 0 && format <= 2);
    const at::Tensor *codes = a.tensor(0, format == DVDQ_CODES_INT8 ? at::kChar : at::kByte), *scale = a.tensor(1, at::kFloat),
                     *w = a.tensor(2, at::kByte), *ws = a.tensor(3, at::kFloat), *bias = a.tensor(6, at::kBFloat16, true),
                     *zero = a.tensor(10, at::kChar, true), *rowsum = a.tensor(11, at::kInt, true);
    if (!a.ok || ws->dim() < 1) Py_RETURN_NONE;
    int64_t M, K;
    if (format == DVDQ_CODES_FP6) {
        K = a.integer(12);
        if (!a.ok || scale->dim() != 1) Py_RETURN_NONE;
        M = scale->size(0);
        if (codes->numel() < (int64_t)p_codes_bytes(M, K, DVDQ_CODES_FP6)) Py_RETURN_NONE;
    } else {
        if (codes->dim() != 2) Py_RETURN_NONE;
        M = codes->size(0);
        K = codes->size(1) * (format == DVDQ_CODES_PACKED4 ? 2 : 1);
    }
    const int64_t N = ws->size(0);
    if (!vector_of(scale, M) || !weights_fit(*w, layout, N, K) || (bias && !vector_of(bias, N)) || (zero && !vector_of(zero, N)) ||
        (zero && !rowsum) || (rowsum && !vector_of(rowsum, M)))
        Py_RETURN_NONE;
    const at::Tensor y = a.output(7, at::kBFloat16, {M, N}, *codes);
    void *stream = a.stream(8);
    if (!a.ok) Py_RETURN_NONE;
    const int rc = unlocked([&] {
        return p_w4ax_gemm((const int8_t *)ptr(codes), (const float *)ptr(scale), (const uint8_t *)ptr(w), (const float *)ptr(ws),
                           (const int8_t *)ptr(zero), (const int32_t *)ptr(rowsum), ptr(bias), M, N, K, bits, format, layout,
                           y.data_ptr(), nullptr, stream);
    });
    if (rc != 0) return PyLong_FromLong(rc);
    return object(args[7], y);
    END_HANDLE_TH_ERRORS
}

// state, bits, stream -> status
PyObject *gbs_reset(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Args a(args, n, 3);
    const at::Tensor *state = a.tensor(0, at::kByte);
    const int bits = a.small(1);
    void *stream = a.stream(2);
    if (!a.ok) Py_RETURN_NONE;
    return PyLong_FromLong(unlocked([&] { return p_gbs_reset(state->data_ptr(), bits, stream); }));
    END_HANDLE_TH_ERRORS
}

// f_t, f_prev, delta, b_low, b_high, state, workspace, stream -> status
PyObject *gbs_step(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Args a(args, n, 8);
    const at::Tensor *f_t = a.tensor(0, at::kBFloat16), *f_prev = a.tensor(1, at::kBFloat16), *state = a.tensor(5, at::kByte),
                     *workspace = a.tensor(6, at::kByte);
    const int b_low = a.small(3), b_high = a.small(4);
    void *stream = a.stream(7);
    if (!a.ok || !PyFloat_CheckExact(args[2]) || f_t->sizes() != f_prev->sizes()) Py_RETURN_NONE;
    const float delta = (float)PyFloat_AS_DOUBLE(args[2]);
    return PyLong_FromLong(unlocked([&] {
        return p_gbs_step(f_t->data_ptr(), f_prev->data_ptr(), f_t->numel(), delta, b_low, b_high, state->data_ptr(),
                          workspace->data_ptr(), (size_t)workspace->numel(), stream);
    }));
    END_HANDLE_TH_ERRORS
}

// torch._C._cuda_getDevice and _cuda_getCurrentRawStream, then the addresses of the C functions in the library that the binding has
// loaded, in this order.
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n) {
    void **const to[] = {(void **)&p_rotate_quant, (void **)&p_rotate_quant_blockwise, (void **)&p_w4ax_gemm, (void **)&p_qlinear,
                         (void **)&p_gbs_reset, (void **)&p_gbs_step, (void **)&p_codes_bytes, (void **)&p_qlinear_workspace_bytes,
                         (void **)&p_w4_native_bytes, (void **)&p_w4_native_fp6_bytes};
    constexpr Py_ssize_t kFunctions = sizeof(to) / sizeof(to[0]);
    if (n != 2 + kFunctions) {
        PyErr_SetString(PyExc_TypeError, "bind: two callables and ten addresses");
        return nullptr;
    }
    Py_INCREF(args[0]);
    Py_INCREF(args[1]);
    get_device = args[0];
    get_raw_stream = args[1];
    for (Py_ssize_t i = 0; i < kFunctions; ++i) {
        *to[i] = PyLong_AsVoidPtr(args[2 + i]);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_RETURN_NONE;
}

#define DVDQ_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {DVDQ_METHOD(bind), DVDQ_METHOD(qlinear), DVDQ_METHOD(rotate_quant), DVDQ_METHOD(rotate_quant_blockwise),
                         DVDQ_METHOD(w4ax_gemm), DVDQ_METHOD(gbs_reset), DVDQ_METHOD(gbs_step), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
