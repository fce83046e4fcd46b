// The eager calls of ops.py and decoder.py in native code: allocate the outputs, take the pointers and the current stream, call
// the library.  The same calls through torch's Python functions and ctypes cost 8 to 10 us each -- more than most of the
// kernels they launch (a 1536 x 1536 product of one token with its quantizer: 20.9 us a pass for 6.7 us of kernels).
//
// Nothing is decided or checked here that the Python side does not check as well: whatever these functions do not take as it is
// (an operand that is not a plain device tensor, a shape, a dtype) they answer with None BEFORE the library is called, and the
// Python function goes through its own checks and the ctypes binding, which raise what they always raised.  Once the library has
// been called, a status other than BL_OK is the answer, an int that the Python function raises: a second call could do twice
// what the first did in part (the residual form of bl_norm_quant adds into its input).  Nothing is kept between calls.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/TracerMode.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "bitlinear.h"
#include "bitlinear_decoder.h"

namespace {

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// A plain device tensor (torch's own class or its Parameter, no subclass, which may have a word in every torch function, nor any
// while a mode has one; no functorch wrapper), or nullptr.
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o) || at::impl::torch_function_mode_enabled() || c10::impl::dispatch_mode_enabled()) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    const c10::DispatchKeySet keys = t.unsafeGetTensorImpl()->key_set();
    if (!t.is_cuda() || t.layout() != at::kStrided || keys.has(c10::DispatchKey::Python) || keys.has(c10::DispatchKey::FuncTorchBatched) ||
        keys.has(c10::DispatchKey::FuncTorchGradWrapper) || keys.has(c10::DispatchKey::Functionalize))
        return nullptr;
    return &t;
}

// The same, contiguous and of one dtype.
const at::Tensor* plain(PyObject* o, at::ScalarType type) {
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == type && t->is_contiguous() ? t : nullptr;
}

// An output, every byte of which the library writes: straight from the allocator that at::empty asks (plain() has made sure that no mode
// or wrapper has a word in it; a trace still gets to see it).  At four outputs a pass the dispatcher's 0.25 us each were 8 % of a small product with its
// quantizer (11.3 -> 10.4 us).
at::Tensor fresh(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like) {
    if (at::tracer::impl::is_dispatch_enabled()) return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
    return at::Tensor(at::detail::empty_cuda(shape, type, like.device(), std::nullopt));
}

// Memory of a ctypes object (a descriptor, an argument struct, an array of items) for the time of one call.
struct Memory {
    Py_buffer view{};
    bool ok;
    explicit Memory(PyObject* o, size_t least = 1) : ok(PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) == 0) {
        if (!ok) PyErr_Clear();
        else if ((size_t)view.len < least) { PyBuffer_Release(&view); ok = false; }
    }
    ~Memory() { if (ok) PyBuffer_Release(&view); }
    template <typename T> T* as() const { return static_cast<T*>(view.buf); }
};

struct WithoutGil {   // a full queue makes a launch wait
    PyThreadState* state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

// Quantization outputs for M rows of K, either given (all three) or fresh.
struct Quant {
    at::Tensor q, a_scale, q_sum;
    bool take(PyObject* const* given, int64_t M, int64_t K, const at::Tensor& like) {
        if (given[0] == Py_None) {
            const int64_t Kp = bl_padded_k(K);
            if (Kp < 0 || M < 1) return false;
            q = fresh({M, Kp}, at::kChar, like);
            a_scale = fresh({M}, at::kFloat, like);
            q_sum = fresh({M}, at::kInt, like);
            return true;
        }
        const at::Tensor *a = plain(given[0]), *b = plain(given[1]), *c = plain(given[2]);
        if (!a || !b || !c) return false;
        q = *a; a_scale = *b; q_sum = *c;
        return true;
    }
    PyObject* wrap() const {
        PyObject* r = PyTuple_New(3);
        if (!r) return nullptr;
        PyTuple_SET_ITEM(r, 0, THPVariable_Wrap(q));
        PyTuple_SET_ITEM(r, 1, THPVariable_Wrap(a_scale));
        PyTuple_SET_ITEM(r, 2, THPVariable_Wrap(q_sum));
        return r;
    }
};

#define BL_NEEDS(n)                                             \
    if (nargs != (n)) {                                         \
        PyErr_SetString(PyExc_TypeError, "wrong argument count"); \
        return nullptr;                                         \
    }

// quant_act(x, q, a_scale, q_sum) -> (q, a_scale, q_sum); the last three all None for fresh ones
PyObject* quant_act(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    BL_NEEDS(4)
    const at::Tensor* x = plain(args[0]);
    if (!x || x->dim() != 2 || x->stride(1) != 1) Py_RETURN_NONE;
    bl_dtype dt;
    if (x->scalar_type() == at::kFloat) dt = BL_F32;
    else if (x->scalar_type() == at::kBFloat16) dt = BL_BF16;
    else Py_RETURN_NONE;
    const int64_t M = x->size(0), K = x->size(1);
    Quant out;
    if (!out.take(args + 1, M, K, *x)) Py_RETURN_NONE;
    bl_status status;
    void* stream = current_stream();
    {
        WithoutGil release;
        status = bl_quant_act(x->data_ptr(), dt, M, K, x->stride(0), static_cast<int8_t*>(out.q.data_ptr()),
                              static_cast<float*>(out.a_scale.data_ptr()), static_cast<int32_t*>(out.q_sum.data_ptr()), stream);
    }
    if (status != BL_OK) return PyLong_FromLong(status);
    return out.wrap();
    END_HANDLE_TH_ERRORS
}

// product(gemm, blob, desc, q, a_scale, q_sum, out, want_acc) -> (out, acc or None); out may be None
PyObject* product(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    BL_NEEDS(8)
    const bool gemm = args[0] == Py_True, want_acc = PyObject_IsTrue(args[7]) == 1;
    const at::Tensor *blob = plain(args[1]), *q = plain(args[3]), *a = plain(args[4]), *s = plain(args[5]);
    Memory desc(args[2], sizeof(bl_packed_desc));
    if (!blob || !q || !a || !s || !desc.ok || q->dim() != 2) Py_RETURN_NONE;
    const bl_packed_desc* d = desc.as<const bl_packed_desc>();
    const int64_t M = q->size(0), N = d->N;
    if (M < 1 || N < 1) Py_RETURN_NONE;
    at::Tensor out, acc;
    if (args[6] == Py_None) {
        out = fresh({M, N}, at::kFloat, *blob);
    } else {
        const at::Tensor* given = plain(args[6]);
        if (!given) Py_RETURN_NONE;
        out = *given;
    }
    if (want_acc) acc = fresh({M, N}, at::kInt, *blob);
    bl_status status;
    void* stream = current_stream();
    {
        WithoutGil release;
        status = (gemm ? bl_gemm : bl_gemv)(blob->data_ptr(), d, static_cast<const int8_t*>(q->data_ptr()), static_cast<const float*>(a->data_ptr()),
                                            static_cast<const int32_t*>(s->data_ptr()), M, static_cast<float*>(out.data_ptr()),
                                            want_acc ? static_cast<int32_t*>(acc.data_ptr()) : nullptr, stream);
    }
    if (status != BL_OK) return PyLong_FromLong(status);
    PyObject* r = PyTuple_New(2);
    if (!r) return nullptr;
    PyTuple_SET_ITEM(r, 0, THPVariable_Wrap(out));
    if (want_acc) PyTuple_SET_ITEM(r, 1, THPVariable_Wrap(acc));
    else { Py_INCREF(Py_None); PyTuple_SET_ITEM(r, 1, Py_None); }
    return r;
    END_HANDLE_TH_ERRORS
}

// gemm_batch([blob, desc, blob, desc, ...], q, a_scale, q_sum) -> [out, ...]
PyObject* gemm_batch(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    BL_NEEDS(4)
    const at::Tensor *q = plain(args[1]), *a = plain(args[2]), *s = plain(args[3]);
    if (!PyList_Check(args[0]) || !q || !a || !s || q->dim() != 2) Py_RETURN_NONE;
    const Py_ssize_t count = PyList_GET_SIZE(args[0]) / 2;
    if (count < 1 || count > BL_MAX_GEMM_BATCH) Py_RETURN_NONE;
    const int64_t M = q->size(0);
    bl_gemv_item items[BL_MAX_GEMM_BATCH];
    bl_packed_desc descs[BL_MAX_GEMM_BATCH];
    at::Tensor outs[BL_MAX_GEMM_BATCH];
    for (Py_ssize_t i = 0; i < count; ++i) {
        const at::Tensor* blob = plain(PyList_GET_ITEM(args[0], 2 * i));
        Memory desc(PyList_GET_ITEM(args[0], 2 * i + 1), sizeof(bl_packed_desc));
        if (!blob || !desc.ok) Py_RETURN_NONE;
        descs[i] = *desc.as<const bl_packed_desc>();
        if (M < 1 || descs[i].N < 1) Py_RETURN_NONE;
        outs[i] = fresh({M, descs[i].N}, at::kFloat, *q);
        items[i] = {blob->data_ptr(), &descs[i], static_cast<const int8_t*>(q->data_ptr()), static_cast<const float*>(a->data_ptr()),
                    static_cast<const int32_t*>(s->data_ptr()), static_cast<float*>(outs[i].data_ptr()), nullptr};
    }
    bl_status status;
    void* stream = current_stream();
    {
        WithoutGil release;
        status = bl_gemm_batch(items, (int32_t)count, M, stream);
    }
    if (status != BL_OK) return PyLong_FromLong(status);
    PyObject* r = PyList_New(count);
    if (!r) return nullptr;
    for (Py_ssize_t i = 0; i < count; ++i) PyList_SET_ITEM(r, i, THPVariable_Wrap(outs[i]));
    return r;
    END_HANDLE_TH_ERRORS
}

// norm_quant(mode, gamma, eps, a, b, h, q, a_scale, q_sum, y, quantize, scratch) -> (q, a_scale, q_sum), or True without a
// quantizer.  The plain, residual and gated modes; tensors may be None.
PyObject* norm_quant(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    BL_NEEDS(12)
    const long mode = PyLong_AsLong(args[0]);
    const double eps = PyFloat_AsDouble(args[2]);
    if (PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
    if (mode != BL_NORM_PLAIN && mode != BL_NORM_RESIDUAL && mode != BL_NORM_GATED) Py_RETURN_NONE;
    const at::Tensor* ref = plain(args[mode == BL_NORM_RESIDUAL ? 5 : 3], at::kFloat);
    const at::Tensor* gamma = plain(args[1], at::kFloat);
    if (!ref || !gamma || ref->dim() != 2) Py_RETURN_NONE;
    const int64_t M = ref->size(0), K = ref->size(1);
    if (M < 1 || M > INT32_MAX || gamma->dim() != 1 || gamma->size(0) != K) Py_RETURN_NONE;
    bl_norm_quant_args p{};
    void* rows[4] = {nullptr, nullptr, nullptr, nullptr};
    const int at_arg[4] = {3, 4, 5, 9};   // a, b, h, y
    for (int i = 0; i < 4; ++i) {
        if (args[at_arg[i]] == Py_None) continue;
        const at::Tensor* t = plain(args[at_arg[i]], at::kFloat);
        if (!t || t->sizes() != ref->sizes()) Py_RETURN_NONE;
        rows[i] = t->data_ptr();
    }
    if (args[11] != Py_None) {
        const at::Tensor* scratch = plain(args[11]);
        if (!scratch || scratch->numel() * scratch->element_size() < M * BL_NORM_SCRATCH_BYTES) Py_RETURN_NONE;
        p.scratch_dev = scratch->data_ptr();
    }
    const bool quantize = PyObject_IsTrue(args[10]) == 1;
    Quant out;
    if (quantize) {
        if (!out.take(args + 6, M, K, *ref) || out.q.dim() != 2) Py_RETURN_NONE;
        p.q_dev = static_cast<int8_t*>(out.q.data_ptr());
        p.a_scale_dev = static_cast<float*>(out.a_scale.data_ptr());
        p.q_sum_dev = static_cast<int32_t*>(out.q_sum.data_ptr());
        p.Kp = out.q.size(1);
    }
    p.mode = (int32_t)mode;
    p.M = (int32_t)M;
    p.K = K;
    p.a_dev = static_cast<const float*>(rows[0]);
    p.b_dev = static_cast<const float*>(rows[1]);
    p.h_dev = static_cast<float*>(rows[2]);
    p.y_dev = static_cast<float*>(rows[3]);
    p.gamma_dev = static_cast<const float*>(gamma->data_ptr());
    p.eps = (float)eps;
    bl_status status;
    void* stream = current_stream();
    {
        WithoutGil release;
        status = bl_norm_quant(&p, stream);
    }
    if (status != BL_OK) return PyLong_FromLong(status);
    if (!quantize) Py_RETURN_TRUE;
    return out.wrap();
    END_HANDLE_TH_ERRORS
}

// final_norm(h, delta or None, h_out or None, gamma, eps, y, pos, pos_set) -> True
PyObject* final_norm(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    BL_NEEDS(8)
    const double eps = PyFloat_AsDouble(args[4]);
    const long pos_set = PyLong_AsLong(args[7]);
    if (PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
    const at::Tensor *h = plain(args[0], at::kFloat), *gamma = plain(args[3], at::kFloat), *pos = plain(args[6], at::kInt);
    if (!h || !gamma || !pos || h->dim() != 2 || pos->numel() != 1 || pos_set > INT32_MAX) Py_RETURN_NONE;
    const int64_t M = h->size(0), K = h->size(1);
    if (M < 1 || M > INT32_MAX || gamma->dim() != 1 || gamma->size(0) != K) Py_RETURN_NONE;
    void* rows[3] = {nullptr, nullptr, nullptr};
    const int at_arg[3] = {1, 2, 5};   // delta, h_out, y
    for (int i = 0; i < 3; ++i) {
        if (args[at_arg[i]] == Py_None) continue;
        const at::Tensor* t = plain(args[at_arg[i]], at::kFloat);
        if (!t || t->sizes() != h->sizes()) Py_RETURN_NONE;
        rows[i] = t->data_ptr();
    }
    const bl_final_norm_args p{static_cast<const float*>(h->data_ptr()), static_cast<const float*>(rows[0]), static_cast<float*>(rows[1]),
                               static_cast<const float*>(gamma->data_ptr()), static_cast<float*>(rows[2]), K, (int32_t)M, (float)eps,
                               static_cast<int32_t*>(pos->data_ptr()), pos_set < 0 ? -1 : (int32_t)pos_set};
    bl_status status;
    void* stream = current_stream();
    {
        WithoutGil release;
        status = bl_final_norm(&p, stream);
    }
    if (status != BL_OK) return PyLong_FromLong(status);
    Py_RETURN_TRUE;
    END_HANDLE_TH_ERRORS
}

// The prepared launches: launch(which, items, M, workspace) -> bl_status, on the current stream; None if `items`, a ctypes array (for
// the last one the argument struct), does not hold whole ones of that launch's.
enum { kGemvBatch, kDecodeBatch, kQuantBatch, kDecodeNormBatch, kTl2Batch, kAttnDecode, kLaunches };

PyObject* launch(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    BL_NEEDS(4)
    const long which = PyLong_AsLong(args[0]), M = PyLong_AsLong(args[2]);
    void* workspace = PyLong_AsVoidPtr(args[3]);
    if (PyErr_Occurred()) return nullptr;
    constexpr size_t kSizes[kLaunches] = {sizeof(bl_gemv_item), sizeof(bl_decode_item), sizeof(bl_quant_item),
                                          sizeof(bl_decode_norm_item), sizeof(bl_gemv_item), sizeof(bl_attn_args)};
    if (which < 0 || which >= kLaunches) Py_RETURN_NONE;
    Memory items(args[1], kSizes[which]);
    if (!items.ok || items.view.len % kSizes[which] != 0 || items.view.len / kSizes[which] > INT32_MAX) Py_RETURN_NONE;
    const int32_t n = (int32_t)(items.view.len / kSizes[which]);
    void* stream = current_stream();
    bl_status status = BL_ERR_SHAPE;
    {
        WithoutGil release;
        switch (which) {
            case kGemvBatch: status = bl_gemv_batch(items.as<const bl_gemv_item>(), n, M, workspace, stream); break;
            case kDecodeBatch: status = bl_decode_batch(items.as<const bl_decode_item>(), n, M, workspace, stream); break;
            case kQuantBatch: status = bl_quant_act_batch(items.as<const bl_quant_item>(), n, stream); break;
            case kDecodeNormBatch: status = bl_decode_norm_batch(items.as<const bl_decode_norm_item>(), n, workspace, stream); break;
            case kTl2Batch: status = bl_tl2_gemv_batch(items.as<const bl_gemv_item>(), n, workspace, stream); break;
            case kAttnDecode: status = bl_attn_decode(items.as<const bl_attn_args>(), stream); break;
        }
    }
    return PyLong_FromLong(status);
    END_HANDLE_TH_ERRORS
}

PyObject* stream(PyObject*, PyObject*) {
    HANDLE_TH_ERRORS
    return PyLong_FromVoidPtr(current_stream());
    END_HANDLE_TH_ERRORS
}

#define BL_FAST(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {BL_FAST(quant_act), BL_FAST(product), BL_FAST(gemm_batch), BL_FAST(norm_quant), BL_FAST(final_norm), BL_FAST(launch),
                         {"stream", stream, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
