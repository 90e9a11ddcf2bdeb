// The per-call half of binding.py in C++: checks the tensors, allocates the results, takes torch's current
// stream and calls the C ABI (include/morph.h), whose addresses bind() hands over once at load time.
//
// A decode linear lasts 5 to 20 us on the device; the same marshalling in Python (attribute look-ups, ctypes
// conversions, torch.empty) took about 10 us of host time per call, so that calls in a row were paced by the
// host.  Here it is 1 us on top of the launch itself: M = 1, 4096 x 4096, 4-bit went from 10.5 to 5.7 us a call.
//
// Every function returns its result, or None when anything is not as the call wants it (type, device, shape,
// contiguity, or the library refuses it: nothing was launched then); binding.py goes through its checked
// path on None, which names what is wrong.  MORPH_ERR_DEVICE is no refusal: something may have been launched, and the
// error is the runtime's last, which asking has cleared.  It is raised here; a second call would run the work again and report success.
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>

#include "../../include/morph.h"

namespace {

using DenseFn = decltype(&morph_linear_fp16);
using QuantFn = decltype(&morph_linear_w8a16);
using NativeFn = decltype(&morph_linear_w4a16_native);

enum { F_DENSE = 0, F_W4, F_W8, F_NATIVE, F_DENSE_BF, F_W4_BF, F_W8_BF, F_NATIVE_BF, F_GLUE, F_GLUE_BF, F_COSINE, F_COSINE_BF,
       F_QUANT_W4, F_QUANT_W8, F_QUANT_NATIVE, F_DEQ_W4, F_DEQ_W8, F_DEQ_NATIVE, F_NATIVE_BYTES, F_COUNT };
const char* const kName[F_COUNT] = {
    "morph_linear_fp16", "morph_linear_w4a16", "morph_linear_w8a16", "morph_linear_w4a16_native",
    "morph_linear_bf16", "morph_linear_w4a16_bf16", "morph_linear_w8a16_bf16", "morph_linear_w4a16_native_bf16",
    "morph_glue", "morph_glue_bf16", "morph_cosine_rows", "morph_cosine_rows_bf16",
    "morph_quantize_layer", "morph_quantize_layer_w8", "morph_quantize_layer_native_only",
    "morph_dequantize_w4", "morph_dequantize_w8", "morph_dequantize_w4_native", "morph_w4_native_bytes"};
void* g_fn[F_COUNT];
PyObject* g_error;                                       // binding.MorphError
constexpr int64_t kGroup = MORPH_GROUP_SIZE;
constexpr int64_t kMaxInt = 0x7FFFFFFF;

inline void* stream_now() { return c10::hip::getCurrentHIPStream().stream(); }

inline const at::Tensor* tensor_of(PyObject* o) { return THPVariable_Check(o) ? &THPVariable_Unpack(o) : nullptr; }

inline bool usable(const at::Tensor* t, at::ScalarType dt)
{
    return t && t->is_cuda() && t->scalar_type() == dt && t->is_contiguous();
}

inline at::Tensor fresh(at::IntArrayRef size, at::ScalarType dt, const at::Tensor& like)
{
    return at::Tensor(at::detail::empty_cuda(size, dt, like.device(), std::nullopt));
}

inline PyObject* none()
{
    PyErr_Clear();
    Py_RETURN_NONE;
}

// a status other than MORPH_OK: None after a refusal, the exception after a failure
PyObject* refused(int rc, long which)
{
    if (rc != MORPH_ERR_DEVICE) return none();
    PyErr_Clear();
    if (!g_error) PyErr_Format(PyExc_RuntimeError, "%s: status %d", kName[which], rc);
    else if (PyObject* e = PyObject_CallFunction(g_error, "is", rc, kName[which])) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

// The C ABI runs without the interpreter's lock, as under ctypes: a launch that waits for room in a full queue
// must not stop the thread whose work would empty it.
template <class Fn, class... Args>
int unlocked(Fn fn, Args... args)
{
    PyThreadState* ts = PyEval_SaveThread();
    const int rc = fn(args...);                          // (C functions: nothing is thrown)
    PyEval_RestoreThread(ts);
    return rc;
}

// A C++ exception (an allocation that fails) becomes Python's in the checked path, which meets it again.
template <class F>
PyObject* guarded(F&& f)
{
    try {
        return f();
    } catch (...) {
        return none();
    }
}

bool dtype_code(at::ScalarType dt, int* code)
{
    switch (dt) {
        case at::kFloat: *code = MORPH_DTYPE_F32; return true;
        case at::kHalf: *code = MORPH_DTYPE_F16; return true;
        case at::kBFloat16: *code = MORPH_DTYPE_BF16; return true;
        default: return false;
    }
}

// linear(which, x, w, scales, qzeros, ws, out, group_size): which = F_DENSE .. F_NATIVE_BF; scales and qzeros None for dense weights
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        if (n != 8) return none();
        const long which = PyLong_AsLong(a[0]);
        if (which < F_DENSE || which > F_NATIVE_BF) return none();
        const bool bf = which >= F_DENSE_BF;
        const int  kind = (int)which & 3;
        const at::ScalarType act = bf ? at::kBFloat16 : at::kHalf;
        const at::Tensor *x = tensor_of(a[1]), *w = tensor_of(a[2]);
        if (!usable(x, act) || x->dim() != 2) return none();
        const int64_t M = x->size(0), K = x->size(1);
        int64_t N;
        const at::Tensor *s = nullptr, *z = nullptr;
        if (kind == F_DENSE) {
            if (!usable(w, act) || w->dim() != 2 || w->size(0) != K) return none();
            N = w->size(1);
        } else {
            s = tensor_of(a[3]);
            z = tensor_of(a[4]);
            if (!usable(s, at::kHalf) || s->dim() != 2 || !usable(z, at::kInt)) return none();
            N = s->size(1);
            if (K > kMaxInt || N > kMaxInt) return none();
            if (kind == F_NATIVE) {
                if (!usable(w, at::kByte) || (size_t)w->numel() != ((decltype(&morph_w4_native_bytes))g_fn[F_NATIVE_BYTES])((int)K, (int)N)) return none();
            } else if (!usable(w, at::kInt) || w->dim() != 2 || w->size(0) != K || w->size(1) != N / (kind == F_W4 ? 8 : 4)) return none();
        }
        if (M > kMaxInt || K > kMaxInt || N > kMaxInt) return none();
        void*  wp = nullptr;
        size_t wb = 0;
        if (a[5] != Py_None) {
            const at::Tensor* ws = tensor_of(a[5]);
            if (!ws || ws->element_size() != 1) return none();
            wp = ws->data_ptr();
            wb = (size_t)ws->numel();
        }
        const long group = PyLong_AsLong(a[7]);
        at::Tensor made;
        const at::Tensor* y;
        if (a[6] == Py_None) {
            made = fresh({M, N}, act, *x);
            y = &made;
        } else {
            y = tensor_of(a[6]);
            if (!usable(y, act)) return none();
        }
        int rc;
        if (kind == F_DENSE)
            rc = unlocked((DenseFn)g_fn[which], x->data_ptr(), w->data_ptr(), y->data_ptr(), (int)M, (int)K, (int)N, wp, wb, stream_now());
        else if (kind == F_NATIVE)
            rc = unlocked((NativeFn)g_fn[which], x->data_ptr(), w->data_ptr(), s->data_ptr(), (const int32_t*)z->data_ptr(), y->data_ptr(), (int)M,
                                         (int)K, (int)N, (int)group, wp, wb, stream_now());
        else
            rc = unlocked((QuantFn)g_fn[which], x->data_ptr(), (const int32_t*)w->data_ptr(), s->data_ptr(), (const int32_t*)z->data_ptr(), y->data_ptr(),
                                        (int)M, (int)K, (int)N, (int)group, wp, wb, stream_now());
        if (rc != MORPH_OK) return refused(rc, which);
        if (a[6] != Py_None) {
            Py_INCREF(a[6]);
            return a[6];
        }
        return THPVariable_Wrap(std::move(made));
    });
}

// glue(op, a, b, H): b and H may be None
PyObject* glue(PyObject*, PyObject* const* v, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        if (n != 4) return none();
        const long op = PyLong_AsLong(v[0]);
        const at::Tensor *a = tensor_of(v[1]), *b = v[2] == Py_None ? nullptr : tensor_of(v[2]);
        if (!a || a->dim() != 2 || (v[2] != Py_None && !b)) return none();
        const at::ScalarType dt = a->scalar_type();
        if ((dt != at::kHalf && dt != at::kBFloat16) || !usable(a, dt) || (b && !usable(b, dt))) return none();
        const int64_t M = a->size(0);
        const int64_t H = v[3] == Py_None ? a->size(1) / (op == MORPH_GLUE_QKV ? 3 : op == MORPH_GLUE_SWIGLU ? 2 : 1) : PyLong_AsLong(v[3]);
        if (M > kMaxInt || H < 0 || H > kMaxInt) return none();
        at::Tensor out = fresh({M, H}, dt, *a);
        const int which = dt == at::kBFloat16 ? F_GLUE_BF : F_GLUE;
        const int rc = unlocked((decltype(&morph_glue))g_fn[which],
            (int)op, a->data_ptr(), b ? b->data_ptr() : nullptr, out.data_ptr(), (int)M, (int)H, stream_now());
        return rc == MORPH_OK ? THPVariable_Wrap(std::move(out)) : refused(rc, which);
    });
}

// cosine_rows(a, b) -> (cos, mean)
PyObject* cosine_rows(PyObject*, PyObject* const* v, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        if (n != 2) return none();
        const at::Tensor *a = tensor_of(v[0]), *b = tensor_of(v[1]);
        if (!a || !b || a->dim() != 2 || b->dim() != 2) return none();
        const at::ScalarType dt = a->scalar_type();
        if ((dt != at::kHalf && dt != at::kBFloat16) || !usable(a, dt) || !usable(b, dt) || a->sizes() != b->sizes()) return none();
        const int64_t M = a->size(0), H = a->size(1);
        if (M > kMaxInt || H > kMaxInt) return none();
        at::Tensor cos = fresh({M}, at::kFloat, *a), mean = fresh({1}, at::kFloat, *a);
        const int which = dt == at::kBFloat16 ? F_COSINE_BF : F_COSINE;
        const int rc = unlocked((decltype(&morph_cosine_rows))g_fn[which],
            a->data_ptr(), b->data_ptr(), (float*)cos.data_ptr(), (float*)mean.data_ptr(), (int)M, (int)H, stream_now());
        if (rc != MORPH_OK) return refused(rc, which);
        PyObject* t = PyTuple_New(2);
        if (!t) return nullptr;
        PyTuple_SET_ITEM(t, 0, THPVariable_Wrap(std::move(cos)));
        PyTuple_SET_ITEM(t, 1, THPVariable_Wrap(std::move(mean)));
        return t;
    });
}

// quantize(which, w, group_size) -> (codes, scales, zeros): which = F_QUANT_W4, _W8, _NATIVE
PyObject* quantize(PyObject*, PyObject* const* v, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        if (n != 3) return none();
        const long which = PyLong_AsLong(v[0]), group = PyLong_AsLong(v[2]);
        if (which < F_QUANT_W4 || which > F_QUANT_NATIVE) return none();
        const at::Tensor* w = tensor_of(v[1]);
        int code;
        if (!w || !dtype_code(w->scalar_type(), &code) || !usable(w, w->scalar_type()) || w->dim() != 2) return none();
        const int64_t K = w->size(0), N = w->size(1), per_word = which == F_QUANT_W8 ? 4 : 8;
        if (K < kGroup || K % kGroup || N < 8 || N % 8 || K > kMaxInt || N > kMaxInt) return none();
        at::Tensor q, s = fresh({K / kGroup, N}, at::kHalf, *w), z = fresh({K / kGroup, N / per_word}, at::kInt, *w);
        int rc;
        if (which == F_QUANT_NATIVE) {
            q = fresh({(int64_t)((decltype(&morph_w4_native_bytes))g_fn[F_NATIVE_BYTES])((int)K, (int)N)}, at::kByte, *w);
            rc = unlocked((decltype(&morph_quantize_layer_native_only))g_fn[which], w->data_ptr(), code, q.data_ptr(), s.data_ptr(), (int32_t*)z.data_ptr(),
                                                                            (int)K, (int)N, (int)group, stream_now());
        } else {
            q = fresh({K, N / per_word}, at::kInt, *w);
            rc = unlocked((decltype(&morph_quantize_layer))g_fn[which], w->data_ptr(), code, (int32_t*)q.data_ptr(), s.data_ptr(), (int32_t*)z.data_ptr(),
                                                                (int)K, (int)N, (int)group, stream_now());
        }
        if (rc != MORPH_OK) return refused(rc, which);
        PyObject* t = PyTuple_New(3);
        if (!t) return nullptr;
        PyTuple_SET_ITEM(t, 0, THPVariable_Wrap(std::move(q)));
        PyTuple_SET_ITEM(t, 1, THPVariable_Wrap(std::move(s)));
        PyTuple_SET_ITEM(t, 2, THPVariable_Wrap(std::move(z)));
        return t;
    });
}

// dequantize(which, codes, scales, zeros, dtype code, group_size) -> [K, N]: which = F_DEQ_W4, _W8, _NATIVE
PyObject* dequantize(PyObject*, PyObject* const* v, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        if (n != 6) return none();
        const long which = PyLong_AsLong(v[0]), code = PyLong_AsLong(v[4]), group = PyLong_AsLong(v[5]);
        if (which < F_DEQ_W4 || which > F_DEQ_NATIVE || code < MORPH_DTYPE_F32 || code > MORPH_DTYPE_BF16) return none();
        const at::Tensor *q = tensor_of(v[1]), *s = tensor_of(v[2]), *z = tensor_of(v[3]);
        if (!usable(q, which == F_DEQ_NATIVE ? at::kByte : at::kInt) || !usable(s, at::kHalf) || s->dim() != 2 || !usable(z, at::kInt)) return none();
        const int64_t N = s->size(1), K = s->size(0) * kGroup;
        if (K > kMaxInt || N > kMaxInt || (which != F_DEQ_NATIVE && (q->dim() != 2 || q->size(0) != K))) return none();
        at::Tensor out = fresh({K, N}, code == MORPH_DTYPE_F32 ? at::kFloat : code == MORPH_DTYPE_F16 ? at::kHalf : at::kBFloat16, *q);
        int rc;
        if (which == F_DEQ_NATIVE)
            rc = unlocked((decltype(&morph_dequantize_w4_native))g_fn[which], q->data_ptr(), s->data_ptr(), (const int32_t*)z->data_ptr(), out.data_ptr(),
                                                                      (int)code, (int)K, (int)N, (int)group, stream_now());
        else
            rc = unlocked((decltype(&morph_dequantize_w4))g_fn[which], (const int32_t*)q->data_ptr(), s->data_ptr(), (const int32_t*)z->data_ptr(),
                                                               out.data_ptr(), (int)code, (int)K, (int)N, (int)group, stream_now());
        return rc == MORPH_OK ? THPVariable_Wrap(std::move(out)) : refused(rc, which);
    });
}

// bind(addresses): the C ABI functions in the order of the enumeration above
PyObject* bind(PyObject*, PyObject* list)
{
    if (!PyList_Check(list) || PyList_GET_SIZE(list) != F_COUNT) {
        PyErr_SetString(PyExc_ValueError, "bind() takes a list of the library's function addresses");
        return nullptr;
    }
    void* got[F_COUNT];
    for (int i = 0; i < F_COUNT; i++) {
        got[i] = PyLong_AsVoidPtr(PyList_GET_ITEM(list, i));
        if (!got[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind(): a NULL address");
            return nullptr;
        }
    }
    for (int i = 0; i < F_COUNT; i++) g_fn[i] = got[i];
    Py_RETURN_NONE;
}

// errors(cls): the exception that a failure raises, called with the status and the function's name
PyObject* errors(PyObject*, PyObject* cls)
{
    Py_INCREF(cls);
    PyObject* was = g_error;
    g_error = cls;
    Py_XDECREF(was);
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"bind", bind, METH_O, nullptr},
    {"errors", errors, METH_O, nullptr},
    {"linear", (PyCFunction)(void*)linear, METH_FASTCALL, nullptr},
    {"glue", (PyCFunction)(void*)glue, METH_FASTCALL, nullptr},
    {"cosine_rows", (PyCFunction)(void*)cosine_rows, METH_FASTCALL, nullptr},
    {"quantize", (PyCFunction)(void*)quantize, METH_FASTCALL, nullptr},
    {"dequantize", (PyCFunction)(void*)dequantize, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_call_path", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call_path(void) { return PyModule_Create(&kModule); }
