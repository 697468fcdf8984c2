// The launching calls of binding.py with their arguments taken apart natively: a torch tensor's address, sizes, strides and type
// are read from the tensor itself instead of through half a dozen Python calls and a ctypes descriptor each, and the library
// function is called directly.  What these calls decide is only how the arguments travel: every check of shapes and types is the
// library's, and anything out of the ordinary -- an argument that is not exactly a tensor or a parameter with memory on the GPU, a
// type the library has no code for, a stream object, an active torch function mode -- is declined (None), and binding.py's own
// marshalling takes the call or raises as it always has.
// Measured (256 x 256 x 256 fp16, enqueued back to back): 5.6 us a call through ctypes, of which 1.4 were marshalling.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../../include/nt.h"
#include "without_lock.h"

namespace {

// the library's functions, handed over by binding.py from the library it has loaded
decltype(&nt_gemm) p_gemm, p_bmm;
decltype(&nt_addmm) p_addmm;
decltype(&nt_addmm_act) p_addmm_act;
decltype(&nt_conv2d_implicit) p_conv;
decltype(&nt_sdpa) p_sdpa;
decltype(&nt_softmax) p_softmax;
decltype(&nt_rms_norm) p_rms_norm;
decltype(&nt_add) p_add;
decltype(&nt_silu) p_silu;

struct Operand {
    void *p;
    nt_tensor_desc d;
    nt_dtype dtype;
};

// false: not a plain GPU tensor of a type the library knows
bool take(PyObject *o, Operand *out)
{
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || !t.has_storage()) return false;
    const c10::TensorImpl *impl = t.unsafeGetTensorImpl();
    if (impl->has_symbolic_sizes_strides() || impl->key_set().has(c10::DispatchKey::Python)) return false;
    switch (t.scalar_type()) {
    case at::kHalf: out->dtype = NT_F16; break;
    case at::kBFloat16: out->dtype = NT_BF16; break;
    case at::kFloat: out->dtype = NT_F32; break;
    default: return false;
    }
    const int64_t n = t.dim();
    if (n < 1 || n > NT_MAX_DIMS) return false;
    const auto sizes = t.sizes(), strides = t.strides();
    out->d.ndim = (int32_t)n;
    for (int64_t i = 0; i < n; ++i) {
        out->d.size[i] = sizes[i];
        out->d.stride[i] = strides[i];
    }
    out->p = t.data_ptr();
    return true;
}

bool integer(PyObject *o, int32_t *v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long x = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || x < INT32_MIN || x > INT32_MAX) return false;
    *v = (int32_t)x;
    return true;
}

bool real(PyObject *o, float *v)
{
    if (!PyFloat_CheckExact(o)) return false;
    *v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}

// a tuple or list of `n` ints
bool integers(PyObject *o, int n, int32_t *v)
{
    const bool tuple = PyTuple_CheckExact(o);
    if (!tuple && !PyList_CheckExact(o)) return false;
    if ((tuple ? PyTuple_GET_SIZE(o) : PyList_GET_SIZE(o)) != n) return false;
    for (int i = 0; i < n; ++i)
        if (!integer(tuple ? PyTuple_GET_ITEM(o, i) : PyList_GET_ITEM(o, i), &v[i])) return false;
    return true;
}

bool tile_of(PyObject *o, nt_tile_cfg *cfg)
{
    int32_t v[3] = {0, 0, 0};
    if (o != Py_None && !integers(o, 3, v)) return false;
    *cfg = nt_tile_cfg{v[0], v[1], v[2]};
    return true;
}

// the current device's current stream; false: a stream object was given
bool stream_of(PyObject *o, void **s)
{
    if (o != Py_None) return false;
    *s = (void *)c10::hip::getCurrentHIPStream().stream();
    return true;
}

bool modes_active() { return at::impl::torch_function_mode_enabled(); }

PyObject *declined() { Py_RETURN_NONE; }

// C++ exceptions must not cross into the interpreter.  One from taking the arguments apart: the general path repeats the call and reports
// what it finds.  (Not a catch-all, see without_lock.h.)
template <typename F>
PyObject *guarded(F f)
{
    try {
        return modes_active() ? declined() : f();
    } catch (const std::exception &) {
        return declined();
    }
}

PyObject *product(decltype(p_gemm) fn, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        Operand A, B, C;
        nt_tile_cfg cfg;
        void *s;
        if (!fn || n != 5 || !take(a[0], &A) || !take(a[1], &B) || !take(a[2], &C) || !tile_of(a[3], &cfg) || !stream_of(a[4], &s)) return declined();
        return without_lock([&] { return fn(A.p, &A.d, B.p, &B.d, C.p, &C.d, A.dtype, C.dtype, cfg, s); });
    });
}
PyObject *gemm(PyObject *, PyObject *const *a, Py_ssize_t n) { return product(p_gemm, a, n); }
PyObject *bmm(PyObject *, PyObject *const *a, Py_ssize_t n) { return product(p_bmm, a, n); }

// addmm(input, A, B, C, alpha, beta, act code, tile, stream); the input of C's shape, or one row of it
PyObject *addmm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        Operand D, A, B, C;
        float alpha, beta;
        int32_t act;
        nt_tile_cfg cfg;
        void *s;
        if (!p_addmm_act || n != 9 || !take(a[0], &D) || !take(a[1], &A) || !take(a[2], &B) || !take(a[3], &C) || !real(a[4], &alpha) || !real(a[5], &beta) ||
            !integer(a[6], &act) || !tile_of(a[7], &cfg) || !stream_of(a[8], &s))
            return declined();
        if (D.dtype != C.dtype || C.d.ndim != 2) return declined();
        if (D.d.ndim == 1) {
            if (D.d.size[0] != C.d.size[1] || C.d.size[0] < 2 || C.d.size[1] < 2) return declined();
            D.d = nt_tensor_desc{2, {C.d.size[0], C.d.size[1]}, {0, D.d.stride[0]}};
        } else if (D.d.ndim != 2 || D.d.size[0] != C.d.size[0] || D.d.size[1] != C.d.size[1]) {
            return declined();
        }
        if (act) return without_lock([&] { return p_addmm_act(D.p, &D.d, A.p, &A.d, B.p, &B.d, C.p, &C.d, alpha, beta, (nt_activation)act, A.dtype, C.dtype, cfg, s); });
        return without_lock([&] { return p_addmm(D.p, &D.d, A.p, &A.d, B.p, &B.d, C.p, &C.d, alpha, beta, A.dtype, C.dtype, cfg, s); });
    });
}

// conv2d(x, w, y, stride, pad, tile, stream)
PyObject *conv2d(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        Operand x, w, y;
        int32_t stride[2], pad[2];
        nt_tile_cfg cfg;
        void *s;
        if (!p_conv || n != 7 || !take(a[0], &x) || !take(a[1], &w) || !take(a[2], &y) || !integers(a[3], 2, stride) || !integers(a[4], 2, pad) ||
            !tile_of(a[5], &cfg) || !stream_of(a[6], &s))
            return declined();
        return without_lock([&] { return p_conv(x.p, &x.d, w.p, &w.d, y.p, &y.d, stride[0], stride[1], pad[0], pad[1], x.dtype, y.dtype, cfg, s); });
    });
}

PyObject *sdpa(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        Operand q, k, v, o;
        float scale;
        void *s;
        if (!p_sdpa || n != 6 || !take(a[0], &q) || !take(a[1], &k) || !take(a[2], &v) || !take(a[3], &o) || !real(a[4], &scale) || !stream_of(a[5], &s)) return declined();
        return without_lock([&] { return p_sdpa(q.p, &q.d, k.p, &k.d, v.p, &v.d, o.p, &o.d, scale, q.dtype, s); });
    });
}

PyObject *softmax(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        Operand x, o;
        void *s;
        if (!p_softmax || n != 3 || !take(a[0], &x) || !take(a[1], &o) || !stream_of(a[2], &s)) return declined();
        return without_lock([&] { return p_softmax(x.p, &x.d, o.p, &o.d, x.dtype, s); });
    });
}

PyObject *rms_norm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        Operand x, o;
        float eps;
        void *s;
        if (!p_rms_norm || n != 4 || !take(a[0], &x) || !take(a[1], &o) || !real(a[2], &eps) || !stream_of(a[3], &s)) return declined();
        return without_lock([&] { return p_rms_norm(x.p, &x.d, o.p, &o.d, eps, x.dtype, s); });
    });
}

PyObject *add(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        Operand x, y, o;
        int32_t block;
        void *s;
        if (!p_add || n != 5 || !take(a[0], &x) || !take(a[1], &y) || !take(a[2], &o) || !integer(a[3], &block) || !stream_of(a[4], &s)) return declined();
        return without_lock([&] { return p_add(x.p, &x.d, y.p, &y.d, o.p, &o.d, x.dtype, block, s); });
    });
}

PyObject *silu(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        Operand x, o;
        int32_t block;
        void *s;
        if (!p_silu || n != 4 || !take(a[0], &x) || !take(a[1], &o) || !integer(a[2], &block) || !stream_of(a[3], &s)) return declined();
        return without_lock([&] { return p_silu(x.p, &x.d, o.p, &o.d, x.dtype, block, s); });
    });
}

// bind(addresses of nt_gemm, nt_bmm, nt_addmm, nt_addmm_act, nt_conv2d_implicit, nt_sdpa, nt_softmax, nt_rms_norm, nt_add, nt_silu)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 10) {
        PyErr_SetString(PyExc_TypeError, "ten addresses wanted");
        return nullptr;
    }
    void *p[10];
    for (int i = 0; i < 10; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
            return nullptr;
        }
    }
    p_gemm = (decltype(p_gemm))p[0]; p_bmm = (decltype(p_bmm))p[1]; p_addmm = (decltype(p_addmm))p[2]; p_addmm_act = (decltype(p_addmm_act))p[3];
    p_conv = (decltype(p_conv))p[4]; p_sdpa = (decltype(p_sdpa))p[5]; p_softmax = (decltype(p_softmax))p[6]; p_rms_norm = (decltype(p_rms_norm))p[7];
    p_add = (decltype(p_add))p[8]; p_silu = (decltype(p_silu))p[9];
    Py_RETURN_NONE;
}

#define NT_CALL(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {NT_CALL(gemm), NT_CALL(bmm), NT_CALL(addmm), NT_CALL(conv2d), NT_CALL(sdpa), NT_CALL(softmax), NT_CALL(rms_norm),
                         NT_CALL(add), NT_CALL(silu), NT_CALL(bind), {nullptr, nullptr, 0, nullptr}};
#undef NT_CALL
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_nt_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__nt_calls(void) { return PyModule_Create(&module); }
