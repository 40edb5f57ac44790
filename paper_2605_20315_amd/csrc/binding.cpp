// Marshalling of the common call forms in native code: torch tensors to the C ABI of include/mixquant.h.
//
// A small product is over in a few microseconds on the GPU, so what bounds such a call is the host.  Through ctypes
// an nvfp4_linear call takes 11.7 us with its outputs given and 16.7 with them allocated, of which the two launches are 4.4 to
// 4.8: the rest are attribute look-ups on eight tensors and argument conversion.  Here a tensor is unpacked in nanoseconds, and the
// call takes 5.2 and 7.6 us; a small bf16_gemm_ws 2.7 and 3.6 us instead of 6.3 and 7.9, of which its launch is 2.2.
//
// Every function returns None, before anything has been enqueued, for a call that is not of the plain form (another
// type, shape or stride than the kernels take, a tensor subclass, a tensor that is not on the GPU, a
// function mode, a value that does not fit): ops.py then takes its general path, which accepts or refuses it
// with its own message.  A status other than MQ_OK goes to the `check` callable, which raises.
// The functions are called through addresses that ops.py hands over, so there is one loaded library.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "../../include/mixquant.h"

namespace {

decltype(&::nvfp4_global_scale) p_global_scale;
decltype(&::nvfp4_quantize) p_quantize;
decltype(&::nvfp4_quantize_silu_mul) p_quantize_silu_mul;
decltype(&::nvfp4_quantize_rmsnorm) p_quantize_rmsnorm;
decltype(&::nvfp4_relayout) p_relayout;
decltype(&::nvfp4_gemm_ws) p_gemm_ws;
decltype(&::bf16_gemm_ws) p_bf16_gemm_ws;
PyObject *g_check;

// "Not of the plain form" is a return value (false, a null pointer, None) and no C++ exception: one of those takes 3.7 us, as
// much as the general path's own marshalling.
PyObject *general() { Py_RETURN_NONE; }

void *current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

const at::Tensor *tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    const bool plain = t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage() &&
                       !t.unsafeGetTensorImpl()->is_python_dispatch();
    return plain ? &t : nullptr;
}

const at::Tensor *typed(PyObject *o, at::ScalarType type)
{
    const at::Tensor *t = tensor(o);
    return t && t->scalar_type() == type ? t : nullptr;
}

bool integer(PyObject *o, int &value)  // (an int, or one of its subclasses such as an IntEnum member)
{
    if (!PyLong_Check(o)) return false;
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    value = (int)v;
    return !overflow && v >= INT32_MIN && v <= INT32_MAX;
}

bool real(PyObject *o, float &value)
{
    int i;
    if (PyFloat_CheckExact(o)) return value = (float)PyFloat_AS_DOUBLE(o), true;
    return integer(o, i) ? (value = (float)i, true) : false;
}

// rows, columns and row stride of a 2-D tensor whose last dimension is contiguous
struct Rows {
    int64_t rows, K, ld;
    bool read(const at::Tensor &t)
    {
        if (t.dim() != 2 || t.stride(1) != 1) return false;
        rows = t.size(0), K = t.size(1);
        ld = rows > 1 ? t.stride(0) : std::max(t.stride(0), K);
        return true;
    }
};

at::Tensor make(int64_t rows, int64_t cols, at::ScalarType type, const at::Tensor &like)
{
    return at::empty({rows, cols}, at::TensorOptions().dtype(type).device(like.device()));
}

PyObject *new_ref(PyObject *o)
{
    Py_INCREF(o);
    return o;
}

// an output that the caller may have passed: kept as the same Python object
struct Out {
    PyObject *obj = nullptr;
    at::Tensor made;
    const at::Tensor *t = nullptr;
    bool read(PyObject *o)
    {
        if (o == Py_None) return true;
        obj = o;
        return (t = tensor(o));
    }
    bool read_bytes(PyObject *o) { return read(o) && (!obj || t->is_contiguous()); }
};
void allocate(Out &o, int64_t rows, int64_t cols, at::ScalarType type, const at::Tensor &like)
{
    if (o.obj) return;
    o.made = make(rows, cols, type, like);
    o.t = &o.made;
}
PyObject *give(const Out &o) { return o.obj ? new_ref(o.obj) : THPVariable_Wrap(o.made); }

// what the C entry points want of a product's output and workspace
struct Product {
    Out y;
    int64_t ldy, ws_bytes = 0;
    void *ws = nullptr;
    int out;
    bool read(PyObject *workspace, PyObject *out_o, PyObject *y_o)
    {
        if (!integer(out_o, out) || !y.read(y_o)) return false;
        if (y.obj && y.t->dim() != 2 && y.t->dim() != 1) return false;  // (one row may come as a vector)
        if (workspace == Py_None) return true;
        const at::Tensor *t = tensor(workspace);
        if (!t || !t->is_contiguous()) return false;
        ws = t->data_ptr();
        ws_bytes = t->numel() * t->element_size();
        return true;
    }
    void allocate_y(int64_t M, int64_t N, const at::Tensor &like)
    {
        allocate(y, M, N, out == MQ_OUT_BF16 ? at::kBFloat16 : at::kFloat, like);
        ldy = M > 1 ? y.t->stride(0) : std::max(y.t->stride(0), N);
    }
};

// Runs `call` without the interpreter lock; false when it has raised.
template <class F>
bool enqueue(const char *what, F &&call)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    if (rc == MQ_OK) return true;
    PyObject *r = PyObject_CallFunction(g_check, "is", rc, what);
    Py_XDECREF(r);
    return false;
}

struct Quant {
    const at::Tensor *x, *alpha;
    Rows r;
    Out codes, scales;
    int layout;
    int64_t K;
    bool read(PyObject *xo, PyObject *ao, PyObject *codes_o, PyObject *scales_o, PyObject *layout_o, int per = 1)
    {
        if (!(x = typed(xo, at::kBFloat16)) || !(alpha = typed(ao, at::kFloat)) || !r.read(*x)) return false;
        K = r.K / per;
        return r.K % (per * 16) == 0 && integer(layout_o, layout) && codes.read_bytes(codes_o) && scales.read_bytes(scales_o);
    }
    void allocate_outputs()
    {
        allocate(codes, r.rows, K / 2, at::kByte, *x);
        allocate(scales, r.rows, K / 16, at::kByte, *x);
    }
    uint8_t *codes_ptr() const { return static_cast<uint8_t *>(codes.t->data_ptr()); }
    uint8_t *scales_ptr() const { return static_cast<uint8_t *>(scales.t->data_ptr()); }
    const float *alpha_ptr() const { return static_cast<const float *>(alpha->data_ptr()); }
    PyObject *result() const
    {
        PyObject *c = give(codes), *s = c ? give(scales) : nullptr;
        PyObject *t = s ? PyTuple_Pack(2, c, s) : nullptr;
        Py_XDECREF(c);
        Py_XDECREF(s);
        return t;
    }
};

// weights (or activations) of the block-scaled product: codes [rows, K/2], scales [rows, K/16]
struct Packed {
    const at::Tensor *c, *s;
    int64_t rows, K;
    bool read(PyObject *co, PyObject *so)
    {
        if (!(c = typed(co, at::kByte)) || !(s = typed(so, at::kByte))) return false;
        if (c->dim() != 2 || s->dim() != 2 || !c->is_contiguous() || !s->is_contiguous()) return false;
        rows = c->size(0), K = c->size(1) * 2;
        return s->size(0) == rows && s->size(1) == K / 16;
    }
    const uint8_t *codes() const { return static_cast<const uint8_t *>(c->data_ptr()); }
    const uint8_t *scales() const { return static_cast<const uint8_t *>(s->data_ptr()); }
};

// Entry points take positional arguments only (the keyword forms are those of ops.py) and end here.
template <class F>
PyObject *entry(Py_ssize_t n, Py_ssize_t want, F &&body)
{
    if (n != want) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
        return nullptr;
    }
    if (!g_check || at::impl::torch_function_mode_enabled()) return general();
    try {
        return body();
    } catch (python_error &e) {  // raised by Python code that an allocation went through (a dispatch mode): the call's answer
        e.restore();
        return nullptr;
    } catch (const std::exception &) {  // nothing has been enqueued: the general path meets the same and reports it
        return PyErr_Occurred() ? nullptr : general();
    }
}

PyObject *global_scale(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return entry(n, 2, [&]() -> PyObject * {
        const at::Tensor *x = typed(a[0], at::kBFloat16);
        Rows r;
        Out alpha;
        if (!x || !r.read(*x) || !alpha.read(a[1])) return general();
        if (!alpha.obj) {
            alpha.made = at::empty({1}, at::TensorOptions().dtype(at::kFloat).device(x->device()));
            alpha.t = &alpha.made;
        }
        void *const st = current_stream();
        const void *xp = x->data_ptr();
        float *ap = static_cast<float *>(alpha.t->data_ptr());
        if (!enqueue("nvfp4_global_scale", [&] { return p_global_scale(xp, r.rows, r.K, r.ld, ap, st); })) return nullptr;
        return give(alpha);
    });
}

PyObject *quantize(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return entry(n, 5, [&]() -> PyObject * {
        Quant q;
        if (!q.read(a[0], a[1], a[2], a[3], a[4])) return general();
        q.allocate_outputs();
        void *const st = current_stream();
        const void *xp = q.x->data_ptr();
        const float *ap = q.alpha_ptr();
        uint8_t *cp = q.codes_ptr(), *sp = q.scales_ptr();
        if (!enqueue("nvfp4_quantize", [&] { return p_quantize(xp, q.r.rows, q.K, q.r.ld, ap, cp, sp, q.layout, st); }))
            return nullptr;
        return q.result();
    });
}

PyObject *quantize_silu_mul(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return entry(n, 5, [&]() -> PyObject * {
        Quant q;
        if (!q.read(a[0], a[1], a[2], a[3], a[4], 2)) return general();
        q.allocate_outputs();
        void *const st = current_stream();
        const void *xp = q.x->data_ptr();
        const float *ap = q.alpha_ptr();
        uint8_t *cp = q.codes_ptr(), *sp = q.scales_ptr();
        if (!enqueue("nvfp4_quantize_silu_mul", [&] {
                return p_quantize_silu_mul(xp, q.r.rows, q.K, q.r.ld, ap, cp, sp, q.layout, nullptr, q.K, st);
            }))
            return nullptr;
        return q.result();
    });
}

PyObject *quantize_rmsnorm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return entry(n, 7, [&]() -> PyObject * {
        Quant q;
        float eps;
        const at::Tensor *w = typed(a[1], at::kBFloat16);
        if (!w || !real(a[2], eps) || !q.read(a[0], a[3], a[4], a[5], a[6])) return general();
        if (w->dim() != 1 || w->size(0) != q.K || !w->is_contiguous() || q.K % 64) return general();
        q.allocate_outputs();
        void *const st = current_stream();
        const void *xp = q.x->data_ptr(), *wp = w->data_ptr();
        const float *ap = q.alpha_ptr();
        uint8_t *cp = q.codes_ptr(), *sp = q.scales_ptr();
        if (!enqueue("nvfp4_quantize_rmsnorm", [&] {
                return p_quantize_rmsnorm(xp, q.r.rows, q.K, q.r.ld, wp, eps, ap, cp, sp, q.layout, nullptr, q.K, st);
            }))
            return nullptr;
        return q.result();
    });
}

PyObject *relayout(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return entry(n, 4, [&]() -> PyObject * {
        Packed p;
        int from, to;
        if (!p.read(a[0], a[1]) || !integer(a[2], from) || !integer(a[3], to)) return general();
        Out c, s;
        allocate(c, p.rows, p.K / 2, at::kByte, *p.c);
        allocate(s, p.rows, p.K / 16, at::kByte, *p.s);
        void *const st = current_stream();
        const uint8_t *pc = p.codes(), *ps = p.scales();
        uint8_t *oc = static_cast<uint8_t *>(c.t->data_ptr()), *os = static_cast<uint8_t *>(s.t->data_ptr());
        if (!enqueue("nvfp4_relayout", [&] { return p_relayout(pc, ps, oc, os, p.rows, p.K, from, to, st); })) return nullptr;
        PyObject *po = give(c), *so = po ? give(s) : nullptr, *t = so ? PyTuple_Pack(2, po, so) : nullptr;
        Py_XDECREF(po);
        Py_XDECREF(so);
        return t;
    });
}

PyObject *gemm_ws(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return entry(n, 10, [&]() -> PyObject * {
        Packed pa, pb;
        Product p;
        int layout;
        const at::Tensor *aa = tensor(a[2]), *ba = tensor(a[5]);
        if (!aa || !ba || !pa.read(a[0], a[1]) || !pb.read(a[3], a[4]) || pa.K != pb.K) return general();
        if (!p.read(a[6], a[7], a[8]) || !integer(a[9], layout)) return general();
        const int64_t M = pa.rows, N = pb.rows, K = pa.K;
        p.allocate_y(M, N, *pa.c);
        void *const st = current_stream(), *const y = p.y.t->data_ptr();
        const uint8_t *ac = pa.codes(), *as = pa.scales(), *bc = pb.codes(), *bs = pb.scales();
        const float *aap = static_cast<const float *>(aa->data_ptr()), *bap = static_cast<const float *>(ba->data_ptr());
        if (!enqueue("nvfp4_gemm_ws", [&] {
                return p_gemm_ws(ac, as, aap, bc, bs, bap, M, N, K, y, p.ldy, p.out, layout, p.ws, p.ws_bytes, st);
            }))
            return nullptr;
        return give(p.y);
    });
}

// The quantizer and the product of one layer.  What the two native forms ask of their arguments is asked in front of the first
// launch; what the library refuses by a status (an unknown `out`, a misaligned y or weight) it refuses call by call, so a
// refused product comes behind an enqueued quantizer, as it does in the general path.
PyObject *linear(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return entry(n, 11, [&]() -> PyObject * {
        // x, alpha_x, w_codes, w_scales, alpha_w, out, y, codes, scales, layout, workspace
        Quant q;
        Packed pb;
        Product p;
        const at::Tensor *ba = tensor(a[4]);
        if (!ba || !q.read(a[0], a[1], a[7], a[8], a[9]) || !pb.read(a[2], a[3]) || !p.read(a[10], a[5], a[6])) return general();
        const int64_t M = q.r.rows, N = pb.rows, K = q.K;
        if (pb.K != K) return general();
        auto matches = [&](const Out &o, int64_t cols) {  // what the product asks of the quantizer's outputs
            return !o.obj || (o.t->scalar_type() == at::kByte && o.t->dim() == 2 && o.t->size(0) == M && o.t->size(1) == cols);
        };
        if (!matches(q.codes, K / 2) || !matches(q.scales, K / 16)) return general();
        q.allocate_outputs();
        p.allocate_y(M, N, *q.codes.t);
        void *const st = current_stream(), *const y = p.y.t->data_ptr();
        const void *xp = q.x->data_ptr();
        const float *ap = q.alpha_ptr(), *bap = static_cast<const float *>(ba->data_ptr());
        uint8_t *cp = q.codes_ptr(), *sp = q.scales_ptr();
        const uint8_t *bc = pb.codes(), *bs = pb.scales();
        const char *what = "nvfp4_quantize";
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = p_quantize(xp, M, K, q.r.ld, ap, cp, sp, q.layout, st);
        if (rc == MQ_OK) {
            what = "nvfp4_gemm_ws";
            rc = p_gemm_ws(cp, sp, ap, bc, bs, bap, M, N, K, y, p.ldy, p.out, q.layout, p.ws, p.ws_bytes, st);
        }
        Py_END_ALLOW_THREADS
        if (rc != MQ_OK) {
            Py_XDECREF(PyObject_CallFunction(g_check, "is", rc, what));
            return nullptr;
        }
        return give(p.y);
    });
}

PyObject *bf16_gemm_ws(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return entry(n, 5, [&]() -> PyObject * {
        const at::Tensor *x = typed(a[0], at::kBFloat16), *w = typed(a[1], at::kBFloat16);
        Rows rx, rw;
        Product p;
        if (!x || !w || !rx.read(*x) || !rw.read(*w) || rx.K != rw.K || !p.read(a[2], a[3], a[4])) return general();
        const int64_t M = rx.rows, N = rw.rows;
        p.allocate_y(M, N, *x);
        void *const st = current_stream(), *const y = p.y.t->data_ptr();
        const void *xp = x->data_ptr(), *wp = w->data_ptr();
        if (!enqueue("bf16_gemm_ws", [&] {
                return p_bf16_gemm_ws(xp, rx.ld, wp, rw.ld, M, N, rx.K, y, p.ldy, p.out, p.ws, p.ws_bytes, st);
            }))
            return nullptr;
        return give(p.y);
    });
}

// bind(check, addresses by name): where the library's functions are
PyObject *bind(PyObject *, PyObject *args)
{
    PyObject *check, *addresses;
    if (!PyArg_ParseTuple(args, "OO!", &check, &PyDict_Type, &addresses)) return nullptr;
    bool ok = true;
    auto get = [&](const char *name, auto &fn) {
        PyObject *v = PyDict_GetItemString(addresses, name);  // borrowed
        void *p = v ? PyLong_AsVoidPtr(v) : nullptr;
        if (!p) ok = false;
        fn = reinterpret_cast<std::remove_reference_t<decltype(fn)>>(p);
    };
    get("nvfp4_global_scale", p_global_scale);
    get("nvfp4_quantize", p_quantize);
    get("nvfp4_quantize_silu_mul", p_quantize_silu_mul);
    get("nvfp4_quantize_rmsnorm", p_quantize_rmsnorm);
    get("nvfp4_relayout", p_relayout);
    get("nvfp4_gemm_ws", p_gemm_ws);
    get("bf16_gemm_ws", p_bf16_gemm_ws);
    if (!ok) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, "bind: a function of the library is missing");
        return nullptr;
    }
    g_check = new_ref(check);
    Py_RETURN_NONE;
}

#define MQ_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {MQ_FAST(global_scale), MQ_FAST(quantize), MQ_FAST(quantize_silu_mul), MQ_FAST(quantize_rmsnorm),
                         MQ_FAST(relayout),     MQ_FAST(gemm_ws),  MQ_FAST(linear),            MQ_FAST(bf16_gemm_ws),
                         {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "Plain-form calls of the mixquant library.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
