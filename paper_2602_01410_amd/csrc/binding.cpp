// Native half of snip.py: takes torch tensors and QTensor objects apart and calls the C ABI of include/snip.h.  Argument
// marshalling only, like the Python half; the library is called through its exported symbols, looked up once by bind().
//
// A call of the C ABI takes about 3 us of host time, most of it the launch.  Marshalled in Python (attribute reads, one
// ctypes structure per operand, torch.cuda.current_stream()) a call took 8.8-9.5 us, more than the kernels of a small
// training step; the functions below take about 1 us around the launch.
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <cstring>
#include "../../include/snip.h"

namespace {

decltype(&snip_quantize) p_quantize;
decltype(&snip_quantize_both) p_quantize_both;
decltype(&snip_quantize_sr_fp4) p_quantize_sr_fp4;
decltype(&snip_gemm_fwd) p_gemm[3];
decltype(&snip_gemm_fwd_norm) p_gemm_norm[3];
decltype(&snip_quantize_paper) p_quantize_paper;
decltype(&snip_gemm_paper) p_gemm_paper;
decltype(&snip_quant_error_stats) p_stats;
decltype(&snip_quant_error_stats_both) p_stats_both;
decltype(&snip_adamw_sensitivity) p_adamw;

PyObject *s_codes, *s_scales, *s_scales_g4, *s_rows, *s_cols, *s_fmt;      // interned attribute names

// Every helper returns false (or -1) with a Python exception set when an argument is not what it should be.
bool tensor(PyObject* o, const at::Tensor*& t)
{
    if (!THPVariable_Check(o)) { PyErr_SetString(PyExc_TypeError, "expected a torch.Tensor"); return false; }
    t = &THPVariable_Unpack(o);
    return true;
}
bool pointer(PyObject* o, void*& p)                 // None: null
{
    p = nullptr;
    if (o == Py_None) return true;
    const at::Tensor* t;
    if (!tensor(o, t)) return false;
    p = t->data_ptr();
    return true;
}
bool integer(PyObject* o, int64_t& v) { v = PyLong_AsLongLong(o); return !(v == -1 && PyErr_Occurred()); }

struct Source { void* p; int64_t rows, cols, ld; };
bool source(PyObject* o, Source& s)
{
    const at::Tensor* t;
    if (!tensor(o, t)) return false;
    if (t->dim() != 2 || t->element_size() != 2 || !t->is_cuda()) {
        PyErr_SetString(PyExc_ValueError, "expected a 2-D CUDA tensor of bf16 (or its uint16/int16 bit patterns)");
        return false;
    }
    if (t->stride(1) != 1) { PyErr_SetString(PyExc_ValueError, "rows must be contiguous"); return false; }
    s = {t->data_ptr(), t->size(0), t->size(1), t->stride(0)};
    return true;
}
bool attr_int(PyObject* o, PyObject* name, int64_t& v)
{
    PyObject* a = PyObject_GetAttr(o, name);
    if (!a) return false;
    const bool ok = integer(a, v);
    Py_DECREF(a);
    return ok;
}
bool attr_ptr(PyObject* o, PyObject* name, void*& p)
{
    PyObject* a = PyObject_GetAttr(o, name);
    if (!a) return false;
    const bool ok = pointer(a, p);                  // (the object keeps the tensor alive)
    Py_DECREF(a);
    return ok;
}
bool qtensor(PyObject* o, snip_qtensor& q)
{
    void *c, *s, *g;
    int64_t fmt;
    if (!attr_ptr(o, s_codes, c) || !attr_ptr(o, s_scales, s) || !attr_ptr(o, s_scales_g4, g) || !attr_int(o, s_rows, q.rows) ||
        !attr_int(o, s_cols, q.cols) || !attr_int(o, s_fmt, fmt))
        return false;
    q.codes = c; q.scales = (uint8_t*)s; q.scales_g4 = (uint8_t*)g; q.fmt = (int32_t)fmt;
    return true;
}
bool workspace(PyObject* o, void*& p, size_t& n)    // a uint8 tensor or None
{
    p = nullptr; n = 0;
    if (o == Py_None) return true;
    const at::Tensor* t;
    if (!tensor(o, t)) return false;
    p = t->data_ptr(); n = (size_t)t->numel();
    return true;
}
bool stream(PyObject* o, void*& s)                  // None: the current stream of the current device
{
    if (o == Py_None) { s = (void*)c10::hip::getCurrentHIPStream().stream(); return true; }
    s = PyLong_AsVoidPtr(o);
    return !(s == nullptr && PyErr_Occurred());
}
bool plan(PyObject* o, snip_layer_plan& p)          // the ctypes structure of snip.make_plan
{
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return false;
    const bool ok = b.len == (Py_ssize_t)sizeof(p);
    if (ok) std::memcpy(&p, b.buf, sizeof(p));
    PyBuffer_Release(&b);
    if (!ok) PyErr_SetString(PyExc_TypeError, "expected a plan");
    return ok;
}
bool count(Py_ssize_t n, Py_ssize_t want)
{
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    return false;
}

template <class F> PyObject* call(F f)
{
    snip_status st;
    Py_BEGIN_ALLOW_THREADS
    st = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
}

// (x, fmt, axis, rule, out, stats, workspace, stream)
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Source x; int64_t fmt, axis, rule; snip_qtensor q; void *st, *ws, *s; size_t wn;
    if (!count(n, 8) || !source(a[0], x) || !integer(a[1], fmt) || !integer(a[2], axis) || !integer(a[3], rule) || !qtensor(a[4], q) ||
        !pointer(a[5], st) || !workspace(a[6], ws, wn) || !stream(a[7], s))
        return nullptr;
    return call([&] { return p_quantize(x.p, x.rows, x.cols, x.ld, (snip_fmt)fmt, (snip_axis)axis, (snip_scale_rule)rule, &q, (snip_stats*)st, ws, wn, s); });
}
// (x, rule, out_row, out_col, stats_row, stats_col, scope, workspace, stream)
PyObject* quantize_both(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Source x; int64_t rule, scope; snip_qtensor qr, qc; void *sr, *sc, *ws, *s; size_t wn;
    if (!count(n, 9) || !source(a[0], x) || !integer(a[1], rule) || !qtensor(a[2], qr) || !qtensor(a[3], qc) || !pointer(a[4], sr) ||
        !pointer(a[5], sc) || !integer(a[6], scope) || !workspace(a[7], ws, wn) || !stream(a[8], s))
        return nullptr;
    return call([&] { return p_quantize_both(x.p, x.rows, x.cols, x.ld, (snip_scale_rule)rule, &qr, &qc, (snip_stats*)sr, (snip_stats*)sc,
                                             (snip_stats_scope)scope, ws, wn, s); });
}
// (x, axis, rule, seed, out, stream)
PyObject* quantize_sr_fp4(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Source x; int64_t axis, rule; snip_qtensor q; void* s;
    if (!count(n, 6) || !source(a[0], x) || !integer(a[1], axis) || !integer(a[2], rule)) return nullptr;
    const unsigned long long seed = PyLong_AsUnsignedLongLong(a[3]);
    if (seed == (unsigned long long)-1 && PyErr_Occurred()) return nullptr;
    if (!qtensor(a[4], q) || !stream(a[5], s)) return nullptr;
    return call([&] { return p_quantize_sr_fp4(x.p, x.rows, x.cols, x.ld, (snip_axis)axis, (snip_scale_rule)rule, seed, &q, s); });
}
struct Output { void* p; int64_t ld; };
bool output(PyObject* o, Output& out)
{
    const at::Tensor* t;
    if (!tensor(o, t)) return false;
    if (t->dim() < 1) { PyErr_SetString(PyExc_ValueError, "expected a matrix as output"); return false; }
    out = {t->data_ptr(), t->stride(0)};
    return true;
}
bool which_gemm(PyObject* o, int64_t& w)
{
    if (!integer(o, w)) return false;
    if (w < 0 || w > 2) { PyErr_SetString(PyExc_ValueError, "no such GEMM"); return false; }
    return true;
}
// (which, plan, a, b, out, out_dtype, stream)
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    int64_t w, dt; snip_layer_plan p; snip_qtensor qa, qb; Output o; void* s;
    if (!count(n, 7) || !which_gemm(a[0], w) || !plan(a[1], p) || !qtensor(a[2], qa) || !qtensor(a[3], qb) || !output(a[4], o) ||
        !integer(a[5], dt) || !stream(a[6], s))
        return nullptr;
    return call([&] { return p_gemm[w](&p, &qa, &qb, o.p, o.ld, (snip_out_dtype)dt, nullptr, 0, s); });
}
// (which, plan, a, b, out, out_dtype, sum_sq, workspace, stream)
PyObject* gemm_norm(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    int64_t w, dt; snip_layer_plan p; snip_qtensor qa, qb; Output o; void *ss, *ws, *s; size_t wn;
    if (!count(n, 9) || !which_gemm(a[0], w) || !plan(a[1], p) || !qtensor(a[2], qa) || !qtensor(a[3], qb) || !output(a[4], o) ||
        !integer(a[5], dt) || !pointer(a[6], ss) || !workspace(a[7], ws, wn) || !stream(a[8], s))
        return nullptr;
    return call([&] { return p_gemm_norm[w](&p, &qa, &qb, o.p, o.ld, (snip_out_dtype)dt, (double*)ss, ws, wn, s); });
}
// (x, fmt, axis, group, codes, scales, stream)
PyObject* quantize_paper(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Source x; int64_t fmt, axis, group; void *c, *sc, *s;
    if (!count(n, 7) || !source(a[0], x) || !integer(a[1], fmt) || !integer(a[2], axis) || !integer(a[3], group) || !pointer(a[4], c) ||
        !pointer(a[5], sc) || !stream(a[6], s))
        return nullptr;
    return call([&] { return p_quantize_paper(x.p, x.rows, x.cols, x.ld, (snip_fmt)fmt, (snip_axis)axis, (snip_group)group, c, (float*)sc, s); });
}
bool ptensor(PyObject* const* a, snip_ptensor& q)   // codes, scales, fmt, group
{
    const at::Tensor* c;
    int64_t fmt, group;
    void* sc;
    if (!tensor(a[0], c) || !pointer(a[1], sc) || !integer(a[2], fmt) || !integer(a[3], group)) return false;
    if (c->dim() != 2) { PyErr_SetString(PyExc_ValueError, "expected 2-D codes"); return false; }
    q.codes = c->data_ptr(); q.scales = (const float*)sc; q.rows = c->size(0);
    q.cols = fmt == SNIP_FP8_E4M3 ? c->size(1) : 2 * c->size(1); q.fmt = (int32_t)fmt; q.group = (int32_t)group;
    return true;
}
// (a_codes, a_scales, a_fmt, a_group, b_codes, b_scales, b_fmt, b_group, out, out_dtype, stream)
PyObject* gemm_paper(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    snip_ptensor pa, pb; Output o; int64_t dt; void* s;
    if (!count(n, 11) || !ptensor(a, pa) || !ptensor(a + 4, pb) || !output(a[8], o) || !integer(a[9], dt) || !stream(a[10], s)) return nullptr;
    return call([&] { return p_gemm_paper(&pa, &pb, o.p, o.ld, (snip_out_dtype)dt, s); });
}
// (x, axis, rule, out, per_line, workspace, stream)
PyObject* stats(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Source x; int64_t axis, rule; void *o, *pl, *ws, *s; size_t wn;
    if (!count(n, 7) || !source(a[0], x) || !integer(a[1], axis) || !integer(a[2], rule) || !pointer(a[3], o) || !pointer(a[4], pl) ||
        !workspace(a[5], ws, wn) || !stream(a[6], s))
        return nullptr;
    return call([&] { return p_stats(x.p, x.rows, x.cols, x.ld, (snip_axis)axis, (snip_scale_rule)rule, (snip_stats*)o, (float*)pl, ws, wn, s); });
}
// (x, rule, out_row, out_col, workspace, stream)
PyObject* stats_both(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Source x; int64_t rule; void *r, *c, *ws, *s; size_t wn;
    if (!count(n, 6) || !source(a[0], x) || !integer(a[1], rule) || !pointer(a[2], r) || !pointer(a[3], c) || !workspace(a[4], ws, wn) || !stream(a[5], s))
        return nullptr;
    return call([&] { return p_stats_both(x.p, x.rows, x.cols, x.ld, (snip_scale_rule)rule, (snip_stats*)r, (snip_stats*)c, ws, wn, s); });
}
// (m, v, g, g_dtype, n, beta1, beta2, eps, out, workspace, stream)
PyObject* adamw(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    void *m, *v, *g, *o, *ws, *s; int64_t dt, cnt; size_t wn;
    if (!count(n, 11) || !pointer(a[0], m) || !pointer(a[1], v) || !pointer(a[2], g) || !integer(a[3], dt) || !integer(a[4], cnt)) return nullptr;
    const double b1 = PyFloat_AsDouble(a[5]), b2 = PyFloat_AsDouble(a[6]), eps = PyFloat_AsDouble(a[7]);
    if (PyErr_Occurred() || !pointer(a[8], o) || !workspace(a[9], ws, wn) || !stream(a[10], s)) return nullptr;
    return call([&] { return p_adamw((const float*)m, (const float*)v, g, (snip_out_dtype)dt, cnt, (float)b1, (float)b2, (float)eps, (double*)o, ws, wn, s); });
}

template <class F> bool find(void* lib, const char* name, F& f)
{
    f = (F)dlsym(lib, name);
    if (!f) PyErr_Format(PyExc_RuntimeError, "the library has no symbol %s", name);
    return f != nullptr;
}
// (path of the library)
PyObject* bind(PyObject*, PyObject* arg)
{
    const char* path = PyUnicode_AsUTF8(arg);
    if (!path) return nullptr;
    void* lib = dlopen(path, RTLD_NOW | RTLD_LOCAL);
    if (!lib) { PyErr_Format(PyExc_RuntimeError, "%s", dlerror()); return nullptr; }
    if (!find(lib, "snip_quantize", p_quantize) || !find(lib, "snip_quantize_both", p_quantize_both) ||
        !find(lib, "snip_quantize_sr_fp4", p_quantize_sr_fp4) || !find(lib, "snip_gemm_fwd", p_gemm[0]) || !find(lib, "snip_gemm_dgrad", p_gemm[1]) ||
        !find(lib, "snip_gemm_wgrad", p_gemm[2]) || !find(lib, "snip_gemm_fwd_norm", p_gemm_norm[0]) ||
        !find(lib, "snip_gemm_dgrad_norm", p_gemm_norm[1]) || !find(lib, "snip_gemm_wgrad_norm", p_gemm_norm[2]) ||
        !find(lib, "snip_quantize_paper", p_quantize_paper) || !find(lib, "snip_gemm_paper", p_gemm_paper) ||
        !find(lib, "snip_quant_error_stats", p_stats) || !find(lib, "snip_quant_error_stats_both", p_stats_both) ||
        !find(lib, "snip_adamw_sensitivity", p_adamw))
        return nullptr;
    Py_RETURN_NONE;
}

// torch reports errors (no device, a tensor without storage) as C++ exceptions
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    try {
        return F(self, a, n);
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}
#define SNIP_FAST(name) {#name, (PyCFunction)(void (*)(void))guarded<name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", bind, METH_O, nullptr}, SNIP_FAST(quantize), SNIP_FAST(quantize_both), SNIP_FAST(quantize_sr_fp4),
                         SNIP_FAST(gemm), SNIP_FAST(gemm_norm), SNIP_FAST(quantize_paper), SNIP_FAST(gemm_paper), SNIP_FAST(stats),
                         SNIP_FAST(stats_both), SNIP_FAST(adamw), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_snip_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__snip_binding(void)
{
    s_codes = PyUnicode_InternFromString("codes");
    s_scales = PyUnicode_InternFromString("scales");
    s_scales_g4 = PyUnicode_InternFromString("scales_g4");
    s_rows = PyUnicode_InternFromString("rows");
    s_cols = PyUnicode_InternFromString("cols");
    s_fmt = PyUnicode_InternFromString("fmt");
    return PyModule_Create(&module);
}
