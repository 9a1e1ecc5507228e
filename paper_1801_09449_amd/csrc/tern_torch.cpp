// The per-call path of the Python binding in native code: argument checks, output allocation and the C
// call for torch tensors.  A launch of the smallest layers takes 7 us of GPU time and its Python binding
// (ctypes structures, a dozen attribute look-ups per tensor) took 9-12 us of host time; a chain of
// fourteen modules 80 us more.  Every function here handles the plain case only: plain tensors of the
// right type, device, layout and size.  For anything else it returns None before anything is launched, and
// the Python function that called it goes through its own checks, which name what is wrong.
// Results: the output tensor (0 from a network without a prediction layer); None (not the plain case); or an
// int, the C entry point's negative status.
// Nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "tern.h"

namespace {

// "Not the plain case": unwinds to the entry point, which returns None.
struct Other {};

PyObject* g_raw_stream = nullptr;    // torch._C._cuda_getCurrentRawStream
struct Names {
    PyObject *c_in, *c_out, *w_bank, *thr_lo, *thr_hi, *k, *stride, *pad, *dil, *skip_from, *up, *pool;
} g_names;

// A borrowed tensor argument that a kernel can take: exact torch.Tensor with storage on a GPU, contiguous,
// conjugation and negation resolved.
const at::Tensor& tensor(PyObject* o, at::ScalarType type)
{
    if (!THPVariable_CheckExact(o)) throw Other();
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || t.layout() != at::kStrided ||
        !t.unsafeGetTensorImpl()->has_storage() || !t.is_contiguous() || t.is_neg() || t.is_conj())
        throw Other();
    return t;
}

struct Ref {                          // owned reference
    PyObject* o;
    explicit Ref(PyObject* p) : o(p)
    {
        if (!p) { PyErr_Clear(); throw Other(); }
    }
    ~Ref() { Py_XDECREF(o); }
    Ref(const Ref&) = delete;
    Ref& operator=(const Ref&) = delete;
};

// Sequences, numpy's integers and booleans are handled here too: leaving a call to the Python path costs an
// exception on top of it (3 us; lists for k, stride and pad made a call 12.4 -> 15.0 us).
int32_t int_of(PyObject* o)
{
    Ref i(PyNumber_Index(o));         // (an int itself is only counted)
    int over = 0;
    const long long v = PyLong_AsLongLongAndOverflow(i.o, &over);
    if (over || v < INT32_MIN || v > INT32_MAX) throw Other();
    return (int32_t)v;
}

// A list or tuple, as a tuple of its own (attributes of its items are looked up, which may run Python code).
PyObject* items(PyObject* o)
{
    if (!PyList_Check(o) && !PyTuple_Check(o)) throw Other();
    return PySequence_Tuple(o);
}

// An int or three ints.
void triple(PyObject* o, int32_t (&out)[3])
{
    if (PyLong_Check(o)) {
        out[0] = out[1] = out[2] = int_of(o);
        return;
    }
    Ref t(items(o));
    if (PyTuple_GET_SIZE(t.o) != 3) throw Other();
    for (int a = 0; a < 3; ++a) out[a] = int_of(PyTuple_GET_ITEM(t.o, a));
}

void attr_triple(PyObject* o, PyObject* name, int32_t (&out)[3])
{
    Ref r(PyObject_GetAttr(o, name));
    triple(r.o, out);
}
int32_t attr_int(PyObject* o, PyObject* name)
{
    Ref r(PyObject_GetAttr(o, name));
    return int_of(r.o);
}

void* stream_of(const at::Tensor& t)
{
    Ref i(PyLong_FromLong(t.device().index()));
    Ref r(PyObject_CallOneArg(g_raw_stream, i.o));
    void* s = PyLong_AsVoidPtr(r.o);
    if (!s && PyErr_Occurred()) { PyErr_Clear(); throw Other(); }
    return s;
}

int32_t dim32(int64_t v)
{
    if (v < 0 || v > INT32_MAX) throw Other();
    return (int32_t)v;
}
tern_dims dims5(const at::Tensor& t)
{
    if (t.dim() != 5) throw Other();
    const auto s = t.sizes();
    return {dim32(s[0]), dim32(s[1]), dim32(s[2]), dim32(s[3]), dim32(s[4])};
}

// `o`, checked to hold exactly the packed form of `d`, or a new tensor for None.
at::Tensor packed_out(PyObject* o, const tern_dims& d, const at::Tensor& like)
{
    if (o == Py_None)
        return at::empty({d.n, d.d, d.h, d.w, 2, tern_words(d.c)}, like.options().dtype(at::kInt));
    const at::Tensor& t = tensor(o, at::kInt);
    const size_t need = tern_packed_bytes(d);
    if (need == 0 || (size_t)t.numel() * 4 != need) throw Other();
    return t;
}

// Other Python threads run while a launch is queued.
struct Unlocked {
    PyThreadState* s = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(s); }
};
template <typename F>
int launch(F f)
{
    Unlocked u;
    return f();
}

PyObject* result(int rc, PyObject* given, const at::Tensor& out)
{
    if (rc != TERN_OK) return PyLong_FromLong(rc);
    if (given != Py_None) {
        Py_INCREF(given);
        return given;
    }
    return THPVariable_Wrap(out);
}

template <typename F>
PyObject* guarded(F f)
{
    try {
        return f();
    } catch (...) {                   // Other, or anything torch throws: the Python path says what it is
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

#define TERN_ARGS(N)                                                              \
    if (nargs != N) {                                                             \
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");           \
        return nullptr;                                                           \
    }

// conv(binary, in_packed, c_in, w_bank, c_out, k, stride, pad, dil, thr_lo, thr_hi, out)
PyObject* conv(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    TERN_ARGS(12)
    return guarded([&]() -> PyObject* {
        const bool binary = a[0] == Py_True;
        const at::Tensor& in = tensor(a[1], at::kInt);
        const at::Tensor& bank = tensor(a[3], at::kInt);
        const int32_t c_in = int_of(a[2]), c_out = int_of(a[4]);
        if (in.dim() != 6) throw Other();
        const auto e = in.sizes();
        if (c_in < 1 || e[4] != 2 || e[5] != tern_words(c_in)) throw Other();
        const tern_dims id = {dim32(e[0]), c_in, dim32(e[1]), dim32(e[2]), dim32(e[3])};
        tern_conv_geom g;
        triple(a[5], g.k); triple(a[6], g.stride); triple(a[7], g.pad); triple(a[8], g.dil);
        const size_t need = binary ? tern_binary_bank_bytes(c_out, c_in, g.k[0], g.k[1], g.k[2])
                                   : tern_filter_bank_bytes(c_out, c_in, g.k[0], g.k[1], g.k[2]);
        if (need == 0 || (size_t)bank.numel() * 4 != need) throw Other();
        tern_dims o;
        if (tern_conv_out_dims(id, c_out, g, &o) != TERN_OK) throw Other();
        const auto call = binary ? tern_conv3d_binary : tern_conv3d;
        if (a[9] != Py_None || a[10] != Py_None) {
            const at::Tensor& lo = tensor(a[9], at::kInt);
            const at::Tensor& hi = tensor(a[10], at::kInt);
            if (lo.numel() != c_out || hi.numel() != c_out) throw Other();
            const at::Tensor out = packed_out(a[11], o, in);
            const auto *pi = (const uint32_t*)in.data_ptr(), *pb = (const uint32_t*)bank.data_ptr();
            const auto *pl = (const int32_t*)lo.data_ptr(), *ph = (const int32_t*)hi.data_ptr();
            auto* po = (uint32_t*)out.data_ptr();
            void* s = stream_of(in);
            return result(launch([&] { return call(pi, id, pb, c_out, g, pl, ph, nullptr, po, s); }), a[11], out);
        }
        at::Tensor out;
        if (a[11] == Py_None) {
            out = at::empty({o.n, o.c, o.d, o.h, o.w}, in.options());
        } else {
            out = tensor(a[11], at::kInt);
            if (out.sizes() != at::IntArrayRef({o.n, o.c, o.d, o.h, o.w})) throw Other();
        }
        const auto *pi = (const uint32_t*)in.data_ptr(), *pb = (const uint32_t*)bank.data_ptr();
        auto* po = (int32_t*)out.data_ptr();
        void* s = stream_of(in);
        return result(launch([&] { return call(pi, id, pb, c_out, g, nullptr, nullptr, po, nullptr, s); }), a[11], out);
    });
}

// pack(src, out)
PyObject* pack(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    TERN_ARGS(2)
    return guarded([&]() -> PyObject* {
        const at::Tensor& src = tensor(a[0], at::kChar);
        const tern_dims d = dims5(src);
        if (tern_packed_bytes(d) == 0) throw Other();
        const at::Tensor out = packed_out(a[1], d, src);
        const auto* ps = (const int8_t*)src.data_ptr();
        auto* po = (uint32_t*)out.data_ptr();
        void* s = stream_of(src);
        return result(launch([&] { return tern_pack(ps, d, po, s); }), a[1], out);
    });
}

// threshold_pack(src, thr_lo, thr_hi, out)
PyObject* threshold_pack(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    TERN_ARGS(4)
    return guarded([&]() -> PyObject* {
        if (!THPVariable_CheckExact(a[0])) throw Other();
        const at::ScalarType type = THPVariable_Unpack(a[0]).scalar_type();
        if (type != at::kInt && type != at::kFloat) throw Other();
        const at::Tensor& src = tensor(a[0], type);
        const at::Tensor& lo = tensor(a[1], type);
        const at::Tensor& hi = tensor(a[2], type);
        const tern_dims d = dims5(src);
        if (tern_packed_bytes(d) == 0 || lo.numel() != d.c || hi.numel() != d.c) throw Other();
        const at::Tensor out = packed_out(a[3], d, src);
        const void *ps = src.data_ptr(), *pl = lo.data_ptr(), *ph = hi.data_ptr();
        auto* po = (uint32_t*)out.data_ptr();
        void* s = stream_of(src);
        const tern_src_type t = type == at::kInt ? TERN_SRC_I32 : TERN_SRC_F32;
        return result(launch([&] { return tern_threshold_pack(ps, t, d, pl, ph, po, s); }), a[3], out);
    });
}

// A workspace tensor of at least `need` bytes, or a new one for None.
at::Tensor workspace_of(PyObject* o, size_t need, const at::Tensor& like)
{
    if (o == Py_None) return at::empty({(int64_t)need}, like.options().dtype(at::kByte));
    return tensor(o, at::kByte);
}

// fcn(x, in_lo, in_hi, layers, workspace, out)
PyObject* fcn(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    TERN_ARGS(6)
    return guarded([&]() -> PyObject* {
        const at::Tensor& x = tensor(a[0], at::kFloat);
        const at::Tensor& lo = tensor(a[1], at::kFloat);
        const at::Tensor& hi = tensor(a[2], at::kFloat);
        const tern_dims d = dims5(x);
        if (lo.numel() != d.c || hi.numel() != d.c) throw Other();
        Ref list(items(a[3]));
        const Py_ssize_t n = PyTuple_GET_SIZE(list.o);
        if (n < 1 || n > 1024) throw Other();
        std::vector<tern_layer> layers((size_t)n);
        tern_dims cur = d;
        for (Py_ssize_t i = 0; i < n; ++i) {
            PyObject* L = PyTuple_GET_ITEM(list.o, i);
            tern_layer& l = layers[(size_t)i];
            l.c_in = attr_int(L, g_names.c_in);
            l.c_out = attr_int(L, g_names.c_out);
            attr_triple(L, g_names.k, l.g.k); attr_triple(L, g_names.stride, l.g.stride);
            attr_triple(L, g_names.pad, l.g.pad); attr_triple(L, g_names.dil, l.g.dil);
            Ref bank(PyObject_GetAttr(L, g_names.w_bank)), tl(PyObject_GetAttr(L, g_names.thr_lo)),
                th(PyObject_GetAttr(L, g_names.thr_hi));
            const at::Tensor& b = tensor(bank.o, at::kInt);
            const at::Tensor& t0 = tensor(tl.o, at::kInt);
            const at::Tensor& t1 = tensor(th.o, at::kInt);
            const size_t need = tern_filter_bank_bytes(l.c_out, l.c_in, l.g.k[0], l.g.k[1], l.g.k[2]);
            if (need == 0 || (size_t)b.numel() * 4 != need || t0.numel() != l.c_out || t1.numel() != l.c_out) throw Other();
            l.w_bank = (const uint32_t*)b.data_ptr();
            l.thr_lo = (const int32_t*)t0.data_ptr();
            l.thr_hi = (const int32_t*)t1.data_ptr();
            tern_dims o;
            if (l.c_in != cur.c || tern_conv_out_dims(cur, l.c_out, l.g, &o) != TERN_OK) throw Other();
            cur = o;
        }
        const size_t need = tern_fcn_workspace_bytes(d, layers.data(), (int32_t)n);
        if (need == 0) throw Other();
        const at::Tensor ws = workspace_of(a[4], need, x);
        const at::Tensor out = packed_out(a[5], cur, x);
        const auto *px = (const float*)x.data_ptr(), *pl = (const float*)lo.data_ptr(), *ph = (const float*)hi.data_ptr();
        void *pw = ws.data_ptr(), *s = stream_of(x);
        const size_t have = (size_t)ws.numel();
        auto* po = (uint32_t*)out.data_ptr();
        return result(launch([&] {
                          return tern_fcn_forward(px, d, pl, ph, layers.data(), (int32_t)n, pw, have, po, nullptr, nullptr, s);
                      }), a[5], out);
    });
}

// net(x, in_lo, in_hi, mods, head_w, head_b, head_stride, head_pad, head_dil, workspace, head_out)
PyObject* net(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    TERN_ARGS(11)
    return guarded([&]() -> PyObject* {
        const at::Tensor& x = tensor(a[0], at::kFloat);
        const at::Tensor& lo = tensor(a[1], at::kFloat);
        const at::Tensor& hi = tensor(a[2], at::kFloat);
        const tern_dims d = dims5(x);
        if (lo.numel() < d.c || hi.numel() < d.c) throw Other();
        Ref list(items(a[3]));
        const Py_ssize_t n = PyTuple_GET_SIZE(list.o);
        if (n < 1 || n > 1024) throw Other();
        std::vector<tern_module> mods((size_t)n);
        std::vector<tern_dims> outs((size_t)n);
        tern_dims cur = d;
        for (Py_ssize_t i = 0; i < n; ++i) {
            PyObject* M = PyTuple_GET_ITEM(list.o, i);
            tern_module& m = mods[(size_t)i];
            m.c_out = attr_int(M, g_names.c_out);
            m.skip_from = attr_int(M, g_names.skip_from);
            attr_triple(M, g_names.k, m.g.k); attr_triple(M, g_names.stride, m.g.stride);
            attr_triple(M, g_names.pad, m.g.pad); attr_triple(M, g_names.dil, m.g.dil);
            attr_triple(M, g_names.up, m.up); attr_triple(M, g_names.pool, m.pool);
            Ref bank(PyObject_GetAttr(M, g_names.w_bank)), tl(PyObject_GetAttr(M, g_names.thr_lo)),
                th(PyObject_GetAttr(M, g_names.thr_hi));
            const at::Tensor& b = tensor(bank.o, at::kInt);
            const at::Tensor& t0 = tensor(tl.o, at::kInt);
            const at::Tensor& t1 = tensor(th.o, at::kInt);
            m.w_bank = (const uint32_t*)b.data_ptr();
            m.thr_lo = (const int32_t*)t0.data_ptr();
            m.thr_hi = (const int32_t*)t1.data_ptr();
            // extents, as the library walks them
            if (m.skip_from >= i || m.skip_from < -1) throw Other();
            int64_t e[4] = {cur.c, cur.d, cur.h, cur.w};
            for (int k = 0; k < 3; ++k) {
                if (m.up[k] < 1 || m.up[k] > 1024 || m.pool[k] < 1 || m.pool[k] > 4) throw Other();
                e[1 + k] *= m.up[k];
            }
            if (m.skip_from >= 0) e[0] += outs[(size_t)m.skip_from].c;
            if (m.pool[0] > 1 || m.pool[1] > 1 || m.pool[2] > 1) {
                e[0] = 64 * ((e[0] + 31) / 32);
                for (int k = 0; k < 3; ++k) e[1 + k] /= m.pool[k];
            }
            const tern_dims in = {cur.n, dim32(e[0]), dim32(e[1]), dim32(e[2]), dim32(e[3])};
            if (tern_conv_out_dims(in, m.c_out, m.g, &cur) != TERN_OK) throw Other();
            outs[(size_t)i] = cur;
            // the library reads this much of each (larger ones were always accepted)
            if ((size_t)b.numel() * 4 < tern_filter_bank_bytes(m.c_out, in.c, m.g.k[0], m.g.k[1], m.g.k[2]) ||
                t0.numel() < m.c_out || t1.numel() < m.c_out)
                throw Other();
        }
        const size_t need = tern_net_workspace_bytes(d, mods.data(), (int32_t)n);
        if (need == 0) throw Other();
        const at::Tensor ws = workspace_of(a[9], need, x);
        const auto *px = (const float*)x.data_ptr(), *pl = (const float*)lo.data_ptr(), *ph = (const float*)hi.data_ptr();
        const float *pw = nullptr, *pb = nullptr;
        float* po = nullptr;
        int32_t head_c_out = 0;
        tern_conv_geom g = {};
        at::Tensor out;
        if (a[4] == Py_None) {
            if (a[10] != Py_None) throw Other();
        } else {
            const at::Tensor& w = tensor(a[4], at::kFloat);
            const tern_dims wd = dims5(w);
            head_c_out = wd.n;
            g.k[0] = wd.d; g.k[1] = wd.h; g.k[2] = wd.w;
            triple(a[6], g.stride); triple(a[7], g.pad); triple(a[8], g.dil);
            if (wd.c != cur.c) throw Other();
            if (a[5] != Py_None) {
                const at::Tensor& bias = tensor(a[5], at::kFloat);
                if (bias.numel() < head_c_out) throw Other();
                pb = (const float*)bias.data_ptr();
            }
            tern_dims o;
            if (tern_conv_out_dims(cur, head_c_out, g, &o) != TERN_OK) throw Other();
            if (a[10] == Py_None) {
                out = at::empty({o.n, o.c, o.d, o.h, o.w}, x.options());
            } else {
                out = tensor(a[10], at::kFloat);
                if (out.numel() < (int64_t)o.n * o.c * o.d * o.h * o.w) throw Other();
            }
            pw = (const float*)w.data_ptr();
            po = (float*)out.data_ptr();
        }
        void *pws = ws.data_ptr(), *s = stream_of(x);
        const size_t have = (size_t)ws.numel();
        const int rc = launch([&] {
            return tern_net_forward(px, d, pl, ph, mods.data(), (int32_t)n, pw, pb, head_c_out, g, pws, have, po, nullptr,
                                    nullptr, nullptr, s);
        });
        if (!pw) return PyLong_FromLong(rc);
        return result(rc, a[10], out);
    });
}

#define TERN_METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {TERN_METHOD(conv), TERN_METHOD(pack), TERN_METHOD(threshold_pack), TERN_METHOD(fcn),
                          TERN_METHOD(net), {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_tern_torch", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tern_torch()
{
    PyObject* c = PyImport_ImportModule("torch._C");
    if (!c) return nullptr;
    g_raw_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
    Py_DECREF(c);
    if (!g_raw_stream) return nullptr;
    g_names = {PyUnicode_InternFromString("c_in"), PyUnicode_InternFromString("c_out"), PyUnicode_InternFromString("w_bank"),
               PyUnicode_InternFromString("thr_lo"), PyUnicode_InternFromString("thr_hi"), PyUnicode_InternFromString("k"),
               PyUnicode_InternFromString("stride"), PyUnicode_InternFromString("pad"), PyUnicode_InternFromString("dil"),
               PyUnicode_InternFromString("skip_from"), PyUnicode_InternFromString("up"), PyUnicode_InternFromString("pool")};
    return PyModule_Create(&kModule);
}
