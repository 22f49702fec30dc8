// The hot calls of sar.py: tensors checked and handed over to the C entry points.
//
// A short step is bound by the host: written in Python over ctypes, a call cost 2.5 to 3 us beside the entry point's own
// (HIP launches, 3 us each), and an all-blocks call another 1 to 2 us for every block, whose tensors were looked at attribute
// by attribute.  The functions here take the arguments of sar.py's functions of the same names, in their order, and check
// what those state; they keep nothing between calls.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdarg>
#include <cstdio>
#include <string>
#include <vector>

#include "../../include/sar_mi355x.h"

namespace {

// A Python error is set.
struct Raised {};

// What the library, or a check here, refuses: sar.SarError with this code and text.
struct Refused {
    int code;
    std::string text;
};

[[noreturn]] void raise_sar(int code, const std::string& text) { throw Refused{code, text}; }

// SarError is that of the package this module was imported as a part of, whatever its name.
void set_error(PyObject* self, const Refused& r)
{
    const char* own = PyModule_GetName(self);
    if (!own) return;
    std::string name(own);
    name.erase(name.rfind('.') + 1);
    PyObject* m = PyImport_ImportModule((name + "sar").c_str());
    PyObject* type = m ? PyObject_GetAttrString(m, "SarError") : nullptr;
    PyObject* e = type ? PyObject_CallFunction(type, "is", r.code, r.text.c_str()) : nullptr;
    if (e) PyErr_SetObject(type, e);
    Py_XDECREF(e);
    Py_XDECREF(type);
    Py_XDECREF(m);
}

[[noreturn]] void refuse(const char* fmt, ...) __attribute__((format(printf, 1, 2)));
void refuse(const char* fmt, ...)
{
    char text[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(text, sizeof text, fmt, ap);
    va_end(ap);
    raise_sar(SAR_ERR_INVALID_ARG, text);
}

void check(int rc)
{
    if (rc != SAR_OK) raise_sar(rc, sar_last_error());
}

// ---- arguments

const at::Tensor& tensor(PyObject* o)
{
    if (!THPVariable_Check(o)) {
        // (None has none of a tensor's attributes, and says so)
        PyErr_Format(o == Py_None ? PyExc_AttributeError : PyExc_TypeError, "expected a tensor, got %s", Py_TYPE(o)->tp_name);
        throw Raised{};
    }
    return THPVariable_Unpack(o);
}

template <typename T = void>
T* ptr_of(const at::Tensor& t)
{
    if (!t.is_contiguous()) {
        PyErr_SetString(PyExc_AssertionError, "tensors passed to the library must be contiguous");
        throw Raised{};
    }
    return static_cast<T*>(t.data_ptr());
}

// the address of a tensor, or null for None
template <typename T = void>
T* ptr(PyObject* o)
{
    return o == Py_None ? nullptr : ptr_of<T>(tensor(o));
}

// an address given as a number, or null for None
template <typename T>
T* address(PyObject* o)
{
    if (o == Py_None) return nullptr;
    PyObject* n = PyLong_Check(o) ? (Py_INCREF(o), o) : PyObject_GetAttrString(o, "value");   // (ctypes.c_void_p)
    if (!n) throw Raised{};
    void* p = n == Py_None ? nullptr : PyLong_AsVoidPtr(n);
    Py_DECREF(n);
    if (PyErr_Occurred()) throw Raised{};
    return static_cast<T*>(p);
}

int64_t integer(PyObject* o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
}

float real(PyObject* o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Raised{};
    return (float)v;
}

int truth(PyObject* o)
{
    PyObject* n = PyNumber_Long(o);
    if (!n) throw Raised{};
    const long long v = PyLong_AsLongLong(n);
    Py_DECREF(n);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v != 0;
}

std::string type_name(at::ScalarType t)
{
    return std::string("torch.") + c10::getDtypeNames(t).first;
}

int dtype_code(at::ScalarType t)
{
    if (t == at::kFloat) return SAR_F32;
    if (t == at::kBFloat16) return SAR_BF16;
    raise_sar(SAR_ERR_UNSUPPORTED, "dtype " + type_name(t));
}

size_t bytes_of(PyObject* o) { return tensor(o).numel() * tensor(o).element_size(); }

// ... of scratch that a call may do without
size_t bytes_if(PyObject* o) { return o == Py_None ? 0 : bytes_of(o); }

std::string shape_text(const at::Tensor& t)
{
    std::string s = "(";
    for (int64_t d = 0; d < t.dim(); ++d) s += (d ? ", " : "") + std::to_string(t.size(d));
    return s + (t.dim() == 1 ? ",)" : ")");
}

// The C side takes one size for both.
void same_shape(const at::Tensor& a, PyObject* o)
{
    if (o == Py_None) return;
    const at::Tensor& b = tensor(o);
    if (a.sizes() != b.sizes() || a.scalar_type() != b.scalar_type())
        raise_sar(SAR_ERR_INVALID_ARG, "tensors of shape " + shape_text(a) + " " + type_name(a.scalar_type()) + " and " +
                                           shape_text(b) + " " + type_name(b.scalar_type()) + " must match");
}

// The sizes of a tensor of `N` dimensions.
template <int N>
void unpack_sizes(const at::Tensor& t, int64_t (&out)[N])
{
    if (t.dim() != N) {
        PyErr_Format(PyExc_ValueError, "expected a tensor of %d dimensions, got %lld", N, (long long)t.dim());
        throw Raised{};
    }
    for (int d = 0; d < N; ++d) out[d] = t.size(d);
}

// torch.cuda.<what>()
PyObject* cuda(const char* what)
{
    PyObject* m = PyImport_ImportModule("torch.cuda");
    PyObject* r = m ? PyObject_CallMethod(m, what, nullptr) : nullptr;
    Py_XDECREF(m);
    if (!r) throw Raised{};
    Py_DECREF(r);                    // (True, False, or an object that is not looked at)
    return r;
}

// The stream work is sent to: torch's current one, which sets up the device where nothing has; null where there is none.
void* stream()
{
    static bool ready = false;       // torch.cuda.is_initialized() does not go back
    if (!ready) {
        if (cuda("is_initialized") != Py_True) {
            if (cuda("is_available") != Py_True) return nullptr;
            cuda("current_stream");
        }
        ready = true;
    }
    return c10::hip::getCurrentHIPStream().stream();
}

// A sar.Blocks object.
struct Blocks {
    const sar_blocks_t* h;
    int P = 0;
    int64_t n_dst = 0;
    bool compact;
    explicit Blocks(PyObject* b)
    {
        static PyObject *const addr = PyUnicode_InternFromString("_addr"), *const flags = PyUnicode_InternFromString("flags");
        PyObject* a = PyObject_GetAttr(b, addr);
        if (!a) throw Raised{};
        if (a == Py_None) {
            Py_DECREF(a);
            raise_sar(SAR_ERR_STATE, "blocks handle already freed");
        }
        h = static_cast<const sar_blocks_t*>(PyLong_AsVoidPtr(a));
        Py_DECREF(a);
        if (PyErr_Occurred()) throw Raised{};
        PyObject* f = PyObject_GetAttr(b, flags);
        if (!f) throw Raised{};
        compact = (PyLong_AsLong(f) & SAR_BUILD_COMPACT) != 0;
        Py_DECREF(f);
        if (PyErr_Occurred()) throw Raised{};
        check(sar_blocks_info(h, &P, &n_dst));
    }
    sar_block_view view(int64_t q) const
    {
        sar_block_view v;
        check(sar_blocks_get(h, (int)q, &v));
        return v;
    }
    void rows(int64_t q, PyObject* o) const
    {
        if (o == Py_None) return;
        const int64_t n = view(q).n_src, has = tensor(o).size(0);
        if (has != n) refuse("block %lld has %lld sources, tensor has %lld rows", (long long)q, (long long)n, (long long)has);
    }
    void err_rows(int64_t q, PyObject* o) const
    {
        if (o == Py_None) return;
        const sar_block_view v = view(q);
        const int64_t n = compact ? v.n_t_rows : v.n_src, has = tensor(o).size(0);
        if (has != n) refuse("block %lld's error has %lld rows, tensor has %lld", (long long)q, (long long)n, (long long)has);
    }
    void dst(PyObject* o) const
    {
        if (o == Py_None) return;
        const int64_t has = tensor(o).size(0);
        if (has != n_dst) refuse("handle has %lld destinations, tensor has %lld rows", (long long)n_dst, (long long)has);
    }
};

// One tensor per block (or None): their addresses, for the calls that reinterpret the memory.
struct List {
    PyObject* items = nullptr;
    std::vector<void*> p;
    List() = default;
    List(const List&) = delete;
    ~List() { Py_XDECREF(items); }
    void open(PyObject* seq)
    {
        // by position: a set has no order, and an iterator is at its end after one look
        if (!PySequence_Check(seq) && !THPVariable_Check(seq)) {
            PyErr_Format(PyExc_TypeError, "expected one tensor per block, got %s", Py_TYPE(seq)->tp_name);
            throw Raised{};
        }
        items = PySequence_Fast(seq, "expected one tensor per block");
        if (!items) throw Raised{};
    }
    PyObject* at(int64_t q) const
    {
        if (q >= PySequence_Fast_GET_SIZE(items)) {
            PyErr_SetString(PyExc_IndexError, "list index out of range");
            throw Raised{};
        }
        return PySequence_Fast_GET_ITEM(items, q);
    }
    void take(const char* what, at::ScalarType dtype, int64_t row_values)
    {
        const Py_ssize_t n = PySequence_Fast_GET_SIZE(items);
        p.assign(n, nullptr);
        for (Py_ssize_t k = 0; k < n; ++k) {
            PyObject* o = PySequence_Fast_GET_ITEM(items, k);
            if (o == Py_None) continue;
            const at::Tensor& t = tensor(o);
            if (!t.is_cuda() || !t.is_contiguous()) refuse("%s[%d] must be a contiguous device tensor", what, (int)k);
            if (t.scalar_type() != dtype)
                refuse("%s[%d] is %s, the call needs %s", what, (int)k, type_name(t.scalar_type()).c_str(),
                       type_name(dtype).c_str());
            if (t.numel() != t.size(0) * row_values)
                refuse("%s[%d] has %lld values per row, the call needs %lld", what, (int)k,
                       (long long)(t.numel() / std::max<int64_t>(t.size(0), 1)), (long long)row_values);
            p[k] = t.data_ptr();
        }
    }
    template <typename T>
    T* const* as() const
    {
        return items ? reinterpret_cast<T* const*>(p.data()) : nullptr;
    }
};

// ---- calls

// The entry point, without Python's lock, as ctypes makes a call.
template <typename F>
void call(F&& f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    check(rc);
}

template <int N, typename F>
PyObject* entry(PyObject* self, PyObject* const* a, Py_ssize_t n, F&& f)
{
    HANDLE_TH_ERRORS
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
        return nullptr;
    }
    try {
        f(a);
    } catch (const Raised&) {
        return nullptr;
    } catch (const Refused& r) {
        set_error(self, r);
        return nullptr;
    }
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}
#define SAR_CALL(name, n_args) \
    PyObject* name(PyObject* self, PyObject* const* args, Py_ssize_t n) { return entry<n_args>(self, args, n, [](PyObject* const* a) {
#define SAR_CALL_END }); }

// b, Zq, mean, out, residual, act
SAR_CALL(spmm_all, 6)
    const Blocks b(a[0]);
    List Z;
    Z.open(a[1]);
    for (int q = 0; q < b.P; ++q) b.rows(q, Z.at(q));
    b.dst(a[3]);
    const at::Tensor& out = tensor(a[3]);
    same_shape(out, a[4]);
    const int64_t F = out.size(-1);
    Z.take("Zq", out.scalar_type(), F);
    const int dt = dtype_code(out.scalar_type()), mean = truth(a[2]), act = (int)integer(a[5]);
    void *const r = ptr(a[4]), *const o = ptr_of(out), *const st = stream();
    call([&] { return sar_spmm_all(b.h, Z.as<const void>(), dt, (int)F, mean, r, act, o, st); });
SAR_CALL_END

// h, dH, act, G
SAR_CALL(act_bwd, 4)
    const at::Tensor& h = tensor(a[0]);
    same_shape(h, a[1]);
    same_shape(h, a[3]);
    void *const p = ptr_of(h), *const d = ptr(a[1]), *const g = ptr(a[3]), *const st = stream();
    const int dt = dtype_code(h.scalar_type()), act = (int)integer(a[2]);
    const int64_t count = h.numel();
    call([&] { return sar_act_bwd(p, d, act, g, dt, count, st); });
SAR_CALL_END

// b, G, mean, dZq
SAR_CALL(spmm_bwd_all, 4)
    const Blocks b(a[0]);
    List dZ;
    dZ.open(a[3]);
    for (int q = 0; q < b.P; ++q) b.err_rows(q, dZ.at(q));
    b.dst(a[1]);
    const at::Tensor& G = tensor(a[1]);
    const int64_t F = G.size(-1);
    dZ.take("dZq", G.scalar_type(), F);
    const int dt = dtype_code(G.scalar_type()), mean = truth(a[2]);
    void *const g = ptr_of(G), *const st = stream();
    call([&] { return sar_spmm_bwd_all(b.h, g, mean, dt, (int)F, dZ.as<void>(), st); });
SAR_CALL_END

// Eq, t_rank, accumulate, Ep
SAR_CALL(error_add, 4)
    const at::Tensor& Ep = tensor(a[3]);
    const int64_t rows = Ep.size(0), F = Ep.numel() / std::max<int64_t>(rows, 1);
    if (a[0] != Py_None) {
        const at::Tensor& Eq = tensor(a[0]);
        if (Eq.scalar_type() != Ep.scalar_type() || Eq.numel() != Eq.size(0) * F)
            refuse("Eq and Ep must have the same row width and type");
    }
    void *const e = ptr(a[0]), *const p = ptr_of(Ep), *const st = stream();
    const int32_t* const rank = address<const int32_t>(a[1]);
    const int acc = truth(a[2]), dt = dtype_code(Ep.scalar_type());
    call([&] { return sar_error_add(e, rank, acc, p, dt, rows, (int)F, st); });
SAR_CALL_END

// Z, a, score
SAR_CALL(gat_scores, 3)
    const at::Tensor& Z = tensor(a[0]);
    int64_t hd[2];
    unpack_sizes(tensor(a[1]), hd);
    void *const z = ptr_of(Z), *const st = stream();
    float *const v = ptr<float>(a[1]), *const s = ptr<float>(a[2]);
    const int dt = dtype_code(Z.scalar_type());
    const int64_t rows = Z.size(0);
    call([&] { return sar_gat_scores(z, dt, rows, (int)hd[0], (int)hd[1], v, s, st); });
SAR_CALL_END

// m, l, acc
SAR_CALL(gat_fwd_begin, 3)
    int64_t nhd[3];
    unpack_sizes(tensor(a[2]), nhd);
    float *const m = ptr<float>(a[0]), *const l = ptr<float>(a[1]), *const acc = ptr<float>(a[2]);
    void* const st = stream();
    call([&] { return sar_gat_fwd_begin(m, l, acc, nhd[0], (int)nhd[1], (int)nhd[2], st); });
SAR_CALL_END

// b, q, Zq, s, tq, a_l, slope, m, l, acc
SAR_CALL(gat_fwd_block, 10)
    const Blocks b(a[0]);
    const int64_t q = integer(a[1]);
    int64_t nhd[3];
    unpack_sizes(tensor(a[9]), nhd);
    b.rows(q, a[2]);
    b.rows(q, a[4]);
    for (int k : {3, 7, 8, 9}) b.dst(a[k]);
    void *const z = ptr(a[2]), *const st = stream();
    float *const s = ptr<float>(a[3]), *const t = ptr<float>(a[4]), *const al = ptr<float>(a[5]);
    float *const m = ptr<float>(a[7]), *const l = ptr<float>(a[8]), *const acc = ptr<float>(a[9]);
    const int dt = dtype_code(tensor(a[2]).scalar_type());
    const float slope = real(a[6]);
    call([&] { return sar_gat_fwd_block(b.h, (int)q, z, s, t, al, dt, (int)nhd[1], (int)nhd[2], slope, m, l, acc, st); });
SAR_CALL_END

// m, l, acc, out, L, act
SAR_CALL(gat_fwd_end, 6)
    int64_t nhd[3];
    unpack_sizes(tensor(a[2]), nhd);
    float *const m = ptr<float>(a[0]), *const l = ptr<float>(a[1]), *const acc = ptr<float>(a[2]), *const L = ptr<float>(a[4]);
    void *const out = ptr(a[3]), *const st = stream();
    const int act = (int)integer(a[5]), dt = dtype_code(tensor(a[3]).scalar_type());
    call([&] { return sar_gat_fwd_end(m, l, acc, act, out, L, dt, nhd[0], (int)nhd[1], (int)nhd[2], st); });
SAR_CALL_END

// b, Zq, s, tq, a_l, slope, out, L, act
SAR_CALL(gat_fwd_all, 9)
    const Blocks b(a[0]);
    const at::Tensor& out = tensor(a[6]);
    int64_t nhd[3];
    unpack_sizes(out, nhd);
    List Z, t;
    Z.open(a[1]);
    if (a[3] != Py_None) t.open(a[3]);
    for (int q = 0; q < b.P; ++q) {
        b.rows(q, Z.at(q));
        if (t.items) b.rows(q, t.at(q));
    }
    for (int k : {2, 6, 7}) b.dst(a[k]);
    Z.take("Zq", out.scalar_type(), nhd[1] * nhd[2]);
    if (t.items) t.take("tq", at::kFloat, nhd[1]);
    float *const s = ptr<float>(a[2]), *const al = ptr<float>(a[4]), *const L = ptr<float>(a[7]);
    void *const o = ptr_of(out), *const st = stream();
    const int dt = dtype_code(out.scalar_type()), act = (int)integer(a[8]);
    const float slope = real(a[5]);
    call([&] {
        return sar_gat_fwd_all(b.h, Z.as<const void>(), s, t.as<const float>(), al, dt, (int)nhd[1], (int)nhd[2], slope, act, o,
                               L, st);
    });
SAR_CALL_END

// G, out, s, L, rec, ds, act, Gact
SAR_CALL(gat_bwd_begin, 8)
    const at::Tensor& G = tensor(a[0]);
    int64_t nhd[3];
    unpack_sizes(G, nhd);
    same_shape(G, a[1]);
    same_shape(G, a[7]);
    void *const g = ptr_of(G), *const o = ptr(a[1]), *const ga = ptr(a[7]), *const st = stream();
    float *const s = ptr<float>(a[2]), *const L = ptr<float>(a[3]), *const rec = ptr<float>(a[4]), *const ds = ptr<float>(a[5]);
    const int act = (int)integer(a[6]), dt = dtype_code(G.scalar_type());
    call([&] { return sar_gat_bwd_begin(g, o, s, L, act, ga, dt, rec, ds, nhd[0], (int)nhd[1], (int)nhd[2], st); });
SAR_CALL_END

// b, q, Zq, G, tq, rec, a_l, slope, dZq, dtq, ds, da_l, work
SAR_CALL(gat_bwd_block, 13)
    const Blocks b(a[0]);
    const int64_t q = integer(a[1]);
    int64_t hd[2];
    unpack_sizes(tensor(a[6]), hd);
    b.rows(q, a[2]);
    b.rows(q, a[4]);
    b.err_rows(q, a[8]);
    b.err_rows(q, a[9]);
    for (int k : {3, 5, 10}) b.dst(a[k]);
    void *const z = ptr(a[2]), *const g = ptr(a[3]), *const dz = ptr(a[8]), *const work = ptr(a[12]), *const st = stream();
    float *const t = ptr<float>(a[4]), *const rec = ptr<float>(a[5]), *const al = ptr<float>(a[6]), *const dt_q = ptr<float>(a[9]);
    float *const ds = ptr<float>(a[10]), *const da = ptr<float>(a[11]);
    const int dt = dtype_code(tensor(a[3]).scalar_type());
    const float slope = real(a[7]);
    const size_t wb = bytes_of(a[12]);
    call([&] {
        return sar_gat_bwd_block(b.h, (int)q, z, g, t, rec, al, dt, (int)hd[0], (int)hd[1], slope, dz, dt_q, ds, da, work, wb, st);
    });
SAR_CALL_END

// b, Zq, G, tq, rec, a_l, slope, dZq, dtq, ds, da_l, work
SAR_CALL(gat_bwd_all, 12)
    const Blocks b(a[0]);
    int64_t hd[2];
    unpack_sizes(tensor(a[5]), hd);
    List Z, t, dZ, dt_q;
    Z.open(a[1]);
    if (a[3] != Py_None) t.open(a[3]);
    dZ.open(a[7]);
    if (a[8] != Py_None) dt_q.open(a[8]);
    for (int q = 0; q < b.P; ++q) {
        b.rows(q, Z.at(q));
        if (t.items) b.rows(q, t.at(q));
        b.err_rows(q, dZ.at(q));
        if (dt_q.items) b.err_rows(q, dt_q.at(q));
    }
    for (int k : {2, 4, 9}) b.dst(a[k]);
    const at::Tensor& G = tensor(a[2]);
    Z.take("Zq", G.scalar_type(), hd[0] * hd[1]);
    if (t.items) t.take("tq", at::kFloat, hd[0]);
    dZ.take("dZq", G.scalar_type(), hd[0] * hd[1]);
    if (dt_q.items) dt_q.take("dtq", at::kFloat, hd[0]);
    void *const g = ptr_of(G), *const work = ptr(a[11]), *const st = stream();
    float *const rec = ptr<float>(a[4]), *const al = ptr<float>(a[5]), *const ds = ptr<float>(a[9]), *const da = ptr<float>(a[10]);
    const int dt = dtype_code(G.scalar_type());
    const float slope = real(a[6]);
    const size_t wb = bytes_of(a[11]);
    call([&] {
        return sar_gat_bwd_all(b.h, Z.as<const void>(), g, t.as<const float>(), rec, al, dt, (int)hd[0], (int)hd[1], slope,
                               dZ.as<void>(), dt_q.as<float>(), ds, da, work, wb, st);
    });
SAR_CALL_END

// Zdst, ds, a_r, dZadd, dZdst, da_r, work, dZadd_rank
SAR_CALL(gat_bwd_end, 8)
    const at::Tensor& Z = tensor(a[0]);
    int64_t hd[2];
    unpack_sizes(tensor(a[2]), hd);
    void *const z = ptr_of(Z), *const add = ptr(a[3]), *const out = ptr(a[4]), *const work = ptr(a[6]), *const st = stream();
    float *const ds = ptr<float>(a[1]), *const ar = ptr<float>(a[2]), *const da = ptr<float>(a[5]);
    const int32_t* const rank = address<const int32_t>(a[7]);
    const int dt = dtype_code(Z.scalar_type());
    const int64_t rows = Z.size(0);
    const size_t wb = bytes_of(a[6]);
    call([&] {
        return sar_gat_bwd_end(z, ds, ar, add, rank, out, da, dt, rows, (int)hd[0], (int)hd[1], work, wb, st);
    });
SAR_CALL_END

// X, W, Z, a_score, score, a_score2, score2
SAR_CALL(linear_fwd, 7)
    const at::Tensor &X = tensor(a[0]), &W = tensor(a[1]);
    int64_t nk[2], hd[2] = {0, 0};
    unpack_sizes(X, nk);
    const int64_t F = W.size(1);
    if (a[3] != Py_None) unpack_sizes(tensor(a[3]), hd);
    void *const x = ptr_of(X), *const z = ptr(a[2]), *const st = stream();
    float* const w = ptr_of<float>(W);
    float *const a1 = ptr<float>(a[3]), *const s1 = ptr<float>(a[4]), *const a2 = ptr<float>(a[5]), *const s2 = ptr<float>(a[6]);
    const int dt = dtype_code(X.scalar_type());
    call([&] {
        return sar_linear_fwd(x, w, z, dt, nk[0], (int)nk[1], (int)F, (int)hd[0], (int)hd[1], a1, s1, a2, s2, st);
    });
SAR_CALL_END

int64_t inner(PyObject* X, PyObject* W) { return X != Py_None ? tensor(X).size(1) : tensor(W).size(0); }

// X, dZ, W, dW, dX, work
SAR_CALL(linear_bwd, 6)
    const at::Tensor& dZ = tensor(a[1]);
    const int64_t rows = dZ.size(0), F = dZ.numel() / std::max<int64_t>(rows, 1), K = inner(a[0], a[2]);
    void *const x = ptr(a[0]), *const dz = ptr_of(dZ), *const dx = ptr(a[4]), *const work = ptr(a[5]), *const st = stream();
    float *const w = ptr<float>(a[2]), *const dw = ptr<float>(a[3]);
    const int dt = dtype_code(dZ.scalar_type());
    const size_t wb = bytes_if(a[5]);
    call([&] { return sar_linear_bwd(x, dz, w, dw, dx, dt, rows, (int)K, (int)F, work, wb, st); });
SAR_CALL_END

// X, E, E_rank, ds, a_r, H, D, W, dW, dX, n, dtype code, work, rows
SAR_CALL(linear_bwd_rows, 14)
    const int64_t K = inner(a[0], a[7]), n_E = a[1] == Py_None ? 0 : tensor(a[1]).size(0), n_rows = integer(a[10]);
    void *const x = ptr(a[0]), *const e = ptr(a[1]), *const dx = ptr(a[9]), *const rows = ptr(a[13]), *const work = ptr(a[12]);
    const int32_t* const rank = address<const int32_t>(a[2]);
    float *const ds = ptr<float>(a[3]), *const ar = ptr<float>(a[4]), *const w = ptr<float>(a[7]), *const dw = ptr<float>(a[8]);
    const int H = (int)integer(a[5]), D = (int)integer(a[6]), dt = (int)integer(a[11]);
    void* const st = stream();
    const size_t wb = bytes_if(a[12]);
    call([&] {
        return sar_linear_bwd_rows(x, e, rank, n_E, ds, ar, H, D, w, dw, dx, dt, n_rows, (int)K, rows, work, wb, st);
    });
SAR_CALL_END

#define SAR_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    SAR_METHOD(spmm_all), SAR_METHOD(act_bwd), SAR_METHOD(spmm_bwd_all), SAR_METHOD(error_add), SAR_METHOD(gat_scores),
    SAR_METHOD(gat_fwd_begin), SAR_METHOD(gat_fwd_block), SAR_METHOD(gat_fwd_end), SAR_METHOD(gat_fwd_all),
    SAR_METHOD(gat_bwd_begin), SAR_METHOD(gat_bwd_block), SAR_METHOD(gat_bwd_all), SAR_METHOD(gat_bwd_end),
    SAR_METHOD(linear_fwd), SAR_METHOD(linear_bwd), SAR_METHOD(linear_bwd_rows), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding()
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", SAR_BUILT_FOR) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
