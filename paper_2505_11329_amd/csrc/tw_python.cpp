// CPython module over libtw: takes torch tensors and streams from Python, checks
// them, fills the argument structs of tw.h and calls the library. binding.py holds
// the public signatures and forwards to it.
//
// A decode-sized fused step keeps the GPU busy for 4 us, and checking its twelve
// tensors one Python attribute at a time took 13 us of the 17 us a call cost the
// host; read through torch's C++ objects the checks are a few loads each.
// Measured on MI355X, back-to-back calls of 16 rows, H = 8192, P = 8: 16.7 us a
// call through Python attributes and ctypes; through this module 3.3 us of host time in
// a long train of calls (3.9 in bursts of 40 after a synchronisation), while the device
// takes 4.1 us a step.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <new>
#include <vector>

#include "tw.h"

namespace {

PyObject *g_error;  // binding.TwError(status, what)

// Thrown with a Python exception set.
struct PyFail {};

[[noreturn]] void fail() { throw PyFail(); }

template <typename... A>
[[noreturn]] void fail(PyObject *type, const char *fmt, A... a)
{
    PyErr_Format(type, fmt, a...);
    throw PyFail();
}

struct Ref {  // an owned reference
    PyObject *o = nullptr;
    Ref() {}
    explicit Ref(PyObject *p) : o(p) {}
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
    Ref(Ref &&r) noexcept : o(r.o) { r.o = nullptr; }
    Ref &operator=(Ref &&r) noexcept
    {
        PyObject *old = o;
        o = r.o;
        r.o = nullptr;
        Py_XDECREF(old);
        return *this;
    }
    ~Ref() { Py_XDECREF(o); }
    PyObject *release()
    {
        PyObject *p = o;
        o = nullptr;
        return p;
    }
};

int64_t as_int(PyObject *o)
{
    if (PyLong_CheckExact(o)) {
        const int64_t v = PyLong_AsLongLong(o);
        if (v == -1 && PyErr_Occurred()) fail();
        return v;
    }
    Ref n(PyNumber_Long(o));
    if (!n.o) fail();
    const int64_t v = PyLong_AsLongLong(n.o);
    if (v == -1 && PyErr_Occurred()) fail();
    return v;
}
int as_c_int(PyObject *o) { return static_cast<int>(as_int(o)); }
float as_float(PyObject *o)
{
    if (PyFloat_CheckExact(o)) return static_cast<float>(PyFloat_AS_DOUBLE(o));
    Ref n(PyNumber_Float(o));
    if (!n.o) fail();
    return static_cast<float>(PyFloat_AS_DOUBLE(n.o));
}
int as_bool(PyObject *o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) fail();
    return v;
}

// The layout that equals o, as Python compares: 1.0 is one, 0.5 and "0" are none.
int64_t b_layout(PyObject *o)
{
    for (const int64_t layout : {int64_t(TW_B_NK), int64_t(TW_B_KN)}) {
        Ref v(PyLong_FromLongLong(layout));
        const int same = v.o ? PyObject_RichCompareBool(o, v.o, Py_EQ) : -1;
        if (same < 0) fail();
        if (same) return layout;
    }
    fail(PyExc_ValueError, "b_layout must be B_NK or B_KN");
}

// hipStream_t of a torch stream; None means torch's current stream.
void *stream_handle(PyObject *o)
{
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    static PyObject *name = PyUnicode_InternFromString("cuda_stream");
    Ref h(PyObject_GetAttr(o, name));
    if (!h.o) fail();
    const size_t v = PyLong_AsSize_t(h.o);
    if (v == static_cast<size_t>(-1) && PyErr_Occurred()) fail();
    return reinterpret_cast<void *>(v);
}

// What a tensor argument is called in error messages: a name, or name[index].
struct Name {
    const char *s;
    int i = -1;
    PyObject *py() const { return i < 0 ? PyUnicode_FromString(s) : PyUnicode_FromFormat("%s[%d]", s, i); }
};

[[noreturn]] void bad_tensor(PyObject *type, const char *fmt, const Name &n, PyObject *what = nullptr,
                             PyObject *what2 = nullptr)
{
    Ref name(n.py());
    if (!name.o) fail();
    PyErr_Format(type, fmt, name.o, what, what2);
    throw PyFail();
}

const at::Tensor &gpu_tensor(PyObject *o, const Name &n)
{
    if (!THPVariable_Check(o) || !THPVariable_Unpack(o).is_cuda())
        bad_tensor(PyExc_TypeError, "%U must be a GPU tensor", n);
    return THPVariable_Unpack(o);
}

Ref attr_str(PyObject *o, const char *attr)
{
    Ref a(PyObject_GetAttrString(o, attr));
    if (!a.o) fail();
    return a;
}

// Device pointer of a contiguous bf16 GPU tensor; with ndim >= 0 its shape must be the given one.
void *bf16_ptr(PyObject *o, const Name &n, int ndim = -1, int64_t d0 = 0, int64_t d1 = 0)
{
    const at::Tensor &t = gpu_tensor(o, n);
    if (t.scalar_type() != at::kBFloat16) {
        Ref dt = attr_str(o, "dtype");
        bad_tensor(PyExc_TypeError, "%U must be bfloat16, got %S", n, dt.o);
    }
    if (!t.is_contiguous()) bad_tensor(PyExc_ValueError, "%U must be contiguous", n);
    if (ndim >= 0) {
        const auto s = t.sizes();
        if (static_cast<int>(s.size()) != ndim || (ndim > 0 && s[0] != d0) || (ndim > 1 && s[1] != d1)) {
            Ref sh = attr_str(o, "shape");
            Ref got(PySequence_Tuple(sh.o));
            Ref want(ndim == 1 ? Py_BuildValue("(L)", static_cast<long long>(d0))
                               : Py_BuildValue("(LL)", static_cast<long long>(d0), static_cast<long long>(d1)));
            if (!got.o || !want.o) fail();
            bad_tensor(PyExc_ValueError, "%U has shape %S, expected %S", n, got.o, want.o);
        }
    }
    return t.data_ptr();
}

// A required 2-D tensor whose sizes other arguments are checked against.
const at::Tensor &matrix(PyObject *o, const char *name, const char *message)
{
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "%s must be a GPU tensor", name);
    const at::Tensor &t = THPVariable_Unpack(o);
    if (t.dim() != 2) fail(PyExc_ValueError, "%s", message);
    return t;
}

// The given tensor, or a new [rows x cols] one like `like` when None was given.
Ref given_or_new(PyObject *o, const at::Tensor &like, int64_t rows, int64_t cols)
{
    if (o != Py_None) {
        Py_INCREF(o);
        return Ref(o);
    }
    Ref t(THPVariable_Wrap(at::empty({rows, cols}, like.options().dtype(at::kBFloat16))));
    if (!t.o) fail();
    return t;
}

// The items of a sequence that has a length, as a tuple nobody else can change. Room for the
// items is made by length, so one that iterates over another number of them is refused.
Ref items(PyObject *o, const char *name)
{
    const Py_ssize_t n = PyObject_Size(o);
    if (n < 0) fail();
    Ref t(PySequence_Tuple(o));
    if (!t.o) fail();
    if (PyTuple_GET_SIZE(t.o) != n)
        fail(PyExc_ValueError, "%s has a length of %zd and iterates over %zd", name, n, PyTuple_GET_SIZE(t.o));
    return t;
}

// ---- argument structs ----

struct PointerArray {  // the caller's, for the partials' device pointers
    void **p;
    size_t capacity;
};

struct Fused {
    tw_fused_args a;
    void *few[TW_MAX_P];
    std::vector<void *> many;  // more partials than the library takes: it is the one to refuse them
    Ref seq, out, residual_out;
    int64_t rows = 0, H = 0;

    void **room(Py_ssize_t P)
    {
        if (P <= TW_MAX_P) return few;
        many.resize(static_cast<size_t>(P));
        return many.data();
    }
    // given: where the partials' pointers go; without one, into this object
    void fill(PyObject *partials, PyObject *residual, PyObject *weight, PyObject *eps, PyObject *budget, PyObject *o,
              PyObject *ro, const PointerArray *given = nullptr)
    {
        const at::Tensor &res = matrix(residual, "residual", "residual must be [N, H]");
        rows = res.size(0);
        H = res.size(1);
        if (o == Py_None || ro == Py_None) gpu_tensor(residual, {"residual"});
        out = o == Py_None ? like(res) : given_or_new(o, res, rows, H);
        residual_out = ro == Py_None ? like(res) : given_or_new(ro, res, rows, H);
        seq = items(partials, "partials");
        const Py_ssize_t P = PyTuple_GET_SIZE(seq.o);
        if (given && static_cast<size_t>(P) > given->capacity)
            fail(PyExc_ValueError, "the pointer array has room for %zd of %zd partials",
                 static_cast<Py_ssize_t>(given->capacity), P);
        void **ptrs = given ? given->p : room(P);
        for (Py_ssize_t p = 0; p < P; ++p)
            ptrs[p] = bf16_ptr(PyTuple_GET_ITEM(seq.o, p), {"partials", static_cast<int>(p)}, 2, rows, H);
        a.partials = ptrs;
        a.residual = bf16_ptr(residual, {"residual"});
        a.weight = bf16_ptr(weight, {"weight"}, 1, H);
        a.eps = as_float(eps);
        a.N = rows;
        a.H = H;
        a.P = static_cast<int>(P);
        a.cu_budget = as_c_int(budget);
        a.out = bf16_ptr(out.o, {"out"}, 2, rows, H);
        a.residual_out = bf16_ptr(residual_out.o, {"residual_out"}, 2, rows, H);
    }
    static Ref like(const at::Tensor &t)
    {
        Ref r(THPVariable_Wrap(at::empty_like(t)));
        if (!r.o) fail();
        return r;
    }
};

struct Gemm {
    tw_gemm_args g;
    Ref C;
    void fill(PyObject *A, PyObject *B, PyObject *c, PyObject *layout, PyObject *budget)
    {
        const at::Tensor &a = matrix(A, "A", "A and B must be matrices"), &b = matrix(B, "B", "A and B must be matrices");
        const int64_t M = a.size(0), K = a.size(1), lay = b_layout(layout);
        const int64_t N = lay == TW_B_NK ? b.size(0) : b.size(1);
        g.B = lay == TW_B_NK ? bf16_ptr(B, {"B"}, 2, N, K) : bf16_ptr(B, {"B"}, 2, K, N);
        C = given_or_new(c, a, M, N);
        g.A = bf16_ptr(A, {"A"});
        g.C = bf16_ptr(C.o, {"C"}, 2, M, N);
        g.M = M;
        g.N = N;
        g.K = K;
        g.b_layout = static_cast<int>(lay);
        g.cu_budget = as_c_int(budget);
    }
};

struct Layer {
    Fused f;
    Ref Y;
    void fill(tw_layer_args &l, PyObject *X1, PyObject *W1, PyObject *partials, PyObject *residual, PyObject *weight,
              PyObject *eps, PyObject *W2, PyObject *fused_budget, PyObject *gemm_budget, PyObject *out, PyObject *ro,
              PyObject *y, PyObject *schedule, const PointerArray *given = nullptr)
    {
        f.fill(partials, residual, weight, eps, fused_budget, out, ro, given);
        const int64_t K1 = matrix(X1, "X1", "X1 must be [T, K1]").size(1);
        const int64_t N2 = matrix(W2, "W2", "W2 must be [N2, H]").size(0);
        Y = given_or_new(y, THPVariable_Unpack(residual), f.rows, N2);
        l.X1 = bf16_ptr(X1, {"X1"}, 2, f.rows, K1);
        l.W1 = bf16_ptr(W1, {"W1"}, 2, f.H, K1);
        l.K1 = K1;
        l.fused = f.a;
        l.W2 = bf16_ptr(W2, {"W2"}, 2, N2, f.H);
        l.N2 = N2;
        l.Y = bf16_ptr(Y.o, {"Y"}, 2, f.rows, N2);
        l.gemm_cu_budget = as_c_int(gemm_budget);
        l.schedule = as_c_int(schedule);
    }
};

// the streams of a cross-stream call
struct Parent {
    void *stream;
    int set, join;
    Parent(PyObject *parent, PyObject *use_parent, PyObject *join_)
        : stream(nullptr), set(as_bool(use_parent)), join(as_bool(join_))
    {
        if (set) stream = stream_handle(parent);
    }
};

// Calls the library without the interpreter lock, and raises TwError for a status that is not TW_OK.
template <typename F>
void call(const char *what, F &&f)
{
    tw_status s;
    Py_BEGIN_ALLOW_THREADS;
    s = f();
    Py_END_ALLOW_THREADS;
    if (s == TW_OK) return;
    Ref e(PyObject_CallFunction(g_error, "is", static_cast<int>(s), what));
    if (e.o) PyErr_SetObject(g_error, e.o);
    fail();
}

PyObject *pair(Ref &a, Ref &b)
{
    PyObject *t = PyTuple_New(2);
    if (!t) fail();
    PyTuple_SET_ITEM(t, 0, a.release());
    PyTuple_SET_ITEM(t, 1, b.release());
    return t;
}

// d[key], of a dict or any other mapping, the way Python looks it up.
Ref item(PyObject *d, const char *key)
{
    Ref k(PyUnicode_InternFromString(key));
    if (!k.o) fail();
    Ref v(PyObject_GetItem(d, k.o));
    if (!v.o) fail();
    return v;
}
// d.get(key, otherwise)
Ref item(PyObject *d, const char *key, PyObject *otherwise)
{
    static PyObject *get = PyUnicode_InternFromString("get");
    Ref k(PyUnicode_InternFromString(key));
    if (!k.o) fail();
    if (!PyDict_CheckExact(d)) {
        Ref v(PyObject_CallMethodObjArgs(d, get, k.o, otherwise, nullptr));
        if (!v.o) fail();
        return v;
    }
    PyObject *v = PyDict_GetItemWithError(d, k.o);
    if (!v && PyErr_Occurred()) fail();
    if (!v) v = otherwise;
    Py_INCREF(v);
    return Ref(v);
}

// Runs one entry of the module: n positional arguments, C++ and Python errors kept apart.
template <typename F>
PyObject *entry(const char *name, Py_ssize_t got, Py_ssize_t want, F &&f)
{
    if (got != want) return PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, got %zd", name, want, got);
    try {
        return f();
    } catch (const PyFail &) {
    } catch (const std::bad_alloc &) {
        PyErr_NoMemory();
    } catch (const c10::OutOfMemoryError &e) {
        Ref torch(PyImport_ImportModule("torch"));
        Ref type(torch.o ? PyObject_GetAttrString(torch.o, "OutOfMemoryError") : nullptr);
        if (type.o) PyErr_SetString(type.o, e.what_without_backtrace());
    } catch (const c10::Error &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

// ---- entry points (positional arguments in the order of binding.py's functions) ----

PyObject *py_reduce_add_rmsnorm(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("reduce_add_rmsnorm", n, 8, [&] {
        Fused f;
        f.fill(v[0], v[1], v[2], v[3], v[4], v[5], v[6]);
        void *s = stream_handle(v[7]);
        const tw_fused_args &a = f.a;
        call("tw_reduce_add_rmsnorm", [&] {
            return tw_reduce_add_rmsnorm(a.partials, a.residual, a.weight, a.eps, a.N, a.H, a.P, a.cu_budget, a.out,
                                         a.residual_out, s);
        });
        return pair(f.out, f.residual_out);
    });
}

PyObject *py_split_launch(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("split_launch", n, 13, [&] {
        Fused f;
        f.fill(v[0], v[1], v[2], v[3], v[7], v[8], v[9]);
        const int64_t row = as_int(v[4]);
        void *sa = stream_handle(v[5]), *sb = stream_handle(v[6]);
        const Parent p(v[10], v[11], v[12]);
        call("tw_split_launch", [&] { return tw_split_launch(&f.a, row, sa, sb, p.stream, p.set, p.join); });
        return pair(f.out, f.residual_out);
    });
}

PyObject *py_gemm_bf16(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("gemm_bf16", n, 6, [&] {
        Gemm m;
        m.fill(v[0], v[1], v[2], v[3], v[4]);
        void *s = stream_handle(v[5]);
        const tw_gemm_args &g = m.g;
        call("tw_gemm_bf16",
             [&] { return tw_gemm_bf16(g.A, g.B, g.C, g.M, g.N, g.K, g.b_layout, g.cu_budget, s); });
        return m.C.release();
    });
}

PyObject *py_overlap_launch(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("overlap_launch", n, 7, [&]() -> PyObject * {
        Fused f;
        Gemm m;
        Ref zero(PyLong_FromLong(0)), nk(PyLong_FromLong(TW_B_NK));
        const bool has_f = v[0] != Py_None, has_g = v[1] != Py_None;
        Ref of_f[7], of_g[5];  // held until the call has been made
        if (has_f) {
            of_f[0] = item(v[0], "partials");
            of_f[1] = item(v[0], "residual");
            of_f[2] = item(v[0], "weight");
            of_f[3] = item(v[0], "eps");
            of_f[4] = item(v[0], "cu_budget", zero.o);
            of_f[5] = item(v[0], "out", Py_None);
            of_f[6] = item(v[0], "residual_out", Py_None);
            f.fill(of_f[0].o, of_f[1].o, of_f[2].o, of_f[3].o, of_f[4].o, of_f[5].o, of_f[6].o);
        }
        if (has_g) {
            of_g[0] = item(v[1], "A");
            of_g[1] = item(v[1], "B");
            of_g[2] = item(v[1], "C", Py_None);
            of_g[3] = item(v[1], "b_layout", nk.o);
            of_g[4] = item(v[1], "cu_budget", zero.o);
            m.fill(of_g[0].o, of_g[1].o, of_g[2].o, of_g[3].o, of_g[4].o);
        }
        void *comm = stream_handle(v[2]), *compute = stream_handle(v[3]);
        const Parent p(v[4], v[5], v[6]);
        call("tw_overlap_launch", [&] {
            return tw_overlap_launch(has_f ? &f.a : nullptr, has_g ? &m.g : nullptr, comm, compute, p.stream, p.set,
                                     p.join);
        });
        return PyTuple_Pack(3, has_f ? f.out.o : Py_None, has_f ? f.residual_out.o : Py_None, has_g ? m.C.o : Py_None);
    });
}

// X1, W1, partials, residual, weight, eps, W2, stream_compute, stream_comm, fused_cu_budget, gemm_cu_budget, out,
// residual_out, Y, parent, use_parent, join, schedule, then the call's own: split_row | cuts | threshold, multiple
constexpr int kLayerArgs = 18;
struct LayerCall {
    Layer l;
    tw_layer_args a;
    void *sx, *sc;
    Parent p;
    explicit LayerCall(PyObject *const *v) : p(v[14], v[15], v[16])
    {
        l.fill(a, v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[9], v[10], v[11], v[12], v[13], v[17]);
        sx = stream_handle(v[7]);
        sc = stream_handle(v[8]);
    }
    PyObject *outputs(PyObject *last = nullptr)
    {
        return last ? PyTuple_Pack(4, l.f.out.o, l.f.residual_out.o, l.Y.o, last)
                    : PyTuple_Pack(3, l.f.out.o, l.f.residual_out.o, l.Y.o);
    }
};

PyObject *py_weave_layer(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("weave_layer", n, kLayerArgs + 1, [&] {
        LayerCall c(v);
        const int64_t row = as_int(v[kLayerArgs]);
        call("tw_weave_layer",
             [&] { return tw_weave_layer(&c.a, row, c.sx, c.sc, c.p.stream, c.p.set, c.p.join); });
        return c.outputs();
    });
}

PyObject *py_weave_layer_cuts(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("weave_layer_cuts", n, kLayerArgs + 1, [&] {
        LayerCall c(v);
        Ref seq(PySequence_Tuple(v[kLayerArgs]));
        if (!seq.o) fail();
        std::vector<int64_t> cuts(static_cast<size_t>(PyTuple_GET_SIZE(seq.o)));
        for (size_t i = 0; i < cuts.size(); ++i) cuts[i] = as_int(PyTuple_GET_ITEM(seq.o, i));
        const int n_cuts = static_cast<int>(cuts.size());
        cuts.push_back(0);  // never an empty array
        call("tw_weave_layer_cuts", [&] {
            return tw_weave_layer_cuts(&c.a, cuts.data(), n_cuts, c.sx, c.sc, c.p.stream, c.p.set, c.p.join);
        });
        return c.outputs();
    });
}

PyObject *py_weave_layer_auto(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("weave_layer_auto", n, kLayerArgs + 2, [&] {
        LayerCall c(v);
        const int64_t threshold = as_int(v[kLayerArgs]), multiple = as_int(v[kLayerArgs + 1]);
        int64_t taken = -1;
        call("tw_weave_layer_auto", [&] {
            return tw_weave_layer_auto(&c.a, threshold, multiple, c.sx, c.sc, c.p.stream, c.p.set, c.p.join, &taken);
        });
        Ref t(PyLong_FromLongLong(taken));
        if (!t.o) fail();
        return c.outputs(t.o);
    });
}

// boundaries, split_row, stream_compute, stream_comm, parent, use_parent, join, fused_cu_budget, gemm_cu_budget, schedule
PyObject *py_weave_train(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("weave_train", n, 10, [&]() -> PyObject * {
        const Ref seq = items(v[0], "boundaries");
        const size_t count = static_cast<size_t>(PyTuple_GET_SIZE(seq.o));
        struct Boundary {
            Ref of[10];  // the items of its dict, held until the call has been made
            Layer l;
        };
        static const char *const kKeys[10] = {"X1", "W1", "partials", "residual", "weight", "eps", "W2", "out", "residual_out", "Y"};
        std::vector<Boundary> boundaries(count);
        std::vector<tw_layer_args> args(count + 1);
        for (size_t i = 0; i < count; ++i) {
            Ref *of = boundaries[i].of;
            for (int j = 0; j < 10; ++j) of[j] = item(PyTuple_GET_ITEM(seq.o, i), kKeys[j]);
            // an output made here would be gone before the kernels that write it have run
            for (int j = 7; j < 10; ++j)
                if (of[j].o == Py_None) fail(PyExc_TypeError, "%s must be a GPU tensor", kKeys[j]);
            boundaries[i].l.fill(args[i], of[0].o, of[1].o, of[2].o, of[3].o, of[4].o, of[5].o, of[6].o, v[7], v[8], of[7].o,
                                 of[8].o, of[9].o, v[9]);
        }
        const int64_t row = as_int(v[1]);
        void *sx = stream_handle(v[2]), *sc = stream_handle(v[3]);
        const Parent p(v[4], v[5], v[6]);
        call("tw_weave_train", [&] {
            return tw_weave_train(args.data(), static_cast<int>(count), row, sx, sc, p.stream, p.set, p.join);
        });
        Py_RETURN_NONE;
    });
}

// ---- for the entry points that binding.py calls through ctypes ----

struct Buffer {
    Py_buffer b;
    Buffer(PyObject *o, size_t bytes)
    {
        if (PyObject_GetBuffer(o, &b, PyBUF_WRITABLE) < 0) fail();
        if (static_cast<size_t>(b.len) < bytes) {
            PyBuffer_Release(&b);
            fail(PyExc_ValueError, "the argument struct is too small");
        }
    }
    ~Buffer() { PyBuffer_Release(&b); }
    PointerArray pointers() const { return {static_cast<void **>(b.buf), static_cast<size_t>(b.len) / sizeof(void *)}; }
};

// fill_fused(struct, pointer_array, partials, residual, weight, eps, cu_budget, out, residual_out) -> (out, residual_out)
PyObject *py_fill_fused(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("fill_fused", n, 9, [&] {
        Buffer s(v[0], sizeof(tw_fused_args));
        Buffer ptrs(v[1], 0);
        Fused f;
        const PointerArray to = ptrs.pointers();
        f.fill(v[2], v[3], v[4], v[5], v[6], v[7], v[8], &to);
        *static_cast<tw_fused_args *>(s.b.buf) = f.a;
        return pair(f.out, f.residual_out);
    });
}

// fill_layer(struct, pointer_array, X1, W1, partials, residual, weight, eps, W2, fused_cu_budget, gemm_cu_budget, out,
// residual_out, Y, schedule) -> (out, residual_out, Y)
PyObject *py_fill_layer(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("fill_layer", n, 15, [&] {
        Buffer s(v[0], sizeof(tw_layer_args));
        Buffer ptrs(v[1], 0);
        const PointerArray to = ptrs.pointers();
        Layer l;
        l.fill(*static_cast<tw_layer_args *>(s.b.buf), v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10], v[11],
               v[12], v[13], v[14], &to);
        return PyTuple_Pack(3, l.f.out.o, l.f.residual_out.o, l.Y.o);
    });
}

// bf16_ptr(tensor, name, rows, cols) -> int
PyObject *py_bf16_ptr(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("bf16_ptr", n, 4, [&] {
        const char *name = PyUnicode_AsUTF8(v[1]);
        if (!name) fail();
        return PyLong_FromVoidPtr(bf16_ptr(v[0], {name}, 2, as_int(v[2]), as_int(v[3])));
    });
}

PyObject *py_stream_handle(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("stream_handle", n, 1, [&] { return PyLong_FromVoidPtr(stream_handle(v[0])); });
}

PyObject *py_set_error(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    return entry("set_error", n, 1, [&]() -> PyObject * {
        Py_INCREF(v[0]);
        Py_XSETREF(g_error, v[0]);
        Py_RETURN_NONE;
    });
}

#define TW_METHOD(name)                                                                                            \
    {                                                                                                              \
        #name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr      \
    }
PyMethodDef g_methods[] = {TW_METHOD(reduce_add_rmsnorm), TW_METHOD(split_launch),     TW_METHOD(gemm_bf16),
                           TW_METHOD(overlap_launch),     TW_METHOD(weave_layer),      TW_METHOD(weave_layer_cuts),
                           TW_METHOD(weave_layer_auto),   TW_METHOD(weave_train),      TW_METHOD(fill_fused),
                           TW_METHOD(fill_layer),         TW_METHOD(bf16_ptr),         TW_METHOD(stream_handle),
                           TW_METHOD(set_error),          {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_twpy", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__twpy(void) { return PyModule_Create(&g_module); }
