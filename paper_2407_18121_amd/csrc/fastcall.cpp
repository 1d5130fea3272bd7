// The usual calls of binding.py without its way through Python and ctypes: the same checks of every tensor, one call each.
// Whatever is not usual -- a tensor subclass, a wrong type, shape, device or layout, a number that is neither int nor float --
// makes a function return None, and binding.py, which knows what to say about it, goes its own way.  Nothing is kept from call to
// call but the addresses of the library's functions.
//
// Host time of a call, us, through ctypes -> here: a generation step 8.2 -> 4.7, a prompt's attention (three launches) 12.2 -> 8.6, all of a
// small prompt's layer (five launches in three calls) 25 -> 15.4, where the GPU needs 24.7.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstring>
#include <initializer_list>

#include <torch/csrc/autograd/python_variable.h>

namespace {

struct Functions {
    int (*prefill_score)(const void*, const void*, const void*, void*, float*, float*, int, int, int, int, int, int, float, void*, size_t, void*);
    int (*prefill_score_varlen)(const void*, const void*, const void*, void*, float*, float*, const int32_t*, int, int, int, int, int, int, float, void*,
                                size_t, void*);
    int (*chunk_score)(const void*, const void*, const void*, void*, float*, float*, int, int, int, int, int, int, int, int, float, void*, size_t, void*);
    int (*select_anchors)(const float*, int, int, int, int, int, int, int32_t*, void*, size_t, void*);
    int (*merge_compact)(const void*, const void*, const int32_t*, int, int, int, int, int, int, int, int, void*, void*, int, int32_t*, int32_t*,
                         int32_t*, void*);
    int (*remerge_compact)(const void*, const void*, int, const int32_t*, const int32_t*, const int32_t*, int, int, int, int, int, int, int, int, void*,
                           void*, int, int32_t*, int32_t*, int32_t*, void*);
    int (*decode_step)(const void*, const void*, const void*, void*, void*, int32_t*, int, int, int, int, int, int, int, int32_t, float, int, void*,
                       void*, size_t, void*);
    int (*decode_step_varlen)(const void*, const void*, const void*, void*, void*, int32_t*, const int32_t*, const int32_t*, const int32_t*, int, int,
                              int, int, int, float, int, void*, void*, size_t, void*);
    int (*decode_score_step)(const void*, const void*, const void*, void*, void*, int32_t*, float*, int, int, int, int, int, int, int32_t, float, int,
                             void*, void*, size_t, void*);
    int (*evict_min)(void*, void*, int32_t*, float*, int, int, int, int, int, int, int, int, int, int32_t*, void*);
} fn;
PyObject *raw_stream, *current_device;  // of torch: the current stream's handle, the current device's number

struct Unusual {};  // thrown for whatever binding.py has to look at

const at::Tensor* tensor(PyObject* o)
{
    if (o == Py_None) return nullptr;
    if (Py_TYPE(o) != reinterpret_cast<PyTypeObject*>(THPVariableClass)) throw Unusual{};
    return &THPVariable_Unpack(o);
}
const at::Tensor& required(PyObject* o, int64_t dims)
{
    const at::Tensor* t = tensor(o);
    if (!t || t->dim() != dims) throw Unusual{};
    return *t;
}
void* here(const at::Tensor& t)
{
    if (!t.is_cuda() || !t.is_contiguous()) throw Unusual{};
    return t.data_ptr();
}
template <typename T = void> T* fits(const at::Tensor* t, at::ScalarType type, std::initializer_list<int64_t> shape)
{
    if (!t || t->scalar_type() != type || !t->sizes().equals(at::IntArrayRef(shape.begin(), shape.size()))) throw Unusual{};
    return static_cast<T*>(here(*t));
}
template <typename T = void> T* fits(PyObject* o, at::ScalarType type, std::initializer_list<int64_t> shape) { return fits<T>(tensor(o), type, shape); }
template <typename T = void> T* may_fit(PyObject* o, at::ScalarType type, std::initializer_list<int64_t> shape)
{
    return o == Py_None ? nullptr : fits<T>(o, type, shape);
}
int32_t* counters(PyObject* o, int64_t n, bool optional = false)
{
    const at::Tensor* t = tensor(o);
    if (!t && optional) return nullptr;
    if (!t || t->scalar_type() != at::kInt || t->numel() != n) throw Unusual{};
    return static_cast<int32_t*>(here(*t));
}
int type_code(const at::Tensor& t)
{
    if (t.scalar_type() == at::kFloat) return 0;
    if (t.scalar_type() == at::kBFloat16) return 1;
    throw Unusual{};
}
int integer(PyObject* o)
{
    if (!PyLong_Check(o)) throw Unusual{};
    int overflow = 0;
    const long x = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || x != static_cast<int>(x)) throw Unusual{};
    return static_cast<int>(x);
}
float number(PyObject* o)
{
    if (!PyFloat_Check(o) && !PyLong_Check(o)) throw Unusual{};  // numpy's float64 is a float
    const double x = PyFloat_AsDouble(o);
    if (x == -1.0 && PyErr_Occurred()) throw Unusual{};
    return static_cast<float>(x);
}
int size(int64_t n)
{
    if (n != static_cast<int>(n)) throw Unusual{};
    return static_cast<int>(n);
}
int64_t groups(int64_t G, int64_t H)
{
    if (G != 1 && G != H) throw Unusual{};
    return G;
}
struct Workspace {
    void* p = nullptr;
    size_t bytes = 0;
    explicit Workspace(PyObject* o)
    {
        if (const at::Tensor* t = tensor(o)) p = here(*t), bytes = t->nbytes();
    }
};
void* stream()
{
    PyObject* device = PyObject_CallNoArgs(current_device);
    PyObject* handle = device ? PyObject_CallOneArg(raw_stream, device) : nullptr;
    Py_XDECREF(device);
    if (!handle) throw Unusual{};
    void* s = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    if (!s && PyErr_Occurred()) throw Unusual{};
    return s;
}

// Runs `f(args)`, which does the checks and returns the call to make; the call itself is made without the interpreter's lock.
template <int N, typename F> PyObject* entry(PyObject* const* args, Py_ssize_t n, F&& f)
{
    int rc;
    try {
        if (n != N) throw Unusual{};
        const auto call = f(args);
        Py_BEGIN_ALLOW_THREADS
        rc = call();
        Py_END_ALLOW_THREADS
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(rc);
}

PyObject* prefill_score(PyObject*, PyObject* const* args, Py_ssize_t n)  // q k v out lse score scale ws
{
    return entry<8>(args, n, [](PyObject* const* a) {
        const at::Tensor &q = required(a[0], 4), &score = required(a[5], 3);
        const int64_t B = q.size(0), H = q.size(1), T = q.size(2), D = q.size(3), G = groups(score.size(1), H);
        const auto dt = q.scalar_type();
        const Workspace ws(a[7]);
        return [=, qp = fits(&q, dt, {B, H, T, D}), k = fits(a[1], dt, {B, H, T, D}), v = fits(a[2], dt, {B, H, T, D}),
                out = may_fit(a[3], dt, {B, H, T, D}), lse = may_fit<float>(a[4], at::kFloat, {B, H, T}),
                sp = fits<float>(&score, at::kFloat, {B, G, T}), code = type_code(q), scale = number(a[6]), s = stream(), iB = size(B), iH = size(H),
                iG = size(G), iT = size(T), iD = size(D)] {
            return fn.prefill_score(qp, k, v, out, lse, sp, iB, iH, iG, iT, iD, code, scale, ws.p, ws.bytes, s);
        };
    });
}

PyObject* prefill_score_varlen(PyObject*, PyObject* const* args, Py_ssize_t n)  // q k v out lse score seq_len scale ws
{
    return entry<9>(args, n, [](PyObject* const* a) {
        const at::Tensor &q = required(a[0], 4), &score = required(a[5], 3);
        const int64_t B = q.size(0), H = q.size(1), T = q.size(2), D = q.size(3), G = groups(score.size(1), H);
        const auto dt = q.scalar_type();
        const Workspace ws(a[8]);
        return [=, qp = fits(&q, dt, {B, H, T, D}), k = fits(a[1], dt, {B, H, T, D}), v = fits(a[2], dt, {B, H, T, D}),
                out = may_fit(a[3], dt, {B, H, T, D}), lse = may_fit<float>(a[4], at::kFloat, {B, H, T}),
                sp = fits<float>(&score, at::kFloat, {B, G, T}), len = counters(a[6], B), code = type_code(q), scale = number(a[7]), s = stream(),
                iB = size(B), iH = size(H), iG = size(G), iT = size(T), iD = size(D)] {
            return fn.prefill_score_varlen(qp, k, v, out, lse, sp, len, iB, iH, iG, iT, iD, code, scale, ws.p, ws.bytes, s);
        };
    });
}

PyObject* chunk_score(PyObject*, PyObject* const* args, Py_ssize_t n)  // q k v P out lse score scale ws
{
    return entry<9>(args, n, [](PyObject* const* a) {
        const at::Tensor &q = required(a[0], 4), &k = required(a[1], 4), &score = required(a[6], 3);
        const int64_t B = q.size(0), H = q.size(1), T = q.size(2), D = q.size(3), rows = k.size(2), G = groups(score.size(1), H);
        const int P = integer(a[3]);
        const auto dt = q.scalar_type();
        const Workspace ws(a[8]);
        return [=, qp = fits(&q, dt, {B, H, T, D}), kp = fits(&k, dt, {B, H, rows, D}), v = fits(a[2], dt, {B, H, rows, D}),
                out = may_fit(a[4], dt, {B, H, T, D}), lse = may_fit<float>(a[5], at::kFloat, {B, H, T}),
                sp = fits<float>(&score, at::kFloat, {B, G, P + T}), code = type_code(q), scale = number(a[7]), s = stream(), iB = size(B),
                iH = size(H), iG = size(G), iT = size(T), ir = size(rows), iD = size(D)] {
            return fn.chunk_score(qp, kp, v, out, lse, sp, iB, iH, iG, iT, P, ir, iD, code, scale, ws.p, ws.bytes, s);
        };
    });
}

PyObject* select_anchors(PyObject*, PyObject* const* args, Py_ssize_t n)  // score n_anchor protect_first protect_last anchor_idx
{
    return entry<5>(args, n, [](PyObject* const* a) {
        const at::Tensor& score = required(a[0], 3);
        const int64_t B = score.size(0), G = score.size(1), T = score.size(2);
        const int n_anchor = integer(a[1]);
        return [=, sp = fits<float>(&score, at::kFloat, {B, G, T}), idx = fits<int32_t>(a[4], at::kInt, {B, G, n_anchor}), first = integer(a[2]),
                last = integer(a[3]), s = stream(), iB = size(B), iG = size(G), iT = size(T)] {
            return fn.select_anchors(sp, iB, iG, iT, n_anchor, first, last, idx, nullptr, 0, s);
        };
    });
}

PyObject* merge_compact(PyObject*, PyObject* const* args, Py_ssize_t n)  // k v anchor_idx k_cache v_cache counts assign pos merge_mode
{
    return entry<9>(args, n, [](PyObject* const* a) {
        const at::Tensor &k = required(a[0], 4), &idx = required(a[2], 3), &kc = required(a[3], 4);
        const int64_t B = k.size(0), H = k.size(1), T = k.size(2), D = k.size(3), G = groups(idx.size(1), H), N = idx.size(2), cap = kc.size(2);
        const auto dt = k.scalar_type();
        return [=, kp = fits(&k, dt, {B, H, T, D}), v = fits(a[1], dt, {B, H, T, D}), ip = fits<int32_t>(&idx, at::kInt, {B, G, N}),
                kcp = fits(&kc, dt, {B, H, cap, D}), vc = fits(a[4], dt, {B, H, cap, D}), counts = may_fit<int32_t>(a[5], at::kInt, {B, G, N}),
                assign = may_fit<int32_t>(a[6], at::kInt, {B, G, T}), pos = may_fit<int32_t>(a[7], at::kInt, {B, G, cap}), mode = integer(a[8]),
                code = type_code(k), s = stream(), iB = size(B), iH = size(H), iG = size(G), iT = size(T), iD = size(D), iN = size(N), ic = size(cap)] {
            return fn.merge_compact(kp, v, ip, iB, iH, iG, iT, iD, iN, code, mode, kcp, vc, ic, counts, assign, pos, s);
        };
    });
}

PyObject* remerge_compact(PyObject*, PyObject* const* args, Py_ssize_t n)  // k v L anchor_idx k_cache v_cache weights src_pos counts assign pos merge_mode
{
    return entry<12>(args, n, [](PyObject* const* a) {
        const at::Tensor &k = required(a[0], 4), &idx = required(a[3], 3), &kc = required(a[4], 4);
        const int64_t B = k.size(0), H = k.size(1), rows = k.size(2), D = k.size(3), G = groups(idx.size(1), H), N = idx.size(2), cap = kc.size(2);
        const int L = integer(a[2]);
        const auto dt = k.scalar_type();
        return [=, kp = fits(&k, dt, {B, H, rows, D}), v = fits(a[1], dt, {B, H, rows, D}), weights = may_fit<int32_t>(a[6], at::kInt, {B, G, L}),
                src = may_fit<int32_t>(a[7], at::kInt, {B, G, L}), ip = fits<int32_t>(&idx, at::kInt, {B, G, N}), kcp = fits(&kc, dt, {B, H, cap, D}),
                vc = fits(a[5], dt, {B, H, cap, D}), counts = may_fit<int32_t>(a[8], at::kInt, {B, G, N}),
                assign = may_fit<int32_t>(a[9], at::kInt, {B, G, L}), pos = may_fit<int32_t>(a[10], at::kInt, {B, G, cap}), mode = integer(a[11]),
                code = type_code(k), s = stream(), iB = size(B), iH = size(H), iG = size(G), ir = size(rows), iD = size(D), iN = size(N), ic = size(cap)] {
            return fn.remerge_compact(kp, v, ir, weights, src, ip, iB, iH, iG, L, iD, iN, code, mode, kcp, vc, ic, counts, assign, pos, s);
        };
    });
}

// The tensors of every generation step: q k_new v_new k_cache v_cache pos, and out.
struct Step {
    int64_t B, H, G, D, cap;
    int code;
    void *q, *kn, *vn, *kc, *vc, *out;
    int32_t* pos;
    Step(PyObject* const* a, PyObject* out_, PyObject* G_)
    {
        const at::Tensor& k = required(a[3], 4);
        B = k.size(0), H = k.size(1), cap = k.size(2), D = k.size(3);
        if (G_ != Py_None)
            G = integer(G_);
        else
            G = a[5] != Py_None ? required(a[5], 3).size(1) : 1;
        groups(G, H);
        const auto dt = k.scalar_type();
        q = fits(a[0], dt, {B, H, D}), kn = fits(a[1], dt, {B, H, D}), vn = fits(a[2], dt, {B, H, D});
        kc = fits(&k, dt, {B, H, cap, D}), vc = fits(a[4], dt, {B, H, cap, D});
        pos = may_fit<int32_t>(a[5], at::kInt, {B, G, cap});
        out = fits(out_, dt, {B, H, D});
        code = type_code(k);
        size(B), size(H), size(D), size(cap);
    }
};

PyObject* decode_step(PyObject*, PyObject* const* args, Py_ssize_t n)  // .. cache_len evict_idx new_pos scale out ws G
{
    return entry<13>(args, n, [](PyObject* const* a) {
        const Step t(a, a[10], a[12]);
        const Workspace ws(a[11]);
        return [=, len = integer(a[6]), evict = integer(a[7]), new_pos = integer(a[8]), scale = number(a[9]), s = stream()] {
            return fn.decode_step(t.q, t.kn, t.vn, t.kc, t.vc, t.pos, t.B, t.H, t.G, t.D, t.cap, len, evict, new_pos, scale, t.code, t.out, ws.p,
                                  ws.bytes, s);
        };
    });
}

PyObject* decode_step_varlen(PyObject*, PyObject* const* args, Py_ssize_t n)  // .. cache_len_b evict_idx_b new_pos_b scale out G ws
{
    return entry<13>(args, n, [](PyObject* const* a) {
        const Step t(a, a[10], a[11]);
        const Workspace ws(a[12]);
        return [=, len = counters(a[6], t.B), evict = counters(a[7], t.B, true), new_pos = counters(a[8], t.B, true), scale = number(a[9]),
                s = stream()] {
            return fn.decode_step_varlen(t.q, t.kn, t.vn, t.kc, t.vc, t.pos, len, evict, new_pos, t.B, t.H, t.G, t.D, t.cap, scale, t.code, t.out, ws.p,
                                         ws.bytes, s);
        };
    });
}

PyObject* decode_score_step(PyObject*, PyObject* const* args, Py_ssize_t n)  // .. freq cache_len new_pos scale out ws
{
    return entry<12>(args, n, [](PyObject* const* a) {
        const at::Tensor& freq = required(a[6], 3);
        PyObject* G = PyLong_FromLongLong(freq.size(1));
        struct Free {
            PyObject* o;
            ~Free() { Py_XDECREF(o); }
        } const free{G};
        const Step t(a, a[10], G);
        const Workspace ws(a[11]);
        return [=, f = fits<float>(&freq, at::kFloat, {t.B, t.G, t.cap}), len = integer(a[7]), new_pos = integer(a[8]), scale = number(a[9]),
                s = stream()] {
            return fn.decode_score_step(t.q, t.kn, t.vn, t.kc, t.vc, t.pos, f, t.B, t.H, t.G, t.D, t.cap, len, new_pos, scale, t.code, t.out, ws.p,
                                        ws.bytes, s);
        };
    });
}

PyObject* evict_min(PyObject*, PyObject* const* args, Py_ssize_t n)  // k_cache v_cache pos freq length protect_first protect_recent victim
{
    return entry<8>(args, n, [](PyObject* const* a) {
        const at::Tensor &k = required(a[0], 4), &freq = required(a[3], 3);
        const int64_t B = k.size(0), H = k.size(1), cap = k.size(2), D = k.size(3), G = groups(freq.size(1), H);
        const auto dt = k.scalar_type();
        return [=, kc = fits(&k, dt, {B, H, cap, D}), vc = fits(a[1], dt, {B, H, cap, D}), pos = may_fit<int32_t>(a[2], at::kInt, {B, G, cap}),
                f = fits<float>(&freq, at::kFloat, {B, G, cap}), len = integer(a[4]), first = integer(a[5]), recent = integer(a[6]),
                victim = fits<int32_t>(a[7], at::kInt, {B, G}), code = type_code(k), s = stream(), iB = size(B), iH = size(H), iG = size(G), iD = size(D),
                ic = size(cap)] { return fn.evict_min(kc, vc, pos, f, iB, iH, iG, iD, ic, len, first, recent, code, victim, s); };
    });
}

// bind(raw_stream, current_device, addresses in the order of Functions)
PyObject* bind(PyObject*, PyObject* args)
{
    PyObject *stream_, *device_, *addresses;
    if (!PyArg_ParseTuple(args, "OOO!", &stream_, &device_, &PyTuple_Type, &addresses)) return nullptr;
    constexpr Py_ssize_t kCount = sizeof(Functions) / sizeof(void*);
    if (PyTuple_GET_SIZE(addresses) != kCount) return PyErr_Format(PyExc_ValueError, "%zd addresses expected", kCount);
    void* at[kCount];
    for (Py_ssize_t i = 0; i < kCount; ++i)
        if (!(at[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i)))) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "no address");
    static_assert(sizeof(Functions) == sizeof(at), "function pointers only");
    memcpy(static_cast<void*>(&fn), at, sizeof(at));
    Py_INCREF(stream_), Py_INCREF(device_);
    raw_stream = stream_, current_device = device_;
    Py_RETURN_NONE;
}

#define EC_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {EC_FAST(prefill_score),   EC_FAST(prefill_score_varlen), EC_FAST(chunk_score),       EC_FAST(select_anchors),
                         EC_FAST(merge_compact),   EC_FAST(remerge_compact),      EC_FAST(decode_step),       EC_FAST(decode_step_varlen),
                         EC_FAST(decode_score_step), EC_FAST(evict_min),          {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall()
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", EC_TORCH_VERSION) < 0) Py_CLEAR(m);
    return m;
}
