// The Python side of the C ABI in native code: each function takes the tensors of one call, checks them, allocates the
// output tensors, and hands their device pointers and the current HIP stream to the entry point of the same name.
// No arithmetic of the method happens here.
//
// Why it is not Python: small batches spend their time here.  64 rows of 1024 fp32 logits (both scores, two poolings) took
// 55 us a pass with ctypes marshalling, all of it host work; the kernels need a third of that.
//
// Every function returns its outputs, or the difr_status as an int if the entry point refused the call, or None if an
// argument is not what it has to be: the Python caller then runs its own checks, which name the argument.
//
// The entry points are not linked: binding.py loads libdifr.so and passes their addresses to bind().
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include "../../include/difr.h"

namespace {

#define DIFR_ENTRIES(X)                                                                                                 \
    X(difr_gumbel_score)                                                                                                \
    X(difr_debug_gumbel_score_unfiltered)                                                                               \
    X(difr_ipt_score)                                                                                                   \
    X(difr_score_both)                                                                                                  \
    X(difr_score_both_peaked)                                                                                           \
    X(difr_score_both_admissible)                                                                                       \
    X(difr_ipt_score_filtered)                                                                                          \
    X(difr_gumbel_likelihood)                                                                                           \
    X(difr_score_both_filtered)                                                                                         \
    X(difr_admissible_count)                                                                                            \
    X(difr_split_workspace_bytes)                                                                                       \
    X(difr_score_split)                                                                                                 \
    X(difr_lmhead_workspace_bytes)                                                                                      \
    X(difr_lmhead_score)                                                                                                \
    X(difr_seq_reduce)                                                                                                  \
    X(difr_classify)

struct Entries {
#define X(name) decltype(&::name) name = nullptr;
    DIFR_ENTRIES(X)
#undef X
} lib;

// dictionary keys, made once
#define DIFR_KEYS(X)                                                                                                    \
    X(margin) X(argmax) X(max_score) X(claimed_score) X(flags) X(logit_rank) X(dist) X(cdf_lo) X(cdf_hi) X(u)           \
    X(ipt_token) X(log_mass) X(count) X(log2_count) X(kept) X(pi) X(log_pi) X(tau) X(active) X(seq_mean) X(seq_max)     \
    X(seq_mismatch) X(seq_flag) X(cls) X(bits)
namespace key {
#define X(name) PyObject *name = nullptr;
DIFR_KEYS(X)
#undef X
}  // namespace key

// An argument that is not what the call needs: the caller gets None.
struct Refused {};

const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_Check(o)) throw Refused();
    return THPVariable_Unpack(o);
}

// contiguous 1-D tensor of n elements (n < 0: any number) on `dev`
void *vec(PyObject *o, at::ScalarType type, int64_t n, const c10::Device &dev)
{
    const at::Tensor &t = tensor(o);
    if (t.scalar_type() != type || t.dim() != 1 || t.device() != dev || (n >= 0 && t.size(0) != n) || !t.is_contiguous()) throw Refused();
    return t.data_ptr();
}
void *vec_or_null(PyObject *o, at::ScalarType type, int64_t n, const c10::Device &dev)
{
    return o == Py_None ? nullptr : vec(o, type, n, dev);
}

double number(PyObject *o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw python_error();
    return v;
}
int64_t whole(PyObject *o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw python_error();
    return v;
}
bool truth(PyObject *o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw python_error();
    return v != 0;
}

// The first eight arguments of every call on stored logits: logits, V, temperature, seeds, seq_ids, positions, claimed,
// temperatures.
struct Rows {
    difr_rows in;
    int64_t N;
    c10::Device dev;

    explicit Rows(PyObject *const *a) : dev(c10::kCUDA)
    {
        const at::Tensor &x = tensor(a[0]);
        if (!x.is_cuda() || x.dim() != 2 || (x.stride(1) != 1 && x.size(1) > 1)) throw Refused();
        if (x.scalar_type() == at::kBFloat16)
            in.dtype = DIFR_BF16;
        else if (x.scalar_type() == at::kFloat)
            in.dtype = DIFR_F32;
        else
            throw Refused();
        dev = x.device();
        N = x.size(0);
        in.logits = x.data_ptr();
        in.N = N;
        in.V = a[1] == Py_None ? x.size(1) : whole(a[1]);
        in.ld = N > 1 ? x.stride(0) : std::max(x.size(1), N ? x.stride(0) : (int64_t)0);
        in.temperature = (float)number(a[2]);
        const at::Tensor &s = tensor(a[3]);
        in.seeds = (const uint64_t *)vec(a[3], at::kLong, -1, dev);
        in.S = s.size(0);
        in.seq_ids = (const int32_t *)vec(a[4], at::kInt, N, dev);
        in.positions = (const uint32_t *)vec(a[5], at::kInt, N, dev);  // uint32 bit patterns held in int32
        in.claimed = (const int32_t *)vec_or_null(a[6], at::kInt, N, dev);
        in.temperatures = (const float *)vec_or_null(a[7], at::kFloat, N, dev);
    }
};
constexpr int kRowArgs = 8;

// One dictionary of output tensors, each in memory of its own, so that a caller may grow, save, keep or record any of them.  A call on
// few tokens has up to twelve: they come from torch's allocator without the way through its dispatcher (64 tokens, both scores and
// pooling, host time: 30 us by at::empty, 23 so; views of one allocation took 17, but one that was grown in place lay over the next).
struct Outputs {
    THPObjectPtr dict;
    c10::Device dev;
    const bool direct;  // nobody watches allocations, and nobody wants them filled
    explicit Outputs(c10::Device d)
        : dict(PyDict_New()), dev(d),
          direct(!c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::globalContext().deterministicAlgorithms())
    {
        if (!dict) throw python_error();
    }
    at::Tensor make(at::ScalarType type, at::IntArrayRef shape)
    {
        if (!direct) return at::empty(shape, at::TensorOptions().dtype(type).device(dev));
        return at::Tensor(at::detail::empty_cuda(shape, type, dev, std::nullopt));
    }
    void *add(PyObject *name, at::ScalarType type, at::IntArrayRef shape)
    {
        at::Tensor t = make(type, shape);
        void *p = t.data_ptr();
        THPObjectPtr w(THPVariable_Wrap(std::move(t)));
        if (!w || PyDict_SetItem(dict, name, w) < 0) throw python_error();
        return p;
    }
    float *f32(PyObject *name, int64_t n) { return (float *)add(name, at::kFloat, {n}); }
    int32_t *i32(PyObject *name, int64_t n) { return (int32_t *)add(name, at::kInt, {n}); }
    uint8_t *u8(PyObject *name, int64_t n) { return (uint8_t *)add(name, at::kByte, {n}); }
};

void *stream_of(const c10::Device &dev) { return (void *)c10::hip::getCurrentHIPStream(dev.index()).stream(); }

// Calls the entry point on the device of its arguments, without the interpreter lock.
template <class F>
int enter(const c10::Device &dev, F &&f)
{
    const c10::DeviceGuard guard(dev);
    void *stream = stream_of(dev);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f(stream);
    Py_END_ALLOW_THREADS
    return rc;
}

PyObject *one(int rc, Outputs &a) { return rc ? PyLong_FromLong(rc) : a.dict.release(); }
PyObject *two(int rc, Outputs &a, Outputs &b) { return rc ? PyLong_FromLong(rc) : PyTuple_Pack(2, a.dict.get(), b.dict.get()); }
PyObject *three(int rc, Outputs &a, Outputs &b, Outputs &c)
{
    return rc ? PyLong_FromLong(rc) : PyTuple_Pack(3, a.dict.get(), b.dict.get(), c.dict.get());
}

// A small batch goes through difr_score_split, with a workspace from torch's allocator that belongs to the call's stream.
// Returns whether it did; the outputs are those of the call in `o`.
bool split(const Rows &r, const int32_t *claimed_ipt, const difr_scores &o, int *rc)
{
    const size_t need = lib.difr_split_workspace_bytes(r.in.N, r.in.V, r.in.dtype, o.count != nullptr);
    if (need == 0) return false;
    const at::Tensor ws = at::empty({(int64_t)need}, at::TensorOptions().dtype(at::kByte).device(r.dev));
    void *p = ws.data_ptr();
    *rc = enter(r.dev, [&](void *s) { return lib.difr_score_split(&r.in, claimed_ipt, &o, p, need, s); });
    return true;
}

// ---- one function per entry point; arguments beyond the row arguments in the comment ----

// claimed_gumbel side of a call that scores both estimators
struct GumbelSide {
    Outputs out;
    float *margin, *max_score, *claimed_score;
    int32_t *argmax, *rank = nullptr;
    uint8_t *flags;
    GumbelSide(c10::Device dev, int64_t N, bool want_rank) : out(dev)
    {
        margin = out.f32(key::margin, N);
        argmax = out.i32(key::argmax, N);
        max_score = out.f32(key::max_score, N);
        claimed_score = out.f32(key::claimed_score, N);
        flags = out.u8(key::flags, N);
        if (want_rank) rank = out.i32(key::logit_rank, N);
    }
};
struct IptSide {
    Outputs out;
    float *dist, *cdf_lo, *cdf_hi, *u, *log_mass = nullptr;
    int32_t *token = nullptr, *kept = nullptr;
    uint8_t *flags;
    IptSide(c10::Device dev, int64_t N, bool want_kept) : out(dev)
    {
        dist = out.f32(key::dist, N);
        cdf_lo = out.f32(key::cdf_lo, N);
        cdf_hi = out.f32(key::cdf_hi, N);
        u = out.f32(key::u, N);
        if (want_kept) kept = out.i32(key::kept, N);
        flags = out.u8(key::flags, N);
    }
};

difr_scores both_sides(const GumbelSide &g, const IptSide &i, double sigma, double eps)
{
    difr_scores sc = {};
    sc.margin = g.margin, sc.argmax = g.argmax, sc.max_score = g.max_score, sc.claimed_score = g.claimed_score;
    sc.flags_gumbel = g.flags, sc.rank_gumbel = g.rank;
    sc.dist = i.dist, sc.cdf_lo = i.cdf_lo, sc.cdf_hi = i.cdf_hi, sc.u = i.u, sc.ipt_token = i.token, sc.sigma = sigma, sc.eps = eps;
    sc.log_mass = i.log_mass, sc.flags_ipt = i.flags;
    return sc;
}

// rows, want_scores, unfiltered, want_rank
PyObject *gumbel_score(PyObject *const *a)
{
    Rows r(a);
    a += kRowArgs;
    Outputs o(r.dev);
    float *margin = o.f32(key::margin, r.N);
    int32_t *argmax = o.i32(key::argmax, r.N);
    uint8_t *flags = o.u8(key::flags, r.N);
    float *max_score = nullptr, *claimed_score = nullptr;
    if (truth(a[0])) {
        max_score = o.f32(key::max_score, r.N);
        claimed_score = o.f32(key::claimed_score, r.N);
    }
    const auto entry = truth(a[1]) ? lib.difr_debug_gumbel_score_unfiltered : lib.difr_gumbel_score;
    int32_t *rank = truth(a[2]) ? o.i32(key::logit_rank, r.N) : nullptr;
    int rc;
    difr_scores sc = {};
    sc.margin = margin, sc.argmax = argmax, sc.max_score = max_score, sc.claimed_score = claimed_score, sc.flags_gumbel = flags;
    sc.rank_gumbel = rank;
    if (entry == lib.difr_gumbel_score && split(r, nullptr, sc, &rc)) return one(rc, o);
    return one(enter(r.dev, [&](void *s) { return entry(&r.in, margin, argmax, max_score, claimed_score, flags, rank, s); }), o);
}

// rows, want_token, want_log_mass, sigma, eps, want_interval, want_rank
PyObject *ipt_score(PyObject *const *a)
{
    Rows r(a);
    a += kRowArgs;
    const double sigma = number(a[2]), eps = number(a[3]);
    Outputs o(r.dev);
    float *dist = o.f32(key::dist, r.N);
    uint8_t *flags = o.u8(key::flags, r.N);
    float *cdf_lo = nullptr, *cdf_hi = nullptr, *u = nullptr;
    if (truth(a[4])) {
        cdf_lo = o.f32(key::cdf_lo, r.N);
        cdf_hi = o.f32(key::cdf_hi, r.N);
        u = o.f32(key::u, r.N);
    }
    int32_t *token = truth(a[0]) ? o.i32(key::ipt_token, r.N) : nullptr;
    float *log_mass = truth(a[1]) ? o.f32(key::log_mass, r.N) : nullptr;
    int32_t *rank = truth(a[5]) ? o.i32(key::logit_rank, r.N) : nullptr;
    int rc;
    difr_scores sc = {};
    sc.dist = dist, sc.cdf_lo = cdf_lo, sc.cdf_hi = cdf_hi, sc.u = u, sc.ipt_token = token, sc.sigma = sigma, sc.eps = eps;
    sc.log_mass = log_mass, sc.flags_ipt = flags, sc.rank_ipt = rank;
    if (split(r, r.in.claimed, sc, &rc)) return one(rc, o);
    return one(enter(r.dev, [&](void *s) {
                   return lib.difr_ipt_score(&r.in, dist, cdf_lo, cdf_hi, u, token, sigma, eps, log_mass, flags, rank, s);
               }), o);
}

// Most peaked rows that are shared.  Shared rows regenerate the noise of all their vectors, the peaked kernel that of few, and is
// the faster one once the rows by themselves keep most of the chip busy.  Logits falling as -3 ln rank, T = 0.6, peaked kernel /
// shared rows, us: V = 151,936 256 rows 42.6 / 34.0, 384 rows 46.5 / 45.5, 512 rows 46.9 / 52.7, 740 rows 52 / 69; V = 100,000
// 256 rows 33.4 / 29.3, 384 rows 35.2 / 36.3; V = 65,000 256 rows 25.5 / 24.5, 310 rows 26.9 / 27.3.
constexpr int64_t kPeakedShared = 320;

// rows, claimed_ipt, peaked, want_rank, want_token, want_log_mass, sigma, eps
PyObject *score_both(PyObject *const *a)
{
    Rows r(a);
    a += kRowArgs;
    const int32_t *ci = (const int32_t *)vec_or_null(a[0], at::kInt, r.N, r.dev);
    const bool peaked = truth(a[1]);
    const auto entry = peaked ? lib.difr_score_both_peaked : lib.difr_score_both;
    const double sigma = number(a[5]), eps = number(a[6]);
    GumbelSide g(r.dev, r.N, truth(a[2]));
    IptSide i(r.dev, r.N, false);
    if (truth(a[3])) i.token = i.out.i32(key::ipt_token, r.N);
    if (truth(a[4])) i.log_mass = i.out.f32(key::log_mass, r.N);
    int rc;
    const bool whole = peaked && !g.rank && r.N > kPeakedShared;  // (with the rank the peaked call is the ordinary one)
    if (!whole && split(r, ci, both_sides(g, i, sigma, eps), &rc)) return two(rc, g.out, i.out);
    return two(enter(r.dev, [&](void *s) {
                   return entry(&r.in, ci, g.margin, g.argmax, g.max_score, g.claimed_score, g.flags, g.rank, i.dist, i.cdf_lo,
                                i.cdf_hi, i.u, i.token, sigma, eps, i.log_mass, i.flags, s);
               }), g.out, i.out);
}

// rows, claimed_ipt, delta
PyObject *score_both_admissible(PyObject *const *a)
{
    Rows r(a);
    a += kRowArgs;
    const int32_t *ci = (const int32_t *)vec_or_null(a[0], at::kInt, r.N, r.dev);
    const float delta = (float)number(a[1]);
    GumbelSide g(r.dev, r.N, false);
    IptSide i(r.dev, r.N, false);
    Outputs o(r.dev);
    int32_t *count = o.i32(key::count, r.N);
    float *log2_count = o.f32(key::log2_count, r.N);
    int rc;
    difr_scores sc = both_sides(g, i, 0.0, 0.0);
    sc.delta = delta, sc.count = count, sc.log2_count = log2_count;
    if (split(r, ci, sc, &rc)) return three(rc, g.out, i.out, o);
    return three(enter(r.dev, [&](void *s) {
                     return lib.difr_score_both_admissible(&r.in, ci, delta, g.margin, g.argmax, g.max_score, g.claimed_score,
                                                           g.flags, i.dist, i.cdf_lo, i.cdf_hi, i.u, i.flags, count, log2_count, s);
                 }), g.out, i.out, o);
}

// rows, max_score, delta, want_log2
PyObject *admissible_count(PyObject *const *a)
{
    Rows r(a);
    a += kRowArgs;
    const float *M = (const float *)vec_or_null(a[0], at::kFloat, r.N, r.dev);
    const float delta = (float)number(a[1]);
    Outputs o(r.dev);
    int32_t *count = o.i32(key::count, r.N);
    float *log2_count = truth(a[2]) ? o.f32(key::log2_count, r.N) : nullptr;
    return one(enter(r.dev, [&](void *s) { return lib.difr_admissible_count(&r.in, M, delta, count, log2_count, s); }), o);
}

// rows, top_k, top_p, want_token, want_log_mass, sigma, eps
PyObject *ipt_score_filtered(PyObject *const *a)
{
    Rows r(a);
    a += kRowArgs;
    const int32_t top_k = (int32_t)whole(a[0]);
    const float top_p = (float)number(a[1]);
    const double sigma = number(a[4]), eps = number(a[5]);
    IptSide i(r.dev, r.N, true);
    if (truth(a[2])) i.token = i.out.i32(key::ipt_token, r.N);
    if (truth(a[3])) i.log_mass = i.out.f32(key::log_mass, r.N);
    return one(enter(r.dev, [&](void *s) {
                   return lib.difr_ipt_score_filtered(&r.in, top_k, top_p, i.dist, i.cdf_lo, i.cdf_hi, i.u, i.token, sigma, eps,
                                                      i.log_mass, i.kept, i.flags, s);
               }), i.out);
}

// the likelihood side of the next two: z, top_k, top_p, s, sigma, want_active
struct Likelihood {
    difr_likelihood_params p;
    Outputs out;
    float *pi, *log_pi, *tau;
    int32_t *active = nullptr;
    uint8_t *flags;
    Likelihood(const Rows &r, PyObject *const *a) : out(r.dev)
    {
        p.z = (const float *)vec(a[0], at::kFloat, -1, r.dev);
        p.M = (int32_t)tensor(a[0]).size(0);
        p.top_k = (int32_t)whole(a[1]);
        p.top_p = (float)number(a[2]);
        const int64_t s = whole(a[3]);
        p.s = (int32_t)s;
        p.sigma = (float)number(a[4]);
        pi = out.f32(key::pi, r.N);
        log_pi = out.f32(key::log_pi, r.N);
        tau = out.f32(key::tau, r.N);
        flags = out.u8(key::flags, r.N);
        if (truth(a[5])) {
            void *q = out.add(key::active, at::kInt, {r.N, std::max(s, (int64_t)0)});
            if (s > 0) active = (int32_t *)q;
        }
    }
};

// rows, likelihood arguments
PyObject *gumbel_likelihood(PyObject *const *a)
{
    Rows r(a);
    Likelihood k(r, a + kRowArgs);
    return one(enter(r.dev, [&](void *s) { return lib.difr_gumbel_likelihood(&r.in, &k.p, k.pi, k.log_pi, k.tau, k.active, k.flags, s); }),
               k.out);
}

// rows, likelihood arguments, claimed_ipt, want_token, want_log_mass, sigma_ipt, eps
PyObject *score_both_filtered(PyObject *const *a)
{
    Rows r(a);
    Likelihood k(r, a + kRowArgs);
    a += kRowArgs + 6;
    const int32_t *ci = (const int32_t *)vec_or_null(a[0], at::kInt, r.N, r.dev);
    const double sigma = number(a[3]), eps = number(a[4]);
    IptSide i(r.dev, r.N, true);
    if (truth(a[1])) i.token = i.out.i32(key::ipt_token, r.N);
    if (truth(a[2])) i.log_mass = i.out.f32(key::log_mass, r.N);
    return two(enter(r.dev, [&](void *s) {
                   return lib.difr_score_both_filtered(&r.in, ci, &k.p, k.pi, k.log_pi, k.tau, k.active, k.flags, i.dist, i.cdf_lo,
                                                       i.cdf_hi, i.u, i.token, sigma, eps, i.log_mass, i.kept, i.flags, s);
               }), k.out, i.out);
}

// hidden, weight, temperature, seeds, seq_ids, positions, claimed_gumbel, claimed_ipt, temperatures, workspace,
// want_rank, want_log_mass, want_token, sigma, eps
PyObject *lmhead_score(PyObject *const *a)
{
    const at::Tensor &h = tensor(a[0]), &w = tensor(a[1]);
    for (const at::Tensor *t : {&h, &w})
        if (!t->is_cuda() || t->scalar_type() != at::kBFloat16 || t->dim() != 2 || (t->size(1) > 1 && t->stride(1) != 1)) throw Refused();
    const c10::Device dev = h.device();
    const int64_t N = h.size(0), d = h.size(1), V = w.size(0);
    if (w.size(1) != d || w.device() != dev) throw Refused();
    difr_lmhead in;
    in.hidden = h.data_ptr();
    in.weight = w.data_ptr();
    in.N = N;
    in.V = V;
    in.d = d;
    in.ldh = N > 1 ? h.stride(0) : d;
    in.ldw = V > 1 ? w.stride(0) : d;
    in.temperature = (float)number(a[2]);
    in.seeds = (const uint64_t *)vec(a[3], at::kLong, -1, dev);
    in.S = tensor(a[3]).size(0);
    in.seq_ids = (const int32_t *)vec(a[4], at::kInt, N, dev);
    in.positions = (const uint32_t *)vec(a[5], at::kInt, N, dev);
    in.claimed_gumbel = (const int32_t *)vec_or_null(a[6], at::kInt, N, dev);
    in.claimed_ipt = (const int32_t *)vec_or_null(a[7], at::kInt, N, dev);
    in.temperatures = (const float *)vec_or_null(a[8], at::kFloat, N, dev);
    const bool want_token = truth(a[12]);
    const double sigma = number(a[13]), eps = number(a[14]);
    at::Tensor ws;
    if (a[9] == Py_None) {
        const int64_t need = (int64_t)lib.difr_lmhead_workspace_bytes(N, V, d, want_token);
        ws = at::empty({std::max(need, (int64_t)8)}, at::TensorOptions().dtype(at::kByte).device(dev));
    } else {
        ws = tensor(a[9]);
        if (ws.device() != dev || ws.scalar_type() != at::kByte || !ws.is_contiguous()) throw Refused();
    }
    void *wsp = ws.data_ptr();
    const size_t wsn = (size_t)ws.numel();
    GumbelSide g(dev, N, truth(a[10]));
    IptSide i(dev, N, false);
    if (truth(a[11])) i.log_mass = i.out.f32(key::log_mass, N);
    if (want_token) i.token = i.out.i32(key::ipt_token, N);
    return two(enter(dev, [&](void *s) {
                   return lib.difr_lmhead_score(&in, g.margin, g.argmax, g.max_score, g.claimed_score, g.flags, g.rank, i.dist,
                                                i.cdf_lo, i.cdf_hi, i.u, i.token, sigma, eps, i.log_mass, i.flags, wsp, wsn, s);
               }), g.out, i.out);
}

// scores, row_flags, seq_offsets, threshold
PyObject *seq_reduce(PyObject *const *a)
{
    const at::Tensor &x = tensor(a[0]);
    if (!x.is_cuda()) throw Refused();
    const c10::Device dev = x.device();
    const float *scores = (const float *)vec(a[0], at::kFloat, -1, dev);
    const int64_t N = x.size(0);
    const uint8_t *flags = (const uint8_t *)vec_or_null(a[1], at::kByte, N, dev);
    const int64_t *off = (const int64_t *)vec(a[2], at::kLong, -1, dev);
    const int64_t S = tensor(a[2]).size(0) - 1;
    if (S < 0) throw Refused();
    const float threshold = (float)number(a[3]);
    Outputs o(dev);
    float *mean = o.f32(key::seq_mean, S), *mx = o.f32(key::seq_max, S);
    int32_t *mis = o.i32(key::seq_mismatch, S);
    uint8_t *fl = o.u8(key::seq_flag, S);
    return one(enter(dev, [&](void *s) { return lib.difr_seq_reduce(scores, flags, off, N, S, threshold, mean, mx, mis, fl, s); }), o);
}

// scores, ranks, tau, rank_cutoff, V, log2_admissible
PyObject *classify(PyObject *const *a)
{
    const at::Tensor &x = tensor(a[0]);
    if (!x.is_cuda()) throw Refused();
    const c10::Device dev = x.device();
    const float *scores = (const float *)vec(a[0], at::kFloat, -1, dev);
    const int64_t N = x.size(0);
    const int32_t *ranks = (const int32_t *)vec_or_null(a[1], at::kInt, N, dev);
    const float tau = (float)number(a[2]);
    const int64_t cutoff = whole(a[3]), V = whole(a[4]);
    const float *log2_adm = (const float *)vec_or_null(a[5], at::kFloat, N, dev);
    Outputs o(dev);
    uint8_t *cls = o.u8(key::cls, N);
    float *bits = o.f32(key::bits, N);
    return one(enter(dev, [&](void *s) { return lib.difr_classify(scores, ranks, N, tau, cutoff, V, log2_adm, cls, bits, s); }), o);
}

// ---- module ----

template <PyObject *(*F)(PyObject *const *), int N>
PyObject *fast(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Refused &) {
        Py_RETURN_NONE;
    }
    END_HANDLE_TH_ERRORS
}

// bind({entry point: address})
PyObject *bind(PyObject *, PyObject *addresses)
{
#define X(name)                                                                                                         \
    {                                                                                                                   \
        PyObject *o = PyDict_GetItemString(addresses, #name);                                                           \
        void *p = o ? PyLong_AsVoidPtr(o) : nullptr;                                                                    \
        if (!p) {                                                                                                       \
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #name);                                              \
            return nullptr;                                                                                             \
        }                                                                                                               \
        lib.name = reinterpret_cast<decltype(&::name)>(p);                                                              \
    }
    DIFR_ENTRIES(X)
#undef X
    Py_RETURN_NONE;
}

template <PyObject *(*F)(PyObject *const *), int N>
constexpr PyMethodDef method(const char *name)
{
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&fast<F, N>)), METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {
    {"bind", bind, METH_O, nullptr},
    method<gumbel_score, kRowArgs + 3>("gumbel_score"),
    method<ipt_score, kRowArgs + 6>("ipt_score"),
    method<score_both, kRowArgs + 7>("score_both"),
    method<score_both_admissible, kRowArgs + 2>("score_both_admissible"),
    method<admissible_count, kRowArgs + 3>("admissible_count"),
    method<ipt_score_filtered, kRowArgs + 6>("ipt_score_filtered"),
    method<gumbel_likelihood, kRowArgs + 6>("gumbel_likelihood"),
    method<score_both_filtered, kRowArgs + 11>("score_both_filtered"),
    method<lmhead_score, 15>("lmhead_score"),
    method<seq_reduce, 4>("seq_reduce"),
    method<classify, 6>("classify"),
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native()
{
#define X(name)                                          \
    key::name = PyUnicode_InternFromString(#name);       \
    if (!key::name) return nullptr;
    DIFR_KEYS(X)
#undef X
    return PyModule_Create(&module);
}
