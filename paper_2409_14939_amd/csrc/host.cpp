// The Python side of the C ABI: CPython functions that check the tensors of a call, allocate what the
// caller did not pass, and enqueue the library call on the current stream of the current device.
//
// Why it is native: a small mini-batch is bound by the host.  Every call marshals 10 to 20 arguments
// around 1 to 6 launches of about 3 us; through ctypes (with torch.cuda.current_stream() at 2.9 us) the
// marshalling cost more than a launch.  One aggregation call without launches: 6.3 us through ctypes, 0.4 us
// here; a 256-seed block (plan, forward, backward: 8 launches) took 46 us of host time and takes 24 us.
//
// Conventions: arguments are positional (binding.py holds the signatures, defaults and documentation);
// None stands for an absent tensor; a violated precondition raises TypeError / ValueError before any
// library call, a status other than FASTGL_OK raises binding.FastglError.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>
#include <new>
#include <vector>

#include "fastgl_agg.h"
#include "fastgl_edge.h"
#include "fastgl_idmap.h"
#include "fastgl_match.h"
#include "fastgl_update.h"

namespace {

PyObject *g_error_class = nullptr;   // binding.FastglError
PyObject *g_handle_name = nullptr;   // interned names: of Plan's handle attribute
PyObject *g_value_name = nullptr;    // and of c_void_p's value

struct Raised {};                    // a Python exception is set

[[noreturn]] void fail(PyObject *type, const char *msg)
{
    PyErr_SetString(type, msg);
    throw Raised{};
}

const at::Tensor &tensor(PyObject *o, const char *name)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
        throw Raised{};
    }
    return THPVariable_Unpack(o);
}

const char *dtype_name(at::ScalarType t)
{
    switch (t) {
        case at::kInt: return "torch.int32";
        case at::kLong: return "torch.int64";
        case at::kFloat: return "torch.float32";
        case at::kBFloat16: return "torch.bfloat16";
        case at::kByte: return "torch.uint8";
        default: return "the right dtype";
    }
}

// A contiguous device tensor of the given type.
const at::Tensor &dev(PyObject *o, at::ScalarType t, const char *name)
{
    const at::Tensor &x = tensor(o, name);
    if (!x.is_cuda() || x.scalar_type() != t || !x.is_contiguous()) {
        PyErr_Format(PyExc_TypeError, "%s must be a contiguous device tensor of %s", name, dtype_name(t));
        throw Raised{};
    }
    return x;
}

fastgl_dtype feat_dtype(const at::Tensor &x)
{
    if (x.scalar_type() == at::kFloat) return FASTGL_F32;
    if (x.scalar_type() == at::kBFloat16) return FASTGL_BF16;
    fail(PyExc_TypeError, "features must be float32 or bfloat16");
}

// Two dimensions, or more of which the others are 1.
bool matrix(const at::Tensor &x) { return x.dim() >= 2 && (x.dim() == 2 || x.numel() == x.size(0) * x.size(1)); }

// Feature matrix: contiguous, on the device, float32 or bfloat16.
const at::Tensor &features(PyObject *o, const char *name)
{
    const at::Tensor &x = tensor(o, name);
    feat_dtype(x);
    dev(o, x.scalar_type(), name);
    if (!matrix(x)) {
        PyErr_Format(PyExc_ValueError, "%s must have two dimensions", name);
        throw Raised{};
    }
    return x;
}

// A size or an enumerator: an int and nothing that int() would round or parse.
int64_t integer(PyObject *o)
{
    if (!PyLong_Check(o)) {
        PyErr_Format(PyExc_TypeError, "an int is expected, not %s", Py_TYPE(o)->tp_name);
        throw Raised{};
    }
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
}

// What int() makes of it.
int64_t to_integer(PyObject *o)
{
    PyObject *i = PyNumber_Long(o);
    if (!i) throw Raised{};
    const long long v = PyLong_AsLongLong(i);
    Py_DECREF(i);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
}

// What float() makes of it.
float to_real(PyObject *o)
{
    PyObject *f = PyNumber_Float(o);
    if (!f) throw Raised{};
    const double v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return (float)v;
}

bool truth(PyObject *o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Raised{};
    return v != 0;
}

bool none(PyObject *o) { return o == Py_None; }

bool shape2(const at::Tensor &x, int64_t a, int64_t b) { return x.dim() == 2 && x.size(0) == a && x.size(1) == b; }
bool shape1(const at::Tensor &x, int64_t a) { return x.dim() == 1 && x.size(0) == a; }

// A tensor to return: the caller's (checked) or a new one.
struct Out {
    at::Tensor t;
    Out() = default;
    Out(PyObject *o, at::ScalarType type, at::IntArrayRef shape, const at::Tensor &like, const char *name)
    {
        if (none(o)) t = at::empty(shape, like.options().dtype(type));
        else t = dev(o, type, name);
    }
    void *p() const { return t.defined() ? t.data_ptr() : nullptr; }
};

// The scratch buffer of a call: the caller's, or `bytes` allocated for this call.  The bytes are only
// asked for when the caller passed none.
struct Scratch {
    at::Tensor t;
    template <class BYTES>
    Scratch(PyObject *o, const at::Tensor &like, BYTES bytes)
    {
        if (none(o)) t = at::empty({(int64_t)bytes()}, like.options().dtype(at::kByte));
        else t = tensor(o, "workspace");
    }
    void *p() const { return t.data_ptr(); }
    size_t n() const { return (size_t)t.numel(); }
};

// The handle of anything with the attribute of that name: None, an address, or a c_void_p around either.
const fastgl_plan *plan_of(PyObject *o)
{
    if (none(o)) return nullptr;
    PyObject *h = PyObject_GetAttr(o, g_handle_name);
    if (h && !none(h) && !PyLong_Check(h)) {
        PyObject *v = PyObject_GetAttr(h, g_value_name);
        Py_DECREF(h);
        h = v;
    }
    if (!h) throw Raised{};
    const void *p = none(h) ? nullptr : PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (!p && PyErr_Occurred()) throw Raised{};
    return static_cast<const fastgl_plan *>(p);
}

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

// The library call, outside the interpreter's lock as ctypes has it.
template <class CALL>
void run(CALL call)
{
    fastgl_status st;
    void *s = stream();
    Py_BEGIN_ALLOW_THREADS
    st = call(s);
    Py_END_ALLOW_THREADS
    if (st == FASTGL_OK) return;
    PyObject *e = PyObject_CallFunction(g_error_class, "is", (int)st, fastgl_last_error());
    if (e) {
        PyErr_SetObject(g_error_class, e);
        Py_DECREF(e);
    }
    throw Raised{};
}

PyObject *wrap(const at::Tensor &t)
{
    if (!t.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(t);
}

PyObject *tuple(std::initializer_list<at::Tensor> ts)
{
    PyObject *r = PyTuple_New((Py_ssize_t)ts.size());
    Py_ssize_t i = 0;
    for (const at::Tensor &t : ts) PyTuple_SET_ITEM(r, i++, wrap(t));
    return r;
}

// Every function: METH_FASTCALL with a fixed number of arguments, exceptions turned into the ones torch raises for
// them (torch.OutOfMemoryError for an allocation that does not fit: programs catch it and go on with less).
typedef PyObject *(*Body)(PyObject *const *);
template <Body BODY, int NARGS>
PyObject *entry(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != NARGS) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, got %zd", NARGS, n);
        return nullptr;
    }
    try {
        return BODY(a);
    } catch (const Raised &) {
        return nullptr;
    } catch (const std::bad_alloc &) {
        return PyErr_NoMemory();
    } catch (const std::exception &) {
        torch::translate_exception_to_python(std::current_exception());
        return nullptr;
    }
}

struct Block {
    const at::Tensor &indptr, &indices;
    int64_t num_dst, num_src, num_edges;
    Block(PyObject *ip, PyObject *ix, PyObject *ns)
        : indptr(dev(ip, at::kInt, "indptr")), indices(dev(ix, at::kInt, "indices")), num_dst(indptr.numel() - 1),
          num_src(integer(ns)), num_edges(indices.numel())
    {
    }
    const int32_t *ip() const { return (const int32_t *)indptr.data_ptr(); }
    const int32_t *ix() const { return (const int32_t *)indices.data_ptr(); }
};

const float *optional_f32(PyObject *o, const char *name)
{
    return none(o) ? nullptr : (const float *)dev(o, at::kFloat, name).data_ptr();
}

// ------------------------------------------------------------------------------------ aggregation
// (backward, indptr, indices, edge_w, num_src, mode, in, out, plan, workspace) -> out
PyObject *aggregate(PyObject *const *a)
{
    const bool backward = a[0] == Py_True;
    const Block b(a[1], a[2], a[4]);
    const float *w = optional_f32(a[3], "edge_w");
    const auto mode = (fastgl_agg_mode)integer(a[5]);
    const at::Tensor &in = features(a[6], "input features");
    const int64_t feat = in.size(1), rows = backward ? b.num_src : b.num_dst;
    if (in.size(0) != (backward ? b.num_dst : b.num_src))
        fail(PyExc_ValueError, backward ? "grad_out must have num_dst rows" : "X must have num_src rows");
    const Out out(a[7], in.scalar_type(), {rows, feat}, in, "output features");
    if (!shape2(out.t, rows, feat))
        fail(PyExc_ValueError, backward ? "grad_X must be [num_src, feat]" : "out must be [num_dst, feat]");
    const fastgl_dtype dt = feat_dtype(in);
    const fastgl_plan *p = plan_of(a[8]);
    const Scratch ws(a[9], in,
                     [&] { return fastgl_block_workspace_bytes(b.num_dst, b.num_src, b.num_edges, feat, dt); });
    const auto fn = backward ? fastgl_block_aggregate_bwd : fastgl_block_aggregate_fwd;
    run([&](void *s) {
        return fn(b.ip(), b.ix(), w, b.num_dst, b.num_src, b.num_edges, feat, mode, dt, in.data_ptr(), out.p(), p, ws.p(),
                  ws.n(), s);
    });
    return wrap(out.t);
}

// (indptr, indices, edge_w, num_src, mode, X, out) -> out
PyObject *aggregate_static(PyObject *const *a)
{
    const Block b(a[0], a[1], a[3]);
    const float *w = optional_f32(a[2], "edge_w");
    const auto mode = (fastgl_agg_mode)integer(a[4]);
    const at::Tensor &X = features(a[5], "X");
    const at::Tensor &out = dev(a[6], X.scalar_type(), "out");
    if (X.size(0) != b.num_src || !shape2(out, b.num_dst, X.size(1)))
        fail(PyExc_ValueError, "X must be [num_src, feat] and out [num_dst, feat]");
    run([&](void *s) {
        return fastgl_block_aggregate_fwd_static(b.ip(), b.ix(), w, b.num_dst, b.num_src, b.num_edges, X.size(1), mode,
                                                 feat_dtype(X), X.data_ptr(), out.data_ptr(), s);
    });
    return wrap(out);
}

// (blocks: sequence of (indptr, indices, num_src), parts, plan_mems: indexed by block, or None) -> [(handle, memory)]
PyObject *plan_create_many(PyObject *const *a)
{
    const int parts = (int)integer(a[1]);
    struct Seq {                             // no iterators: binding.py goes through the blocks once more
        PyObject *s;
        explicit Seq(PyObject *o) : s(nullptr)
        {
            if (!PySequence_Check(o)) fail(PyExc_TypeError, "blocks must be a sequence of (indptr, indices, num_src)");
            s = PySequence_Fast(o, "a sequence is expected");
            if (!s) throw Raised{};
        }
        ~Seq() { Py_DECREF(s); }
        Py_ssize_t n() const { return PySequence_Fast_GET_SIZE(s); }
        PyObject *at(Py_ssize_t i) const { return PySequence_Fast_GET_ITEM(s, i); }
    };
    const Seq blocks(a[0]);
    const Py_ssize_t n = blocks.n();
    std::vector<fastgl_block_desc> desc((size_t)n);
    std::vector<at::Tensor> mem((size_t)n);
    std::vector<fastgl_plan *> out((size_t)n, nullptr);
    struct Ref { PyObject *o; ~Ref() { Py_XDECREF(o); } };
    for (Py_ssize_t i = 0; i < n; ++i) {
        const Seq item(blocks.at(i));
        if (item.n() != 3) fail(PyExc_ValueError, "a block is (indptr, indices, num_src)");
        const Block b(item.at(0), item.at(1), item.at(2));
        if (!none(a[2])) {
            const Ref index{PyLong_FromSsize_t(i)}, m{index.o ? PyObject_GetItem(a[2], index.o) : nullptr};
            if (!m.o) throw Raised{};
            mem[i] = tensor(m.o, "plan memory");
        } else
            mem[i] = at::empty({(int64_t)fastgl_block_plan_bytes(b.num_dst, b.num_src, b.num_edges)},
                               b.indptr.options().dtype(at::kByte));
        fastgl_block_desc &d = desc[(size_t)i];
        d.indptr = b.ip(); d.indices = b.ix();
        d.num_dst = b.num_dst; d.num_src = b.num_src; d.num_edges = b.num_edges;
        d.parts = parts; d.plan_mem = mem[i].data_ptr(); d.plan_bytes = (size_t)mem[i].numel();
    }
    run([&](void *s) { return fastgl_block_plan_create_many((int)n, desc.data(), s, out.data()); });
    PyObject *r = PyList_New(n);
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject *t = PyTuple_New(2);
        PyTuple_SET_ITEM(t, 0, PyLong_FromVoidPtr(out[(size_t)i]));
        PyTuple_SET_ITEM(t, 1, wrap(mem[(size_t)i]));
        PyList_SET_ITEM(r, i, t);
    }
    return r;
}

// (table, ids, out) -> out
PyObject *gather_rows(PyObject *const *a)
{
    const at::Tensor &table = features(a[0], "table"), &ids = dev(a[1], at::kLong, "ids");
    const int64_t n = ids.numel(), feat = table.size(1);
    const Out out(a[2], table.scalar_type(), {n, feat}, table, "out");
    run([&](void *s) {
        return fastgl_gather_rows(table.data_ptr(), table.size(0), (const int64_t *)ids.data_ptr(), n, feat,
                                  feat_dtype(table), out.p(), s);
    });
    return wrap(out.t);
}

// ----------------------------------------------------------------------------------- update phase
// (H, W, bias, relu, Y) -> Y
PyObject *update_fwd(PyObject *const *a)
{
    const at::Tensor &H = features(a[0], "H"), &W = dev(a[1], H.scalar_type(), "W");
    const int64_t M = H.size(0), K = H.size(1);
    if (H.dim() != 2 || !matrix(W) || W.size(0) != K) fail(PyExc_ValueError, "W must be [K,N] and bias [N]");
    const int64_t N = W.size(1);
    const int relu = truth(a[3]);
    if (!none(a[2]) && !shape1(tensor(a[2], "bias"), N)) fail(PyExc_ValueError, "W must be [K,N] and bias [N]");
    const float *bias = optional_f32(a[2], "bias");
    const Out Y(a[4], H.scalar_type(), {M, N}, H, "Y");
    if (!shape2(Y.t, M, N)) fail(PyExc_ValueError, "Y must be [M,N]");
    run([&](void *s) {
        if (H.scalar_type() == at::kFloat)
            return fastgl_update_fwd((const float *)H.data_ptr(), (const float *)W.data_ptr(), bias, M, K, N, relu,
                                     (float *)Y.p(), s);
        return fastgl_update_fwd_bf16((const uint16_t *)H.data_ptr(), (const uint16_t *)W.data_ptr(), bias, M, K, N, relu,
                                      (uint16_t *)Y.p(), s);
    });
    return wrap(Y.t);
}

// (indptr, indices, edge_w, num_src, mode, X, W, bias, relu, H, Y, want_H, plan, workspace) -> (H, Y)
PyObject *layer_fwd(PyObject *const *a)
{
    const Block b(a[0], a[1], a[3]);
    const float *w = optional_f32(a[2], "edge_w");
    const auto mode = (fastgl_agg_mode)integer(a[4]);
    const at::Tensor &X = features(a[5], "X"), &W = dev(a[6], X.scalar_type(), "W");
    const int64_t K = X.size(1);
    if (X.size(0) != b.num_src || !matrix(W) || W.size(0) != K ||
        (!none(a[7]) && !shape1(tensor(a[7], "bias"), W.size(1))))
        fail(PyExc_ValueError, "X must be [num_src,K], W [K,N], bias [N]");
    const int64_t N = W.size(1);
    const float *bias = optional_f32(a[7], "bias");
    const int relu = truth(a[8]);
    Out H;
    if (!none(a[9]) || truth(a[11])) H = Out(a[9], X.scalar_type(), {b.num_dst, K}, X, "H");
    const Out Y(a[10], X.scalar_type(), {b.num_dst, N}, X, "Y");
    const fastgl_dtype dt = feat_dtype(X);
    const fastgl_plan *p = plan_of(a[12]);
    const Scratch ws(a[13], X, [&] { return fastgl_block_workspace_bytes(b.num_dst, b.num_src, b.num_edges, K, dt); });
    run([&](void *s) {
        return fastgl_layer_fwd(b.ip(), b.ix(), w, b.num_dst, b.num_src, b.num_edges, K, mode, dt, X.data_ptr(),
                                W.data_ptr(), bias, N, relu, H.p(), Y.p(), p, ws.p(), ws.n(), s);
    });
    return tuple({H.t, Y.t});
}

// (H, W, Y, dY, relu, want_dH, want_dW, want_db, dH, dW, db, workspace) -> (dH, dW, db)
PyObject *update_bwd(PyObject *const *a)
{
    const at::Tensor &H = features(a[0], "H"), &W = dev(a[1], H.scalar_type(), "W"), &dY = dev(a[3], H.scalar_type(), "dY");
    const void *Y = none(a[2]) ? nullptr : dev(a[2], H.scalar_type(), "Y").data_ptr();
    const int64_t M = H.size(0), K = H.size(1);
    const bool fits = H.dim() == 2 && matrix(W) && W.size(0) == K && shape2(dY, M, W.size(1)) &&
                      (none(a[2]) || shape2(tensor(a[2], "Y"), M, W.size(1)));
    if (!fits) fail(PyExc_ValueError, "shapes must be H [M,K], W [K,N], Y and dY [M,N]");
    const int64_t N = W.size(1);
    const int relu = truth(a[4]);
    Out dH, dW, db;
    if (!none(a[8]) || truth(a[5])) dH = Out(a[8], H.scalar_type(), {M, K}, H, "dH");
    if (!none(a[9]) || truth(a[6])) dW = Out(a[9], at::kFloat, {K, N}, H, "dW");
    if (!none(a[10]) || truth(a[7])) db = Out(a[10], at::kFloat, {N}, H, "db");
    if (dH.t.defined() && !shape2(dH.t, M, K)) fail(PyExc_ValueError, "dH must have the shape of H");
    if (dW.t.defined() && !shape2(dW.t, K, N)) fail(PyExc_ValueError, "dW must have the shape of W");
    if (db.t.defined() && !shape1(db.t, N)) fail(PyExc_ValueError, "db must have shape [N]");
    const Scratch ws(a[11], H, [&] {
        const size_t n = fastgl_update_bwd_workspace_bytes(M, K, N);
        return n < 256 ? (size_t)256 : n;
    });
    run([&](void *s) {
        if (H.scalar_type() == at::kFloat)
            return fastgl_update_bwd((const float *)H.data_ptr(), (const float *)W.data_ptr(), (const float *)Y,
                                     (const float *)dY.data_ptr(), M, K, N, relu, (float *)dH.p(), (float *)dW.p(),
                                     (float *)db.p(), ws.p(), ws.n(), s);
        return fastgl_update_bwd_bf16((const uint16_t *)H.data_ptr(), (const uint16_t *)W.data_ptr(), (const uint16_t *)Y,
                                      (const uint16_t *)dY.data_ptr(), M, K, N, relu, (uint16_t *)dH.p(), (float *)dW.p(),
                                      (float *)db.p(), ws.p(), ws.n(), s);
    });
    return tuple({dH.t, dW.t, db.t});
}

// --------------------------------------------------------------------------- ID map, Match, reorder
// (dst_gid, nbr_gid, mode, local_nbr, unique_gid, result, workspace) -> (local_nbr, unique_gid, result)
PyObject *idmap(PyObject *const *a)
{
    const at::Tensor &dst = dev(a[0], at::kLong, "dst_gid"), &nbr = dev(a[1], at::kLong, "nbr_gid");
    const int64_t nd = dst.numel(), nn = nbr.numel();
    const auto mode = (fastgl_idmap_mode)integer(a[2]);
    const Out local(a[3], at::kInt, {nn}, dst, "local_nbr");
    const Out uniq(a[4], at::kLong, {nd + nn > 0 ? nd + nn : 1}, dst, "unique_gid");
    const Out result(a[5], at::kInt, {2}, dst, "result");
    if (local.t.numel() < nn || uniq.t.numel() < nd + nn || result.t.numel() < 2)
        fail(PyExc_ValueError, "output arrays too small");
    const Scratch ws(a[6], dst, [&] { return fastgl_idmap_workspace_bytes(nd, nn); });
    run([&](void *s) {
        return fastgl_idmap((const int64_t *)dst.data_ptr(), nd, (const int64_t *)nbr.data_ptr(), nn, mode,
                            (int32_t *)local.p(), (int64_t *)uniq.p(), (int32_t *)result.p(), ws.p(), ws.n(), s);
    });
    return tuple({local.t, uniq.t, result.t});
}

// (prev_gid, new_gid, src_row, load_pos, load_gid, result, workspace) -> (src_row, load_pos, load_gid, result)
PyObject *match(PyObject *const *a)
{
    const at::Tensor &prev = dev(a[0], at::kLong, "prev_gid"), &next = dev(a[1], at::kLong, "new_gid");
    const int64_t np = prev.numel(), nn = next.numel();
    const Out row(a[2], at::kInt, {nn}, next, "src_row"), pos(a[3], at::kInt, {nn}, next, "load_pos");
    const Out gid(a[4], at::kLong, {nn}, next, "load_gid"), result(a[5], at::kInt, {2}, next, "result");
    if (row.t.numel() < nn || pos.t.numel() < nn || gid.t.numel() < nn || result.t.numel() < 2)
        fail(PyExc_ValueError, "output arrays too small");
    const Scratch ws(a[6], next, [&] { return fastgl_match_workspace_bytes(np, nn); });
    run([&](void *s) {
        return fastgl_match((const int64_t *)prev.data_ptr(), np, (const int64_t *)next.data_ptr(), nn, (int32_t *)row.p(),
                            (int32_t *)pos.p(), (int64_t *)gid.p(), (int32_t *)result.p(), ws.p(), ws.n(), s);
    });
    return tuple({row.t, pos.t, gid.t, result.t});
}

// (X_prev, X_load, src_row, n_load, out) -> out
PyObject *assemble_rows(PyObject *const *a)
{
    const at::Tensor &prev = features(a[0], "X_prev"), &load = dev(a[1], prev.scalar_type(), "X_load");
    const at::Tensor &row = dev(a[2], at::kInt, "src_row");
    const int64_t feat = prev.size(1), n = row.numel(), n_load = integer(a[3]);
    if (!matrix(load) || load.size(1) != feat || load.size(0) < n_load)
        fail(PyExc_ValueError, "X_load must be [>= n_load, feat]");
    const Out out(a[4], prev.scalar_type(), {n, feat}, prev, "out");
    if (!shape2(out.t, n, feat)) fail(PyExc_ValueError, "out must be [n_new, feat]");
    run([&](void *s) {
        return fastgl_assemble_rows(prev.data_ptr(), prev.size(0), load.data_ptr(), n_load, (const int32_t *)row.data_ptr(),
                                    n, feat, feat_dtype(prev), out.p(), s);
    });
    return wrap(out.t);
}

// (gid, offsets: sequence of ints, workspace) -> (counts, violations)
PyObject *overlap_counts(PyObject *const *a)
{
    const at::Tensor &gid = dev(a[0], at::kLong, "gid");
    PyObject *seq = PySequence_Fast(a[1], "offsets must be a sequence");
    if (!seq) throw Raised{};
    struct Drop { PyObject *o; ~Drop() { Py_DECREF(o); } } drop{seq};
    std::vector<int64_t> off;
    for (Py_ssize_t i = 0; i < PySequence_Fast_GET_SIZE(seq); ++i) off.push_back(to_integer(PySequence_Fast_GET_ITEM(seq, i)));
    if (off.empty()) fail(PyExc_ValueError, "offsets must hold at least one entry");
    const int n = (int)off.size() - 1;
    const at::Tensor counts = at::empty({n, n}, gid.options()), viol = at::empty({1}, gid.options().dtype(at::kInt));
    const Scratch ws(a[2], gid, [&] { return fastgl_overlap_workspace_bytes(gid.numel()); });
    run([&](void *s) {
        return fastgl_overlap_counts((const int64_t *)gid.data_ptr(), off.data(), n, (int64_t *)counts.data_ptr(),
                                     (int32_t *)viol.data_ptr(), ws.p(), ws.n(), s);
    });
    return tuple({counts, viol});
}

// ------------------------------------------------------------------------------------ edge weights
// (indptr, indices, num_src, mode, X, grad_out, plan, grad_w, workspace) -> grad_w
PyObject *edge_weight_grad(PyObject *const *a)
{
    const Block b(a[0], a[1], a[2]);
    const auto mode = (fastgl_agg_mode)integer(a[3]);
    const at::Tensor &X = features(a[4], "X"), &G = dev(a[5], X.scalar_type(), "grad_out");
    if (X.size(0) != b.num_src || !shape2(G, b.num_dst, X.size(1)))
        fail(PyExc_ValueError, "X must be [num_src, feat] and grad_out [num_dst, feat]");
    const fastgl_plan *p = plan_of(a[6]);
    const Out w(a[7], at::kFloat, {b.num_edges}, X, "grad_w");
    if (w.t.numel() != b.num_edges) fail(PyExc_ValueError, "grad_w must have one entry per edge");
    const Scratch ws(a[8], X, [&] { return fastgl_edge_workspace_bytes(b.num_dst, b.num_edges); });
    run([&](void *s) {
        return fastgl_edge_weight_grad(b.ip(), b.ix(), b.num_dst, b.num_src, b.num_edges, X.size(1), mode, feat_dtype(X),
                                       X.data_ptr(), G.data_ptr(), p, (float *)w.p(), ws.p(), ws.n(), s);
    });
    return wrap(w.t);
}

// (indptr, score, alpha, workspace) -> alpha
PyObject *edge_softmax_fwd(PyObject *const *a)
{
    const at::Tensor &ip = dev(a[0], at::kInt, "indptr"), &score = dev(a[1], at::kFloat, "score");
    const int64_t nd = ip.numel() - 1, E = score.numel();
    const Out alpha(a[2], at::kFloat, score.sizes(), score, "alpha");
    if (alpha.t.numel() != E) fail(PyExc_ValueError, "alpha must have one entry per edge");
    const Scratch ws(a[3], score, [&] { return fastgl_edge_workspace_bytes(nd, E); });
    run([&](void *s) {
        return fastgl_edge_softmax_fwd((const int32_t *)ip.data_ptr(), nd, E, (const float *)score.data_ptr(),
                                       (float *)alpha.p(), ws.p(), ws.n(), s);
    });
    return wrap(alpha.t);
}

// (indptr, alpha, grad_alpha, grad_score, workspace) -> grad_score
PyObject *edge_softmax_bwd(PyObject *const *a)
{
    const at::Tensor &ip = dev(a[0], at::kInt, "indptr"), &alpha = dev(a[1], at::kFloat, "alpha");
    const at::Tensor &da = dev(a[2], at::kFloat, "grad_alpha");
    const int64_t nd = ip.numel() - 1, E = alpha.numel();
    const Out ds(a[3], at::kFloat, alpha.sizes(), alpha, "grad_score");
    if (da.numel() != E || ds.t.numel() != E) fail(PyExc_ValueError, "per-edge arrays must have one entry per edge");
    const Scratch ws(a[4], alpha, [&] { return fastgl_edge_workspace_bytes(nd, E); });
    run([&](void *s) {
        return fastgl_edge_softmax_bwd((const int32_t *)ip.data_ptr(), nd, E, (const float *)alpha.data_ptr(),
                                       (const float *)da.data_ptr(), (float *)ds.p(), ws.p(), ws.n(), s);
    });
    return wrap(ds.t);
}

// (indptr, indices, el, er, slope, score) -> score
PyObject *edge_score_fwd(PyObject *const *a)
{
    const at::Tensor &ip = dev(a[0], at::kInt, "indptr"), &ix = dev(a[1], at::kInt, "indices");
    const at::Tensor &el = dev(a[2], at::kFloat, "el"), &er = dev(a[3], at::kFloat, "er");
    const int64_t nd = ip.numel() - 1, E = ix.numel();
    if (el.numel() != nd) fail(PyExc_ValueError, "el must have one entry per destination node");
    const float slope = to_real(a[4]);
    const Out score(a[5], at::kFloat, {E}, el, "score");
    if (score.t.numel() != E) fail(PyExc_ValueError, "score must have one entry per edge");
    run([&](void *s) {
        return fastgl_edge_score_fwd((const int32_t *)ip.data_ptr(), (const int32_t *)ix.data_ptr(), nd, er.numel(), E,
                                     (const float *)el.data_ptr(), (const float *)er.data_ptr(), slope,
                                     (float *)score.p(), s);
    });
    return wrap(score.t);
}

// (indptr, indices, el, er, slope, grad_score, plan, want_el, want_er, grad_el, grad_er) -> (grad_el, grad_er)
PyObject *edge_score_bwd(PyObject *const *a)
{
    const at::Tensor &ip = dev(a[0], at::kInt, "indptr"), &ix = dev(a[1], at::kInt, "indices");
    const at::Tensor &el = dev(a[2], at::kFloat, "el"), &er = dev(a[3], at::kFloat, "er");
    const float slope = to_real(a[4]);
    const at::Tensor &g = dev(a[5], at::kFloat, "grad_score");
    const int64_t nd = ip.numel() - 1, E = ix.numel();
    if (el.numel() != nd || g.numel() != E)
        fail(PyExc_ValueError, "el must have one entry per destination node, grad_score one per edge");
    const fastgl_plan *p = plan_of(a[6]);
    Out gl, gr;
    if (!none(a[9]) || truth(a[7])) gl = Out(a[9], at::kFloat, el.sizes(), el, "grad_el");
    if (!none(a[10]) || truth(a[8])) gr = Out(a[10], at::kFloat, er.sizes(), er, "grad_er");
    if (gl.t.defined() && gl.t.numel() != el.numel()) fail(PyExc_ValueError, "grad_el must have one entry per node");
    if (gr.t.defined() && gr.t.numel() != er.numel()) fail(PyExc_ValueError, "grad_er must have one entry per node");
    run([&](void *s) {
        return fastgl_edge_score_bwd((const int32_t *)ip.data_ptr(), (const int32_t *)ix.data_ptr(), nd, er.numel(), E,
                                     (const float *)el.data_ptr(), (const float *)er.data_ptr(), slope,
                                     (const float *)g.data_ptr(), p, (float *)gl.p(), (float *)gr.p(), s);
    });
    return tuple({gl.t, gr.t});
}

// (error class): called once by binding.py
PyObject *set_error_class(PyObject *const *a)
{
    Py_INCREF(a[0]);
    Py_XDECREF(g_error_class);
    g_error_class = a[0];
    Py_RETURN_NONE;
}

#define FN(name, nargs) {#name, (PyCFunction)(void (*)(void))entry<name, nargs>, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    FN(aggregate, 10), FN(aggregate_static, 7), FN(plan_create_many, 3), FN(gather_rows, 3),
    FN(update_fwd, 5), FN(layer_fwd, 14), FN(update_bwd, 12), FN(idmap, 7), FN(match, 7), FN(assemble_rows, 5),
    FN(overlap_counts, 3), FN(edge_weight_grad, 9), FN(edge_softmax_fwd, 4), FN(edge_softmax_bwd, 5),
    FN(edge_score_fwd, 6), FN(edge_score_bwd, 11), FN(set_error_class, 1), {nullptr, nullptr, 0, nullptr}};
#undef FN

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_host", "Native marshalling of the C ABI's calls.", -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host(void)
{
    g_handle_name = PyUnicode_InternFromString("handle");
    g_value_name = PyUnicode_InternFromString("value");
    return g_handle_name && g_value_name ? PyModule_Create(&g_module) : nullptr;
}
