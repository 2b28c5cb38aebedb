// The Python binding's hot half: tensors in, one library call, tensors out.
//
// What bounds it: the short calls of a decoding step (verification, cache append, one drafting step) run 2-10 us on
// the GPU, and marshalled by ctypes each cost the host 8-15 us -- parameter structs, eleven converted arguments, one
// Python call per data pointer and stride, three allocations through the dispatcher.  Here the same checks, sizes and
// pointers are taken from the tensors in C++, so that a call costs the host little more than its kernel launches
// (about 2.4 us each).  Nothing is computed here; argument rules and error texts are those the binding always had.
//
// Every function returns the library's status (0 = ok) alone or ahead of its results; api.py raises on it.  The GIL is
// released around library calls, as ctypes does.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "internal.h"
#include "opttree.h"

namespace {

struct PyErrSet {};                      // a Python error has been set: unwind to the entry point

[[noreturn]] void fail(PyObject* type, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    PyErr_FormatV(type, fmt, ap);
    va_end(ap);
    throw PyErrSet();
}

const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a torch.Tensor, got %s", Py_TYPE(o)->tp_name);
    return THPVariable_Unpack(o);
}
const at::Tensor* tensor_or_null(PyObject* o) { return o == Py_None ? nullptr : &tensor(o); }
void* ptr(const at::Tensor& t) { return t.data_ptr(); }
void* ptr(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }
size_t bytes_of(const at::Tensor& t) { return (size_t)t.numel(); }          // workspaces are uint8 tensors

int32_t as_int(PyObject* o) {
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw PyErrSet();
    if (v != (int32_t)v) fail(PyExc_OverflowError, "%ld does not fit 32 bits", v);
    return (int32_t)v;
}
double as_double(PyObject* o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw PyErrSet();
    return v;
}
int32_t dtype_code(const at::Tensor& t) {
    if (t.scalar_type() == at::kFloat) return OT_F32;
    if (t.scalar_type() == at::kBFloat16) return OT_BF16;
    PyErr_Format(PyExc_TypeError, "unsupported dtype %s", c10::toString(t.scalar_type()));
    throw PyErrSet();
}
void* current_stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

// Data pointers are taken before the GIL is released: a tensor without storage (functorch wrappers, sparse, fake) answers
// data_ptr() with an exception, which becomes a Python error only under the GIL.
struct NoGil {
    PyThreadState* const state = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(state); }
};
template <typename F>
int without_gil(F&& f) {
    const NoGil released;
    return f();
}

struct Ref {                             // owned reference
    PyObject* p;
    explicit Ref(PyObject* q) : p(q) { if (!q) throw PyErrSet(); }
    Ref(const Ref&) = delete;
    ~Ref() { Py_XDECREF(p); }
    PyObject* release() { PyObject* q = p; p = nullptr; return q; }
};

at::Tensor new_tensor(at::IntArrayRef sizes, at::ScalarType st, const at::Device& dev) {
    return at::empty(sizes, at::TensorOptions().dtype(st).device(dev));
}
PyObject* wrap(const at::Tensor& t) { return THPVariable_Wrap(t); }

// interned attribute names, made when the module is
struct Names {
    PyObject *token, *parent, *depth, *score, *mask, *n_out, *expect;
    PyObject *p, *step, *ws, *frontier_token, *frontier_parent, *frontier_count, *esub, *go;
} names;

ot_build_params copy_params(PyObject* ctypes_struct) {
    Py_buffer buf;
    if (PyObject_GetBuffer(ctypes_struct, &buf, PyBUF_SIMPLE)) throw PyErrSet();
    ot_build_params p;
    const bool ok = buf.len == (Py_ssize_t)sizeof(p);
    if (ok) memcpy(&p, buf.buf, sizeof(p));
    PyBuffer_Release(&buf);
    if (!ok) fail(PyExc_TypeError, "BuildParams expected");
    return p;
}

// a Tree's seven tensors; `cls` builds one when the caller brought none
ot_tree_out tree_pointers(PyObject* tree) {
    auto get = [&](PyObject* name) { Ref a(PyObject_GetAttr(tree, name)); return ptr(tensor(a.p)); };
    return ot_tree_out{(int32_t*)get(names.token), (int32_t*)get(names.parent), (int32_t*)get(names.depth),
                       (float*)get(names.score), (uint64_t*)get(names.mask), (int32_t*)get(names.n_out),
                       (double*)get(names.expect)};
}
PyObject* new_tree(PyObject* cls, int64_t B, int64_t n, const at::Device& dev) {
    const int64_t W = (n + 63) / 64;
    Ref token(wrap(new_tensor({B, n}, at::kInt, dev))), parent(wrap(new_tensor({B, n}, at::kInt, dev)));
    Ref depth(wrap(new_tensor({B, n}, at::kInt, dev))), score(wrap(new_tensor({B, n}, at::kFloat, dev)));
    Ref mask(wrap(new_tensor({B, n, W}, at::kLong, dev))), n_out(wrap(new_tensor({B}, at::kInt, dev)));
    Ref expect(wrap(new_tensor({B}, at::kDouble, dev)));
    PyObject* tree = PyObject_CallFunctionObjArgs(cls, token.p, parent.p, depth.p, score.p, mask.p, n_out.p, expect.p, nullptr);
    if (!tree) throw PyErrSet();
    return tree;
}

// frontier width of step `step` and the widest one before step `depth` (F_0 = 1, F_{t+1} = min(n, k F_t))
void frontier(int k, int n, int step, int depth, int64_t& at_step, int64_t& widest) {
    int64_t F = 1;
    at_step = widest = 1;
    for (int t = 0; t < depth; ++t) {
        if (t == step) at_step = F;
        widest = F > widest ? F : widest;
        F = std::min<int64_t>(n, (int64_t)k * F);
    }
}

ot_build_params build_params(const at::Tensor& x, int32_t k, int32_t n, int32_t depth) {
    if (x.dim() != 4 || x.stride(3) != 1) fail(PyExc_ValueError, "logits must be [B, depth, n, V] with a contiguous last dimension");
    int64_t unused, need = 1;
    if (depth >= 1 && k >= 1 && n >= 1) frontier(k, n, 0, depth, unused, need);
    if (x.size(1) < depth || x.size(2) < need)
        fail(PyExc_ValueError, "logits tensor [%lld, %lld, %lld, %lld] smaller than (depth %d, widest frontier %lld)", (long long)x.size(0),
             (long long)x.size(1), (long long)x.size(2), (long long)x.size(3), (int)depth, (long long)need);
    ot_build_params p;
    p.batch = (int32_t)x.size(0); p.vocab = (int32_t)x.size(3); p.depth = depth; p.k = k; p.n = n;
    p.logits_dtype = dtype_code(x);
    p.stride_seq = x.stride(0); p.stride_depth = x.stride(1); p.stride_row = x.stride(2);
    return p;
}

ot_attn_params attn_params(const at::Tensor& Q, const at::Tensor* Kp, const at::Tensor* Vp, const at::Tensor& Kt, const at::Tensor& Vt,
                           const at::Tensor& O, float scale) {
    if (Q.dim() != 4 || Kt.dim() != 4) fail(PyExc_ValueError, "Q and K_tree must have four dimensions");
    ot_attn_params p;
    p.batch = (int32_t)Q.size(0); p.q_heads = (int32_t)Q.size(1); p.kv_heads = (int32_t)Kt.size(1);
    p.head_dim = (int32_t)Q.size(3); p.n = (int32_t)Q.size(2);
    p.max_prefix = Kp ? (int32_t)Kp->size(2) : 0;
    p.dtype = dtype_code(Q);
    p.softmax_scale = scale;
    auto st = [&](const at::Tensor* t, int64_t* s) {
        if (!t) { s[0] = 0; s[1] = 0; s[2] = p.head_dim; return; }
        if (t->dim() != 4) fail(PyExc_ValueError, "attention tensors have four dimensions");
        if (t->stride(3) != 1) fail(PyExc_ValueError, "last dimension must be contiguous");
        s[0] = t->stride(0); s[1] = t->stride(1); s[2] = t->stride(2);
    };
    st(&Q, p.q_strides); st(Kp, p.kp_strides); st(Vp, p.vp_strides); st(&Kt, p.kt_strides); st(&Vt, p.vt_strides);
    st(&O, p.o_strides);
    const int32_t keys = (int32_t)Kt.size(2);
    p.n_keys = keys == p.n ? 0 : keys;
    return p;
}

void want_args(Py_ssize_t got, Py_ssize_t want) {
    if (got != want) fail(PyExc_TypeError, "%zd arguments expected, got %zd", want, got);
}

// ---- entry points: (arguments) -> result object, errors as exceptions ------------------------------------------------

// (logits, k, n, depth, out | None, workspace | None, Tree) -> (status, tree)
PyObject* build_tree(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 7);
    const at::Tensor& x = tensor(a[0]);
    const ot_build_params p = build_params(x, as_int(a[1]), as_int(a[2]), as_int(a[3]));
    const size_t need = ot_build_workspace_bytes(&p);
    const void* const px = ptr(x);
    if (need == 0) return Py_BuildValue("iO", ot_build_tree(&p, px, nullptr, 0, nullptr, nullptr), Py_None);
    at::Tensor own;
    const at::Tensor* ws = tensor_or_null(a[5]);
    if (!ws) { own = new_tensor({(int64_t)need}, at::kByte, x.device()); ws = &own; }
    Ref tree(a[4] == Py_None ? new_tree(a[6], p.batch, p.n, x.device()) : (Py_INCREF(a[4]), a[4]));
    const ot_tree_out o = tree_pointers(tree.p);
    void* const pw = ptr(*ws);
    const size_t nw = bytes_of(*ws);
    void* s = current_stream();
    const int st = without_gil([&] { return ot_build_tree(&p, px, pw, nw, &o, s); });
    return Py_BuildValue("iO", st, tree.p);
}

// (logits, k, n, depth, delta, out | None, workspace | None, Tree) -> (status, tree, steps, e_sub)
PyObject* build_tree_adaptive(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 8);
    const at::Tensor& x = tensor(a[0]);
    const ot_build_params p = build_params(x, as_int(a[1]), as_int(a[2]), as_int(a[3]));
    const double delta = as_double(a[4]);
    const size_t need = ot_build_workspace_bytes(&p);
    if (need == 0) return Py_BuildValue("iOOO", OT_ERR_UNSUPPORTED, Py_None, Py_None, Py_None);
    at::Tensor own;
    const at::Tensor* ws = tensor_or_null(a[6]);
    if (!ws) { own = new_tensor({(int64_t)need}, at::kByte, x.device()); ws = &own; }
    Ref tree(a[5] == Py_None ? new_tree(a[7], p.batch, p.n, x.device()) : (Py_INCREF(a[5]), a[5]));
    const ot_tree_out o = tree_pointers(tree.p);
    const at::Tensor steps = new_tensor({p.batch}, at::kInt, x.device()), e = new_tensor({p.batch}, at::kDouble, x.device());
    const void* const px = ptr(x);
    void* const pw = ptr(*ws);
    const size_t nw = bytes_of(*ws);
    int32_t* const psteps = (int32_t*)ptr(steps);
    double* const pe = (double*)ptr(e);
    void* s = current_stream();
    const int st = without_gil([&] { return ot_build_tree_adaptive(&p, delta, px, pw, nw, &o, psteps, pe, s); });
    Ref ws_(wrap(steps)), we_(wrap(e));
    return Py_BuildValue("iOOO", st, tree.p, ws_.p, we_.p);
}

// (BuildParams, device) -> (status, workspace, frontier_token, frontier_parent, frontier_count)
PyObject* stream_begin(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 2);
    const ot_build_params p = copy_params(a[0]);
    const size_t need = ot_build_workspace_bytes(&p);
    if (need == 0) return Py_BuildValue("iOOOO", ot_tree_begin(&p, nullptr, 0, nullptr), Py_None, Py_None, Py_None, Py_None);
    at::Device dev(at::kCUDA);
    if (THPDevice_Check(a[1])) dev = reinterpret_cast<THPDevice*>(a[1])->device;
    else if (PyUnicode_Check(a[1])) dev = at::Device(std::string(PyUnicode_AsUTF8(a[1])));
    else dev = at::Device(at::kCUDA, (c10::DeviceIndex)as_int(a[1]));
    const at::Tensor ws = new_tensor({(int64_t)need}, at::kByte, dev);
    const at::Tensor tok = new_tensor({p.batch, p.n}, at::kInt, dev), par = new_tensor({p.batch, p.n}, at::kInt, dev);
    const at::Tensor cnt = new_tensor({p.batch}, at::kInt, dev);
    void* const pw = ptr(ws);
    int32_t *const pt = (int32_t*)ptr(tok), *const pp = (int32_t*)ptr(par), *const pc = (int32_t*)ptr(cnt);
    void* s = current_stream();
    // one small kernel sets the loop state and the frontier arrays (tokens and parents -1, counts 0)
    const int st = without_gil([&] { return ot_internal_tree_begin(&p, pw, need, pt, pp, pc, s); });
    Ref w(wrap(ws)), t(wrap(tok)), q(wrap(par)), c(wrap(cnt));
    return Py_BuildValue("iOOOO", st, w.p, t.p, q.p, c.p);
}

// (TreeStream, rows) -> (status, frontier_token, frontier_parent)
PyObject* stream_expand(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 2);
    PyObject* self = a[0];
    const at::Tensor& rows = tensor(a[1]);
    if (rows.dim() != 3 || rows.stride(2) != 1) fail(PyExc_ValueError, "rows must be [B, F, V] with a contiguous last dimension");
    Ref po(PyObject_GetAttr(self, names.p)), so(PyObject_GetAttr(self, names.step));
    const ot_build_params p = copy_params(po.p);
    const int step = as_int(so.p);
    if (step >= p.depth) fail(PyExc_ValueError, "all %d drafting steps have been fed", (int)p.depth);
    int64_t need, widest;
    frontier(p.k, p.n, step, p.depth, need, widest);
    if (rows.size(0) < p.batch || rows.size(1) < need || rows.size(2) < p.vocab)
        fail(PyExc_ValueError, "rows (%lld, %lld, %lld) smaller than [batch %d, F_%d = %lld, vocab %d]", (long long)rows.size(0),
             (long long)rows.size(1), (long long)rows.size(2), (int)p.batch, step, (long long)need, (int)p.vocab);
    Ref ws(PyObject_GetAttr(self, names.ws)), tok(PyObject_GetAttr(self, names.frontier_token));
    Ref par(PyObject_GetAttr(self, names.frontier_parent)), cnt(PyObject_GetAttr(self, names.frontier_count));
    const at::Tensor& w = tensor(ws.p);
    int32_t *pt = (int32_t*)ptr(tensor(tok.p)), *pp = (int32_t*)ptr(tensor(par.p)), *pc = (int32_t*)ptr(tensor(cnt.p));
    const void* const pr = ptr(rows);
    void* const pw = ptr(w);
    const size_t nw = bytes_of(w);
    const int64_t stride_seq = rows.stride(0), stride_row = rows.stride(1);
    void* s = current_stream();
    const int st = without_gil([&] { return ot_tree_expand(&p, step, pr, stride_seq, stride_row, pw, nw, pt, pp, pc, s); });
    if (st == OT_OK) {
        Ref next(PyLong_FromLong(step + 1));
        if (PyObject_SetAttr(self, names.step, next.p)) throw PyErrSet();
    }
    return Py_BuildValue("iOO", st, tok.p, par.p);
}

// (TreeStream) -> (status, mask)
PyObject* stream_mask(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 1);
    Ref po(PyObject_GetAttr(a[0], names.p)), so(PyObject_GetAttr(a[0], names.step)), ws(PyObject_GetAttr(a[0], names.ws));
    const ot_build_params p = copy_params(po.p);
    const int step = as_int(so.p);
    const at::Tensor& w = tensor(ws.p);
    const at::Tensor m = new_tensor({p.batch, p.n, ((int64_t)p.depth * p.n + 63) / 64}, at::kLong, w.device());
    void* const pw = ptr(w);
    const size_t nw = bytes_of(w);
    uint64_t* const pm = (uint64_t*)ptr(m);
    void* s = current_stream();
    const int st = without_gil([&] { return ot_tree_frontier_mask(&p, step, pw, nw, pm, s); });
    Ref mo(wrap(m));
    return Py_BuildValue("iO", st, mo.p);
}

// (TreeStream, delta) -> (status, e_sub, go_on); the two result tensors belong to the stream object and are made once
PyObject* stream_esub(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 2);
    const double delta = as_double(a[1]);
    Ref po(PyObject_GetAttr(a[0], names.p)), so(PyObject_GetAttr(a[0], names.step)), ws(PyObject_GetAttr(a[0], names.ws));
    const ot_build_params p = copy_params(po.p);
    const int step = as_int(so.p);
    const at::Tensor& w = tensor(ws.p);
    if (!PyObject_HasAttr(a[0], names.esub)) {
        Ref e(wrap(new_tensor({p.batch}, at::kDouble, w.device()))), g(wrap(new_tensor({p.batch}, at::kInt, w.device())));
        if (PyObject_SetAttr(a[0], names.esub, e.p) || PyObject_SetAttr(a[0], names.go, g.p)) throw PyErrSet();
    }
    Ref e(PyObject_GetAttr(a[0], names.esub)), g(PyObject_GetAttr(a[0], names.go));
    double* pe = (double*)ptr(tensor(e.p));
    int32_t* pg = (int32_t*)ptr(tensor(g.p));
    void* const pw = ptr(w);
    const size_t nw = bytes_of(w);
    void* s = current_stream();
    const int st = without_gil([&] { return ot_tree_esub(&p, step, delta, pw, nw, pe, pg, s); });
    return Py_BuildValue("iOO", st, e.p, g.p);
}

// (TreeStream, out | None, Tree) -> (status, tree)
PyObject* stream_finalize(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 3);
    Ref po(PyObject_GetAttr(a[0], names.p)), so(PyObject_GetAttr(a[0], names.step)), ws(PyObject_GetAttr(a[0], names.ws));
    const ot_build_params p = copy_params(po.p);
    const int step = as_int(so.p);
    const at::Tensor& w = tensor(ws.p);
    Ref tree(a[1] == Py_None ? new_tree(a[2], p.batch, p.n, w.device()) : (Py_INCREF(a[1]), a[1]));
    const ot_tree_out o = tree_pointers(tree.p);
    void* const pw = ptr(w);
    const size_t nw = bytes_of(w);
    void* s = current_stream();
    const int st = without_gil([&] { return ot_tree_finalize(&p, step, pw, nw, &o, s); });
    return Py_BuildValue("iO", st, tree.p);
}

// (Q, K_prefix | None, V_prefix | None, K_tree, V_tree, prefix_len, mask, out | None, workspace, scale) -> (status, out)
PyObject* attention(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 10);
    const at::Tensor &Q = tensor(a[0]), &Kt = tensor(a[3]), &Vt = tensor(a[4]);
    const at::Tensor *Kp = tensor_or_null(a[1]), *Vp = tensor_or_null(a[2]), *len = tensor_or_null(a[5]), *mask = tensor_or_null(a[6]);
    at::Tensor own;
    const at::Tensor* O = tensor_or_null(a[7]);
    if (!O) { own = at::empty_like(Q); O = &own; }
    const at::Tensor& w = tensor(a[8]);
    const ot_attn_params p = attn_params(Q, Kp, Vp, Kt, Vt, *O, (float)as_double(a[9]));
    const void *const q = ptr(Q), *const kp = ptr(Kp), *const vp = ptr(Vp), *const kt = ptr(Kt), *const vt = ptr(Vt);
    const int32_t* const pl = (const int32_t*)ptr(len);
    const uint64_t* const pm = (const uint64_t*)ptr(mask);
    void *const po = ptr(*O), *const pw = ptr(w);
    const size_t nw = bytes_of(w);
    void* s = current_stream();
    const int st = without_gil([&] { return ot_tree_verify_attention(&p, q, kp, vp, kt, vt, pl, pm, po, pw, nw, s); });
    Ref o(wrap(*O));
    return Py_BuildValue("iO", st, o.p);
}

// as attention, with (k_scale, v_scale) ahead of prefix_len
PyObject* attention_fp8kv(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 12);
    const at::Tensor &Q = tensor(a[0]), &Kt = tensor(a[3]), &Vt = tensor(a[4]);
    const at::Tensor *Kp = tensor_or_null(a[1]), *Vp = tensor_or_null(a[2]), *len = tensor_or_null(a[7]), *mask = tensor_or_null(a[8]);
    const at::Tensor* kv[4] = {Kp, Vp, &Kt, &Vt};
    for (const at::Tensor* t : kv)
        if (t && t->scalar_type() != at::kByte) fail(PyExc_TypeError, "the 8-bit cache is passed as uint8 tensors");
    const at::Tensor* sc[2] = {&tensor(a[5]), &tensor(a[6])};
    for (const at::Tensor* t : sc)
        if (t->scalar_type() != at::kFloat || !t->is_contiguous() || t->dim() != 2 || Q.dim() != 4 || Kt.dim() != 4 ||
            t->size(0) != Q.size(0) || t->size(1) != Kt.size(1))
            fail(PyExc_ValueError, "scales must be contiguous float32 [B, Hkv]");
    at::Tensor own;
    const at::Tensor* O = tensor_or_null(a[9]);
    if (!O) { own = at::empty_like(Q); O = &own; }
    const at::Tensor& w = tensor(a[10]);
    const ot_attn_params p = attn_params(Q, Kp, Vp, Kt, Vt, *O, (float)as_double(a[11]));
    const void *const q = ptr(Q), *const kp = ptr(Kp), *const vp = ptr(Vp), *const kt = ptr(Kt), *const vt = ptr(Vt);
    const float *const ks = (const float*)ptr(sc[0]), *const vs = (const float*)ptr(sc[1]);
    const int32_t* const pl = (const int32_t*)ptr(len);
    const uint64_t* const pm = (const uint64_t*)ptr(mask);
    void *const po = ptr(*O), *const pw = ptr(w);
    const size_t nw = bytes_of(w);
    void* s = current_stream();
    const int st = without_gil([&] { return ot_tree_verify_attention_fp8kv(&p, q, kp, vp, kt, vt, ks, vs, pl, pm, po, pw, nw, s); });
    Ref o(wrap(*O));
    return Py_BuildValue("iO", st, o.p);
}

// (target_logits, u | None, temperature, token, parent, n_out, workspace | None) -> (status, length, node, token);
// u None: greedy
PyObject* verify(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 7);
    const at::Tensor& x = tensor(a[0]);
    if (x.dim() != 3 || x.stride(2) != 1) fail(PyExc_ValueError, "target_logits must be [B, n + 1, V] with a contiguous last dimension");
    const int64_t B = x.size(0), rows = x.size(1), n = rows - 1;
    const at::Tensor* u = tensor_or_null(a[1]);
    if (u && (u->scalar_type() != at::kFloat || u->dim() != 2 || u->size(0) != B || u->size(1) != rows || !u->is_contiguous()))
        fail(PyExc_ValueError, "u must be a contiguous float32 tensor [B, n + 1]");
    const float T = u ? (float)as_double(a[2]) : 0.f;
    ot_verify_params p;
    p.batch = (int32_t)B; p.vocab = (int32_t)x.size(2); p.n = (int32_t)n; p.logits_dtype = dtype_code(x);
    p.stride_seq = x.stride(0); p.stride_row = x.stride(1);
    const size_t need = u ? ot_verify_sample_workspace_bytes(&p) : ot_verify_workspace_bytes(&p);
    if (need == 0) return Py_BuildValue("iOOO", 1, Py_None, Py_None, Py_None);         // (the query rejects the shape)
    const at::Tensor &tok = tensor(a[3]), &par = tensor(a[4]), &n_out = tensor(a[5]);
    at::Tensor own;
    const at::Tensor* ws = tensor_or_null(a[6]);
    if (!ws) { own = new_tensor({(int64_t)need}, at::kByte, x.device()); ws = &own; }
    const at::Tensor len = new_tensor({B}, at::kInt, x.device()), node = new_tensor({B, n}, at::kInt, x.device());
    const at::Tensor out = new_tensor({B, rows}, at::kInt, x.device());
    const int32_t *pt = (const int32_t*)ptr(tok), *pp = (const int32_t*)ptr(par), *pn = (const int32_t*)ptr(n_out);
    int32_t *ol = (int32_t*)ptr(len), *on = (int32_t*)ptr(node), *ot = (int32_t*)ptr(out);
    const void* const px = ptr(x);
    const float* const pu = (const float*)ptr(u);
    void* const pw = ptr(*ws);
    const size_t nw = bytes_of(*ws);
    void* s = current_stream();
    const int st = without_gil([&] {
        return u ? ot_verify_sample(&p, T, px, pu, pt, pp, pn, pw, nw, ol, on, ot, s)
                 : ot_verify_greedy(&p, px, pt, pp, pn, pw, nw, ol, on, ot, s);
    });
    Ref l(wrap(len)), d(wrap(node)), o(wrap(out));
    return Py_BuildValue("iOOO", st, l.p, d.p, o.p);
}

// (K_prefix, V_prefix, K_tree, V_tree, prefix_len, accept_len, accept_node) -> (status, new_len)
PyObject* kv_append(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 7);
    const at::Tensor &Kp = tensor(a[0]), &Vp = tensor(a[1]), &Kt = tensor(a[2]), &Vt = tensor(a[3]);
    const at::Tensor &len = tensor(a[4]), &alen = tensor(a[5]), &anode = tensor(a[6]);
    const ot_attn_params p = attn_params(Kt, &Kp, &Vp, Kt, Vt, Kt, 0.f);
    const at::Tensor nl = new_tensor({p.batch}, at::kInt, Kt.device());
    void *const kp = ptr(Kp), *const vp = ptr(Vp);
    const void *const kt = ptr(Kt), *const vt = ptr(Vt);
    const int32_t *const pl = (const int32_t*)ptr(len), *const pa = (const int32_t*)ptr(alen), *const pn = (const int32_t*)ptr(anode);
    int32_t* const po = (int32_t*)ptr(nl);
    void* s = current_stream();
    const int st = without_gil([&] { return ot_kv_append(&p, kp, vp, kt, vt, pl, pa, pn, po, s); });
    Ref o(wrap(nl));
    return Py_BuildValue("iO", st, o.p);
}

// ---- prepared calls: everything but the stream fixed beforehand; called as f(stream) -> status -----------------------
struct PreparedBuild {
    ot_build_params p; const void* logits; void* ws; size_t bytes; ot_tree_out out;
};
struct PreparedAttention {
    ot_attn_params p; const void *Q, *Kp, *Vp, *Kt, *Vt; const int32_t* len; const uint64_t* mask; void *O, *ws; size_t bytes;
};
template <typename S>
S* state_of(PyObject* capsule) { return (S*)PyCapsule_GetPointer(capsule, nullptr); }
template <typename S>
PyObject* capsule_of(const S& s) {
    return PyCapsule_New(new S(s), nullptr, [](PyObject* c) { delete (S*)PyCapsule_GetPointer(c, nullptr); });
}
void* as_pointer(PyObject* o) {
    if (o == Py_None) return nullptr;
    void* v = PyLong_AsVoidPtr(o);
    if (!v && PyErr_Occurred()) throw PyErrSet();
    return v;
}
PyObject* run_prepared_build(PyObject* self, PyObject* stream) {
    try {
        const PreparedBuild* b = state_of<PreparedBuild>(self);
        void* s = as_pointer(stream);
        return PyLong_FromLong(without_gil([&] { return ot_build_tree(&b->p, b->logits, b->ws, b->bytes, &b->out, s); }));
    } catch (const PyErrSet&) { return nullptr; }
}
PyObject* run_prepared_attention(PyObject* self, PyObject* stream) {
    try {
        const PreparedAttention* t = state_of<PreparedAttention>(self);
        void* s = as_pointer(stream);
        return PyLong_FromLong(without_gil([&] {
            return ot_tree_verify_attention(&t->p, t->Q, t->Kp, t->Vp, t->Kt, t->Vt, t->len, t->mask, t->O, t->ws, t->bytes, s);
        }));
    } catch (const PyErrSet&) { return nullptr; }
}
PyMethodDef run_build_def = {"run", run_prepared_build, METH_O, nullptr};
PyMethodDef run_attention_def = {"run", run_prepared_attention, METH_O, nullptr};

// (logits, k, n, depth, workspace, tree) -> callable
PyObject* prepare_build(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 6);
    const at::Tensor &x = tensor(a[0]), &w = tensor(a[4]);
    const PreparedBuild b{build_params(x, as_int(a[1]), as_int(a[2]), as_int(a[3])), ptr(x), ptr(w), bytes_of(w), tree_pointers(a[5])};
    Ref c(capsule_of(b));
    return PyCFunction_New(&run_build_def, c.p);
}
// (Q, K_prefix | None, V_prefix | None, K_tree, V_tree, prefix_len, mask, out, workspace, scale) -> callable
PyObject* prepare_attention(PyObject* const* a, Py_ssize_t na) {
    want_args(na, 10);
    const at::Tensor &Q = tensor(a[0]), &Kt = tensor(a[3]), &Vt = tensor(a[4]), &O = tensor(a[7]), &w = tensor(a[8]);
    const at::Tensor *Kp = tensor_or_null(a[1]), *Vp = tensor_or_null(a[2]), *len = tensor_or_null(a[5]), *mask = tensor_or_null(a[6]);
    const PreparedAttention t{attn_params(Q, Kp, Vp, Kt, Vt, O, (float)as_double(a[9])), ptr(Q), ptr(Kp), ptr(Vp), ptr(Kt), ptr(Vt),
                              (const int32_t*)ptr(len), (const uint64_t*)ptr(mask), ptr(O), ptr(w), bytes_of(w)};
    Ref c(capsule_of(t));
    return PyCFunction_New(&run_attention_def, c.p);
}

template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    try {
        return F(args, nargs);
    } catch (const PyErrSet&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}
#define OT_METHOD(name) {#name, (PyCFunction)(void (*)(void))entry<name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {OT_METHOD(build_tree), OT_METHOD(build_tree_adaptive), OT_METHOD(stream_begin), OT_METHOD(stream_expand),
                         OT_METHOD(stream_mask), OT_METHOD(stream_esub), OT_METHOD(stream_finalize), OT_METHOD(attention),
                         OT_METHOD(attention_fp8kv), OT_METHOD(verify), OT_METHOD(kv_append), OT_METHOD(prepare_build),
                         OT_METHOD(prepare_attention), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
    auto s = [](const char* t) { return PyUnicode_InternFromString(t); };
    names = Names{s("token"), s("parent"), s("depth"), s("score"), s("mask"), s("n_out"), s("expect"), s("p"), s("step"), s("ws"),
                  s("frontier_token"), s("frontier_parent"), s("frontier_count"), s("_esub"), s("_go")};
    return PyModule_Create(&module);
}
