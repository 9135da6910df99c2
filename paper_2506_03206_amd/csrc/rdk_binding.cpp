// CPython side of the binding: the per-step calls of the library, taken from torch tensors without ctypes.
//
// A decoding step of a small batch is a handful of launches of a few microseconds each, so the host path counts: through
// ctypes, Python attribute reads and one object per argument a call cost 10-15 us of host time before its first launch.
// Here a call reads tensor pointers, strides and dtypes from the tensor objects themselves, asks the library for the
// workspace size, and launches; nothing is kept between calls but the workspaces that the Python objects own.
// Other Python threads run while a call allocates or launches (a launch waits when the queue is full): everything that is
// taken from Python objects is taken before, and what a call uses is held by it.
//
// Every function returns the library's status as an int; argument mistakes that the Python layer used to assert raise
// AssertionError.  Positional arguments only: rdk.py holds the signatures and defaults.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "rdk.h"

namespace {

struct PyFail {};   // a Python exception is set

[[noreturn]] void fail(const char *what)
{
    PyErr_SetString(PyExc_AssertionError, what);
    throw PyFail{};
}

void need(bool ok, const char *what)
{
    if (!ok) fail(what);
}

const at::Tensor &tensor(PyObject *o, const char *what)
{
    if (!THPVariable_Check(o)) fail(what);
    return THPVariable_Unpack(o);
}

void *ptr(const at::Tensor &t) { return t.data_ptr(); }

int64_t integer(PyObject *o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw PyFail{};
    return v;
}

int32_t int32_of(PyObject *o)
{
    const int64_t v = integer(o);
    need(v >= INT32_MIN && v <= INT32_MAX, "an integer argument is out of range");
    return (int32_t)v;
}

uint64_t word(PyObject *o)   // seeds and counters: modulo 2^64, as an unsigned C argument takes them
{
    PyObject *i = PyNumber_Index(o);   // numpy integers too
    if (!i) throw PyFail{};
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) throw PyFail{};
    return v;
}

// what a [B, len] tensor holds: probabilities, or logits of its dtype
rdk_input_kind_t kind_of(const at::Tensor &t, PyObject *kind)
{
    if (PyUnicode_Check(kind) && PyUnicode_CompareWithASCIIString(kind, "prob") == 0) {
        need(t.scalar_type() == at::kFloat, "probabilities are float32");
        return RDK_PROB_F32;
    }
    if (t.scalar_type() == at::kBFloat16) return RDK_LOGIT_BF16;
    need(t.scalar_type() == at::kFloat, "logits are float32 or bfloat16");
    return RDK_LOGIT_F32;
}

int64_t rows(const at::Tensor &t)   // leading dimension of a row-major [B, len] device tensor
{
    need(t.dim() == 2 && t.stride(1) == 1 && t.is_cuda(), "rows: a two-dimensional device tensor with unit stride along its rows");
    return t.stride(0);
}

struct Rows {   // a [B, len] input
    void *p;
    rdk_input_kind_t kind;
    int64_t ld;
    Rows(const at::Tensor &t, PyObject *k) : p(ptr(t)), kind(kind_of(t, k)), ld(rows(t)) {}
};

struct Names {
    PyObject *h, *ws, *draft_ws, *fused_ws, *out_ws, *draft_ids, *accept, *alpha, *resid_mass, *resid_ids, *n_accepted, *out_tokens,
        *cand_ids, *accepted, *token, *B, *N, *gamma;
} g;

struct Ref {   // an owned reference
    PyObject *o;
    explicit Ref(PyObject *x) : o(x)
    {
        if (!x) throw PyFail{};
    }
    ~Ref() { Py_XDECREF(o); }
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
};

void *device_attr(PyObject *obj, PyObject *name)   // data pointer of a tensor attribute, NULL for None
{
    Ref a(PyObject_GetAttr(obj, name));
    if (a.o == Py_None) return nullptr;
    return ptr(tensor(a.o, "an output buffer is not a tensor"));
}

int64_t int_attr(PyObject *obj, PyObject *name)
{
    Ref a(PyObject_GetAttr(obj, name));
    return integer(a.o);
}

const rdk_kernel_t *handle(PyObject *kernel)
{
    Ref a(PyObject_GetAttr(kernel, g.h));
    return (const rdk_kernel_t *)PyLong_AsVoidPtr(a.o);
}

// Runs f without the interpreter lock; f touches no Python object.
template <class F>
auto unlocked(const F &f)
{
    struct Release {
        PyThreadState *state = PyEval_SaveThread();
        ~Release() { PyEval_RestoreThread(state); }
    } release;
    return f();
}

struct Scratch {
    at::Tensor t;   // held for the call: another thread may put a larger one in its place meanwhile
    void *p;
    size_t bytes;
};

// The uint8 tensor that `owner` keeps under `name`, replaced by a larger one when the call needs more.
Scratch workspace(PyObject *owner, PyObject *name, size_t bytes, const at::Tensor &like)
{
    {
        Ref a(PyObject_GetAttr(owner, name));
        if (a.o != Py_None) {
            const at::Tensor &t = tensor(a.o, "a workspace is not a tensor");
            if ((size_t)t.numel() >= bytes) return {t, ptr(t), (size_t)t.numel()};
        }
    }
    const at::TensorOptions opt = at::TensorOptions().dtype(at::kByte).device(like.device());
    const at::Tensor t = unlocked([&] { return at::empty({(int64_t)bytes}, opt); });
    Ref w(THPVariable_Wrap(t));
    if (PyObject_SetAttr(owner, name, w.o) != 0) throw PyFail{};
    return {t, ptr(t), bytes};
}

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

PyObject *status(rdk_status_t rc) { return PyLong_FromLong((long)rc); }

struct VerifyTargets {
    int32_t *draft_ids;
    uint8_t *accept;
    float *alpha, *resid_mass;
    int32_t *resid_ids, *n_accepted, *out_tokens;
};

VerifyTargets verify_targets(PyObject *o)
{
    VerifyTargets v;
    v.draft_ids = (int32_t *)device_attr(o, g.draft_ids);
    v.accept = (uint8_t *)device_attr(o, g.accept);
    v.alpha = (float *)device_attr(o, g.alpha);
    v.resid_mass = (float *)device_attr(o, g.resid_mass);
    v.resid_ids = (int32_t *)device_attr(o, g.resid_ids);
    v.n_accepted = (int32_t *)device_attr(o, g.n_accepted);
    v.out_tokens = (int32_t *)device_attr(o, g.out_tokens);
    return v;
}

// the verification descriptor of target rows p; the outputs must have been made for the same batch
rdk_verify_desc_t verify_desc(const at::Tensor &p, PyObject *outputs, int32_t gamma, bool sample, uint64_t seed, uint64_t offset)
{
    need(p.dim() == 2 && p.size(0) <= INT32_MAX && p.size(1) <= INT32_MAX, "p is a [B, N] tensor");
    rdk_verify_desc_t d;
    d.B = (int32_t)p.size(0);
    d.N = (int32_t)p.size(1);
    d.gamma = gamma;
    d.sample_draft = sample ? 1 : 0;
    d.seed = seed;
    d.offset = offset;
    need(int_attr(outputs, g.B) == d.B && int_attr(outputs, g.N) == d.N && int_attr(outputs, g.gamma) == gamma,
         "the outputs were made for another batch shape");
    return d;
}

template <PyObject *(*F)(PyObject *const *), Py_ssize_t COUNT>
PyObject *guarded(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != COUNT) {
        PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", COUNT, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const PyFail &) {
    } catch (const std::exception &) {   // as torch's own bindings raise it (torch.OutOfMemoryError for a workspace)
        torch::translate_exception_to_python(std::current_exception());
    }
    return nullptr;
}

// kernel, mode, p, q, seed, offset, gamma, p_kind, q_kind, sample, outputs, q_prime
PyObject *redistribute_verify(PyObject *const *a)
{
    const rdk_kernel_t *k = handle(a[0]);
    const rdk_linear_mode_t mode = (rdk_linear_mode_t)int32_of(a[1]);
    const at::Tensor &p = tensor(a[2], "p is not a tensor"), &q = tensor(a[3], "q is not a tensor");
    PyObject *o = a[10];
    const rdk_verify_desc_t d = verify_desc(p, o, int32_of(a[6]), PyObject_IsTrue(a[9]) == 1, word(a[4]), word(a[5]));
    size_t bytes = 0;
    rdk_status_t rc = rdk_redistribute_verify_workspace_bytes(k, mode, &d, &bytes);
    if (rc != RDK_OK) return status(rc);
    const Scratch w = workspace(o, g.fused_ws, bytes, p);
    float *out = nullptr;
    int64_t ldo = 0;
    if (a[11] != Py_None) {
        const at::Tensor &t = tensor(a[11], "q_prime is not a tensor");
        ldo = rows(t);
        out = (float *)ptr(t);
    }
    const VerifyTargets v = verify_targets(o);
    const Rows pi(p, a[7]), qi(q, a[8]);
    void *st = stream();
    return status(unlocked([&] {
        return rdk_redistribute_verify(k, mode, &d, pi.p, pi.kind, pi.ld, qi.p, qi.kind, qi.ld, out, ldo, v.draft_ids, v.accept, v.alpha,
                                       v.resid_mass, v.resid_ids, v.n_accepted, v.out_tokens, w.p, w.bytes, st);
    }));
}

// p, q_prime, seed, offset, gamma, p_kind, sample, outputs, use_workspace
PyObject *verify_sample(PyObject *const *a)
{
    const at::Tensor &p = tensor(a[0], "p is not a tensor");
    PyObject *o = a[7];
    const rdk_verify_desc_t d = verify_desc(p, o, int32_of(a[4]), PyObject_IsTrue(a[6]) == 1, word(a[2]), word(a[3]));
    const float *q = nullptr;
    int64_t ldq = 0;
    if (a[1] != Py_None) {
        const at::Tensor &t = tensor(a[1], "q_prime is not a tensor");
        ldq = rows(t);
        q = (const float *)ptr(t);
    }
    const VerifyTargets v = verify_targets(o);
    const Rows pi(p, a[5]);
    void *st = stream();
    if (PyObject_IsTrue(a[8]) != 1)
        return status(unlocked([&] {
            return rdk_verify_sample_static(&d, pi.p, pi.kind, pi.ld, q, ldq, v.draft_ids, v.accept, v.alpha, v.resid_mass, v.resid_ids,
                                            v.n_accepted, v.out_tokens, st);
        }));
    Ref ws(PyObject_GetAttr(o, g.out_ws));
    const at::Tensor &w = tensor(ws.o, "the workspace is not a tensor");
    void *wp = ptr(w);
    const size_t bytes = (size_t)w.numel();
    return status(unlocked([&] {
        return rdk_verify_sample(&d, pi.p, pi.kind, pi.ld, q, ldq, v.draft_ids, v.accept, v.alpha, v.resid_mass, v.resid_ids,
                                 v.n_accepted, v.out_tokens, wp, bytes, st);
    }));
}

Scratch kernel_workspace(PyObject *kernel, const rdk_kernel_t *k, int32_t B, const at::Tensor &like, rdk_status_t &rc)
{
    size_t bytes = 0;
    rc = rdk_workspace_bytes(k, B, &bytes);
    return rc == RDK_OK ? workspace(kernel, g.ws, bytes, like) : Scratch{at::Tensor(), nullptr, 0};
}

// kernel, q, q_kind, out
PyObject *redistribute_exact(PyObject *const *a)
{
    const rdk_kernel_t *k = handle(a[0]);
    const at::Tensor &q = tensor(a[1], "q is not a tensor"), &out = tensor(a[3], "out is not a tensor");
    const int64_t ldo = rows(out);
    const Rows qi(q, a[2]);
    const int32_t B = (int32_t)q.size(0);
    rdk_status_t rc;
    const Scratch w = kernel_workspace(a[0], k, B, q, rc);
    if (rc != RDK_OK) return status(rc);
    float *dst = (float *)ptr(out);
    void *st = stream();
    return status(unlocked([&] { return rdk_redistribute_exact(k, qi.p, qi.kind, qi.ld, B, dst, ldo, w.p, w.bytes, st); }));
}

// kernel, mode, q, q_kind, p, p_kind, out
PyObject *redistribute_linear(PyObject *const *a)
{
    const rdk_kernel_t *k = handle(a[0]);
    const rdk_linear_mode_t mode = (rdk_linear_mode_t)int32_of(a[1]);
    const at::Tensor &q = tensor(a[2], "q is not a tensor"), &out = tensor(a[6], "out is not a tensor");
    const int64_t ldo = rows(out);
    const Rows qi(q, a[3]);
    const int32_t B = (int32_t)q.size(0);
    const void *p = nullptr;
    rdk_input_kind_t pk = RDK_PROB_F32;
    int64_t ldp = 0;
    if (a[4] != Py_None) {
        const at::Tensor &t = tensor(a[4], "p is not a tensor");
        p = ptr(t);
        pk = kind_of(t, a[5]);
        ldp = rows(t);
    }
    rdk_status_t rc;
    const Scratch w = kernel_workspace(a[0], k, B, q, rc);
    if (rc != RDK_OK) return status(rc);
    float *dst = (float *)ptr(out);
    void *st = stream();
    return status(unlocked([&] {
        return rdk_redistribute_linear(k, mode, p, pk, ldp, qi.p, qi.kind, qi.ld, B, dst, ldo, w.p, w.bytes, st);
    }));
}

// kernel, q, seed, offset, q_kind, q_prime, draft_ids, q_draft
PyObject *sample_draft(PyObject *const *a)
{
    const rdk_kernel_t *k = handle(a[0]);
    const at::Tensor &q = tensor(a[1], "q is not a tensor");
    const Rows qi(q, a[4]);
    const int32_t B = (int32_t)q.size(0);
    size_t bytes = 0;
    const rdk_status_t rc = rdk_sample_draft_workspace_bytes(k, B, &bytes);
    if (rc != RDK_OK) return status(rc);
    const Scratch w = workspace(a[0], g.draft_ws, bytes, q);
    float *out = nullptr;
    int64_t ldo = 0;
    if (a[5] != Py_None) {
        const at::Tensor &t = tensor(a[5], "q_prime is not a tensor");
        ldo = rows(t);
        out = (float *)ptr(t);
    }
    const uint64_t seed = word(a[2]), offset = word(a[3]);
    int32_t *ids = (int32_t *)ptr(tensor(a[6], "draft_ids is not a tensor"));
    float *qd = (float *)ptr(tensor(a[7], "q_draft is not a tensor"));
    void *st = stream();
    return status(unlocked([&] {
        return rdk_sample_draft(k, qi.p, qi.kind, qi.ld, B, seed, offset, ids, qd, out, ldo, w.p, w.bytes, st);
    }));
}

// p, q_prime, C, seed, offset, p_kind, sample, outputs
PyObject *verify_multi(PyObject *const *a)
{
    const at::Tensor &p = tensor(a[0], "p is not a tensor"), &q = tensor(a[1], "q_prime is not a tensor");
    need(p.dim() == 2 && p.size(0) <= INT32_MAX && p.size(1) <= INT32_MAX, "p is a [B, N] tensor");
    PyObject *o = a[7];
    rdk_multi_desc_t d;
    d.B = (int32_t)p.size(0);
    d.N = (int32_t)p.size(1);
    d.C = int32_of(a[2]);
    d.seed = word(a[3]);
    d.offset = word(a[4]);
    d.sample_candidates = PyObject_IsTrue(a[6]) == 1 ? 1 : 0;
    const Rows pi(p, a[5]);
    size_t bytes = 0;
    const rdk_status_t rc = rdk_verify_multi_workspace_bytes(&d, pi.kind, &bytes);
    if (rc != RDK_OK) return status(rc);
    const Scratch w = workspace(o, g.out_ws, bytes, p);
    const float *qp = (const float *)ptr(q);
    const int64_t ldq = rows(q);
    int32_t *cand = (int32_t *)device_attr(o, g.cand_ids), *acc = (int32_t *)device_attr(o, g.accepted),
            *tok = (int32_t *)device_attr(o, g.token);
    float *mass = (float *)device_attr(o, g.resid_mass);
    void *st = stream();
    return status(unlocked([&] {
        return rdk_verify_multi(&d, pi.p, pi.kind, pi.ld, qp, ldq, cand, acc, tok, mass, w.p, w.bytes, st);
    }));
}

// child_node, accepted, token -> (status, n_accepted, out_tokens)
PyObject *tree_walk(PyObject *const *a)
{
    const at::Tensor &child = tensor(a[0], "child_node is not a tensor"), &acc = tensor(a[1], "accepted is not a tensor"),
                     &tok = tensor(a[2], "token is not a tensor");
    need(child.dim() == 3 && child.is_contiguous(), "child_node is a contiguous [S, nodes, C] tensor");
    const int64_t S = child.size(0), nodes = child.size(1), C = child.size(2);
    need(acc.numel() == S * nodes && tok.numel() == S * nodes, "accepted and token hold one value per node");
    need(S <= INT32_MAX && nodes <= INT32_MAX && C <= INT32_MAX, "too many trees, nodes or children");
    const at::TensorOptions opt = at::TensorOptions().dtype(at::kInt).device(child.device());
    at::Tensor n_acc, out;
    const rdk_status_t rc = unlocked([&] {
        n_acc = at::empty({S}, opt);
        out = at::empty({S, nodes}, opt);   // the walk writes every element
        return rdk_tree_walk((int32_t)S, (int32_t)nodes, (int32_t)C, (const int32_t *)ptr(child), (const int32_t *)ptr(acc),
                             (const int32_t *)ptr(tok), (int32_t *)ptr(n_acc), (int32_t *)ptr(out), stream());
    });
    PyObject *t = PyTuple_New(3);
    if (!t) throw PyFail{};
    PyTuple_SET_ITEM(t, 0, status(rc));
    PyTuple_SET_ITEM(t, 1, THPVariable_Wrap(n_acc));
    PyTuple_SET_ITEM(t, 2, THPVariable_Wrap(out));
    return t;
}

#define RDK_METHOD(NAME, COUNT) {#NAME, (PyCFunction)(void (*)(void))(&guarded<NAME, COUNT>), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {RDK_METHOD(redistribute_verify, 12), RDK_METHOD(verify_sample, 9),  RDK_METHOD(redistribute_exact, 4),
                         RDK_METHOD(redistribute_linear, 7),  RDK_METHOD(sample_draft, 8),   RDK_METHOD(verify_multi, 8),
                         RDK_METHOD(tree_walk, 3),            {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_rdk_binding", "Per-step calls of the RDK library on torch tensors.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__rdk_binding(void)
{
    PyObject **slot[] = {&g.h, &g.ws, &g.draft_ws, &g.fused_ws, &g.out_ws, &g.draft_ids, &g.accept, &g.alpha, &g.resid_mass,
                         &g.resid_ids, &g.n_accepted, &g.out_tokens, &g.cand_ids, &g.accepted, &g.token, &g.B, &g.N, &g.gamma};
    const char *name[] = {"_h", "_ws", "_draft_ws", "fused_ws", "ws", "draft_ids", "accept", "alpha", "resid_mass",
                          "resid_ids", "n_accepted", "out_tokens", "cand_ids", "accepted", "token", "B", "N", "gamma"};
    for (size_t i = 0; i < sizeof(slot) / sizeof(slot[0]); ++i) {
        *slot[i] = PyUnicode_InternFromString(name[i]);
        if (!*slot[i]) return nullptr;
    }
    return PyModule_Create(&module);
}
