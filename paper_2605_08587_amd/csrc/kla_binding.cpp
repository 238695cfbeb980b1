// The launching half of the Python binding: checks the tensors of a call, allocates what the caller did not pass, and
// calls the C ABI on the current stream, without going through Python objects for every pointer and extent.  A decode step
// of one sequence is 4 us of kernel; marshalled in Python its call cost the host 13 us.
//
// Every entry returns None for arguments it does not take (wrong extents or types, tensors that are not plain dense GPU
// tensors, subclasses): the Python code then goes through the same call step by step and raises what there is to raise.
// A refusal by the library itself comes back as its status code (an int).  The functions are called through the addresses
// that bind() was given, so that they are those of the library the package has loaded.
#include <Python.h>

#include <pybind11/pybind11.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <climits>
#include <initializer_list>
#include <optional>

#include "../../include/kla.h"

namespace {

struct Api {
    decltype(&kla_decode_step_opts) decode;
    decltype(&kla_decode_step_diag_opts) decode_diag;
    decltype(&kla_chunk_fwd_workspace_bytes_opts) fwd_bytes;
    decltype(&kla_chunk_fwd_opts) fwd;
    decltype(&kla_chunk_fwd_diag_workspace_bytes) fwd_diag_bytes;
    decltype(&kla_chunk_fwd_diag_opts) fwd_diag;
    decltype(&kla_chunk_bwd_workspace_bytes_opts) bwd_bytes;
    decltype(&kla_chunk_bwd_opts) bwd;
    decltype(&kla_chunk_saved_bytes) saved_bytes;
    decltype(&kla_chunk_fwd_save) fwd_save;
    decltype(&kla_chunk_bwd_saved_workspace_bytes) bwd_saved_bytes;
    decltype(&kla_chunk_bwd_saved) bwd_saved;
    PyObject* bwd_by_steps;                              // the Python module's function for a backward that is not taken here
} api = {};

// A plain, dense tensor: torch.Tensor or Parameter itself, strided and contiguous, with memory of its own.  (What
// function transforms and fake modes pass around is not.)
const at::Tensor* dense(const at::Tensor& t)
{
    if (!t.defined() || t.layout() != at::kStrided) return nullptr;
    const c10::TensorImpl* impl = t.unsafeGetTensorImpl();
    const c10::DispatchKeySet ks = impl->key_set();
    if (!impl->has_storage() || impl->is_python_dispatch() || ks.has(c10::DispatchKey::FuncTorchBatched) ||
        ks.has(c10::DispatchKey::FuncTorchGradWrapper) || ks.has(c10::DispatchKey::Functionalize))
        return nullptr;
    return t.is_contiguous() ? &t : nullptr;
}
const at::Tensor* dense(PyObject* o) { return THPVariable_CheckExact(o) ? dense(THPVariable_Unpack(o)) : nullptr; }
template <typename O> const at::Tensor* on_gpu(const O& o)
{
    const at::Tensor* t = dense(o);
    return t && t->is_cuda() ? t : nullptr;
}
// GPU tensor of this element type and these extents
template <typename O> const at::Tensor* gpu(const O& o, at::ScalarType type, at::IntArrayRef shape)
{
    const at::Tensor* t = on_gpu(o);
    return t && t->scalar_type() == type && t->sizes() == shape ? t : nullptr;
}
bool is_none(PyObject* o) { return o == Py_None; }
bool is_none(const at::Tensor& t) { return !t.defined(); }
// the same, or None (then *t stays null); false: neither
template <typename O> bool gpu_or_none(const O& o, at::ScalarType type, at::IntArrayRef shape, const at::Tensor** t)
{
    *t = nullptr;
    if (is_none(o)) return true;
    *t = gpu(o, type, shape);
    return *t != nullptr;
}
// What a forward left behind for the backward of q: bytes on q's device, or none (then *t stays null); false: something else.
// (It comes back through the caller's hands, a hook on saved tensors, and goes to the kernels as a bare pointer.)
template <typename O> bool saved_or_none(const O& o, const at::Tensor& q, const at::Tensor** t)
{
    *t = nullptr;
    if (is_none(o)) return true;
    *t = on_gpu(o);
    return *t && (*t)->scalar_type() == at::kByte && (*t)->device() == q.device();
}
void* ptr(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }
float* fptr(const at::Tensor* t) { return static_cast<float*>(ptr(t)); }

bool type_of(const at::Tensor& q, kla_dtype* dt)
{
    if (q.scalar_type() == at::kBFloat16) *dt = KLA_BF16;
    else if (q.scalar_type() == at::kFloat) *dt = KLA_F32;
    else return false;
    return true;
}
bool number(PyObject* o, double* x)
{
    *x = PyFloat_AsDouble(o);
    if (*x == -1.0 && PyErr_Occurred()) { PyErr_Clear(); return false; }
    return true;
}
bool integer(PyObject* o, long lo, long hi, long* x)
{
    *x = PyLong_AsLong(o);
    if (*x == -1 && PyErr_Occurred()) { PyErr_Clear(); return false; }
    return *x >= lo && *x <= hi;
}
bool ints(std::initializer_list<int64_t> xs)
{
    for (const int64_t x : xs) if (x > INT_MAX) return false;
    return true;
}
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }
// Other threads run while a call allocates and launches (and get their turn back if it throws).
struct NoGil {
    PyThreadState* state = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(state); }
};
PyObject* wrap(const std::optional<at::Tensor>& t)
{
    if (t) return THPVariable_Wrap(*t);
    Py_RETURN_NONE;
}

// What the chunk entry points share.
struct Chunk {
    const at::Tensor *q, *k, *v, *la, *eta, *h0, *cu;
    const int32_t* cu_host;
    int64_t N, T, H, dk, dv, n_states;
    int n_seq;
    double eps;
    kla_dtype dt;
    at::ScalarType type;

    // args: q, k, v, log_alpha, eta, eps, h0, cu_seqlens, cu_seqlens_host
    bool take(PyObject* const* a, bool diag)
    {
        double e;
        return number(a[5], &e) && take(a[0], a[1], a[2], a[3], a[4], a[6], a[7], a[8], e, diag);
    }
    // the same of Python objects (None: not given) or of tensors (undefined: not given)
    template <typename O>
    bool take(const O& q_, const O& k_, const O& v_, const O& la_, const O& eta_, const O& h0_, const O& cu_, const O& host_, double eps_,
              bool diag = false)
    {
        eps = eps_;
        q = on_gpu(q_); v = on_gpu(v_);
        if (!q || !v || q->dim() != 4 || v->dim() != 4 || !type_of(*q, &dt)) return false;
        type = q->scalar_type();
        N = q->size(0); T = q->size(1); H = q->size(2); dk = q->size(3); dv = v->size(3);
        if (!ints({N, T, H, dk, dv}) || v->scalar_type() != type || v->sizes() != at::IntArrayRef({N, T, H, dv})) return false;
        k = gpu(k_, type, q->sizes());
        la = diag ? gpu(la_, at::kFloat, q->sizes()) : gpu(la_, at::kFloat, {N, T, H});
        eta = gpu(eta_, at::kFloat, {N, T, H});
        if (!k || !la || !eta) return false;
        cu = nullptr; cu_host = nullptr; n_seq = 0; n_states = N;
        if (!is_none(cu_)) {
            cu = on_gpu(cu_);
            const at::Tensor* c = dense(host_);
            if (!cu || !c || !c->is_cpu() || cu->scalar_type() != at::kInt || c->scalar_type() != at::kInt || cu->dim() != 1 ||
                c->dim() != 1 || cu->numel() != c->numel() || cu->numel() < 2 || cu->numel() > INT_MAX)
                return false;
            cu_host = static_cast<const int32_t*>(c->data_ptr());
            n_seq = (int)cu->numel() - 1;
            n_states = n_seq;
        } else if (!is_none(host_)) return false;
        return gpu_or_none(h0_, at::kFloat, {n_states, H, dk, dv}, &h0);
    }
    at::Tensor empty(at::IntArrayRef shape, at::ScalarType t) const { return at::empty(shape, q->options().dtype(t).requires_grad(false)); }
};

PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 13 || !PyCallable_Check(a[12])) { PyErr_SetString(PyExc_TypeError, "bind takes twelve addresses and a function"); return nullptr; }
    void* p[12];
    for (int i = 0; i < 12; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address"); return nullptr; }
    }
    api.decode = reinterpret_cast<decltype(api.decode)>(p[0]);
    api.decode_diag = reinterpret_cast<decltype(api.decode_diag)>(p[1]);
    api.fwd_bytes = reinterpret_cast<decltype(api.fwd_bytes)>(p[2]);
    api.fwd = reinterpret_cast<decltype(api.fwd)>(p[3]);
    api.fwd_diag_bytes = reinterpret_cast<decltype(api.fwd_diag_bytes)>(p[4]);
    api.fwd_diag = reinterpret_cast<decltype(api.fwd_diag)>(p[5]);
    api.bwd_bytes = reinterpret_cast<decltype(api.bwd_bytes)>(p[6]);
    api.bwd = reinterpret_cast<decltype(api.bwd)>(p[7]);
    api.saved_bytes = reinterpret_cast<decltype(api.saved_bytes)>(p[8]);
    api.fwd_save = reinterpret_cast<decltype(api.fwd_save)>(p[9]);
    api.bwd_saved_bytes = reinterpret_cast<decltype(api.bwd_saved_bytes)>(p[10]);
    api.bwd_saved = reinterpret_cast<decltype(api.bwd_saved)>(p[11]);
    Py_INCREF(a[12]);
    Py_XDECREF(api.bwd_by_steps);
    api.bwd_by_steps = a[12];
    Py_RETURN_NONE;
}

// decode(q, k, v, log_alpha, eta, eps, S, out, opts, diag) -> out
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 10 || !api.decode) Py_RETURN_NONE;
    const bool diag = a[9] == Py_True;
    const at::Tensor *q = on_gpu(a[0]), *v = on_gpu(a[2]);
    kla_dtype dt;
    double eps;
    long opts;
    if (!q || !v || q->dim() != 3 || v->dim() != 3 || !type_of(*q, &dt) || !number(a[5], &eps) || !integer(a[8], 0, UINT_MAX, &opts))
        Py_RETURN_NONE;
    const int64_t B = q->size(0), H = q->size(1), dk = q->size(2), dv = v->size(2);
    const at::ScalarType type = q->scalar_type();
    const at::Tensor *k = gpu(a[1], type, q->sizes()), *eta = gpu(a[4], at::kFloat, {B, H}), *S = gpu(a[6], at::kFloat, {B, H, dk, dv});
    const at::Tensor* la = diag ? gpu(a[3], at::kFloat, q->sizes()) : gpu(a[3], at::kFloat, {B, H});
    const at::Tensor* out = nullptr;
    if (!ints({B, H, dk, dv}) || !k || !eta || !S || !la || v->scalar_type() != type || v->sizes() != at::IntArrayRef({B, H, dv}) ||
        !gpu_or_none(a[7], type, {B, H, dv}, &out))
        Py_RETURN_NONE;
    at::Tensor o;
    int rc;
    {
        const NoGil no_gil;
        o = out ? *out : at::empty({B, H, dv}, q->options().requires_grad(false));
        rc = (diag ? api.decode_diag : api.decode)(ptr(q), ptr(k), ptr(v), fptr(la), fptr(eta), (float)eps, fptr(S), o.data_ptr(), (int)B,
                                                   (int)H, (int)dk, (int)dv, dt, stream(), (unsigned)opts);
    }
    if (rc != KLA_OK) return PyLong_FromLong(rc);
    return THPVariable_Wrap(o);
    END_HANDLE_TH_ERRORS
}

// chunk_fwd(q, k, v, log_alpha, eta, eps, h0, cu_seqlens, cu_seqlens_host, want_hT, workspace, out, hT, chunk, opts, diag)
// -> (out, hT)
PyObject* chunk_fwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 16 || !api.fwd) Py_RETURN_NONE;
    const bool diag = a[15] == Py_True, want_hT = a[9] == Py_True;
    Chunk c;
    long chunk, opts;
    if (!c.take(a, diag) || !integer(a[13], INT_MIN, INT_MAX, &chunk) || !integer(a[14], 0, UINT_MAX, &opts)) Py_RETURN_NONE;
    const at::Tensor *out_ = nullptr, *hT_ = nullptr, *ws_ = nullptr;
    if (!gpu_or_none(a[11], c.type, {c.N, c.T, c.H, c.dv}, &out_) || !gpu_or_none(a[12], at::kFloat, {c.n_states, c.H, c.dk, c.dv}, &hT_))
        Py_RETURN_NONE;
    if (a[10] != Py_None && !(ws_ = on_gpu(a[10]))) Py_RETURN_NONE;
    const int N = (int)c.N, T = (int)c.T, H = (int)c.H, dk = (int)c.dk, dv = (int)c.dv;
    std::optional<at::Tensor> out, hT;
    at::Tensor ws;
    int rc;
    {
        const NoGil no_gil;
        if (ws_) ws = *ws_;
        else {
            const size_t need = diag ? api.fwd_diag_bytes(N, T, H, dk, dv, (int)chunk, c.dt, c.cu_host, c.n_seq)
                                     : api.fwd_bytes(N, T, H, dk, dv, (int)chunk, c.dt, c.cu_host, c.n_seq, (unsigned)opts & ~3u);
            ws = c.empty({(int64_t)(need < 256 ? 256 : need)}, at::kByte);
        }
        out = out_ ? *out_ : c.empty({c.N, c.T, c.H, c.dv}, c.type);
        if (hT_) hT = *hT_;
        else if (want_hT) hT = c.empty({c.n_states, c.H, c.dk, c.dv}, at::kFloat);
        rc = (diag ? api.fwd_diag : api.fwd)(ptr(c.q), ptr(c.k), ptr(c.v), fptr(c.la), fptr(c.eta), (float)c.eps, fptr(c.h0),
                                             out->data_ptr(), hT ? static_cast<float*>(hT->data_ptr()) : nullptr,
                                             static_cast<const int32_t*>(ptr(c.cu)), c.cu_host, c.n_seq, N, T, H, dk, dv, (int)chunk,
                                             c.dt, ws.data_ptr(), ws.nbytes(), stream(), (unsigned)opts);
    }
    if (rc != KLA_OK) return PyLong_FromLong(rc);
    PyObject* r = PyTuple_New(2);
    if (!r) return nullptr;
    PyTuple_SET_ITEM(r, 0, wrap(out));
    PyTuple_SET_ITEM(r, 1, wrap(hT));
    return r;
    END_HANDLE_TH_ERRORS
}

// The gradients dq, dk, dv, dlog_alpha, deta, dh0 (if wanted), all of them new, and the status of the call.  saved: what a forward with
// the same arguments left behind, or null.
int run_bwd(const Chunk& c, const at::Tensor& d_o, const at::Tensor* d_hT, const at::Tensor* saved, bool want_dh0, int chunk, unsigned opts,
            at::Tensor (&g)[6])
{
    const int N = (int)c.N, T = (int)c.T, H = (int)c.H, dk = (int)c.dk, dv = (int)c.dv;
    const size_t need = (saved ? api.bwd_saved_bytes : api.bwd_bytes)(N, T, H, dk, dv, chunk, c.dt, c.cu_host, c.n_seq, opts & ~3u);
    const at::Tensor ws = c.empty({(int64_t)(need < 256 ? 256 : need)}, at::kByte);
    g[0] = c.empty(c.q->sizes(), c.type);
    g[1] = c.empty(c.q->sizes(), c.type);
    g[2] = c.empty(c.v->sizes(), c.type);
    g[3] = c.empty({c.N, c.T, c.H}, at::kFloat);
    g[4] = c.empty({c.N, c.T, c.H}, at::kFloat);
    if (want_dh0) g[5] = c.empty({c.n_states, c.H, c.dk, c.dv}, at::kFloat);
    float *g_la = static_cast<float*>(g[3].data_ptr()), *g_eta = static_cast<float*>(g[4].data_ptr());
    float* g_h0 = want_dh0 ? static_cast<float*>(g[5].data_ptr()) : nullptr;
    const int32_t* cu = static_cast<const int32_t*>(ptr(c.cu));
    if (saved)
        return api.bwd_saved(ptr(c.q), ptr(c.k), ptr(c.v), fptr(c.la), fptr(c.eta), (float)c.eps, fptr(c.h0), d_o.data_ptr(), fptr(d_hT),
                             g[0].data_ptr(), g[1].data_ptr(), g[2].data_ptr(), g_la, g_eta, g_h0, cu, c.cu_host, c.n_seq, N, T, H, dk, dv,
                             chunk, c.dt, ws.data_ptr(), ws.nbytes(), ptr(saved), saved->nbytes(), stream(), opts);
    return api.bwd(ptr(c.q), ptr(c.k), ptr(c.v), fptr(c.la), fptr(c.eta), (float)c.eps, fptr(c.h0), d_o.data_ptr(), fptr(d_hT),
                   g[0].data_ptr(), g[1].data_ptr(), g[2].data_ptr(), g_la, g_eta, g_h0, cu, c.cu_host, c.n_seq, N, T, H, dk, dv, chunk, c.dt,
                   ws.data_ptr(), ws.nbytes(), stream(), opts);
}

// chunk_bwd(q, k, v, log_alpha, eta, eps, h0, cu_seqlens, cu_seqlens_host, d_o, d_hT, want_dh0, chunk, opts, saved)
// -> (dq, dk, dv, dlog_alpha, deta, dh0)
PyObject* chunk_bwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 15 || !api.bwd) Py_RETURN_NONE;
    const bool want_dh0 = a[11] == Py_True;
    Chunk c;
    long chunk, opts;
    if (!c.take(a, false) || !integer(a[12], INT_MIN, INT_MAX, &chunk) || !integer(a[13], 0, UINT_MAX, &opts)) Py_RETURN_NONE;
    const at::Tensor *d_o = gpu(a[9], c.type, {c.N, c.T, c.H, c.dv}), *d_hT = nullptr, *saved = nullptr;
    if (!d_o || !gpu_or_none(a[10], at::kFloat, {c.n_states, c.H, c.dk, c.dv}, &d_hT)) Py_RETURN_NONE;
    if (!saved_or_none(a[14], *c.q, &saved)) Py_RETURN_NONE;
    at::Tensor g[6];
    int rc;
    {
        const NoGil no_gil;
        rc = run_bwd(c, *d_o, d_hT, saved, want_dh0, (int)chunk, (unsigned)opts, g);
    }
    if (rc != KLA_OK) return PyLong_FromLong(rc);
    PyObject* r = PyTuple_New(6);
    if (!r) return nullptr;
    for (int i = 0; i < 6; ++i) PyTuple_SET_ITEM(r, i, g[i].defined() ? THPVariable_Wrap(g[i]) : Py_NewRef(Py_None));
    return r;
    END_HANDLE_TH_ERRORS
}

// ---- kla_chunk: the two directions as one node of the autograd graph -------------------------------------------------------
// What _KlaChunk of the Python module does, without Python in it: the engine runs a backward on a thread of its own, which would
// have to wait for the interpreter twice.  A step of 2 x 35 tokens, 8 heads (30 us of kernels) 119 -> 57 us.
struct Refused { int code; };                            // by the library, in the forward: handed back as its status code

struct KlaChunk : public torch::autograd::Function<KlaChunk> {
    // c: of these very tensors
    static torch::autograd::variable_list forward(torch::autograd::AutogradContext* ctx, const at::Tensor& q, const at::Tensor& k,
                                                  const at::Tensor& v, const at::Tensor& la, const at::Tensor& eta,
                                                  const std::optional<at::Tensor>& h0,
                                                  const Chunk* c, const at::Tensor* cu_host, int64_t opts, bool wanted, bool save)
    {
        const int N = (int)c->N, T = (int)c->T, H = (int)c->H, dk = (int)c->dk, dv = (int)c->dv, chunk = 64;
        const size_t need = api.fwd_bytes(N, T, H, dk, dv, chunk, c->dt, c->cu_host, c->n_seq, (unsigned)opts & ~3u);
        const size_t keep = wanted && save ? api.saved_bytes(N, T, H, dk, dv, chunk, c->dt, c->cu_host, c->n_seq, (unsigned)opts) : 0;
        const at::Tensor ws = c->empty({(int64_t)(need < 256 ? 256 : need)}, at::kByte);
        const at::Tensor out = c->empty({c->N, c->T, c->H, c->dv}, c->type), hT = c->empty({c->n_states, c->H, c->dk, c->dv}, at::kFloat);
        at::Tensor saved;
        if (keep) {
            // no memory for it: the backward recomputes
            try { saved = c->empty({(int64_t)keep}, at::kByte); } catch (const c10::OutOfMemoryError&) {}
        }
        const int32_t* cu = static_cast<const int32_t*>(ptr(c->cu));
        float* h = static_cast<float*>(hT.data_ptr());
        const int rc = saved.defined()
            ? api.fwd_save(ptr(&q), ptr(&k), ptr(&v), fptr(&la), fptr(&eta), (float)c->eps, fptr(c->h0), out.data_ptr(), h, cu, c->cu_host,
                           c->n_seq, N, T, H, dk, dv, chunk, c->dt, ws.data_ptr(), ws.nbytes(), saved.data_ptr(), keep, stream(), (unsigned)opts)
            : api.fwd(ptr(&q), ptr(&k), ptr(&v), fptr(&la), fptr(&eta), (float)c->eps, fptr(c->h0), out.data_ptr(), h, cu, c->cu_host,
                      c->n_seq, N, T, H, dk, dv, chunk, c->dt, ws.data_ptr(), ws.nbytes(), stream(), (unsigned)opts);
        if (rc != KLA_OK) throw Refused{rc};
        if (wanted) {
            ctx->save_for_backward({q, k, v, la, eta, h0 ? *h0 : at::Tensor(), saved});
            ctx->set_materialize_grads(false);           // the library takes a missing d_hT for zeros
            ctx->saved_data["eps"] = c->eps;
            ctx->saved_data["opts"] = opts;
            if (c->cu) {
                // The plan of the backward and what the forward leaves behind are for these offsets: a host copy of our own (the
                // caller may fill its own anew), and the device's unchanged (an inference tensor does not count its changes)
                const at::Tensor cu = c->cu->is_inference() ? c->cu->clone() : *c->cu;
                ctx->saved_data["cu"] = cu;
                ctx->saved_data["cu_version"] = (int64_t)cu._version();
                ctx->saved_data["cu_host"] = cu_host->clone();
            }
        }
        return {out, hT};
    }

    static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx, torch::autograd::variable_list grads)
    {
        const torch::autograd::variable_list s = ctx->get_saved_variables();
        const auto cu = ctx->saved_data.find("cu");
        at::Tensor cu_dev, cu_host;
        if (cu != ctx->saved_data.end()) {
            cu_dev = cu->second.toTensor();
            cu_host = ctx->saved_data["cu_host"].toTensor();
            TORCH_CHECK((int64_t)cu_dev._version() == ctx->saved_data["cu_version"].toInt(),
                        "one of the variables needed for gradient computation has been modified by an inplace operation: cu_seqlens");
        }
        const double eps = ctx->saved_data["eps"].toDouble();
        const int64_t opts = ctx->saved_data["opts"].toInt();
        const bool want_dh0 = s[5].defined() && ctx->needs_input_grad(5);
        const at::Tensor d_o = grads[0].defined() ? grads[0].contiguous() : at::zeros_like(s[2]);
        const at::Tensor d_hT = grads[1].defined() ? grads[1].contiguous() : at::Tensor();
        Chunk c;
        const at::Tensor *saved, *state_grad;
        at::Tensor g[6];
        // (a hook on saved tensors may hand back others than it was given)
        if (!c.take(s[0], s[1], s[2], s[3], s[4], s[5], cu_dev, cu_host, eps) || !saved_or_none(s[6], *c.q, &saved) ||
            !gpu(d_o, c.type, c.v->sizes()) || !gpu_or_none(d_hT, at::kFloat, {c.n_states, c.H, c.dk, c.dv}, &state_grad) ||
            run_bwd(c, d_o, state_grad, saved, want_dh0, 64, (unsigned)opts, g) != KLA_OK)
            by_steps({s[0], s[1], s[2], s[3], s[4], d_o, s[5], d_hT, cu_dev, cu_host, s[6]}, eps, opts, want_dh0, g);
        return {g[0], g[1], g[2], g[3], g[4], g[5], at::Tensor(), at::Tensor(), at::Tensor(), at::Tensor(), at::Tensor()};
    }

    // A backward that is not taken here, or that the library refuses: the Python function goes through it step by step and raises
    // what there is to raise.  t (undefined: None): q, k, v, log_alpha, eta, d_o, h0, d_hT, the offsets, their host copy, saved
    static void by_steps(std::initializer_list<at::Tensor> t, double eps, int64_t opts, bool want_dh0, at::Tensor (&g)[6])
    {
        const pybind11::gil_scoped_acquire gil;
        pybind11::list args;
        for (const at::Tensor& x : t) {
            PyObject* o = THPVariable_Wrap(x);
            if (!o) raise();
            args.append(pybind11::reinterpret_steal<pybind11::object>(o));
        }
        const auto r = pybind11::reinterpret_steal<pybind11::object>(
            PyObject_CallFunction(api.bwd_by_steps, "OdLO", args.ptr(), eps, (long long)opts, want_dh0 ? Py_True : Py_False));
        if (!r) raise();
        if (!PyTuple_Check(r.ptr()) || PyTuple_GET_SIZE(r.ptr()) != 6) { PyErr_SetString(PyExc_TypeError, "kla_chunk_bwd: six gradients"); raise(); }
        for (int i = 0; i < 6; ++i) {
            PyObject* o = PyTuple_GET_ITEM(r.ptr(), i);
            g[i] = THPVariable_Check(o) ? at::Tensor(THPVariable_Unpack(o)) : at::Tensor();
        }
    }
    // the Python error there is, for the thread that called the engine
    [[noreturn]] static void raise()
    {
        python_error e;
        e.persist();
        throw e;
    }
};

// train(q, k, v, log_alpha, eta, eps, h0, cu_seqlens, cu_seqlens_host, opts, save) -> (out, hT), differentiable
PyObject* train(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 11 || !api.fwd_save) Py_RETURN_NONE;
    const bool save = a[10] == Py_True;
    Chunk c;
    long opts;
    if (!c.take(a, false) || !integer(a[9], 0, UINT_MAX, &opts)) Py_RETURN_NONE;
    torch::autograd::variable_list r;
    try {
        const NoGil no_gil;
        bool wanted = c.h0 && c.h0->requires_grad();
        for (const at::Tensor* t : {c.q, c.k, c.v, c.la, c.eta}) wanted = wanted || t->requires_grad();
        r = KlaChunk::apply(*c.q, *c.k, *c.v, *c.la, *c.eta, c.h0 ? std::optional<at::Tensor>(*c.h0) : std::nullopt, &c, c.cu ? &THPVariable_Unpack(a[8]) : nullptr,
                            (int64_t)opts, wanted, save);
    } catch (const Refused& e) {
        return PyLong_FromLong(e.code);
    }
    PyObject* t = PyTuple_New(2);
    if (!t) return nullptr;
    for (int i = 0; i < 2; ++i) PyTuple_SET_ITEM(t, i, THPVariable_Wrap(r[i]));
    return t;
    END_HANDLE_TH_ERRORS
}

#define KLA_FASTCALL(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {KLA_FASTCALL(bind), KLA_FASTCALL(decode), KLA_FASTCALL(chunk_fwd), KLA_FASTCALL(chunk_bwd),
                         KLA_FASTCALL(train), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "kla_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_kla_binding()
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) < 0) Py_CLEAR(m);   // whose tensors it can read
    return m;
}
