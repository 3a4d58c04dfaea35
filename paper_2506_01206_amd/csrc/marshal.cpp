// Argument marshalling of the Python binding (binding.py): tensor checks, output allocation and the current stream,
// then the C ABI of include/mamba_hip.h.  No computation and no HIP call of its own.
//
// Why it is native: a decode step has 17 tensors to check, and in Python every check (device, layout, dtype, shape,
// pointer) is an attribute access of its own.  Marshalled in Python and through ctypes a conv1d call costs 11 us of
// host time and a fused layer step 12 us, three times what their kernels take; here the same checks are a few
// nanoseconds each and a call costs about what the kernel launch itself does.
//
// The C functions are not linked: binding.py loads the library and hands their addresses over (bind), so that both
// always speak to the same copy of it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>
#include <string>

#include "../../include/mamba_hip.h"

namespace {

// a Python exception is already set
struct PyFailed {};

PyObject *mamba_error = nullptr;      // binding.MambaError(function name, status)
PyObject *out_of_memory = nullptr;    // torch.OutOfMemoryError

struct Api {
    decltype(&::mamba_conv1d_fwd) conv1d_fwd;
    decltype(&::mamba_scan_workspace_bytes) scan_workspace_bytes;
    decltype(&::mamba_scan_fwd) scan_fwd;
    decltype(&::mamba_state_step) state_step;
    decltype(&::mamba_conv_state_step) conv_state_step;
    decltype(&::mamba_state_fork) state_fork;
    decltype(&::mamba_linear_fwd) linear_fwd;
    decltype(&::mamba_rmsnorm_fwd) rmsnorm_fwd;
    decltype(&::mamba_block_workspace_bytes) block_workspace_bytes;
    decltype(&::mamba_block_fwd) block_fwd;
    decltype(&::mamba_block_step) block_step;
    decltype(&::mamba_embedding_fwd) embedding_fwd;
    decltype(&::mamba_topk_fwd) topk_fwd;
    decltype(&::mamba2_ssd_workspace_bytes) ssd_workspace_bytes;
    decltype(&::mamba2_ssd_fwd) ssd_fwd;
    decltype(&::mamba2_state_step) ssd_step;
} api;
constexpr Py_ssize_t kApiCount = sizeof(Api) / sizeof(void *);

typedef std::initializer_list<int64_t> Shape;

[[noreturn]] void fail(PyObject *type, const char *format, const char *name)
{
    PyErr_Format(type, format, name);
    throw PyFailed();
}

const at::Tensor &tensor(PyObject *o, const char *name)
{
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "%s must be a tensor", name);
    return THPVariable_Unpack(o);
}

// sizes of a tensor that has to have `rank` dimensions, or at least as many
at::IntArrayRef sizes(PyObject *o, const char *name, size_t rank, bool or_more = false)
{
    const at::IntArrayRef s = tensor(o, name).sizes();
    if (s.size() < rank || (s.size() > rank && !or_more)) {
        PyErr_Format(PyExc_ValueError, "%s must have %s%zu dimensions, got %zu", name, or_more ? "at least " : "", rank, s.size());
        throw PyFailed();
    }
    return s;
}

void *pointer(const at::Tensor &t) { return t.numel() > 0 ? t.data_ptr() : nullptr; }

void placed(const at::Tensor &t, const char *name)
{
    if (!t.is_cuda()) fail(PyExc_ValueError, "%s must live on the GPU", name);
    if (!t.is_contiguous()) fail(PyExc_ValueError, "%s must be contiguous", name);
}

PyObject *dtype_object(at::ScalarType type) { return reinterpret_cast<PyObject *>(torch::getTHPDtype(type)); }   // borrowed

void typed(const at::Tensor &t, at::ScalarType type, const char *name)
{
    if (t.scalar_type() != type) {
        PyErr_Format(PyExc_TypeError, "%s must be %S, got %S", name, dtype_object(type), dtype_object(t.scalar_type()));
        throw PyFailed();
    }
}

std::string text(at::IntArrayRef shape)   // as Python writes a tuple
{
    std::string s = "(";
    for (size_t i = 0; i < shape.size(); ++i) s += (i ? ", " : "") + std::to_string(shape[i]);
    return s + (shape.size() == 1 ? ",)" : ")");
}

void shaped(const at::Tensor &t, Shape shape, const char *name)
{
    const at::IntArrayRef s = t.sizes();
    if (s == at::IntArrayRef(shape)) return;
    PyErr_Format(PyExc_ValueError, "%s must have shape %s, got %s", name, text(shape).c_str(), text(s).c_str());
    throw PyFailed();
}

// device pointer of a contiguous GPU tensor (None: NULL)
void *ptr(PyObject *o, const char *name)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &t = tensor(o, name);
    placed(t, name);
    return pointer(t);
}
void *ptr(PyObject *o, at::ScalarType type, const char *name)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &t = tensor(o, name);
    placed(t, name);
    typed(t, type, name);
    return pointer(t);
}
void *ptr(PyObject *o, at::ScalarType type, Shape shape, const char *name)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &t = tensor(o, name);
    placed(t, name);
    typed(t, type, name);
    shaped(t, shape, name);
    return pointer(t);
}
float *fptr(PyObject *o, Shape shape, const char *name) { return static_cast<float *>(ptr(o, at::kFloat, shape, name)); }

int io_code(const at::Tensor &t)
{
    if (t.scalar_type() == at::kFloat) return MAMBA_F32;
    if (t.scalar_type() == at::kBFloat16) return MAMBA_BF16;
    PyErr_Format(PyExc_TypeError, "I/O tensors must be float32 or bfloat16, got %S", dtype_object(t.scalar_type()));
    throw PyFailed();
}

int64_t integer(PyObject *o)
{
    const int64_t v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw PyFailed();
    return v;
}
int flag(PyObject *o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw PyFailed();
    return v;
}

// stream: the raw stream as an int, None for the current one
void *stream_of(PyObject *o)
{
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    return reinterpret_cast<void *>(integer(o));
}

// An output: the caller's tensor, or one allocated here (then `owned` keeps it, and the result refers to it).
struct Out {
    PyObject *object;                 // borrowed (caller's tensor or None) until made
    PyObject *owned = nullptr;
    explicit Out(PyObject *o) : object(o) {}
    Out(const Out &) = delete;
    ~Out() { Py_XDECREF(owned); }
    void make(const at::Tensor &like, at::IntArrayRef shape, at::ScalarType type)
    {
        owned = THPVariable_Wrap(at::empty(shape, like.options().dtype(type)));
        if (!owned) throw PyFailed();
        object = owned;
    }
    void make(const at::Tensor &like, Shape shape, at::ScalarType type) { make(like, at::IntArrayRef(shape), type); }
    void unless_given(const at::Tensor &like, at::IntArrayRef shape, at::ScalarType type)
    {
        if (object == Py_None) make(like, shape, type);
    }
    void unless_given(const at::Tensor &like, Shape shape, at::ScalarType type) { unless_given(like, at::IntArrayRef(shape), type); }
};

// Scratch of one call.  The caching allocator may hand the block to later work on the current stream as soon as the
// call returns, so a call on another stream (`stream` given) is marshalled with the workspace binding.py allocates.
struct Workspace {
    at::Tensor own;
    void *data = nullptr;
    size_t bytes = 0;
    Workspace(PyObject *given, size_t need, const at::Tensor &like)
    {
        if (given != Py_None) {
            const at::Tensor &t = tensor(given, "workspace");
            data = ptr(given, "workspace");
            bytes = t.numel() * t.element_size();
        } else if (need > 0) {
            own = at::empty({(int64_t)(need < 16 ? 16 : need)}, like.options().dtype(at::kByte));
            data = own.data_ptr();
            bytes = (size_t)own.numel();
        }
    }
};

// Calls a function of the C ABI, the interpreter lock released meanwhile (a launch can block on a full queue), and
// raises MambaError for a status that is not zero.  A class, to be used with braces: only there are the arguments, which do
// the checks, formed in the order in which they are written (the current stream last, when all tensors are known to be the GPU's).
template <typename F, typename... A> struct Call {
    Call(const char *function, F f, A... args)
    {
        int status;
        Py_BEGIN_ALLOW_THREADS
        status = f(args...);
        Py_END_ALLOW_THREADS
        if (status == 0) return;
        PyObject *e = PyObject_CallFunction(mamba_error, "si", function, status);
        if (e) {
            PyErr_SetObject(mamba_error, e);
            Py_DECREF(e);
        }
        throw PyFailed();
    }
};

PyObject *result(PyObject *const *first, PyObject *const *last)
{
    PyObject *t = PyTuple_New((Py_ssize_t)(last - first));
    if (!t) throw PyFailed();
    for (Py_ssize_t i = 0; i < last - first; ++i) {
        Py_INCREF(first[i]);
        PyTuple_SET_ITEM(t, i, first[i]);
    }
    return t;
}
PyObject *result(std::initializer_list<PyObject *> items) { return result(items.begin(), items.end()); }

// The functions below take the arguments of binding.py's functions of the same names, all of them, by position.
typedef PyObject *const *Args;

PyObject *conv1d_fwd(Args a)
{
    PyObject *x = a[0], *w = a[1], *bias = a[2], *state_in = a[3];
    Out y(a[4]), state_out(a[5]);
    const at::Tensor &xt = tensor(x, "x");
    const auto s = sizes(x, "x", 3);
    const int64_t B = s[0], L = s[1], D = s[2], K = sizes(w, "w", 2)[1];
    const int io = io_code(xt);
    const auto type = xt.scalar_type();
    y.unless_given(xt, s, type);
    if (flag(a[7])) state_out.unless_given(xt, {B, D, K - 1}, type);
    Call{"mamba_conv1d_fwd", api.conv1d_fwd, ptr(x, "x"), fptr(w, {D, K}, "w"), fptr(bias, {D}, "bias"), ptr(state_in, type, {B, D, K - 1}, "conv_state_in"),
         ptr(y.object, type, {B, L, D}, "y"), ptr(state_out.object, type, {B, D, K - 1}, "conv_state_out"), B, L, D,
         (int)K, flag(a[6]), io, stream_of(a[8])};
    return result({y.object, state_out.object});
}

PyObject *scan_fwd(Args a)
{
    PyObject *x = a[0], *A = a[2];
    Out out(a[9]), h_final(a[10]);
    const at::Tensor &xt = tensor(x, "x");
    const auto s = sizes(x, "x", 3);
    const int64_t B = s[0], L = s[1], D = s[2], N = sizes(A, "A", 2)[1], chunk_len = integer(a[12]);
    const int io = io_code(xt);
    const auto type = xt.scalar_type();
    out.unless_given(xt, s, type);
    if (flag(a[14])) h_final.unless_given(xt, {B, D, N}, at::kFloat);
    const Workspace ws(a[11], api.scan_workspace_bytes(B, L, D, N, chunk_len), xt);
    Call{"mamba_scan_fwd", api.scan_fwd, ptr(x, "x"), ptr(a[1], type, {B, L, D}, "dt"), fptr(A, {D, N}, "A"), ptr(a[3], type, {B, L, N}, "Bm"),
         ptr(a[4], type, {B, L, N}, "Cm"), fptr(a[5], {D}, "Dskip"), ptr(a[6], type, {B, L, D}, "z"),
         fptr(a[7], {D}, "dt_bias"), fptr(a[8], {B, D, N}, "h0"), ptr(out.object, type, {B, L, D}, "out"),
         fptr(h_final.object, {B, D, N}, "h_final"), ws.data, ws.bytes, B, L, D, N, chunk_len, flag(a[13]), io,
         stream_of(a[15])};
    return result({out.object, h_final.object});
}

PyObject *state_step(Args a)
{
    PyObject *h_in = a[0], *x = a[1], *parent = a[9];
    Out h_out(a[10]), out(a[11]);
    const at::Tensor &xt = tensor(x, "x");
    const auto s = sizes(h_in, "h_in", 3);
    const int64_t n_in = s[0], D = s[1], N = s[2], n_out = sizes(x, "x", 1, true)[0];
    const int io = io_code(xt);
    const auto type = xt.scalar_type();
    h_out.unless_given(xt, {n_out, D, N}, at::kFloat);
    out.unless_given(xt, xt.sizes(), type);
    Call{"mamba_state_step", api.state_step, fptr(h_out.object, {n_out, D, N}, "h_out"), static_cast<const float *>(ptr(h_in, at::kFloat, "h_in")),
         static_cast<const int32_t *>(ptr(parent, at::kInt, {n_out}, "parent_idx")), ptr(x, "x"),
         ptr(a[2], type, {n_out, D}, "dt"), fptr(a[3], {D, N}, "A"), ptr(a[4], type, {n_out, N}, "Bm"),
         ptr(a[5], type, {n_out, N}, "Cm"), fptr(a[6], {D}, "Dskip"), ptr(a[7], type, {n_out, D}, "z"),
         fptr(a[8], {D}, "dt_bias"), ptr(out.object, type, {n_out, D}, "out"), n_out, n_in, D, N, flag(a[12]), io,
         stream_of(a[13])};
    return result({h_out.object, out.object});
}

PyObject *conv_state_step(Args a)
{
    PyObject *h_in = a[0], *conv_in = a[1], *x = a[2], *conv_w = a[3], *parent = a[12];
    Out h_out(a[13]), conv_out(a[14]), out(a[15]), xc(a[16]);
    const at::Tensor &xt = tensor(x, "x");
    const auto s = sizes(h_in, "h_in", 3);
    const int64_t n_in = s[0], D = s[1], N = s[2], n_out = sizes(x, "x", 1, true)[0], K = sizes(conv_w, "conv_w", 2)[1];
    const int io = io_code(xt);
    const auto type = xt.scalar_type();
    h_out.unless_given(xt, {n_out, D, N}, at::kFloat);
    conv_out.unless_given(xt, {n_out, D, K - 1}, type);
    out.unless_given(xt, xt.sizes(), type);
    if (flag(a[17])) xc.unless_given(xt, xt.sizes(), type);
    Call{"mamba_conv_state_step", api.conv_state_step, fptr(h_out.object, {n_out, D, N}, "h_out"), static_cast<const float *>(ptr(h_in, at::kFloat, "h_in")),
         ptr(conv_out.object, type, {n_out, D, K - 1}, "conv_state_out"),
         ptr(conv_in, type, {n_in, D, K - 1}, "conv_state_in"),
         static_cast<const int32_t *>(ptr(parent, at::kInt, {n_out}, "parent_idx")), ptr(x, "x"),
         fptr(conv_w, {D, K}, "conv_w"), fptr(a[4], {D}, "conv_bias"), ptr(a[5], type, {n_out, D}, "dt"),
         fptr(a[6], {D, N}, "A"), ptr(a[7], type, {n_out, N}, "Bm"), ptr(a[8], type, {n_out, N}, "Cm"),
         fptr(a[9], {D}, "Dskip"), ptr(a[10], type, {n_out, D}, "z"), fptr(a[11], {D}, "dt_bias"),
         ptr(out.object, type, {n_out, D}, "out"), ptr(xc.object, type, {n_out, D}, "xc_out"), n_out, n_in, D, N,
         (int)K, flag(a[18]), flag(a[19]), io, stream_of(a[20])};
    return result({h_out.object, conv_out.object, out.object, xc.object});
}

PyObject *state_fork(Args a)
{
    PyObject *conv_src = a[0], *ssm_src = a[1], *parent = a[2];
    Out conv_dst(a[3]), ssm_dst(a[4]);
    const bool has_conv = conv_src != Py_None, has_ssm = ssm_src != Py_None;
    PyObject *ref = has_conv ? conv_src : ssm_src;
    const at::Tensor &rt = tensor(ref, has_conv ? "conv_src" : "ssm_src");
    const auto s = sizes(ref, has_conv ? "conv_src" : "ssm_src", 4, true);
    const int64_t n_layers = s[0], n_in = s[1], D = s[2], n_out = sizes(parent, "parent_idx", 1, true)[0];
    int64_t K = 1, N = 0;
    int code = MAMBA_F32;
    if (has_conv) {
        K = s[3] + 1;
        code = io_code(rt);
        conv_dst.unless_given(rt, {n_layers, n_out, D, K - 1}, rt.scalar_type());
    }
    if (has_ssm) {
        N = sizes(ssm_src, "ssm_src", 4, true)[3];
        ssm_dst.unless_given(rt, {n_layers, n_out, D, N}, at::kFloat);
    }
    Call{"mamba_state_fork", api.state_fork, ptr(conv_dst.object, "conv_dst"), ptr(conv_src, "conv_src"),
         static_cast<float *>(ptr(ssm_dst.object, at::kFloat, "ssm_dst")),
         static_cast<const float *>(ptr(ssm_src, at::kFloat, "ssm_src")),
         static_cast<const int32_t *>(ptr(parent, at::kInt, "parent_idx")), n_layers, n_out, n_in, D, N, (int)K, code,
         stream_of(a[5])};
    return result({conv_dst.object, ssm_dst.object});
}

PyObject *linear_fwd(Args a)   // x, w, bias, residual, out0, width0, out1, width1, out2, width2, outputs to allocate, stream
{
    PyObject *x = a[0], *w = a[1];
    const at::Tensor &xt = tensor(x, "x");
    const auto s = sizes(x, "x", 2);
    const int64_t M = s[0], K = s[1], N = sizes(w, "w", 2)[0];
    const auto type = xt.scalar_type();
    const int io = io_code(xt);
    const int64_t n0 = integer(a[5]), n1 = integer(a[7]), n2 = integer(a[9]), allocate = integer(a[10]);
    Out o0(a[4]), o1(a[6]), o2(a[8]);
    if (allocate > 0) o0.make(xt, {M, n0}, type);                // (a negative width is refused here, or by the C function)
    if (allocate > 1) o1.make(xt, {M, n1}, type);
    if (allocate > 2) o2.make(xt, {M, n2}, type);
    Call{"mamba_linear_fwd", api.linear_fwd, ptr(x, "x"), ptr(w, type, {N, K}, "w"), fptr(a[2], {N}, "bias"), ptr(a[3], type, {M, N}, "residual"),
         ptr(o0.object, type, {M, n0}, "out0"), n0, ptr(o1.object, type, {M, n1}, "out1"), n1,
         ptr(o2.object, type, {M, n2}, "out2"), n2, M, K, io, stream_of(a[11])};
    PyObject *made[3];
    size_t count = 0;
    for (PyObject *o : {o0.object, o1.object, o2.object})
        if (o != Py_None) made[count++] = o;
    return result(made, made + count);
}

PyObject *rmsnorm_fwd(Args a)
{
    PyObject *x = a[0], *w = a[1];
    Out y(a[3]);
    const at::Tensor &xt = tensor(x, "x");
    const auto s = sizes(x, "x", 2);
    const int64_t M = s[0], C = s[1];
    const double eps = PyFloat_AsDouble(a[2]);
    if (eps == -1.0 && PyErr_Occurred()) throw PyFailed();
    y.unless_given(xt, s, xt.scalar_type());
    Call{"mamba_rmsnorm_fwd", api.rmsnorm_fwd, ptr(x, "x"), fptr(w, {C}, "w"), ptr(y.object, xt.scalar_type(), {M, C}, "y"), M, C,
         (float)eps, io_code(xt), stream_of(a[4])};
    Py_INCREF(y.object);
    return y.object;
}

const mamba_block_params_t *block_params(PyObject *address)
{
    return reinterpret_cast<const mamba_block_params_t *>(integer(address));
}

PyObject *block_fwd(Args a)   // address of the parameters, hidden, hidden_out, conv_state_in, h0, conv_state_out, h_final, workspace, want_state, stream
{
    const mamba_block_params_t *p = block_params(a[0]);
    PyObject *hidden = a[1];
    Out hidden_out(a[2]), conv_out(a[5]), h_final(a[6]);
    const at::Tensor &ht = tensor(hidden, "hidden");
    const auto s = sizes(hidden, "hidden", 3);
    const int64_t B = s[0], L = s[1], dm = s[2], D = p->d_inner, N = p->d_state, K = p->d_conv;
    hidden_out.unless_given(ht, s, ht.scalar_type());
    if (flag(a[8])) {
        conv_out.unless_given(ht, {B, D, K - 1}, ht.scalar_type());
        h_final.unless_given(ht, {B, D, N}, at::kFloat);
    }
    size_t need = api.block_workspace_bytes(p, B, L);
    const Workspace ws(a[7], need < 16 ? 16 : need, ht);
    Call{"mamba_block_fwd", api.block_fwd, p, ptr(hidden, at::kBFloat16, "hidden"), ptr(hidden_out.object, at::kBFloat16, {B, L, dm}, "hidden_out"),
         ptr(a[3], at::kBFloat16, {B, D, K - 1}, "conv_state_in"),
         ptr(conv_out.object, at::kBFloat16, {B, D, K - 1}, "conv_state_out"), fptr(a[4], {B, D, N}, "h0"),
         fptr(h_final.object, {B, D, N}, "h_final"), ws.data, ws.bytes, B, L, stream_of(a[9])};
    return result({hidden_out.object, conv_out.object, h_final.object});
}

PyObject *block_step(Args a)   // address of the parameters, hidden, conv_src, ssm_src, parent_idx, conv_dst, ssm_dst, hidden_out, workspace, stream
{
    const mamba_block_params_t *p = block_params(a[0]);
    PyObject *hidden = a[1], *conv_src = a[2], *ssm_src = a[3], *parent = a[4];
    Out conv_dst(a[5]), ssm_dst(a[6]), hidden_out(a[7]);
    const at::Tensor &ht = tensor(hidden, "hidden");
    const auto s = sizes(hidden, "hidden", 2);
    const int64_t n_out = s[0], dm = s[1], n_in = sizes(conv_src, "conv_src", 1, true)[0], D = p->d_inner, N = p->d_state, K = p->d_conv;
    hidden_out.unless_given(ht, s, ht.scalar_type());
    if (parent == Py_None) {
        conv_dst.object = conv_src;
        ssm_dst.object = ssm_src;
    } else {
        conv_dst.unless_given(ht, {n_out, D, K - 1}, tensor(conv_src, "conv_src").scalar_type());
        ssm_dst.unless_given(ht, {n_out, D, N}, at::kFloat);
    }
    size_t need = api.block_workspace_bytes(p, n_out, 1);
    const Workspace ws(a[8], need < 16 ? 16 : need, ht);
    Call{"mamba_block_step", api.block_step, p, ptr(hidden, at::kBFloat16, "hidden"), ptr(hidden_out.object, at::kBFloat16, {n_out, dm}, "hidden_out"),
         ptr(conv_src, at::kBFloat16, {n_in, D, K - 1}, "conv_src"),
         ptr(conv_dst.object, at::kBFloat16, {n_out, D, K - 1}, "conv_dst"), fptr(ssm_src, {n_in, D, N}, "ssm_src"),
         fptr(ssm_dst.object, {n_out, D, N}, "ssm_dst"),
         static_cast<const int32_t *>(ptr(parent, at::kInt, {n_out}, "parent_idx")), ws.data, ws.bytes, n_out, n_in,
         stream_of(a[9])};
    return result({hidden_out.object, conv_dst.object, ssm_dst.object});
}

PyObject *embedding_fwd(Args a)
{
    PyObject *tokens = a[0], *table = a[1];
    Out out(a[2]);
    const at::Tensor &tt = tensor(table, "table");
    const auto ts = sizes(table, "table", 2);
    const int64_t M = sizes(tokens, "tokens", 1, true)[0], V = ts[0], dm = ts[1];
    out.unless_given(tt, {M, dm}, tt.scalar_type());
    Call{"mamba_embedding_fwd", api.embedding_fwd, static_cast<const int32_t *>(ptr(tokens, at::kInt, {M}, "tokens")), ptr(table, "table"),
         ptr(out.object, tt.scalar_type(), {M, dm}, "out"), M, V, dm, io_code(tt), stream_of(a[3])};
    Py_INCREF(out.object);
    return out.object;
}

PyObject *topk_fwd(Args a)
{
    PyObject *logits = a[0];
    Out idx(a[2]), val(a[3]);
    const at::Tensor &lt = tensor(logits, "logits");
    const auto s = sizes(logits, "logits", 2);
    const int64_t M = s[0], V = s[1], k = integer(a[1]);
    idx.unless_given(lt, {M, k}, at::kInt);
    val.unless_given(lt, {M, k}, at::kFloat);
    Call{"mamba_topk_fwd", api.topk_fwd, ptr(logits, "logits"), static_cast<int32_t *>(ptr(idx.object, at::kInt, {M, k}, "idx")),
         fptr(val.object, {M, k}, "val"), M, V, (int)k, io_code(lt), stream_of(a[4])};
    return result({idx.object, val.object});
}

PyObject *ssd_fwd(Args a)
{
    PyObject *x = a[0], *Bm = a[3];
    Out out(a[9]), h_final(a[10]);
    const at::Tensor &xt = tensor(x, "x");
    const auto s = sizes(x, "x", 4);
    const int64_t B = s[0], L = s[1], H = s[2], P = s[3], N = sizes(Bm, "Bm", 3)[2];
    const auto type = xt.scalar_type();
    out.unless_given(xt, s, type);
    if (flag(a[12])) h_final.unless_given(xt, {B, H, P, N}, at::kFloat);
    size_t need = api.ssd_workspace_bytes(B, L, H, P, N);
    const Workspace ws(a[11], need < 16 ? 16 : need, xt);
    Call{"mamba2_ssd_fwd", api.ssd_fwd, ptr(x, "x"), ptr(a[1], type, {B, L, H}, "dt"), fptr(a[2], {H}, "A"), ptr(Bm, type, {B, L, N}, "Bm"),
         ptr(a[4], type, {B, L, N}, "Cm"), fptr(a[5], {H}, "Dskip"), ptr(a[6], type, {B, L, H, P}, "z"),
         fptr(a[7], {H}, "dt_bias"), fptr(a[8], {B, H, P, N}, "h0"), ptr(out.object, type, {B, L, H, P}, "out"),
         fptr(h_final.object, {B, H, P, N}, "h_final"), ws.data, ws.bytes, B, L, H, P, N, flag(a[13]), io_code(xt),
         stream_of(a[14])};
    return result({out.object, h_final.object});
}

PyObject *ssd_step(Args a)
{
    PyObject *h_in = a[0], *x = a[1], *parent = a[9];
    Out h_out(a[10]), out(a[11]);
    const at::Tensor &xt = tensor(x, "x");
    const auto s = sizes(h_in, "h_in", 4);
    const int64_t n_in = s[0], H = s[1], P = s[2], N = s[3], n_out = sizes(x, "x", 1, true)[0];
    const auto type = xt.scalar_type();
    h_out.unless_given(xt, {n_out, H, P, N}, at::kFloat);
    out.unless_given(xt, xt.sizes(), type);
    Call{"mamba2_state_step", api.ssd_step, fptr(h_out.object, {n_out, H, P, N}, "h_out"), static_cast<const float *>(ptr(h_in, at::kFloat, "h_in")),
         static_cast<const int32_t *>(ptr(parent, at::kInt, {n_out}, "parent_idx")), ptr(x, "x"),
         ptr(a[2], type, {n_out, H}, "dt"), fptr(a[3], {H}, "A"), ptr(a[4], type, {n_out, N}, "Bm"),
         ptr(a[5], type, {n_out, N}, "Cm"), fptr(a[6], {H}, "Dskip"), ptr(a[7], type, {n_out, H, P}, "z"),
         fptr(a[8], {H}, "dt_bias"), ptr(out.object, type, {n_out, H, P}, "out"), n_out, n_in, H, P, N, flag(a[12]),
         io_code(xt), stream_of(a[13])};
    return result({h_out.object, out.object});
}

// argument count, PyFailed and C++ exceptions (an allocation that fails) in one place
template <PyObject *(*F)(Args), int COUNT> PyObject *entry(PyObject *, Args args, Py_ssize_t n)
{
    if (n != COUNT) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, got %zd", COUNT, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const PyFailed &) {
        return nullptr;
    } catch (const c10::OutOfMemoryError &e) {
        PyErr_SetString(out_of_memory, e.what_without_backtrace());
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// bind(MambaError, torch.OutOfMemoryError, address, address, ...): the C functions in the order of Api
PyObject *bind(PyObject *, Args args, Py_ssize_t n)
{
    if (n != 2 + kApiCount) {
        PyErr_SetString(PyExc_TypeError, "bind: two exception classes and one address per function");
        return nullptr;
    }
    void **slot = reinterpret_cast<void **>(&api);
    for (Py_ssize_t i = 0; i < kApiCount; ++i) {
        slot[i] = PyLong_AsVoidPtr(args[2 + i]);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_INCREF(args[0]);
    Py_XSETREF(mamba_error, args[0]);
    Py_INCREF(args[1]);
    Py_XSETREF(out_of_memory, args[1]);
    Py_RETURN_NONE;
}

#define MAMBA_ENTRY(F, COUNT) {#F, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<F, COUNT>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&bind)), METH_FASTCALL, nullptr},
    MAMBA_ENTRY(conv1d_fwd, 9), MAMBA_ENTRY(scan_fwd, 16), MAMBA_ENTRY(state_step, 14), MAMBA_ENTRY(conv_state_step, 21),
    MAMBA_ENTRY(state_fork, 6), MAMBA_ENTRY(linear_fwd, 12), MAMBA_ENTRY(rmsnorm_fwd, 5), MAMBA_ENTRY(block_fwd, 10),
    MAMBA_ENTRY(block_step, 10), MAMBA_ENTRY(embedding_fwd, 4), MAMBA_ENTRY(topk_fwd, 5), MAMBA_ENTRY(ssd_fwd, 15),
    MAMBA_ENTRY(ssd_step, 14), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "argument marshalling of the mamba_hip binding", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
