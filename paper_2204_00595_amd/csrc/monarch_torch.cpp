// Host path of the Python binding: argument checks, output and scratch allocation, the stream, the call into the C
// ABI, and the autograd node, in one native module (_native.so).  No arithmetic and no kernels here.
//
// Why native: a training step of one layer enqueues six kernels of 3 to 30 us; with the marshalling in Python
// (ctypes, a torch.autograd.Function, a dozen torch calls) the host needed 200 us for it, more than the GPU for every
// batch up to about 32768 rows of 768 features.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/core/LegacyTypeDispatch.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/core/Allocator.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/StreamGuard.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cmath>

#include "../../include/monarch.h"

namespace {

using at::Tensor;

PyObject* g_error = nullptr;  // binding.MonarchError

// With or without the GIL (the backward runs on an autograd thread): raises binding.MonarchError(status, where).
[[noreturn]] void raise_status(int status, const char* where)
{
    const PyGILState_STATE gil = PyGILState_Ensure();
    PyObject* e = g_error ? PyObject_CallFunction(g_error, "is", status, where) : nullptr;
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    } else if (!PyErr_Occurred()) {
        PyErr_Format(PyExc_RuntimeError, "%s failed: %d (%s)", where, status, monarch_status_string(status));
    }
    python_error err;
    err.persist();
    PyGILState_Release(gil);
    throw err;
}

// ---- arguments ----

Tensor tensor_arg(PyObject* o, const char* name)
{
    TORCH_CHECK_TYPE(THPVariable_Check(o), name, " must be a tensor, got ", Py_TYPE(o)->tp_name);
    return THPVariable_Unpack(o);
}
Tensor optional_arg(PyObject* o, const char* name) { return o == Py_None ? Tensor() : tensor_arg(o, name); }

unsigned flags_arg(PyObject* o)
{
    const unsigned long v = PyLong_AsUnsignedLongMask(o);
    if (v == (unsigned long)-1 && PyErr_Occurred()) throw python_error();
    return (unsigned)v;
}
bool bool_arg(PyObject* o) { return PyObject_IsTrue(o) == 1; }

// the `stream` argument of a call: None, or a torch.cuda.Stream
struct StreamArg {
    void* raw = nullptr;
    c10::optional<c10::Stream> torch;
};
int64_t int_attr(PyObject* o, const char* name)
{
    PyObject* a = PyObject_GetAttrString(o, name);
    if (!a) throw python_error();
    const long long v = PyLong_AsLongLong(a);
    Py_DECREF(a);
    if (v == -1 && PyErr_Occurred()) throw python_error();
    return v;
}
StreamArg stream_arg(PyObject* o)
{
    StreamArg s;
    if (o == Py_None) return s;
    s.raw = reinterpret_cast<void*>(int_attr(o, "cuda_stream"));
    s.torch = c10::Stream::unpack3(int_attr(o, "stream_id"), (c10::DeviceIndex)int_attr(o, "device_index"),
                                   (c10::DeviceType)int_attr(o, "device_type"));
    return s;
}

void check(const Tensor& t, const char* name, at::IntArrayRef shape, at::ScalarType dtype, c10::Device device)
{
    TORCH_CHECK_VALUE(t.is_cuda() && t.device() == device, name, " must live on ", device);
    TORCH_CHECK_TYPE(t.scalar_type() == dtype, name, ": dtype ", t.scalar_type(), ", expected ", dtype);
    TORCH_CHECK_VALUE(t.sizes() == shape, name, ": shape ", t.sizes(), ", expected ", shape);
    TORCH_CHECK_VALUE(t.is_contiguous(), name, " must be contiguous");
}

// The shape of a multiply, read off its operands: R (k, q, p), L (k, s, q), `rows` (batch, ...).
struct Shape {
    int64_t B = 0, k = 0, p = 0, q = 0, s = 0;
    at::ScalarType dtype;
    c10::Device device;
    Shape(const Tensor& rows, const Tensor& R, const Tensor& L) : dtype(rows.scalar_type()), device(rows.device())
    {
        TORCH_CHECK_VALUE(R.dim() == 3 && L.dim() == 3, "R and L must have three dimensions");
        TORCH_CHECK_VALUE(rows.dim() >= 1, "the operand must have a batch dimension");
        B = rows.size(0);
        k = R.size(0);
        q = R.size(1);
        p = R.size(2);
        s = L.size(1);
    }
    int64_t n_in() const { return k * p; }
    int64_t n_out() const { return k * s; }
    monarch_dtype code() const
    {
        TORCH_CHECK_TYPE(dtype == at::kFloat || dtype == at::kBFloat16, "dtype must be float32 or bfloat16, got ", dtype);
        return dtype == at::kFloat ? MONARCH_F32 : MONARCH_BF16;
    }
    void check_factors(const Tensor& R, const Tensor& L) const
    {
        check(R, "R", {k, q, p}, dtype, device);
        check(L, "L", {k, s, q}, dtype, device);
    }
};

Tensor make(at::IntArrayRef shape, at::ScalarType dtype, c10::Device device)
{
    return at::empty(shape, at::TensorOptions().dtype(dtype).device(device));
}
// the caller's buffer, checked, or a new one
Tensor out(Tensor t, const char* name, at::IntArrayRef shape, at::ScalarType dtype, c10::Device device)
{
    if (!t.defined()) return make(shape, dtype, device);
    check(t, name, shape, dtype, device);
    return t;
}

// Where a call runs: its device made current, the raw stream.  Scratch the call allocates itself belongs to that
// stream (the caching allocator hands its block, once released, only to later work of that same stream).
struct Where {
    at::AutoDispatchBelowADInplaceOrView below;
    c10::DeviceGuard guard;
    const StreamArg& st;
    explicit Where(const Shape& sh, const StreamArg& s) : Where(sh.device, s) {}
    Where(c10::Device d, const StreamArg& s) : guard(d), st(s)
    {
        TORCH_CHECK_VALUE(d.is_cuda(), "the operands must live on a GPU, not on ", d);
    }
    void* stream() const
    {
        return st.torch ? st.raw : (void*)c10::hip::getCurrentHIPStreamMasqueradingAsCUDA().stream();
    }
    Tensor scratch(size_t bytes) const
    {
        if (!st.torch) return make({(int64_t)bytes}, at::kByte, guard.current_device());
        c10::StreamGuard on(*st.torch);
        return make({(int64_t)bytes}, at::kByte, guard.current_device());
    }
    // the same memory without a tensor around it, for the calls whose host time counts (8 rows of a packed forward: 1
    // us less)
    c10::DataPtr block(size_t bytes) const
    {
        if (!bytes) return {};
        c10::OptionalStreamGuard on;
        if (st.torch) on.reset_stream(*st.torch);
        return c10::GetAllocator(c10::DeviceType::CUDA)->allocate(bytes);
    }
};

struct Bytes {  // a buffer handed to the library, possibly none
    void* p = nullptr;
    size_t n = 0;
    Bytes() = default;
    explicit Bytes(const Tensor& t)
    {
        if (!t.defined()) return;
        p = t.data_ptr();
        n = t.nbytes();
    }
};
void* ptr(const Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }

// ---- the calls ----

Tensor fwd(const Tensor& x, const Tensor& R, const Tensor& L, Tensor y, unsigned flags, const StreamArg& st)
{
    const Shape sh(x, R, L);
    const Where w(sh, st);
    check(x, "x", {sh.B, sh.n_in()}, sh.dtype, sh.device);
    sh.check_factors(R, L);
    y = out(y, "y", {sh.B, sh.n_out()}, sh.dtype, sh.device);
    const int rc = monarch_fwd_ex(ptr(x), ptr(R), ptr(L), ptr(y), sh.B, (int)sh.n_in(), (int)sh.k, (int)sh.q, (int)sh.s, sh.code(),
                                  w.stream(), flags);
    if (rc) raise_status(rc, "monarch_fwd");
    return y;
}

Tensor fwd_static(const Tensor& x, const Tensor& R, const Tensor& L, const Tensor& y, unsigned flags, const StreamArg& st)
{
    const Shape sh(x, R, L);
    const Where w(sh, st);
    check(x, "x", {sh.B, sh.n_in()}, sh.dtype, sh.device);
    sh.check_factors(R, L);
    check(y, "y", {sh.B, sh.n_out()}, sh.dtype, sh.device);
    const int rc = monarch_fwd_static(ptr(x), ptr(R), ptr(L), ptr(y), sh.B, (int)sh.n_in(), (int)sh.k, (int)sh.q, (int)sh.s,
                                      sh.code(), w.stream(), flags);
    if (rc) raise_status(rc, "monarch_fwd_static");
    return y;
}

// Forward with a workspace, with or without bias and nonlinearity.
struct Layer {
    Tensor y_pre, y;
};
enum class Act { none, gelu };
Layer fwd_layer(const char* name, const Tensor& x, const Tensor& R, const Tensor& L, const Tensor& bias, Act act, Tensor y_pre,
                bool want_pre, Tensor y, Tensor ws, unsigned flags, const StreamArg& st)
{
    const Shape sh(x, R, L);
    const Where w(sh, st);
    check(x, "x", {sh.B, sh.n_in()}, sh.dtype, sh.device);
    sh.check_factors(R, L);
    if (bias.defined()) check(bias, "bias", {sh.n_out()}, sh.dtype, sh.device);
    y = out(y, "y", {sh.B, sh.n_out()}, sh.dtype, sh.device);
    if (want_pre || y_pre.defined()) y_pre = out(y_pre, "y_pre", {sh.B, sh.n_out()}, sh.dtype, sh.device);
    if (!ws.defined()) {
        if (flags & MONARCH_FLAG_WS_PACKED) {
            // An empty batch asks whether the shape cannot do without a workspace; elsewhere the flag has nothing to
            // refer to.
            const int rc = monarch_fwd_ws(ptr(x), ptr(R), ptr(L), ptr(y), 0, (int)sh.n_in(), (int)sh.k, (int)sh.q, (int)sh.s, sh.code(),
                                          w.stream(), nullptr, 0, flags);
            TORCH_CHECK_VALUE(rc != MONARCH_ERR_WORKSPACE, "MONARCH_FLAG_WS_PACKED needs the workspace of the earlier call");
            if (rc) raise_status(rc, name);
            flags &= ~MONARCH_FLAG_WS_PACKED;
        }
        const size_t need = monarch_fwd_workspace_bytes(sh.B, (int)sh.n_in(), (int)sh.k, (int)sh.q, (int)sh.s, sh.code(), flags);
        if (need) ws = w.scratch(need);
    }
    const Bytes b(ws);
    // a workspace of packed weights is only read (other streams may be using it): the vector between the factors of a
    // short batch goes to memory of this call
    const size_t mid = flags & MONARCH_FLAG_WS_PACKED ? monarch_fwd_packed_scratch_bytes(sh.B, (int)sh.n_in(), (int)sh.k, (int)sh.q,
                                                                                        (int)sh.s, sh.code(), flags)
                                                      : 0;
    const c10::DataPtr scratch = w.block(mid);
    const int rc = mid
        ? monarch_fwd_packed(ptr(x), ptr(R), ptr(L), ptr(bias), act == Act::gelu, ptr(y_pre), ptr(y), sh.B, (int)sh.n_in(), (int)sh.k,
                             (int)sh.q, (int)sh.s, sh.code(), w.stream(), b.p, b.n, scratch.get(), mid, flags)
        : act == Act::gelu
        ? monarch_fwd_bias_gelu(ptr(x), ptr(R), ptr(L), ptr(bias), ptr(y_pre), ptr(y), sh.B, (int)sh.n_in(), (int)sh.k, (int)sh.q,
                                (int)sh.s, sh.code(), w.stream(), b.p, b.n, flags)
        : monarch_fwd_bias(ptr(x), ptr(R), ptr(L), ptr(bias), ptr(y), sh.B, (int)sh.n_in(), (int)sh.k, (int)sh.q, (int)sh.s,
                           sh.code(), w.stream(), b.p, b.n, flags);
    if (rc) raise_status(rc, name);
    return Layer{y_pre, y};
}

Tensor fwd_t(const Tensor& x, const Tensor& R, const Tensor& L, Tensor y, Tensor ws, unsigned flags, const StreamArg& st)
{
    const Shape sh(x, R, L);
    const Where w(sh, st);
    check(x, "x", {sh.B, sh.n_out()}, sh.dtype, sh.device);
    sh.check_factors(R, L);
    y = out(y, "y", {sh.B, sh.n_in()}, sh.dtype, sh.device);
    if (!ws.defined()) {
        const size_t need = monarch_fwd_t_workspace_bytes(sh.B, (int)sh.n_in(), (int)sh.k, (int)sh.q, (int)sh.s, sh.code(), flags);
        if (need) ws = w.scratch(need);
    }
    const Bytes b(ws);
    const int rc = monarch_fwd_t(ptr(x), ptr(R), ptr(L), ptr(y), sh.B, (int)sh.n_in(), (int)sh.k, (int)sh.q, (int)sh.s, sh.code(),
                                 w.stream(), b.p, b.n, flags);
    if (rc) raise_status(rc, "monarch_fwd_t");
    return y;
}

struct Saved {
    Tensor y, saved;
};
// layer: monarch_fwd_keep, which keeps the vector for more shapes
Saved fwd_save(const Tensor& x, const Tensor& R, const Tensor& L, const Tensor& bias, Tensor y, Tensor saved, unsigned flags,
               const StreamArg& st, bool layer = false)
{
    const Shape sh(x, R, L);
    const Where w(sh, st);
    check(x, "x", {sh.B, sh.n_in()}, sh.dtype, sh.device);
    sh.check_factors(R, L);
    if (bias.defined()) check(bias, "bias", {sh.n_out()}, sh.dtype, sh.device);
    y = out(y, "y", {sh.B, sh.n_out()}, sh.dtype, sh.device);
    const size_t need = (layer ? monarch_kept_bytes : monarch_saved_bytes)(sh.B, (int)sh.n_in(), (int)sh.k, (int)sh.q, (int)sh.s, sh.code(), flags);
    if (flags & MONARCH_FLAG_WS_PACKED) raise_status(MONARCH_ERR_INVALID, "monarch_fwd_save");
    // nothing to save for this shape: the forward that has a workspace (fp32, k = 64 blocks of 64, 12000 rows: 6050
    // us without one, which is the SIMT kernels there, 290 with)
    if (!need) return Saved{fwd_layer("monarch_fwd_save", x, R, L, bias, Act::none, {}, false, y, {}, flags, st).y, Tensor()};
    if (!saved.defined()) saved = make({(int64_t)need}, at::kByte, sh.device);
    const Bytes b(saved);
    const int rc = (layer ? monarch_fwd_keep : monarch_fwd_bias_save)(ptr(x), ptr(R), ptr(L), ptr(bias), ptr(y), b.p, b.n, sh.B, (int)sh.n_in(),
                                                                      (int)sh.k, (int)sh.q, (int)sh.s, sh.code(), w.stream(), flags);
    if (rc) raise_status(rc, "monarch_fwd_save");
    return Saved{y, saved};
}

// Every backward: `x_pre` (the layer's input is gelu(x_pre)) and `saved` (the vector between the factors) may be
// missing.
struct Grads {
    Tensor dx, dR, dL, dbias;
};
Grads bwd(const char* name, const Tensor& dy, const Tensor& x, const Tensor& x_pre, const Tensor& saved, const Tensor& R,
          const Tensor& L, Grads g, bool want_dbias, Tensor ws, unsigned flags, const StreamArg& st, bool layer = false)
{
    const Shape sh(x, R, L);
    const Where w(sh, st);
    check(x, "x", {sh.B, sh.n_in()}, sh.dtype, sh.device);
    if (x_pre.defined()) check(x_pre, "x_pre", {sh.B, sh.n_in()}, sh.dtype, sh.device);
    check(dy, "dy", {sh.B, sh.n_out()}, sh.dtype, sh.device);
    sh.check_factors(R, L);
    const at::ScalarType gt = (flags & MONARCH_FLAG_WGRAD_F32) ? at::kFloat : sh.dtype;
    g.dx = out(g.dx, x_pre.defined() ? "dx_pre" : "dx", {sh.B, sh.n_in()}, sh.dtype, sh.device);
    g.dR = out(g.dR, "dR", {sh.k, sh.q, sh.p}, gt, sh.device);
    g.dL = out(g.dL, "dL", {sh.k, sh.s, sh.q}, gt, sh.device);
    if (want_dbias || g.dbias.defined()) g.dbias = out(g.dbias, "dbias", {sh.n_out()}, gt, sh.device);
    if (!ws.defined()) {
        auto bytes = layer && saved.defined() ? monarch_bwd_kept_workspace_bytes : monarch_bwd_workspace_bytes;
        const size_t need = bytes(sh.B, (int)sh.n_in(), (int)sh.k, (int)sh.q, (int)sh.s, sh.code(), flags);
        if (need) ws = w.scratch(need);
    }
    const Bytes b(ws), sv(saved);
    const int rc = x_pre.defined()
        ? monarch_bwd_bias_gelu_in(ptr(dy), ptr(x), ptr(x_pre), ptr(R), ptr(L), ptr(g.dx), ptr(g.dR), ptr(g.dL), ptr(g.dbias), sh.B,
                                   (int)sh.n_in(), (int)sh.k, (int)sh.q, (int)sh.s, sh.code(), w.stream(), b.p, b.n, flags)
        : (layer ? monarch_bwd_kept : monarch_bwd_saved)(ptr(dy), ptr(x), sv.p, sv.n, ptr(R), ptr(L), ptr(g.dx), ptr(g.dR), ptr(g.dL), ptr(g.dbias),
                                                         sh.B, (int)sh.n_in(), (int)sh.k, (int)sh.q, (int)sh.s, sh.code(), w.stream(), b.p, b.n,
                                                         flags);
    if (rc) raise_status(rc, name);
    return g;
}

Tensor to_dense(const Tensor& R, const Tensor& L, Tensor M, unsigned flags, const StreamArg& st)
{
    const Shape sh(R, R, L);
    const Where w(sh, st);
    sh.check_factors(R, L);
    M = out(M, "M", {sh.n_out(), sh.n_in()}, sh.dtype, sh.device);
    const int rc = monarch_to_dense(ptr(R), ptr(L), ptr(M), (int)sh.n_in(), (int)sh.k, (int)sh.q, (int)sh.s, sh.code(), w.stream(), flags);
    if (rc) raise_status(rc, "monarch_to_dense");
    return M;
}

struct Factors {
    Tensor L, R;
};
Factors project(const Tensor& A, Tensor R, Tensor L, const StreamArg& st)
{
    const Where w(A.device(), st);
    TORCH_CHECK_VALUE(A.dim() >= 1, "A must be n x n");
    const int64_t n = A.size(0), m = std::llround(std::sqrt((double)n));
    TORCH_CHECK_VALUE(m * m == n, "A must be n x n with n a perfect square, got ", A.sizes());
    const at::ScalarType dt = A.scalar_type();
    check(A, "A", {n, n}, dt, A.device());
    R = out(R, "R", {m, m, m}, dt, A.device());
    L = out(L, "L", {m, m, m}, dt, A.device());
    TORCH_CHECK_TYPE(dt == at::kFloat || dt == at::kBFloat16, "dtype must be float32 or bfloat16, got ", dt);
    const int rc = monarch_project(ptr(A), ptr(R), ptr(L), (int)n, (int)m, dt == at::kFloat ? MONARCH_F32 : MONARCH_BF16, w.stream(), 0);
    if (rc) raise_status(rc, "monarch_project");
    return Factors{L, R};
}

// complex64: `pass` as in monarch_c64_workspace_bytes (0 forward, 2 conjugate transpose)
Tensor c64_apply(int pass, bool with_ws, const Tensor& x, const Tensor& R, const Tensor& L, Tensor y, Tensor ws, unsigned flags,
                 const StreamArg& st)
{
    Shape sh(x, R, L);
    sh.dtype = at::kComplexFloat;
    const Where w(sh, st);
    const int64_t from = pass == 2 ? sh.n_out() : sh.n_in(), to = pass == 2 ? sh.n_in() : sh.n_out();
    check(x, "x", {sh.B, from}, sh.dtype, sh.device);
    sh.check_factors(R, L);
    y = out(y, "y", {sh.B, to}, sh.dtype, sh.device);
    const int n = (int)sh.n_in(), k = (int)sh.k, q = (int)sh.q, s = (int)sh.s;
    int rc;
    const char* name;
    if (!with_ws) {
        name = pass == 2 ? "monarch_fwd_h_c64" : "monarch_fwd_c64";
        rc = pass == 2 ? monarch_fwd_h_c64(ptr(x), ptr(R), ptr(L), ptr(y), sh.B, n, k, q, s, w.stream(), flags)
                       : monarch_fwd_c64(ptr(x), ptr(R), ptr(L), ptr(y), sh.B, n, k, q, s, w.stream(), flags);
    } else {
        name = pass == 2 ? "monarch_fwd_h_c64_ws" : "monarch_fwd_c64_ws";
        if (!ws.defined()) ws = w.scratch(std::max<size_t>(monarch_c64_workspace_bytes(pass, sh.B, n, k, q, s, flags), 256));
        const Bytes b(ws);
        rc = pass == 2 ? monarch_fwd_h_c64_ws(ptr(x), ptr(R), ptr(L), ptr(y), sh.B, n, k, q, s, w.stream(), b.p, b.n, flags)
                       : monarch_fwd_c64_ws(ptr(x), ptr(R), ptr(L), ptr(y), sh.B, n, k, q, s, w.stream(), b.p, b.n, flags);
    }
    if (rc) raise_status(rc, name);
    return y;
}

Grads c64_bwd(bool with_ws, const Tensor& dy, const Tensor& x, const Tensor& R, const Tensor& L, Grads g, Tensor ws, unsigned flags,
              const StreamArg& st)
{
    Shape sh(x, R, L);
    sh.dtype = at::kComplexFloat;
    const Where w(sh, st);
    check(x, "x", {sh.B, sh.n_in()}, sh.dtype, sh.device);
    check(dy, "dy", {sh.B, sh.n_out()}, sh.dtype, sh.device);
    sh.check_factors(R, L);
    g.dx = out(g.dx, "dx", {sh.B, sh.n_in()}, sh.dtype, sh.device);
    g.dR = out(g.dR, "dR", {sh.k, sh.q, sh.p}, sh.dtype, sh.device);
    g.dL = out(g.dL, "dL", {sh.k, sh.s, sh.q}, sh.dtype, sh.device);
    const int n = (int)sh.n_in(), k = (int)sh.k, q = (int)sh.q, s = (int)sh.s;
    int rc;
    if (with_ws) {
        if (!ws.defined()) ws = w.scratch(std::max<size_t>(monarch_c64_workspace_bytes(1, sh.B, n, k, q, s, flags), 256));
        const Bytes b(ws);
        rc = monarch_bwd_c64_ws(ptr(dy), ptr(x), ptr(R), ptr(L), ptr(g.dx), ptr(g.dR), ptr(g.dL), sh.B, n, k, q, s, w.stream(), b.p,
                                b.n, flags);
    } else {
        rc = monarch_bwd_c64(ptr(dy), ptr(x), ptr(R), ptr(L), ptr(g.dx), ptr(g.dR), ptr(g.dL), sh.B, n, k, q, s, w.stream(), flags);
    }
    if (rc) raise_status(rc, with_ws ? "monarch_bwd_c64_ws" : "monarch_bwd_c64");
    return g;
}

// ---- autograd ----

// y = x M^T (+ bias).  The forward can keep the vector between the factors for the backward (save_intermediate), else
// the backward recomputes it.
struct LinearFn : torch::autograd::Function<LinearFn> {
    // Where keeping the vector pays, by the GPU time of a training step with bias, recomputed and kept: 64 blocks of 64
    // always (16384 rows 329 us and 287, 4096 rows 106 and 89); fp32 and odd blocks always (192 x 192, four blocks, fp32, 12608 rows: one contraction of 53 us of 400 less).  The bf16
    // layers of four blocks that are multiples of 64 have other forwards for the call that keeps nothing.  Those of
    // short batches (256 x 1024: 300 rows 47 and 54 us, 1000 rows 58 and 59) lose their lead between 1500 and 3500
    // rows (256 x 1024: 2000 rows 76 and 73; 192 x 768: 2000 rows 60 and 62, 2500 rows 66 and 63; 192 x 192: 2500
    // rows 50 and 52, 3500 rows 57 and 55; 1024 x 256: 1500 rows 87 and 92, 2500 rows 103 and 95).  Over long batches
    // the packed forward wins for wide outputs, by most in the widest layer (256 x 1024: 4500 rows 107 and 103, 8192
    // rows 131 and 136, 12000 rows 169 and 179); 192 x 768 crosses at 5000 rows (8192 rows 95 and 97, 12000 rows 121
    // and 129), 256 x 768 at 8192 (12000 rows 143 and 150), 192 x 576 and 128 x 512 not up to 12000 (108 and 108; 82
    // and 80): the line between them costs up to 4 % on either side.  Outputs no wider than the input gain at every
    // length (768 x 192, 16384 rows: 166 and 142).
    static bool keeps(const Tensor& x, const Tensor& R, const Tensor& L)
    {
        const int64_t rows = x.size(0), p = R.size(2), q = R.size(1), s = L.size(1);
        if (x.scalar_type() != at::kBFloat16 || R.size(0) != 4 || p % 64 || q % 64 || s % 64) return true;
        return rows > 2048 && (s <= p || rows <= 8192);
    }
    // (rows, width) from any leading dimensions; their product must be the number of rows, else the last one is not
    // `width`
    static Tensor rows_of(const Tensor& t, int64_t width)
    {
        if (t.dim() == 2 && t.size(1) == width && t.is_contiguous()) return t;
        const Tensor rows = t.reshape({-1, width}).contiguous();
        int64_t leading = 1;
        for (int64_t d = 0; d + 1 < t.dim(); ++d) leading *= t.size(d);
        TORCH_CHECK(rows.size(0) == leading, "the last dimension of the input must be ", width, ", got shape ", t.sizes());
        return rows;
    }
    static Tensor forward(torch::autograd::AutogradContext* ctx, const Tensor& x, const Tensor& R, const Tensor& L,
                          const c10::optional<Tensor>& bias, bool save_intermediate)
    {
        TORCH_CHECK_VALUE(R.dim() == 3 && L.dim() == 3, "R and L must have three dimensions");
        const Tensor x2 = rows_of(x, R.size(0) * R.size(2));
        const StreamArg current;
        Saved r;
        if (save_intermediate && keeps(x2, R, L)) r = fwd_save(x2, R, L, bias.value_or(Tensor()), {}, {}, 0, current, true);
        else if (bias.has_value()) r.y = fwd_layer("monarch_fwd_bias", x2, R, L, *bias, Act::none, {}, false, {}, {}, 0, current).y;
        else r.y = fwd_layer("monarch_fwd_ws", x2, R, L, {}, Act::none, {}, false, {}, {}, 0, current).y;
        ctx->save_for_backward({x2, R, L, r.saved});
        if (bias.has_value()) ctx->saved_data["bias"] = true;
        if (x.dim() == 2) return r.y;
        ctx->saved_data["shape"] = x.sizes().vec();
        std::vector<int64_t> shape = x.sizes().vec();
        if (shape.empty()) shape.resize(1);
        shape.back() = r.y.size(1);
        return r.y.view(shape);
    }
    static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx, torch::autograd::variable_list dy)
    {
        const auto saved = ctx->get_saved_variables();
        const Tensor &x2 = saved[0], &R = saved[1], &L = saved[2];
        const bool bias = ctx->saved_data.count("bias") != 0;
        const StreamArg current;
        Grads g = bwd("monarch_bwd_saved", rows_of(dy[0], L.size(0) * L.size(1)), x2, {}, saved[3], R, L, {}, bias, {}, 0, current, true);
        const auto shape = ctx->saved_data.find("shape");
        if (shape != ctx->saved_data.end()) g.dx = g.dx.view(shape->second.toIntVector());
        return {g.dx, g.dR, g.dL, g.dbias, Tensor()};
    }
};

// ---- the Python module ----

PyObject* none_or(const Tensor& t)
{
    if (t.defined()) return THPVariable_Wrap(t);
    Py_RETURN_NONE;
}
PyObject* tuple_of(std::initializer_list<Tensor> ts)
{
    PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
    Py_ssize_t i = 0;
    for (const Tensor& t : ts) PyTuple_SET_ITEM(r, i++, none_or(t));
    return r;
}
// runs f without the GIL (a full hardware queue blocks the launch)
template <typename F>
auto unlocked(F f)
{
    struct Release {
        PyThreadState* s = PyEval_SaveThread();
        ~Release() { PyEval_RestoreThread(s); }
    } release;
    return f();
}

void expect(Py_ssize_t got, Py_ssize_t want)
{
    TORCH_CHECK_TYPE(got == want, "expected ", want, " arguments, got ", got);
}
#define MONARCH_CALL(name, count)                                               \
    PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n)                 \
    {                                                                           \
        HANDLE_TH_ERRORS                                                        \
        expect(n, count);
#define MONARCH_END          \
        END_HANDLE_TH_ERRORS \
    }

MONARCH_CALL(py_fwd, 6)
    const Tensor x = tensor_arg(a[0], "x"), R = tensor_arg(a[1], "R"), L = tensor_arg(a[2], "L"), y = optional_arg(a[3], "y");
    const unsigned flags = flags_arg(a[4]);
    const StreamArg st = stream_arg(a[5]);
    return THPVariable_Wrap(unlocked([&] { return fwd(x, R, L, y, flags, st); }));
MONARCH_END

MONARCH_CALL(py_fwd_static, 6)
    const Tensor x = tensor_arg(a[0], "x"), R = tensor_arg(a[1], "R"), L = tensor_arg(a[2], "L"), y = tensor_arg(a[3], "y");
    const unsigned flags = flags_arg(a[4]);
    const StreamArg st = stream_arg(a[5]);
    return THPVariable_Wrap(unlocked([&] { return fwd_static(x, R, L, y, flags, st); }));
MONARCH_END

MONARCH_CALL(py_fwd_ws, 7)
    const Tensor x = tensor_arg(a[0], "x"), R = tensor_arg(a[1], "R"), L = tensor_arg(a[2], "L"), y = optional_arg(a[3], "y"),
                 ws = optional_arg(a[4], "workspace");
    const unsigned flags = flags_arg(a[5]);
    const StreamArg st = stream_arg(a[6]);
    return THPVariable_Wrap(
        unlocked([&] { return fwd_layer("monarch_fwd_ws", x, R, L, {}, Act::none, {}, false, y, ws, flags, st).y; }));
MONARCH_END

MONARCH_CALL(py_fwd_bias, 8)
    const Tensor x = tensor_arg(a[0], "x"), R = tensor_arg(a[1], "R"), L = tensor_arg(a[2], "L"), bias = tensor_arg(a[3], "bias"),
                 y = optional_arg(a[4], "y"), ws = optional_arg(a[5], "workspace");
    const unsigned flags = flags_arg(a[6]);
    const StreamArg st = stream_arg(a[7]);
    return THPVariable_Wrap(
        unlocked([&] { return fwd_layer("monarch_fwd_bias", x, R, L, bias, Act::none, {}, false, y, ws, flags, st).y; }));
MONARCH_END

MONARCH_CALL(py_fwd_bias_gelu, 10)
    const Tensor x = tensor_arg(a[0], "x"), R = tensor_arg(a[1], "R"), L = tensor_arg(a[2], "L"), bias = optional_arg(a[3], "bias"),
                 y_pre = optional_arg(a[4], "y_pre"), y = optional_arg(a[5], "y"), ws = optional_arg(a[7], "workspace");
    const bool want_pre = bool_arg(a[6]);
    const unsigned flags = flags_arg(a[8]);
    const StreamArg st = stream_arg(a[9]);
    const Layer r = unlocked(
        [&] { return fwd_layer("monarch_fwd_bias_gelu", x, R, L, bias, Act::gelu, y_pre, want_pre, y, ws, flags, st); });
    return tuple_of({r.y_pre, r.y});
MONARCH_END

MONARCH_CALL(py_fwd_t, 7)
    const Tensor x = tensor_arg(a[0], "x"), R = tensor_arg(a[1], "R"), L = tensor_arg(a[2], "L"), y = optional_arg(a[3], "y"),
                 ws = optional_arg(a[4], "workspace");
    const unsigned flags = flags_arg(a[5]);
    const StreamArg st = stream_arg(a[6]);
    return THPVariable_Wrap(unlocked([&] { return fwd_t(x, R, L, y, ws, flags, st); }));
MONARCH_END

MONARCH_CALL(py_fwd_save, 8)
    const Tensor x = tensor_arg(a[0], "x"), R = tensor_arg(a[1], "R"), L = tensor_arg(a[2], "L"), bias = optional_arg(a[3], "bias"),
                 y = optional_arg(a[4], "y"), saved = optional_arg(a[5], "saved");
    const unsigned flags = flags_arg(a[6]);
    const StreamArg st = stream_arg(a[7]);
    const Saved r = unlocked([&] { return fwd_save(x, R, L, bias, y, saved, flags, st); });
    return tuple_of({r.y, r.saved});
MONARCH_END

// bwd(name, dy, x, x_pre, saved, R, L, dx, dR, dL, dbias, want_dbias, workspace, flags, stream)
MONARCH_CALL(py_bwd, 15)
    const char* name = PyUnicode_AsUTF8(a[0]);
    if (!name) throw python_error();
    const Tensor dy = tensor_arg(a[1], "dy"), x = tensor_arg(a[2], "x"), x_pre = optional_arg(a[3], "x_pre"),
                 saved = optional_arg(a[4], "saved"), R = tensor_arg(a[5], "R"), L = tensor_arg(a[6], "L"),
                 ws = optional_arg(a[12], "workspace");
    const Grads g{optional_arg(a[7], "dx"), optional_arg(a[8], "dR"), optional_arg(a[9], "dL"), optional_arg(a[10], "dbias")};
    const bool want_dbias = bool_arg(a[11]);
    const unsigned flags = flags_arg(a[13]);
    const StreamArg st = stream_arg(a[14]);
    const Grads r = unlocked([&] { return bwd(name, dy, x, x_pre, saved, R, L, g, want_dbias, ws, flags, st); });
    return tuple_of({r.dx, r.dR, r.dL, r.dbias});
MONARCH_END

MONARCH_CALL(py_to_dense, 5)
    const Tensor R = tensor_arg(a[0], "R"), L = tensor_arg(a[1], "L"), M = optional_arg(a[2], "M");
    const unsigned flags = flags_arg(a[3]);
    const StreamArg st = stream_arg(a[4]);
    return THPVariable_Wrap(unlocked([&] { return to_dense(R, L, M, flags, st); }));
MONARCH_END

MONARCH_CALL(py_project, 4)
    const Tensor A = tensor_arg(a[0], "A"), R = optional_arg(a[1], "R"), L = optional_arg(a[2], "L");
    const StreamArg st = stream_arg(a[3]);
    const Factors r = unlocked([&] { return project(A, R, L, st); });
    return tuple_of({r.L, r.R});
MONARCH_END

// c64_apply(pass, with_ws, x, R, L, y, workspace, flags, stream)
MONARCH_CALL(py_c64_apply, 9)
    const int pass = (int)flags_arg(a[0]);
    const bool with_ws = bool_arg(a[1]);
    const Tensor x = tensor_arg(a[2], "x"), R = tensor_arg(a[3], "R"), L = tensor_arg(a[4], "L"), y = optional_arg(a[5], "y"),
                 ws = optional_arg(a[6], "workspace");
    const unsigned flags = flags_arg(a[7]);
    const StreamArg st = stream_arg(a[8]);
    return THPVariable_Wrap(unlocked([&] { return c64_apply(pass, with_ws, x, R, L, y, ws, flags, st); }));
MONARCH_END

// c64_bwd(with_ws, dy, x, R, L, dx, dR, dL, workspace, flags, stream)
MONARCH_CALL(py_c64_bwd, 11)
    const bool with_ws = bool_arg(a[0]);
    const Tensor dy = tensor_arg(a[1], "dy"), x = tensor_arg(a[2], "x"), R = tensor_arg(a[3], "R"), L = tensor_arg(a[4], "L"),
                 ws = optional_arg(a[8], "workspace");
    const Grads g{optional_arg(a[5], "dx"), optional_arg(a[6], "dR"), optional_arg(a[7], "dL"), Tensor()};
    const unsigned flags = flags_arg(a[9]);
    const StreamArg st = stream_arg(a[10]);
    const Grads r = unlocked([&] { return c64_bwd(with_ws, dy, x, R, L, g, ws, flags, st); });
    return tuple_of({r.dx, r.dR, r.dL});
MONARCH_END

// linear(x, R, L, bias, save_intermediate)
MONARCH_CALL(py_linear, 5)
    const Tensor x = tensor_arg(a[0], "x"), R = tensor_arg(a[1], "R"), L = tensor_arg(a[2], "L");
    c10::optional<Tensor> bias;
    if (a[3] != Py_None) bias = tensor_arg(a[3], "bias");
    // nothing is kept where no backward follows (LinearFn::forward itself always runs without gradients)
    const bool save = bool_arg(a[4]) && at::GradMode::is_enabled() &&
                      (x.requires_grad() || R.requires_grad() || L.requires_grad() || (bias && bias->requires_grad()));
    return THPVariable_Wrap(unlocked([&] { return LinearFn::apply(x, R, L, bias, save); }));
MONARCH_END

PyObject* py_set_error(PyObject*, PyObject* cls)
{
    Py_INCREF(cls);
    Py_XSETREF(g_error, cls);
    Py_RETURN_NONE;
}

#define MONARCH_ENTRY(name) {#name, (PyCFunction)(void (*)())py_##name, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    MONARCH_ENTRY(fwd), MONARCH_ENTRY(fwd_static), MONARCH_ENTRY(fwd_ws), MONARCH_ENTRY(fwd_bias), MONARCH_ENTRY(fwd_bias_gelu),
    MONARCH_ENTRY(fwd_t), MONARCH_ENTRY(fwd_save), MONARCH_ENTRY(bwd), MONARCH_ENTRY(to_dense), MONARCH_ENTRY(c64_apply),
    MONARCH_ENTRY(c64_bwd), MONARCH_ENTRY(project), MONARCH_ENTRY(linear), {"set_error", py_set_error, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&g_module); }
