// CPython module behind binding.py: the same calls as the C ABI, on torch tensors.
//
// A call checks its tensors (device, type, contiguity, shape), allocates the outputs and the
// workspace that were not passed in, takes torch's current stream and calls the C ABI.  No
// arithmetic of the method and no kernel lives here.  It exists for the small calls: the kernels
// of a decode step or a short prompt run for 5 to 10 us, and the same work in Python (ctypes
// marshalling, shape tuples, stream objects, torch.empty) took 7 to 10 us a call, so the host and
// not the GPU set the pace.  Measured per decode call (two launches), enqueue time: 16.9 us
// through ctypes, 6.8 us here; passes back to back: 17.1 -> 9.6 us.  A launch is 2.2 to 3 us of what is left; memory, 0.3 us of torch's caching
// allocator a piece, is taken from it directly (allocate(), Workspace): enqueue time of a short training step
// (five tensors and a workspace) 15.0 -> 14.1 us, of a decode call 5.1 -> 4.8.
#include <Python.h>

#include <initializer_list>
#include <stdexcept>
#include <string>

#include <ATen/ATen.h>
#include <ATen/EmptyTensor.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/hip/impl/HIPCachingAllocatorMasqueradingAsCUDA.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/sb_attn.h"

namespace {

PyObject* g_error = nullptr;               // binding.SbAttnError
PyObject* g_oom = nullptr;                 // torch.cuda.OutOfMemoryError

struct Failed : std::runtime_error {       // becomes an SbAttnError
    using std::runtime_error::runtime_error;
};
struct Raised {};                          // a Python exception is already set

using Shape = c10::SmallVector<int64_t, 4>;

std::string text(at::IntArrayRef s)
{
    std::string r = "(";
    for (size_t i = 0; i < s.size(); ++i) r += (i ? ", " : "") + std::to_string(s[i]);
    return r + (s.size() == 1 ? ",)" : ")");
}

const char* dtype_name(at::ScalarType t)
{
    switch (t) {
    case at::kBFloat16: return "torch.bfloat16";
    case at::kFloat: return "torch.float32";
    case at::kInt: return "torch.int32";
    case at::kLong: return "torch.int64";
    default: return c10::toString(t);
    }
}

bool none(PyObject* o) { return o == Py_None; }

const at::Tensor& tensor(PyObject* o, const char* name)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a torch.Tensor, got %s", name, Py_TYPE(o)->tp_name);
        throw Raised{};
    }
    return THPVariable_Unpack(o);
}

// what int(o) gives: integers, floats, one-element tensors
int to_int(PyObject* o)
{
    PyObject* i = PyNumber_Long(o);
    if (!i) throw Raised{};
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(i, &overflow);
    Py_DECREF(i);
    if (overflow) throw Failed("integer argument out of range");
    if (v > INT32_MAX || v < INT32_MIN) throw Failed("integer argument out of range");
    return (int)v;
}

bool truth(PyObject* o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Raised{};
    return v != 0;
}

int dim(const at::Tensor& t, int i)
{
    const int64_t v = t.size(i);
    if (v > INT32_MAX) throw Failed("dimension too large");
    return (int)v;
}

// device pointer of a checked tensor, nullptr for None
void* ptr(PyObject* o, at::ScalarType dtype, at::IntArrayRef shape, const char* name)
{
    if (none(o)) return nullptr;
    const at::Tensor& t = tensor(o, name);
    if (!t.is_cuda()) throw Failed(std::string(name) + " must live on the GPU");
    if (t.scalar_type() != dtype)
        throw Failed(std::string(name) + " must be " + dtype_name(dtype) + ", got " + dtype_name(t.scalar_type()));
    if (!t.is_contiguous()) throw Failed(std::string(name) + " must be contiguous");
    if (shape.data() && t.sizes() != shape)
        throw Failed(std::string(name) + " has shape " + text(t.sizes()) + ", expected " + text(shape));
    return t.data_ptr();
}

void* any_shape(PyObject* o, at::ScalarType dtype, const char* name) { return ptr(o, dtype, at::IntArrayRef(), name); }

// where a call launches: stream=, or the current stream where that is None
struct Launch {
    void* stream;
    bool given;
    c10::DeviceIndex device;               // the current one (-1: not asked for)
};
Launch launch_on(PyObject* o)
{
    if (none(o)) {
        const c10::DeviceIndex device = c10::hip::current_device();
        return {c10::hip::getCurrentHIPStream(device).stream(), false, device};
    }
    PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
    if (!h) throw Raised{};
    void* s = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (!s && PyErr_Occurred()) throw Raised{};
    return {s, true, -1};
}

// `stream` as torch's current stream of `device`, for one scope
class OnStream {
public:
    OnStream(void* stream, c10::DeviceIndex device) : before_(c10::hip::getCurrentHIPStream(device))
    {
        c10::hip::setCurrentHIPStream(c10::hip::getStreamFromExternal(static_cast<hipStream_t>(stream), device));
    }
    OnStream(const OnStream&) = delete;
    ~OnStream() { c10::hip::setCurrentHIPStream(before_); }
    const c10::hip::HIPStream& before() const { return before_; }

private:
    c10::hip::HIPStream before_;
};

// Memory for a launch.  torch's caching allocator hands freed memory on in the order of the stream that it was
// allocated on, so that has to be the stream of the launch: memory of the current stream may still be in use by
// earlier work there, which a launch on stream= does not wait for.  What the caller gets back (`shared`) the current
// stream will use as well: dropped, it is not handed on before the work that the current stream then holds is done.
at::Tensor allocate(at::IntArrayRef shape, at::ScalarType dtype, const at::Tensor& like, const Launch& on, bool shared)
{
    const c10::Device dev = like.device();
    if (!on.given) {
        // on the current device what torch's empty does behind its device guard
        if (on.device == dev.index())
            return at::detail::empty_generic(shape, c10::hip::HIPCachingAllocatorMasqueradingAsCUDA::get(), c10::DispatchKeySet(c10::DispatchKey::CUDA), dtype, c10::nullopt);
        return at::detail::empty_cuda(shape, dtype, dev, c10::nullopt);
    }
    OnStream here(on.stream, dev.index());
    at::Tensor t = at::detail::empty_cuda(shape, dtype, dev, c10::nullopt);
    if (shared && here.before().stream() != on.stream)
        c10::hip::HIPCachingAllocator::recordStream(t.storage().data_ptr(), here.before());
    return t;
}

// a new reference to the caller's tensor, or a fresh one where it is None; released unless taken
class Out {
public:
    Out(PyObject* given, at::ScalarType dtype, at::IntArrayRef shape, const at::Tensor& like, const char* name,
        const Launch& on)
    {
        if (none(given)) {
            if (!like.is_cuda()) throw Failed("q must live on the GPU");
            at::Tensor t = allocate(shape, dtype, like, on, true);
            p_ = t.data_ptr();
            o_ = THPVariable_Wrap(std::move(t));
            if (!o_) throw Raised{};
        } else {
            p_ = ptr(given, dtype, shape, name);
            Py_INCREF(given);
            o_ = given;
        }
    }
    Out(const Out&) = delete;
    ~Out() { Py_XDECREF(o_); }
    template <class T = void> T* p() const { return static_cast<T*>(p_); }
    PyObject* take() { PyObject* r = o_; o_ = nullptr; return r; }

private:
    void* p_ = nullptr;
    PyObject* o_ = nullptr;
};

// the caller's workspace, or one of `need` bytes that goes back to torch's caching allocator when
// the call returns, before the kernels have run, unless it is taken (`keep`: it is to be)
class Workspace {
public:
    Workspace(PyObject* given, size_t need, const at::Tensor& like, const Launch& on, bool keep = false)
    {
        if (!none(given)) {
            t_ = tensor(given, "workspace");
        } else if (need == 0 || !like.is_cuda()) {
            return;
        } else if (!keep && !on.given && on.device == like.device().index()) {
            own_ = p_ = c10::hip::HIPCachingAllocatorMasqueradingAsCUDA::raw_alloc_with_stream(need, static_cast<hipStream_t>(on.stream));
            bytes_ = need;
            return;
        } else {
            t_ = allocate({(int64_t)need}, at::kByte, like, on, keep);
        }
        p_ = t_.data_ptr();
        bytes_ = t_.nbytes();
    }
    Workspace(const Workspace&) = delete;
    ~Workspace()
    {
        if (own_) c10::hip::HIPCachingAllocatorMasqueradingAsCUDA::raw_delete(own_);
    }
    void* p() const { return p_; }
    size_t bytes() const { return bytes_; }
    PyObject* take() { return THPVariable_Wrap(std::move(t_)); }      // (None where there is none)

private:
    at::Tensor t_;
    void *own_ = nullptr, *p_ = nullptr;
    size_t bytes_ = 0;
};

template <class F> void call(const char* what, F f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    if (rc != SB_OK)
        throw Failed(std::string(what) + " failed: " + sb_status_string(rc) + " (" + std::to_string(rc) + ")");
}

PyObject* tuple(std::initializer_list<Out*> outs)
{
    PyObject* t = PyTuple_New((Py_ssize_t)outs.size());
    if (!t) throw Raised{};
    Py_ssize_t i = 0;
    for (Out* o : outs) PyTuple_SET_ITEM(t, i++, o->take());
    return t;
}

// [B, H, T, d] of q, and the kv heads of k
struct Dims {
    int B, H, T, d, Hkv;
    Shape q, kv, m, hd;
};

Dims dims(PyObject* qo, PyObject* ko)
{
    const at::Tensor& q = tensor(qo, "q");
    if (q.dim() != 4) throw Failed("expected a [B, H, T, d] tensor");
    Dims s;
    s.B = dim(q, 0); s.H = dim(q, 1); s.T = dim(q, 2); s.d = dim(q, 3);
    s.Hkv = s.H;
    if (ko) {
        const at::Tensor& k = tensor(ko, "k");
        if (k.dim() != 4) throw Failed("expected a [B, H, T, d] tensor");
        s.Hkv = dim(k, 1);
    }
    s.q = {s.B, s.H, s.T, s.d};
    s.kv = {s.B, s.Hkv, s.T, s.d};
    s.m = {s.B, s.H, s.T};
    s.hd = {s.H, s.d};
    return s;
}

// [H, Ttot, d] of a packed batch
Dims dims_packed(PyObject* qo, PyObject* ko)
{
    const at::Tensor& q = tensor(qo, "q");
    const at::Tensor& k = tensor(ko, "k");
    if (q.dim() != 3) throw Failed("q: expected a packed [H, Ttot, d] tensor");
    if (k.dim() != 3) throw Failed("k: expected a packed [H, Ttot, d] tensor");
    Dims s;
    s.B = 1; s.H = dim(q, 0); s.T = dim(q, 1); s.d = dim(q, 2);
    s.Hkv = dim(k, 0);
    s.q = {s.H, s.T, s.d};
    s.kv = {s.Hkv, s.T, s.d};
    s.m = {s.H, s.T};
    s.hd = {s.H, s.d};
    return s;
}

constexpr at::ScalarType BF = at::kBFloat16, F32 = at::kFloat;

// forward(what, grouped, q, k, v, r, o, m, want_m, stream): bf16, every variant without offsets
PyObject* forward(PyObject* const* a)
{
    const char* what = PyUnicode_AsUTF8(a[0]);
    if (!what) throw Raised{};
    const Dims s = dims(a[2], a[1] == Py_True ? a[3] : nullptr);
    const at::Tensor& like = THPVariable_Unpack(a[2]);
    void* q = any_shape(a[2], BF, "q");
    void* k = ptr(a[3], BF, s.kv, "k");
    void* v = ptr(a[4], BF, s.kv, "v");
    void* r = ptr(a[5], BF, s.hd, "r");
    const Launch on = launch_on(a[9]);
    Out o(a[6], BF, s.q, like, "o", on);
    auto go = [&](float* m) {
        call(what, [&] { return sb_attn_fwd_gqa(q, k, v, r, o.p(), m, s.B, s.H, s.Hkv, s.T, s.d, on.stream); });
    };
    if (none(a[7]) && !truth(a[8])) {
        go(nullptr);
        return o.take();
    }
    Out m(a[7], F32, s.m, like, "m", on);
    go(m.p<float>());
    return tuple({&o, &m});
}

// halt(q, k, v, eps, o, tile_counts, stream)
PyObject* halt(PyObject* const* a)
{
    const Dims s = dims(a[0], nullptr);
    const at::Tensor& like = THPVariable_Unpack(a[0]);
    void* q = any_shape(a[0], BF, "q");
    void* k = ptr(a[1], BF, s.q, "k");
    void* v = ptr(a[2], BF, s.q, "v");
    const double eps = PyFloat_AsDouble(a[3]);
    if (eps == -1.0 && PyErr_Occurred()) throw Raised{};
    const Launch on = launch_on(a[6]);
    Out o(a[4], BF, s.q, like, "o", on);
    const int64_t two[1] = {2};
    auto* tc = static_cast<unsigned long long*>(ptr(a[5], at::kLong, two, "tile_counts"));
    call("sb_attn_fwd_halt",
         [&] { return sb_attn_fwd_halt(q, k, v, o.p(), (float)eps, tc, s.B, s.H, s.T, s.d, on.stream); });
    return o.take();
}

// forward_f32(q, k, v, o, m, want_m, stream)
PyObject* forward_f32(PyObject* const* a)
{
    const Dims s = dims(a[0], nullptr);
    const at::Tensor& like = THPVariable_Unpack(a[0]);
    auto* q = static_cast<float*>(any_shape(a[0], F32, "q"));
    auto* k = static_cast<float*>(ptr(a[1], F32, s.q, "k"));
    auto* v = static_cast<float*>(ptr(a[2], F32, s.q, "v"));
    const Launch on = launch_on(a[6]);
    Out o(a[3], F32, s.q, like, "o", on);
    auto go = [&](float* m) {
        call("sb_attn_fwd_f32", [&] { return sb_attn_fwd_f32(q, k, v, o.p<float>(), m, s.B, s.H, s.T, s.d, on.stream); });
    };
    if (none(a[4]) && !truth(a[5])) {
        go(nullptr);
        return o.take();
    }
    Out m(a[4], F32, s.m, like, "m", on);
    go(m.p<float>());
    return tuple({&o, &m});
}

// backward(what, grouped, q, k, v, r, m, dout, dq, dk, dv, dr, workspace, stream)
PyObject* backward(PyObject* const* a)
{
    const char* what = PyUnicode_AsUTF8(a[0]);
    if (!what) throw Raised{};
    const Dims s = dims(a[2], a[1] == Py_True ? a[3] : nullptr);
    const at::Tensor& like = THPVariable_Unpack(a[2]);
    void* q = any_shape(a[2], BF, "q");
    void* k = ptr(a[3], BF, s.kv, "k");
    void* v = ptr(a[4], BF, s.kv, "v");
    void* r = ptr(a[5], BF, s.hd, "r");
    auto* m = static_cast<float*>(ptr(a[6], F32, s.m, "m"));
    void* g = ptr(a[7], BF, s.q, "dout");
    const Launch on = launch_on(a[13]);
    Out dq(a[8], F32, s.q, like, "dq", on), dk(a[9], F32, s.kv, like, "dk", on), dv(a[10], F32, s.kv, like, "dv", on);
    Workspace ws(a[12], sb_attn_bwd_gqa_workspace_bytes(s.B, s.H, s.Hkv, s.T, s.d), like, on);
    auto go = [&](float* dr) {
        call(what, [&] {
            return sb_attn_bwd_gqa(q, k, v, r, m, g, dq.p<float>(), dk.p<float>(), dv.p<float>(), dr, ws.p(), ws.bytes(),
                                   s.B, s.H, s.Hkv, s.T, s.d, on.stream);
        });
    };
    if (!r) {
        go(static_cast<float*>(ptr(a[11], F32, s.hd, "dr")));
        return tuple({&dq, &dk, &dv});
    }
    Out dr(a[11], F32, s.hd, like, "dr", on);
    go(dr.p<float>());
    return tuple({&dq, &dk, &dv, &dr});
}

// backward_dq(q, k, v, m, dout, dq, workspace, stream): (dq, workspace), the workspace for backward_dkdv
PyObject* backward_dq(PyObject* const* a)
{
    const Dims s = dims(a[0], nullptr);
    const at::Tensor& like = THPVariable_Unpack(a[0]);
    void* q = any_shape(a[0], BF, "q");
    void* k = ptr(a[1], BF, s.q, "k");
    void* v = ptr(a[2], BF, s.q, "v");
    auto* m = static_cast<float*>(ptr(a[3], F32, s.m, "m"));
    void* g = ptr(a[4], BF, s.q, "dout");
    const Launch on = launch_on(a[7]);
    Out dq(a[5], F32, s.q, like, "dq", on);
    Workspace ws(a[6], sb_attn_bwd_workspace_bytes(s.B, s.H, s.T, s.d), like, on, true);
    call("sb_attn_bwd_dq",
         [&] { return sb_attn_bwd_dq(q, k, v, m, g, dq.p<float>(), ws.p(), ws.bytes(), s.B, s.H, s.T, s.d, on.stream); });
    return Py_BuildValue("(NN)", dq.take(), ws.take());
}

// backward_dkdv(q, k, v, dout, workspace, dk, dv, stream)
PyObject* backward_dkdv(PyObject* const* a)
{
    const Dims s = dims(a[0], nullptr);
    const at::Tensor& like = THPVariable_Unpack(a[0]);
    void* q = any_shape(a[0], BF, "q");
    void* k = ptr(a[1], BF, s.q, "k");
    void* v = ptr(a[2], BF, s.q, "v");
    void* g = ptr(a[3], BF, s.q, "dout");
    const Launch on = launch_on(a[7]);
    Workspace ws(a[4], sb_attn_bwd_workspace_bytes(s.B, s.H, s.T, s.d), like, on);
    Out dk(a[5], F32, s.q, like, "dk", on), dv(a[6], F32, s.q, like, "dv", on);
    call("sb_attn_bwd_dkdv", [&] {
        return sb_attn_bwd_dkdv(q, k, v, g, dk.p<float>(), dv.p<float>(), ws.p(), ws.bytes(), s.B, s.H, s.T, s.d, on.stream);
    });
    return tuple({&dk, &dv});
}

// varlen_forward(q, k, v, cu_seqlens, max_T, r, o, m, want_m, stream)
PyObject* varlen_forward(PyObject* const* a)
{
    const Dims s = dims_packed(a[0], a[1]);
    const at::Tensor& like = THPVariable_Unpack(a[0]);
    const int nseq = (int)tensor(a[3], "cu_seqlens").numel() - 1;
    const int max_T = to_int(a[4]);
    void* q = any_shape(a[0], BF, "q");
    void* k = ptr(a[1], BF, s.kv, "k");
    void* v = ptr(a[2], BF, s.kv, "v");
    auto* cu = static_cast<const int*>(any_shape(a[3], at::kInt, "cu_seqlens"));
    void* r = ptr(a[5], BF, s.hd, "r");
    const Launch on = launch_on(a[9]);
    Out o(a[6], BF, s.q, like, "o", on);
    auto go = [&](float* m) {
        call("sb_attn_varlen_fwd",
             [&] { return sb_attn_varlen_fwd(q, k, v, r, o.p(), m, cu, nseq, s.H, s.Hkv, s.T, max_T, s.d, on.stream); });
    };
    if (none(a[7]) && !truth(a[8])) {
        go(nullptr);
        return o.take();
    }
    Out m(a[7], F32, s.m, like, "m", on);
    go(m.p<float>());
    return tuple({&o, &m});
}

// varlen_backward(q, k, v, m, dout, cu_seqlens, max_T, r, dq, dk, dv, dr, workspace, stream)
PyObject* varlen_backward(PyObject* const* a)
{
    const Dims s = dims_packed(a[0], a[1]);
    const at::Tensor& like = THPVariable_Unpack(a[0]);
    const int nseq = (int)tensor(a[5], "cu_seqlens").numel() - 1;
    const int max_T = to_int(a[6]);
    void* q = any_shape(a[0], BF, "q");
    void* k = ptr(a[1], BF, s.kv, "k");
    void* v = ptr(a[2], BF, s.kv, "v");
    auto* m = static_cast<float*>(ptr(a[3], F32, s.m, "m"));
    void* g = ptr(a[4], BF, s.q, "dout");
    auto* cu = static_cast<const int*>(any_shape(a[5], at::kInt, "cu_seqlens"));
    void* r = ptr(a[7], BF, s.hd, "r");
    const Launch on = launch_on(a[13]);
    Out dq(a[8], F32, s.q, like, "dq", on), dk(a[9], F32, s.kv, like, "dk", on), dv(a[10], F32, s.kv, like, "dv", on);
    Workspace ws(a[12], sb_attn_varlen_bwd_gqa_workspace_bytes(nseq, s.H, s.Hkv, s.T, max_T, s.d), like, on);
    auto go = [&](float* dr) {
        call("sb_attn_varlen_bwd", [&] {
            return sb_attn_varlen_bwd(q, k, v, r, m, g, dq.p<float>(), dk.p<float>(), dv.p<float>(), dr, cu, nseq,
                                      s.H, s.Hkv, s.T, max_T, s.d, ws.p(), ws.bytes(), on.stream);
        });
    };
    if (!r) {
        go(static_cast<float*>(ptr(a[11], F32, s.hd, "dr")));
        return tuple({&dq, &dk, &dv});
    }
    Out dr(a[11], F32, s.hd, like, "dr", on);
    go(dr.p<float>());
    return tuple({&dq, &dk, &dv, &dr});
}

// decode(q, k, v, T, r, o, m, want_m, workspace, stream, static): q [B,H,d], cache [B,Hkv,Tcap,d]
PyObject* decode(PyObject* const* a)
{
    const at::Tensor& tq = tensor(a[0], "q");
    const at::Tensor& tk = tensor(a[1], "k");
    if (tq.dim() != 3) throw Failed("q: expected [B, H, d]");
    if (tk.dim() != 4) throw Failed("expected a [B, H, T, d] tensor");
    const int B = dim(tq, 0), H = dim(tq, 1), d = dim(tq, 2), Hkv = dim(tk, 1), Tcap = dim(tk, 2);
    const int T = none(a[3]) ? Tcap : to_int(a[3]);
    const Shape sq = {B, H, d}, skv = {B, Hkv, Tcap, d}, sr = {H, d}, sm = {B, H};
    void* q = any_shape(a[0], BF, "q");
    void* k = ptr(a[1], BF, skv, "k");
    void* v = ptr(a[2], BF, skv, "v");
    void* r = ptr(a[4], BF, sr, "r");
    const Launch on = launch_on(a[9]);
    const bool in_static = truth(a[10]);
    if (in_static && none(a[5])) throw Failed("sb_attn_decode_static allocates nothing: o is required");
    Out o(a[5], BF, sq, tq, "o", on);
    auto go = [&](float* m) {
        if (in_static) {
            call("sb_attn_decode_static",
                 [&] { return sb_attn_decode_static(q, k, v, r, o.p(), m, B, H, Hkv, T, Tcap, d, on.stream); });
            return;
        }
        Workspace ws(a[8], sb_attn_decode_workspace_bytes(B, H, T, d), tq, on);
        call("sb_attn_decode",
             [&] { return sb_attn_decode(q, k, v, r, o.p(), m, ws.p(), ws.bytes(), B, H, Hkv, T, Tcap, d, on.stream); });
    };
    if (none(a[6]) && !truth(a[7])) {
        go(nullptr);
        return o.take();
    }
    Out m(a[6], F32, sm, tq, "m", on);
    go(m.p<float>());
    return tuple({&o, &m});
}

// set_errors(SbAttnError, torch.cuda.OutOfMemoryError)
PyObject* set_errors(PyObject* const* a)
{
    Py_INCREF(a[0]);
    Py_INCREF(a[1]);
    g_error = a[0];
    g_oom = a[1];
    Py_RETURN_NONE;
}

// argument count, and C++ exceptions into Python ones
template <PyObject* (*F)(PyObject* const*), int N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Raised&) {
    } catch (const Failed& e) {
        PyErr_SetString(g_error ? g_error : PyExc_RuntimeError, e.what());
    } catch (const c10::OutOfMemoryError& e) {
        PyErr_SetString(g_oom ? g_oom : PyExc_MemoryError, e.what_without_backtrace());
    } catch (const c10::Error& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

#define SB_ENTRY(F, N) {#F, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<F, N>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    SB_ENTRY(set_errors, 2), SB_ENTRY(forward, 10), SB_ENTRY(halt, 7), SB_ENTRY(forward_f32, 7),
    SB_ENTRY(backward, 14), SB_ENTRY(backward_dq, 8), SB_ENTRY(backward_dkdv, 8),
    SB_ENTRY(varlen_forward, 10), SB_ENTRY(varlen_backward, 14), SB_ENTRY(decode, 11),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sbtorch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__sbtorch(void) { return PyModule_Create(&module); }
