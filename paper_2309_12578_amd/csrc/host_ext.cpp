// Native call path of the Python front end (module _spion_host): argument checks, output and workspace
// allocation from torch's caching allocator, and the autograd node, around the entry points of libspion.
// A forward + backward of a small problem is bound by the host: through ctypes and a Python autograd
// function it took 147 us of host time for 20 us of kernels.
//
// Plain CPython calling convention (METH_FASTCALL) and direct allocation: no dispatcher, no argument
// parsing by format strings.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/autocast_mode.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/autograd/saved_variable.h>
#include <torch/csrc/autograd/variable.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include "spion_host.h"

namespace {

PyObject* g_error_class = nullptr;   // SpionError

// Sets SpionError(code, what); always returns nullptr.
PyObject* spion_error(int code, const char* what) {
    PyObject* e = g_error_class ? PyObject_CallFunction(g_error_class, "is", code, what) : nullptr;
    if (e) {
        PyErr_SetObject(g_error_class, e);
        Py_DECREF(e);
    } else if (!PyErr_Occurred()) {
        PyErr_Format(PyExc_RuntimeError, "%s: %s (%d)", what, spion_strerror(code), code);
    }
    return nullptr;
}

struct SpionFailure {   // thrown with the Python error to set
    int code;
    const char* what;
};

struct BadValue {   // thrown for a ValueError
    const char* msg;
};
[[noreturn]] void bad_value(const char* msg) { throw BadValue{msg}; }

void* device_ptr(const at::Tensor& t) {
    if (!t.is_cuda() || !t.is_contiguous()) bad_value("libspion needs contiguous device tensors");
    return t.data_ptr();
}

const at::Tensor& tensor_arg(PyObject* o) {
    if (!THPVariable_Check(o)) bad_value("libspion needs contiguous device tensors");
    return THPVariable_Unpack(o);
}
at::Tensor optional_arg(PyObject* o) { return o == Py_None ? at::Tensor() : tensor_arg(o); }

int int_arg(PyObject* o) {
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw python_error();
    return (int)v;
}
double double_arg(PyObject* o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw python_error();
    return v;
}

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

at::Tensor new_like(const at::Tensor& t) {
    return at::Tensor(at::detail::empty_cuda(t.sizes(), t.scalar_type(), t.device(), std::nullopt));
}
at::Tensor new_bytes(size_t n, const at::Tensor& like) {
    return at::Tensor(at::detail::empty_cuda({(int64_t)(n < 256 ? 256 : n)}, at::kByte, like.device(), std::nullopt));
}

// One pattern index and the parameters of a call.
struct Index {
    at::Tensor row_ptr, col_idx, col_ptr, row_idx, bsr_pos;
    int nnzb = 0, block = 0;
    float scale = 0.f;
    unsigned flags = 0;
};

spion_attn_params params_of(const at::Tensor& q, const Index& ix) {
    if (q.dim() != 4) bad_value("expected tensors of shape [B, H, L, d]");
    spion_attn_params p;
    p.B = (int32_t)q.size(0);
    p.H = (int32_t)q.size(1);
    p.L = (int32_t)q.size(2);
    p.d = (int32_t)q.size(3);
    p.block = ix.block;
    if (q.scalar_type() == at::kFloat) p.dtype = SPION_F32;
    else if (q.scalar_type() == at::kBFloat16) p.dtype = SPION_BF16;
    else bad_value("unsupported dtype");
    p.scale = ix.scale;
    p.flags = ix.flags;
    return p;
}

// The kernels take every size from Q: a smaller tensor beside it would be read or written past its end.  A larger one,
// a buffer kept for several shapes, has its first elements used.
void room_for(const at::Tensor& q, const at::Tensor& t) {
    if (t.numel() < q.numel() || t.scalar_type() != q.scalar_type())
        bad_value("Q's companions must have its dtype and at least as many elements");
}
void room_for_rows(const at::Tensor& q, const at::Tensor& lse) {
    if (lse.numel() * q.size(3) < q.numel() || lse.scalar_type() != at::kFloat)
        bad_value("LSE must be fp32 with at least B * H * L elements");
}

// For the pieces of long rows (spion_attn_fwd_room), of this call alone: back to the allocator, in the order of the stream,
// when the call returns.
struct Room {
    c10::DataPtr memory;
    size_t bytes;
    void* ptr = nullptr;
    Room(const spion_attn_params& p, int nnzb) : bytes(spion_attn_fwd_room_bytes(&p, nnzb)) {
        if (bytes == 0) return;
        memory = c10::hip::HIPCachingAllocator::get()->allocate(bytes);
        ptr = memory.get();
    }
};

void forward(const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, const Index& ix, at::Tensor& o, at::Tensor& lse) {
    device_ptr(q);
    const spion_attn_params p = params_of(q, ix);
    room_for(q, k);
    room_for(q, v);
    if (!o.defined()) o = new_like(q);
    else room_for(q, o);
    if (!lse.defined())
        lse = at::Tensor(at::detail::empty_cuda({q.size(0), q.size(1), q.size(2)}, at::kFloat, q.device(), std::nullopt));
    else room_for_rows(q, lse);
    const Room room(p, ix.nnzb);
    const int rc = spion_attn_fwd_room(device_ptr(q), device_ptr(k), device_ptr(v), device_ptr(o), (float*)device_ptr(lse),
                                       (const int32_t*)device_ptr(ix.row_ptr), (const int32_t*)device_ptr(ix.col_idx),
                                       ix.nnzb, &p, room.ptr, room.bytes, current_stream());
    if (rc != SPION_OK) throw SpionFailure{rc, "spion_attn_fwd"};
}

void backward(const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, const at::Tensor& o, const at::Tensor& grad,
              const at::Tensor& lse, const Index& ix, at::Tensor& dq, at::Tensor& dk, at::Tensor& dv, at::Tensor& ws) {
    device_ptr(q);
    const spion_attn_params p = params_of(q, ix);
    for (const at::Tensor* t : {&k, &v, &o, &grad}) room_for(q, *t);
    room_for_rows(q, lse);
    for (at::Tensor* t : {&dq, &dk, &dv}) {
        if (!t->defined()) *t = new_like(q);
        else room_for(q, *t);
    }
    if (!ws.defined()) {
        const size_t n = spion_attn_workspace_bytes(&p, ix.nnzb, 1);
        if (n == (size_t)-1) throw SpionFailure{SPION_ERR_SHAPE, "spion_attn_workspace_bytes"};
        ws = new_bytes(n, q);
    }
    const int rc = spion_attn_bwd(device_ptr(q), device_ptr(k), device_ptr(v), device_ptr(o), device_ptr(grad),
                                  (const float*)device_ptr(lse), device_ptr(dq), device_ptr(dk), device_ptr(dv),
                                  (const int32_t*)device_ptr(ix.row_ptr), (const int32_t*)device_ptr(ix.col_idx),
                                  (const int32_t*)device_ptr(ix.col_ptr), (const int32_t*)device_ptr(ix.row_idx),
                                  (const int32_t*)device_ptr(ix.bsr_pos), ix.nnzb, &p, device_ptr(ws),
                                  (size_t)ws.nbytes(), current_stream());
    if (rc != SPION_OK) throw SpionFailure{rc, "spion_attn_bwd"};
}

template <class F>
PyObject* torch_guarded(F&& f) {
    HANDLE_TH_ERRORS
    return f();
    END_HANDLE_TH_ERRORS
}
// Runs f with C++ failures turned into Python errors.
template <class F>
PyObject* guarded(F&& f) {
    try {
        return torch_guarded(f);
    } catch (const SpionFailure& e) {
        return spion_error(e.code, e.what);
    } catch (const BadValue& e) {
        PyErr_SetString(PyExc_ValueError, e.msg);
        return nullptr;
    }
}

bool arg_count(Py_ssize_t got, Py_ssize_t want, const char* name) {
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, got %zd", name, want, got);
    return false;
}

PyObject* wrap(const at::Tensor& t) { return THPVariable_Wrap(t); }

// attn_fwd(Q, K, V, row_ptr, col_idx, nnzb, block, scale, flags, O | None, LSE | None) -> (O, LSE)
PyObject* py_attn_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arg_count(n, 11, "attn_fwd")) return nullptr;
    return guarded([&]() -> PyObject* {
        Index ix;
        ix.row_ptr = tensor_arg(a[3]);
        ix.col_idx = tensor_arg(a[4]);
        ix.nnzb = int_arg(a[5]);
        ix.block = int_arg(a[6]);
        ix.scale = (float)double_arg(a[7]);
        ix.flags = (unsigned)int_arg(a[8]);
        at::Tensor o = optional_arg(a[9]), lse = optional_arg(a[10]);
        forward(tensor_arg(a[0]), tensor_arg(a[1]), tensor_arg(a[2]), ix, o, lse);
        PyObject* r = PyTuple_New(2);
        if (!r) return nullptr;
        PyTuple_SET_ITEM(r, 0, wrap(o));
        PyTuple_SET_ITEM(r, 1, wrap(lse));
        return r;
    });
}

// attn_bwd(Q, K, V, O, dO, LSE, row_ptr, col_idx, col_ptr, row_idx, bsr_pos, nnzb, block, scale, flags,
//          dQ | None, dK | None, dV | None, workspace | None) -> (dQ, dK, dV)
PyObject* py_attn_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arg_count(n, 19, "attn_bwd")) return nullptr;
    return guarded([&]() -> PyObject* {
        Index ix;
        ix.row_ptr = tensor_arg(a[6]);
        ix.col_idx = tensor_arg(a[7]);
        ix.col_ptr = tensor_arg(a[8]);
        ix.row_idx = tensor_arg(a[9]);
        ix.bsr_pos = tensor_arg(a[10]);
        ix.nnzb = int_arg(a[11]);
        ix.block = int_arg(a[12]);
        ix.scale = (float)double_arg(a[13]);
        ix.flags = (unsigned)int_arg(a[14]);
        at::Tensor dq = optional_arg(a[15]), dk = optional_arg(a[16]), dv = optional_arg(a[17]), ws = optional_arg(a[18]);
        backward(tensor_arg(a[0]), tensor_arg(a[1]), tensor_arg(a[2]), tensor_arg(a[3]), tensor_arg(a[4]),
                 tensor_arg(a[5]), ix, dq, dk, dv, ws);
        PyObject* r = PyTuple_New(3);
        if (!r) return nullptr;
        PyTuple_SET_ITEM(r, 0, wrap(dq));
        PyTuple_SET_ITEM(r, 1, wrap(dk));
        PyTuple_SET_ITEM(r, 2, wrap(dv));
        return r;
    });
}

// The gradient of sparse_attention.  Saves what the backward entry point takes; one pass computes all three.
struct SparseAttentionBackward : public torch::autograd::Node {
    torch::autograd::SavedVariable q, k, v, o, lse;
    Index ix;

    std::string name() const override { return "SparseAttentionBackward"; }

    void release_variables() override {
        for (torch::autograd::SavedVariable* s : {&q, &k, &v, &o, &lse}) s->reset_data();
    }

    torch::autograd::variable_list apply(torch::autograd::variable_list&& grads) override {
        torch::autograd::variable_list out(3);
        const at::Tensor& g = grads[0];
        if (!g.defined()) return out;
        at::NoGradGuard no_grad;   // the gradients are not differentiated again
        at::Tensor ws;
        try {
            backward(q.unpack(), k.unpack(), v.unpack(), o.unpack(shared_from_this()), g.contiguous(), lse.unpack(), ix,
                     out[0], out[1], out[2], ws);
        } catch (const SpionFailure& e) {
            PyGILState_STATE gil = PyGILState_Ensure();
            spion_error(e.code, e.what);
            python_error err;
            err.persist();
            PyGILState_Release(gil);
            throw err;
        } catch (const BadValue& e) {
            TORCH_CHECK_VALUE(false, e.msg);
        }
        return out;
    }
};

// sparse_attention(Q, K, V, row_ptr, col_idx, col_ptr, row_idx, bsr_pos, nnzb, block, scale, flags) -> O, or None under
// torch.jit.trace: what is allocated and launched here is not seen by the tracer, which would record O as a constant.
PyObject* py_sparse_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arg_count(n, 12, "sparse_attention")) return nullptr;
    return guarded([&]() -> PyObject* {
        if (torch::jit::tracer::isTracing()) Py_RETURN_NONE;
        const at::Tensor &q = tensor_arg(a[0]), &k = tensor_arg(a[1]), &v = tensor_arg(a[2]);
        Index ix;
        ix.row_ptr = tensor_arg(a[3]);
        ix.col_idx = tensor_arg(a[4]);
        ix.nnzb = int_arg(a[8]);
        ix.block = int_arg(a[9]);
        ix.scale = (float)double_arg(a[10]);
        ix.flags = (unsigned)int_arg(a[11]);
        for (const at::Tensor* t : {&q, &k, &v})
            if (t->_fw_grad(0).defined()) {
                PyErr_SetString(PyExc_NotImplementedError, "sparse_attention has no forward-mode derivative");
                return nullptr;
            }
        const bool grad = torch::autograd::compute_requires_grad(q, k, v);
        at::Tensor o, lse, qc, kc, vc;
        {
            at::NoGradGuard no_grad;
            qc = q.contiguous();
            kc = k.contiguous();
            vc = v.contiguous();
            forward(qc, kc, vc, ix, o, lse);
        }
        if (grad) {
            ix.col_ptr = tensor_arg(a[5]);
            ix.row_idx = tensor_arg(a[6]);
            ix.bsr_pos = tensor_arg(a[7]);
            auto node = std::shared_ptr<SparseAttentionBackward>(new SparseAttentionBackward(), torch::autograd::deleteNode);
            node->set_next_edges(torch::autograd::collect_next_edges(q, k, v));
            node->q = torch::autograd::SavedVariable(qc, false);
            node->k = torch::autograd::SavedVariable(kc, false);
            node->v = torch::autograd::SavedVariable(vc, false);
            node->lse = torch::autograd::SavedVariable(lse, false);
            node->ix = std::move(ix);
            torch::autograd::set_history(o, node);
            node->o = torch::autograd::SavedVariable(o, true);
        }
        return wrap(o);
    });
}

// Whether torch is only computing: nobody traces, transforms, casts or watches its operators.
bool nothing_between() {
    using c10::DispatchKey;
    if (c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::torch_function_mode_enabled()) return false;
    for (DispatchKey k : {DispatchKey::FuncTorchDynamicLayerFrontMode, DispatchKey::Functionalize, DispatchKey::Tracer})
        if (c10::impl::tls_is_dispatch_key_included(k)) return false;
    return !at::autocast::is_autocast_enabled(at::kCUDA);
}
// A plain strided tensor on the current device (whose stream the library is given): no subclass, no wrapper of a
// transform, no view whose values are not those in memory, no tangent.
bool plain(const at::Tensor& t) {
    using c10::DispatchKey;
    for (DispatchKey k : {DispatchKey::Python, DispatchKey::Functionalize, DispatchKey::FuncTorchBatched, DispatchKey::Batched,
                          DispatchKey::FuncTorchGradWrapper, DispatchKey::Negative, DispatchKey::ZeroTensor})
        if (t.key_set().has(k)) return false;
    return t.is_cuda() && t.get_device() == c10::hip::current_device() && t.layout() == at::kStrided && !t._fw_grad(0).defined();
}
bool plain(PyObject* o) { return THPVariable_CheckExact(o) && plain(THPVariable_Unpack(o)); }

// Whether a backward pass may compute in kernels of the library: it is not differentiated itself, backward (grad mode)
// or forward (a tangent on the incoming gradient), nor batched over incoming gradients, nor watched.
bool kernels_may_differentiate(const at::Tensor& grad) {
    return !at::GradMode::is_enabled() && nothing_between() && plain(grad);
}

// The gradient of Y = X W^T + b.  The weight's comes from spion_weight_grad where only numbers are wanted, else, as
// the others, from torch operators.
struct ProjectionBackward : public torch::autograd::Node {
    torch::autograd::SavedVariable x, w;
    bool has_bias = false;

    std::string name() const override { return "ProjectionBackward"; }

    void release_variables() override {
        x.reset_data();
        w.reset_data();
    }

    torch::autograd::variable_list apply(torch::autograd::variable_list&& grads) override {
        torch::autograd::variable_list out(has_bias ? 3 : 2);
        if (!grads[0].defined()) return out;
        const at::Tensor X = x.unpack(), W = w.unpack();
        const int64_t N = W.size(0), M = W.size(1);
        const at::Tensor g = grads[0].reshape({-1, N}), x2 = X.reshape({-1, M});
        if (task_should_compute_output(0)) out[0] = at::mm(g, W).view(X.sizes());
        if (task_should_compute_output(1)) {
            const bool kernel = kernels_may_differentiate(grads[0]) && plain(X);
            out[1] = kernel ? weight_grad(g.contiguous(), x2.contiguous()) : at::mm(g.t(), x2);
        }
        if (has_bias && task_should_compute_output(2)) out[2] = g.sum(0);
        return out;
    }

    static at::Tensor weight_grad(const at::Tensor& g, const at::Tensor& x) {
        const int rows = (int)x.size(0), N = (int)g.size(1), M = (int)x.size(1);
        at::Tensor dw(at::detail::empty_cuda({N, M}, x.scalar_type(), x.device(), std::nullopt));
        const at::Tensor ws = new_bytes(spion_weight_grad_workspace_bytes(rows, N, M), x);
        const int rc = spion_weight_grad(g.data_ptr(), x.data_ptr(), dw.data_ptr(), rows, N, M, ws.data_ptr(),
                                         (size_t)ws.nbytes(), current_stream());
        if (rc == SPION_ERR_PARAM) return at::mm(g.t(), x);   // an operand that is not aligned to 16 bytes
        TORCH_CHECK(rc == SPION_OK, "spion_weight_grad: ", spion_strerror(rc));
        return dw;
    }
};

void heads(bool split, const at::Tensor& merged, const at::Tensor* t, int n) {   // see spion_heads
    void* ptr[3];
    for (int i = 0; i < n; ++i) ptr[i] = t[i].data_ptr();
    const int rc = spion_heads(split, merged.data_ptr(), ptr, (int)t[0].size(0), (int)t[0].size(2), (int)t[0].size(1), n,
                               t[0].scalar_type() == at::kFloat ? SPION_F32 : SPION_BF16, current_stream());
    if (rc != SPION_OK) throw SpionFailure{rc, "spion_heads"};
}

at::Tensor new_heads(const at::Tensor& like, int64_t B, int64_t H, int64_t L) {
    return at::Tensor(at::detail::empty_cuda({B, H, L, 64}, like.scalar_type(), like.device(), std::nullopt));
}

// The kernels read and write the heads where the projections have them (spion_heads_attn_*); for other types and block
// sizes a head split and a head merge go around them.  8 x 2048 tokens, 4 heads, block 32: the sub-layer's step moves
// 26 us of copies less.
bool heads_in_place(const at::Tensor& qkv, const Index& ix) {
    return qkv.scalar_type() == at::kBFloat16 && (ix.block == 32 || ix.block == 64);
}
spion_attn_params heads_params(const at::Tensor& qkv, int64_t H, const Index& ix) {
    spion_attn_params p;
    p.B = (int32_t)qkv.size(0);
    p.H = (int32_t)H;
    p.L = (int32_t)qkv.size(1);
    p.d = 64;
    p.block = ix.block;
    p.dtype = SPION_BF16;
    p.scale = ix.scale;
    p.flags = ix.flags;
    return p;
}

// The gradient of heads_attention.
struct HeadsAttentionBackward : public torch::autograd::Node {
    torch::autograd::SavedVariable q, k, v, o, lse;   // in place: q = qkv, o = the node's output, no k and v
    Index ix;
    int64_t H = 0;
    bool in_place = false;

    std::string name() const override { return "HeadsAttentionBackward"; }

    void release_variables() override {
        for (torch::autograd::SavedVariable* s : {&q, &k, &v, &o, &lse}) s->reset_data();
    }

    torch::autograd::variable_list apply(torch::autograd::variable_list&& grads) override {
        torch::autograd::variable_list out(1);
        if (!grads[0].defined()) return out;
        at::NoGradGuard no_grad;   // the gradients are not differentiated again
        at::Tensor g = grads[0].contiguous(), d[3], ws;
        if ((uintptr_t)g.data_ptr() % 16 != 0) g = g.clone();
        const at::Tensor Q = q.unpack(), O = in_place ? o.unpack(shared_from_this()) : o.unpack();
        const int64_t B = Q.size(0), L = Q.size(in_place ? 1 : 2);
        try {
            if (in_place) {
                const spion_attn_params p = heads_params(Q, H, ix);
                const at::Tensor stat = lse.unpack();
                // what saved-tensor hooks hand back is looked at as the node's own tensors were
                if (Q.dim() != 3 || Q.size(2) != 3 * H * 64 || Q.scalar_type() != at::kBFloat16 || 3 * O.numel() != Q.numel() ||
                    O.scalar_type() != at::kBFloat16 || 3 * g.numel() != Q.numel() || g.scalar_type() != at::kBFloat16 ||
                    stat.numel() != B * H * L || stat.scalar_type() != at::kFloat)
                    bad_value("heads_attention: a saved tensor is not the one that was saved");
                const size_t n = spion_attn_workspace_bytes(&p, ix.nnzb, 1);
                if (n == (size_t)-1) throw SpionFailure{SPION_ERR_SHAPE, "spion_attn_workspace_bytes"};
                ws = new_bytes(n, Q);
                out[0] = new_like(Q);
                const int rc = spion_heads_attn_bwd(
                    device_ptr(Q), device_ptr(O), device_ptr(g), (const float*)device_ptr(stat), device_ptr(out[0]),
                    (const int32_t*)device_ptr(ix.row_ptr), (const int32_t*)device_ptr(ix.col_idx),
                    (const int32_t*)device_ptr(ix.col_ptr), (const int32_t*)device_ptr(ix.row_idx), ix.nnzb, &p,
                    device_ptr(ws), (size_t)ws.nbytes(), current_stream());
                if (rc != SPION_OK) throw SpionFailure{rc, "spion_heads_attn_bwd"};
                return out;
            }
            const at::Tensor dO = new_heads(Q, B, H, L);
            heads(true, g, &dO, 1);
            backward(Q, k.unpack(), v.unpack(), O, dO, lse.unpack(), ix, d[0], d[1], d[2], ws);
            out[0] = at::Tensor(at::detail::empty_cuda({B, L, 3 * H * 64}, Q.scalar_type(), Q.device(), std::nullopt));
            heads(false, out[0], d, 3);
        } catch (const SpionFailure& e) {
            PyGILState_STATE gil = PyGILState_Ensure();
            spion_error(e.code, e.what);
            python_error err;
            err.persist();
            PyGILState_Release(gil);
            throw err;
        } catch (const BadValue& e) {
            TORCH_CHECK_VALUE(false, e.msg);
        }
        return out;
    }
};

// heads_attention(qkv [B, L, 3 H 64], H, row_ptr, col_idx, col_ptr, row_idx, bsr_pos, nnzb, block, flags, apart = False)
// -> [B, L, H 64]: every head's attention as one node; None where the steps are to be taken one by one (see projection).
// apart: the node saves copies, so that the caller may let qkv and the result be changed in place before the backward pass.
PyObject* py_heads_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 11 && !arg_count(n, 10, "heads_attention")) return nullptr;
    return guarded([&]() -> PyObject* {
        if (!nothing_between() || !plain(a[0])) Py_RETURN_NONE;
        const at::Tensor& qkv = THPVariable_Unpack(a[0]);
        const int64_t H = int_arg(a[1]);
        const bool f32 = qkv.scalar_type() == at::kFloat;
        if ((!f32 && qkv.scalar_type() != at::kBFloat16) || qkv.dim() != 3 || !qkv.is_contiguous() || H <= 0 ||
            qkv.size(2) != 3 * H * 64 || qkv.size(1) % 4 != 0 || qkv.numel() == 0 ||
            qkv.numel() / (f32 ? 4 : 8) >= 0x7fffffffll || (uintptr_t)qkv.data_ptr() % 16 != 0)
            Py_RETURN_NONE;
        const int64_t B = qkv.size(0), L = qkv.size(1);
        Index ix;
        ix.row_ptr = tensor_arg(a[2]);
        ix.col_idx = tensor_arg(a[3]);
        ix.nnzb = int_arg(a[7]);
        ix.block = int_arg(a[8]);
        ix.flags = (unsigned)int_arg(a[9]);
        const bool grad = torch::autograd::compute_requires_grad(qkv);
        const bool in_place = heads_in_place(qkv, ix) && !(grad && n == 11 && a[10] == Py_True);
        at::Tensor t[3], o, lse, s;
        if (in_place) {
            const spion_attn_params p = heads_params(qkv, H, ix);
            s = at::Tensor(at::detail::empty_cuda({B, L, H * 64}, qkv.scalar_type(), qkv.device(), std::nullopt));
            lse = at::Tensor(at::detail::empty_cuda({B, H, L}, at::kFloat, qkv.device(), std::nullopt));
            const Room room(p, ix.nnzb);
            const int rc = spion_heads_attn_fwd(device_ptr(qkv), device_ptr(s), (float*)device_ptr(lse),
                                                (const int32_t*)device_ptr(ix.row_ptr), (const int32_t*)device_ptr(ix.col_idx),
                                                ix.nnzb, &p, room.ptr, room.bytes, current_stream());
            if (rc != SPION_OK) throw SpionFailure{rc, "spion_heads_attn_fwd"};
        } else {
            at::NoGradGuard no_grad;
            for (at::Tensor& x : t) x = new_heads(qkv, B, H, L);
            heads(true, qkv, t, 3);
            forward(t[0], t[1], t[2], ix, o, lse);
            s = at::Tensor(at::detail::empty_cuda({B, L, H * 64}, qkv.scalar_type(), qkv.device(), std::nullopt));
            heads(false, s, &o, 1);
        }
        if (grad) {
            ix.col_ptr = tensor_arg(a[4]);
            ix.row_idx = tensor_arg(a[5]);
            ix.bsr_pos = tensor_arg(a[6]);
            auto node = std::shared_ptr<HeadsAttentionBackward>(new HeadsAttentionBackward(), torch::autograd::deleteNode);
            node->set_next_edges(torch::autograd::collect_next_edges(qkv));
            node->H = H;
            node->in_place = in_place;
            node->lse = torch::autograd::SavedVariable(lse, false);
            node->ix = std::move(ix);
            torch::autograd::set_history(s, node);
            if (in_place) {
                node->q = torch::autograd::SavedVariable(qkv, false);
                node->o = torch::autograd::SavedVariable(s, true);
            } else {
                node->q = torch::autograd::SavedVariable(t[0], false);
                node->k = torch::autograd::SavedVariable(t[1], false);
                node->v = torch::autograd::SavedVariable(t[2], false);
                node->o = torch::autograd::SavedVariable(o, false);
            }
        }
        return wrap(s);
    });
}

// The gradient of layer_norm, all three in one pass over X and dY; torch's operator where more than numbers is wanted.  A
// second incoming gradient is that of a residual from X (see residual), whose sum with dX the same pass writes.
struct NormBackward : public torch::autograd::Node {
    torch::autograd::SavedVariable x, w, b, mean, rstd;

    std::string name() const override { return "NormBackward"; }

    void release_variables() override {
        for (torch::autograd::SavedVariable* s : {&x, &w, &b, &mean, &rstd}) s->reset_data();
    }

    torch::autograd::variable_list apply(torch::autograd::variable_list&& grads) override {
        torch::autograd::variable_list out(3);
        const at::Tensor dr = grads.size() > 1 ? grads[1] : at::Tensor();
        if (!grads[0].defined()) {
            out[0] = dr;
            return out;
        }
        const at::Tensor X = x.unpack(), W = w.unpack(), m = mean.unpack(), r = rstd.unpack();
        const int64_t D = W.size(0);
        const at::Tensor g = grads[0].contiguous();
        if (!kernels_may_differentiate(grads[0]) || !plain(X) || !plain(W) || (uintptr_t)g.data_ptr() % 16 != 0) {
            std::vector<int64_t> stat(X.sizes().begin(), X.sizes().end());
            stat.back() = 1;
            std::tie(out[0], out[1], out[2]) = at::native_layer_norm_backward(
                g, X, {D}, m.view(stat), r.view(stat), W, b.unpack(),
                {task_should_compute_output(0), task_should_compute_output(1), task_should_compute_output(2)});
            if (dr.defined() && out[0].defined()) out[0] = out[0] + dr;   // X's gradient may not be asked for
            return out;
        }
        const bool add = dr.defined() && plain(dr) && dr.scalar_type() == X.scalar_type() && dr.is_contiguous() &&
                         dr.sizes() == X.sizes() && (uintptr_t)dr.data_ptr() % 16 == 0;
        const int rows = (int)(X.numel() / D);
        for (at::Tensor* t : {&out[0], &out[1], &out[2]}) *t = new_like(t == &out[0] ? X : W);
        const at::Tensor ws = new_bytes(spion_layer_norm_workspace_bytes(rows, (int)D), X);
        const int rc = spion_layer_norm_grad(g.data_ptr(), add ? dr.data_ptr() : nullptr, X.data_ptr(), W.data_ptr(), m.data_ptr<float>(), r.data_ptr<float>(),
                                             out[0].data_ptr(), out[1].data_ptr(), out[2].data_ptr(), rows, (int)D,
                                             X.scalar_type() == at::kFloat ? SPION_F32 : SPION_BF16, ws.data_ptr(),
                                             (size_t)ws.nbytes(), current_stream());
        TORCH_CHECK(rc == SPION_OK, "spion_layer_norm_grad: ", spion_strerror(rc));
        if (dr.defined() && !add) out[0] = out[0] + dr;
        for (int i = 0; i < 3; ++i)
            if (!task_should_compute_output(i)) out[i].reset();
        return out;
    }
};

// layer_norm(X, w, b, eps) -> Y over the last dimension, or None where torch's operator is to be called (see projection).
PyObject* py_layer_norm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arg_count(n, 4, "layer_norm")) return nullptr;
    return guarded([&]() -> PyObject* {
        if (!nothing_between() || !plain(a[0]) || !plain(a[1]) || !plain(a[2])) Py_RETURN_NONE;
        const at::Tensor &x = THPVariable_Unpack(a[0]), &w = THPVariable_Unpack(a[1]), &b = THPVariable_Unpack(a[2]);
        const auto type = x.scalar_type();
        if ((type != at::kFloat && type != at::kBFloat16) || w.scalar_type() != type || b.scalar_type() != type ||
            x.device() != w.device() || x.device() != b.device() || w.dim() != 1 || x.dim() < 2 || x.numel() == 0)
            Py_RETURN_NONE;
        const int64_t D = w.size(0);
        if (b.dim() != 1 || b.size(0) != D || x.size(-1) != D || D % 64 != 0 || D > 2048 || x.numel() / D > 0x40000000 ||
            !x.is_contiguous() || !w.is_contiguous() || !b.is_contiguous() ||
            ((uintptr_t)x.data_ptr() | (uintptr_t)w.data_ptr() | (uintptr_t)b.data_ptr()) % 16 != 0)
            Py_RETURN_NONE;
        const int64_t rows = x.numel() / D;
        at::Tensor y = new_like(x), mean(at::detail::empty_cuda({rows}, at::kFloat, x.device(), std::nullopt)),
                   rstd(at::detail::empty_cuda({rows}, at::kFloat, x.device(), std::nullopt));
        const int rc = spion_layer_norm(x.data_ptr(), w.data_ptr(), b.data_ptr(), y.data_ptr(), mean.data_ptr<float>(),
                                        rstd.data_ptr<float>(), (int)rows, (int)D, (float)double_arg(a[3]),
                                        type == at::kFloat ? SPION_F32 : SPION_BF16, current_stream());
        if (rc != SPION_OK) throw SpionFailure{rc, "spion_layer_norm"};
        if (torch::autograd::compute_requires_grad(x, w, b)) {
            auto node = std::shared_ptr<NormBackward>(new NormBackward(), torch::autograd::deleteNode);
            node->set_next_edges(torch::autograd::collect_next_edges(x, w, b));
            node->x = torch::autograd::SavedVariable(x, false);
            node->w = torch::autograd::SavedVariable(w, false);
            node->b = torch::autograd::SavedVariable(b, false);
            node->mean = torch::autograd::SavedVariable(mean, false);
            node->rstd = torch::autograd::SavedVariable(rstd, false);
            torch::autograd::set_history(y, node);
        }
        return wrap(y);
    });
}

// residual(X, Y) -> X for a residual around Y = layer_norm(X): an alias whose gradient goes to Y's node, which adds it to
// its own, instead of an addition after it; X itself where Y did not come from that node alone.
PyObject* py_residual(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arg_count(n, 2, "residual")) return nullptr;
    return guarded([&]() -> PyObject* {
        auto as_it_is = [&]() {
            Py_INCREF(a[0]);
            return a[0];
        };
        if (!nothing_between() || !plain(a[0]) || !plain(a[1]) || !at::GradMode::is_enabled()) return as_it_is();
        const at::Tensor &x = THPVariable_Unpack(a[0]), &y = THPVariable_Unpack(a[1]);
        if (!x.requires_grad() || !y.grad_fn()) return as_it_is();
        const auto node = std::dynamic_pointer_cast<NormBackward>(y.grad_fn());
        if (!node || node->num_inputs() != 1 || node->next_edge(0) != torch::autograd::impl::gradient_edge(x)) return as_it_is();
        at::Tensor r;
        {
            at::NoGradGuard no_grad;
            r = x.detach();
        }
        torch::autograd::set_history(r, node);
        return wrap(r);
    });
}

// projection(X, W, b | None) -> X W^T + b with the node above, or None where torch's own operator is to be called:
// nothing to differentiate, types or sizes the kernel does not take, or more than plain tensors in play.  Weights of
// more than 2^20 elements are torch's: with that many output tiles its product fills the machine.  Weight gradient,
// kernel / torch's product, us on the GPU: 1024 x 1024 at 4096, 8192, 16384 and 32768 tokens 32 / 29, 42 / 54, 67 / 103,
// 118 / 200; 1536 x 768 40 / 33, 61 / 61, 105 / 118, 193 / 200; 2304 x 768 67 / 35, 113 / 64, 206 / 127, 391 / 297.
// Up to 2048 tokens the product is the faster one on the GPU (1536 x 512 at 2048: 25 / 18; 256 x 256 at 256: 13 / 10), but
// the host takes longer to launch it and sets the pace there: forward and backward of the sub-layer with the product
// instead of the kernel for both weights took 300 us a call in place of 275.
PyObject* py_projection(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arg_count(n, 3, "projection")) return nullptr;
    return guarded([&]() -> PyObject* {
        if (!nothing_between() || !plain(a[0]) || !plain(a[1]) || (a[2] != Py_None && !plain(a[2]))) Py_RETURN_NONE;
        const at::Tensor &x = THPVariable_Unpack(a[0]), &w = THPVariable_Unpack(a[1]), b = optional_arg(a[2]);
        if (x.scalar_type() != at::kBFloat16 || w.scalar_type() != at::kBFloat16 || x.device() != w.device() ||
            x.dim() < 2 || w.dim() != 2 || !w.is_contiguous() || x.size(-1) != w.size(1) || x.numel() == 0 ||
            w.size(0) % 8 != 0 || w.size(1) % 8 != 0 || w.numel() == 0 || w.numel() > (1 << 20) ||
            x.numel() / x.size(-1) > 0x7fffffff - 4096)   // the kernel's row numbers run a little past the last
            Py_RETURN_NONE;
        if (!torch::autograd::compute_requires_grad(w)) Py_RETURN_NONE;
        at::Tensor y;
        {
            at::NoGradGuard no_grad;
            y = at::linear(x, w, b.defined() ? std::optional<at::Tensor>(b) : std::nullopt);
        }
        auto node = std::shared_ptr<ProjectionBackward>(new ProjectionBackward(), torch::autograd::deleteNode);
        node->has_bias = b.defined();
        node->set_next_edges(b.defined() ? torch::autograd::collect_next_edges(x, w, b) : torch::autograd::collect_next_edges(x, w));
        node->x = torch::autograd::SavedVariable(x, false);
        node->w = torch::autograd::SavedVariable(w, false);
        torch::autograd::set_history(y, node);
        return wrap(y);
    });
}

// generate_pattern(A_s, L, block, filter, mode, value, flags, fl_out, row_ptr, col_idx, col_ptr, row_idx, bsr_pos,
//                  nnzb, pool_sum, workspace | None) -> nnzb, after the pattern is complete
PyObject* py_generate_pattern(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arg_count(n, 16, "generate_pattern")) return nullptr;
    return guarded([&]() -> PyObject* {
        const at::Tensor& A = tensor_arg(a[0]);
        device_ptr(A);
        spion_pattern_params p;
        p.L = int_arg(a[1]);
        p.block = int_arg(a[2]);
        p.filter = int_arg(a[3]);
        p.thresh_mode = int_arg(a[4]);
        p.thresh_value = double_arg(a[5]);
        p.flags = (uint32_t)int_arg(a[6]);
        p.reserved = 0;
        void* ptr[8];
        for (int i = 0; i < 8; ++i) ptr[i] = a[7 + i] == Py_None ? nullptr : device_ptr(tensor_arg(a[7 + i]));
        at::Tensor ws = optional_arg(a[15]);
        if (!ws.defined()) ws = new_bytes(spion_pattern_workspace_bytes(p.L, p.block), A);
        void *score = device_ptr(A), *work = device_ptr(ws), *stream = current_stream();
        const size_t work_bytes = (size_t)ws.nbytes();
        int32_t nnzb = -1;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = spion_pattern_wait((const float*)score, &p, (uint8_t*)ptr[0], (int32_t*)ptr[1], (int32_t*)ptr[2],
                                (int32_t*)ptr[3], (int32_t*)ptr[4], (int32_t*)ptr[5], (int32_t*)ptr[6], (int64_t*)ptr[7],
                                work, work_bytes, stream, &nnzb);
        Py_END_ALLOW_THREADS
        if (rc != SPION_OK) throw SpionFailure{rc, "spion_pattern"};
        return PyLong_FromLong(nnzb);
    });
}

PyObject* py_set_error_class(PyObject*, PyObject* cls) {
    Py_INCREF(cls);
    Py_XSETREF(g_error_class, cls);
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"attn_fwd", (PyCFunction)(void*)py_attn_fwd, METH_FASTCALL, nullptr},
    {"attn_bwd", (PyCFunction)(void*)py_attn_bwd, METH_FASTCALL, nullptr},
    {"sparse_attention", (PyCFunction)(void*)py_sparse_attention, METH_FASTCALL, nullptr},
    {"heads_attention", (PyCFunction)(void*)py_heads_attention, METH_FASTCALL, nullptr},
    {"layer_norm", (PyCFunction)(void*)py_layer_norm, METH_FASTCALL, nullptr},
    {"residual", (PyCFunction)(void*)py_residual, METH_FASTCALL, nullptr},
    {"projection", (PyCFunction)(void*)py_projection, METH_FASTCALL, nullptr},
    {"generate_pattern", (PyCFunction)(void*)py_generate_pattern, METH_FASTCALL, nullptr},
    {"set_error_class", py_set_error_class, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_spion_host", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__spion_host(void) { return PyModule_Create(&kModule); }
