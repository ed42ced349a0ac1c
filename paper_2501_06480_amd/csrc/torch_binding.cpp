// Marshalling between torch tensors and the C ABI of libfwa: argument checks, output allocation, the current stream,
// one call.  Nothing is computed here and nothing is kept from call to call.  The same steps in Python took 9 us for a
// forward and 45 us for the forward and backward of a fused qkv tensor (nine views, two dozen attribute reads, two
// calls through ctypes), more than the kernels of the smaller calls run.  The autograd nodes below are native for the
// same reason: a Python function's bookkeeping, and the interpreter that its backward has to enter from the engine's
// thread, left a training step of the smaller calls waiting for the host (stage 3 of Swin-T at batch 128: 92 us a step, 74
// as native nodes, 66 of them kernels).
//
// Each function returns the outputs, or the library's error code as an int for the Python layer to raise.
#include <ATen/ATen.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/utils/pybind.h>

#include <optional>
#include <string>

#include "../../include/fwa.h"

namespace py = pybind11;

namespace {

using OptTensor = std::optional<at::Tensor>;

[[noreturn]] void type_error(const std::string& s) { throw py::type_error(s); }
[[noreturn]] void value_error(const std::string& s) { throw py::value_error(s); }

int dtype_code(const at::Tensor& t) {
    switch (t.scalar_type()) {
        case at::kFloat: return FWA_F32;
        case at::kBFloat16: return FWA_BF16;
        case at::kHalf: return FWA_F16;
        default: type_error("unsupported tensor dtype");
    }
}

void need_gpu(const at::Tensor& t, const char* name) {
    if (!t.is_cuda()) type_error(std::string(name) + " must be a GPU tensor (there is no CPU path)");
}
void need_like(const at::Tensor& t, const char* name, const at::Tensor& q) {
    if (t.sizes() != q.sizes() || t.scalar_type() != q.scalar_type() || t.device() != q.device())
        value_error(std::string(name) + " must match q in shape, dtype and device");
}
const void* dense_ptr(const at::Tensor& t, const char* name, bool f32) {
    need_gpu(t, name);
    if (!t.is_contiguous()) value_error(std::string(name) + " must be contiguous");
    if (f32 && t.scalar_type() != at::kFloat) type_error(std::string(name) + " must be float32");
    return t.data_ptr();
}

// An [N, L, C] tensor whose channels are contiguous and whose token rows are evenly spaced: its device pointer and the
// row stride in elements (C when contiguous).
struct Rows {
    void* p;
    int64_t ld;
};
Rows rows_of(const at::Tensor& t, const char* name, const at::Tensor* like) {
    need_gpu(t, name);
    if (t.dim() != 3) value_error(std::string(name) + " must be [N, L, C]");
    if (like) need_like(t, name, *like);
    const int64_t N = t.size(0), L = t.size(1), C = t.size(2);
    if (t.is_contiguous()) return {t.data_ptr(), C};
    const int64_t s0 = t.stride(0), s1 = t.stride(1), s2 = t.stride(2);
    if ((C > 1 && s2 != 1) || (L > 1 && s1 < C) || (N > 1 && s0 != L * s1))
        value_error(std::string(name) + ": channels must be contiguous and token rows evenly spaced");
    return {t.data_ptr(), L > 1 ? s1 : (N > 1 ? s0 : C)};
}

// The additive terms: bias [heads, L, L] fp32 or bf16, and a dense mask [nW, L, L] or int32 labels [nW, L].
struct Terms {
    const void* bias = nullptr;
    int bias_dtype = FWA_F32;
    const float* mask = nullptr;
    const int32_t* labels = nullptr;
    int nW = 0;
    bool labels_entry() const { return labels != nullptr || bias_dtype == FWA_BF16; }
};
Terms terms_of(const OptTensor& bias, const OptTensor& mask, const OptTensor& labels, int64_t heads, int64_t L) {
    Terms t;
    if (bias) {
        if (bias->dim() != 3 || bias->size(0) != heads || bias->size(1) != L || bias->size(2) != L)
            value_error("bias must be [heads, L, L]");
        if (bias->scalar_type() == at::kBFloat16) t.bias_dtype = FWA_BF16;
        t.bias = dense_ptr(*bias, "bias", t.bias_dtype == FWA_F32);
    }
    if (mask) {
        if (mask->dim() != 3 || mask->size(1) != L || mask->size(2) != L) value_error("mask must be [nW, L, L]");
        if (t.bias_dtype == FWA_BF16)
            value_error("a bf16 bias goes with a mask given as labels (or with no mask), not with a dense mask");
        if (labels) value_error("give the mask either as a dense tensor or as labels, not both");
        t.mask = static_cast<const float*>(dense_ptr(*mask, "mask", true));
        t.nW = (int)mask->size(0);
    }
    if (labels) {
        need_gpu(*labels, "labels");
        if (labels->scalar_type() != at::kInt || labels->dim() != 2 || labels->size(1) != L || !labels->is_contiguous())
            value_error("labels must be a contiguous int32 tensor [nW, L]");
        t.labels = labels->data_ptr<int32_t>();
        t.nW = (int)labels->size(0);
    }
    return t;
}

// Lets other Python threads run during a launch; the autograd engine's threads do not hold the interpreter to begin with.
struct Nogil {
    std::optional<py::gil_scoped_release> released;
    Nogil() { if (PyGILState_Check()) released.emplace(); }
};

void* stream_of(std::optional<uintptr_t> handle, const at::Tensor& t) {
    return handle ? reinterpret_cast<void*>(*handle) : static_cast<void*>(c10::hip::getCurrentHIPStream(t.device().index()).stream());
}

void need_3d(const at::Tensor& q) {
    if (q.dim() != 3) value_error("q must be [N, L, C]");
}

int call_forward(Rows q, Rows k, Rows v, Rows o, const at::Tensor& like, int64_t N, int64_t L, int64_t C, int heads, float scale,
                 const Terms& t, float mask_value, void* stream) {
    if (!(q.ld == k.ld && q.ld == v.ld)) value_error("q, k and v must share one row stride");
    const int dtype = dtype_code(like);
    const c10::DeviceGuard guard(like.device());
    const Nogil nogil;
    if (t.labels_entry())
        return fwa_forward_labels(q.p, k.p, v.p, o.p, N, (int)L, (int)C, heads, scale, q.ld, o.ld, t.bias, t.bias_dtype,
                                  t.labels, mask_value, t.nW, dtype, stream);
    return fwa_forward_strided(q.p, k.p, v.p, o.p, N, (int)L, (int)C, heads, scale, q.ld, o.ld,
                               static_cast<const float*>(t.bias), t.mask, t.nW, dtype, stream);
}

int run_forward(at::Tensor& o, const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, int heads, float scale, const OptTensor& bias,
                const OptTensor& mask, const OptTensor& out, std::optional<uintptr_t> stream, const OptTensor& labels, float mask_value) {
    need_3d(q);
    const int64_t N = q.size(0), L = q.size(1), C = q.size(2);
    need_gpu(q, "q");
    o = out ? *out : at::empty(q.sizes(), q.options());
    const Terms t = terms_of(bias, mask, labels, heads, L);
    return call_forward(rows_of(q, "q", nullptr), rows_of(k, "k", &q), rows_of(v, "v", &q), rows_of(o, "out", &q), q, N, L, C, heads,
                        scale, t, mask_value, stream_of(stream, q));
}
py::object forward(const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, int heads, float scale, const OptTensor& bias,
                   const OptTensor& mask, const OptTensor& out, std::optional<uintptr_t> stream, const OptTensor& labels, float mask_value) {
    at::Tensor o;
    const int rc = run_forward(o, q, k, v, heads, scale, bias, mask, out, stream, labels, mask_value);
    return rc == FWA_OK ? py::cast(o) : py::cast(rc);
}

// q, k, v as the three slices of a contiguous [N, L, 3, heads, d] tensor: slice_of relies on need_qkv
void need_qkv(const at::Tensor& qkv) {
    if (qkv.dim() != 5 || qkv.size(2) != 3 || !qkv.is_contiguous()) value_error("qkv must be a contiguous [N, L, 3, heads, d] tensor");
    need_gpu(qkv, "qkv");
}
Rows slice_of(const at::Tensor& qkv, int which) {
    const int64_t C = qkv.size(3) * qkv.size(4);
    return {static_cast<char*>(qkv.data_ptr()) + which * C * qkv.element_size(), 3 * C};
}

// The library's code, and the output where that is FWA_OK
int run_forward_qkv(at::Tensor& o, const at::Tensor& qkv, float scale, const OptTensor& bias, const OptTensor& mask, const OptTensor& labels,
                    float mask_value) {
    need_qkv(qkv);
    const int64_t N = qkv.size(0), L = qkv.size(1), heads = qkv.size(3), C = heads * qkv.size(4);
    o = at::empty({N, L, C}, qkv.options());
    const Terms t = terms_of(bias, mask, labels, heads, L);
    return call_forward(slice_of(qkv, 0), slice_of(qkv, 1), slice_of(qkv, 2), {o.data_ptr(), C}, qkv, N, L, C, (int)heads, scale, t,
                        mask_value, stream_of(std::nullopt, qkv));
}
py::object forward_qkv(const at::Tensor& qkv, float scale, const OptTensor& bias, const OptTensor& mask, const OptTensor& labels,
                       float mask_value) {
    at::Tensor o;
    const int rc = run_forward_qkv(o, qkv, scale, bias, mask, labels, mask_value);
    return rc == FWA_OK ? py::cast(o) : py::cast(rc);
}

// The workspace of a call when the caller gives none: needed for dBias, and above 64 tokens for the fp32 copy of a bf16 bias
at::Tensor workspace_for(const at::Tensor& like, int64_t N, int64_t L, int64_t C, int heads, bool want_dbias, const Terms& t) {
    if (!want_dbias && !(t.bias_dtype == FWA_BF16 && L > 64)) return at::Tensor();
    const size_t need = fwa_backward_workspace_bytes(N, (int)L, (int)C, heads, dtype_code(like), want_dbias);
    return need ? at::empty({(int64_t)need}, like.options().dtype(at::kByte)) : at::Tensor();
}

int call_backward(const Rows (&r)[7], const at::Tensor& like, const at::Tensor& dbias, int64_t N, int64_t L, int64_t C, int heads,
                  float scale, const Terms& t, float mask_value, const at::Tensor& ws, void* stream) {
    if (!(r[0].ld == r[1].ld && r[0].ld == r[2].ld)) value_error("q, k and v must share one row stride");
    if (!(r[4].ld == r[5].ld && r[4].ld == r[6].ld)) value_error("dq, dk and dv must share one row stride");
    const int dtype = dtype_code(like);
    float* const db = dbias.defined() ? dbias.data_ptr<float>() : nullptr;
    void* const wp = ws.defined() ? ws.data_ptr() : nullptr;
    const size_t wb = ws.defined() ? (size_t)ws.nbytes() : 0;
    const c10::DeviceGuard guard(like.device());
    const Nogil nogil;
    if (t.labels_entry())
        return fwa_backward_labels(r[0].p, r[1].p, r[2].p, r[3].p, r[4].p, r[5].p, r[6].p, db, N, (int)L, (int)C, heads, scale,
                                   r[0].ld, r[3].ld, r[4].ld, t.bias, t.bias_dtype, t.labels, mask_value, t.nW, dtype, wp, wb, stream);
    return fwa_backward_strided(r[0].p, r[1].p, r[2].p, r[3].p, r[4].p, r[5].p, r[6].p, db, N, (int)L, (int)C, heads, scale,
                                r[0].ld, r[3].ld, r[4].ld, static_cast<const float*>(t.bias), t.mask, t.nW, dtype, wp, wb, stream);
}

at::Tensor dbias_like(const at::Tensor& q, int64_t heads, int64_t L, bool want) {
    return want ? at::empty({heads, L, L}, q.options().dtype(at::kFloat)) : at::Tensor();
}
py::object or_none(const at::Tensor& t) { return t.defined() ? py::cast(t) : py::none(); }

struct Grads {
    at::Tensor q, k, v, bias;  // of the fused tensor: q alone
};

int run_backward(Grads& d, const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, const at::Tensor& d_o, int heads, float scale,
                 const OptTensor& bias, const OptTensor& mask, bool want_dbias, const OptTensor& workspace,
                 std::optional<uintptr_t> stream, const OptTensor& dq_out, const OptTensor& dk_out, const OptTensor& dv_out,
                 const OptTensor& labels, float mask_value) {
    need_3d(q);
    const int64_t N = q.size(0), L = q.size(1), C = q.size(2);
    need_gpu(q, "q");
    d.q = dq_out ? *dq_out : at::empty(q.sizes(), q.options());
    d.k = dk_out ? *dk_out : at::empty(q.sizes(), q.options());
    d.v = dv_out ? *dv_out : at::empty(q.sizes(), q.options());
    d.bias = dbias_like(q, heads, L, want_dbias);
    const Terms t = terms_of(bias, mask, labels, heads, L);
    const at::Tensor ws = workspace ? *workspace : workspace_for(q, N, L, C, heads, want_dbias, t);
    const Rows r[7] = {rows_of(q, "q", nullptr), rows_of(k, "k", &q), rows_of(v, "v", &q), rows_of(d_o, "d_o", &q),
                       rows_of(d.q, "dq", &q), rows_of(d.k, "dk", &q), rows_of(d.v, "dv", &q)};
    return call_backward(r, q, d.bias, N, L, C, heads, scale, t, mask_value, ws, stream_of(stream, q));
}
py::object backward(const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, const at::Tensor& d_o, int heads, float scale,
                    const OptTensor& bias, const OptTensor& mask, bool want_dbias, const OptTensor& workspace,
                    std::optional<uintptr_t> stream, const OptTensor& dq_out, const OptTensor& dk_out, const OptTensor& dv_out,
                    const OptTensor& labels, float mask_value) {
    Grads d;
    const int rc = run_backward(d, q, k, v, d_o, heads, scale, bias, mask, want_dbias, workspace, stream, dq_out, dk_out, dv_out, labels, mask_value);
    if (rc != FWA_OK) return py::cast(rc);
    return py::make_tuple(d.q, d.k, d.v, or_none(d.bias));
}

int run_backward_qkv(Grads& d, const at::Tensor& qkv, const at::Tensor& d_o, float scale, const OptTensor& bias, const OptTensor& mask,
                     bool want_dbias, const OptTensor& labels, float mask_value) {
    need_qkv(qkv);
    const int64_t N = qkv.size(0), L = qkv.size(1), heads = qkv.size(3), C = heads * qkv.size(4);
    need_gpu(d_o, "d_o");
    if (d_o.dim() != 3 || d_o.size(0) != N || d_o.size(1) != L || d_o.size(2) != C || d_o.scalar_type() != qkv.scalar_type() ||
        d_o.device() != qkv.device())
        value_error("d_o must match q in shape, dtype and device");
    d.q = at::empty(qkv.sizes(), qkv.options());
    d.bias = dbias_like(qkv, heads, L, want_dbias);
    const Terms t = terms_of(bias, mask, labels, heads, L);
    const at::Tensor ws = workspace_for(qkv, N, L, C, (int)heads, want_dbias, t);
    const Rows r[7] = {slice_of(qkv, 0), slice_of(qkv, 1), slice_of(qkv, 2), rows_of(d_o, "d_o", nullptr),
                       slice_of(d.q, 0), slice_of(d.q, 1), slice_of(d.q, 2)};
    return call_backward(r, qkv, d.bias, N, L, C, (int)heads, scale, t, mask_value, ws, stream_of(std::nullopt, qkv));
}
py::object backward_qkv(const at::Tensor& qkv, const at::Tensor& d_o, float scale, const OptTensor& bias, const OptTensor& mask,
                        bool want_dbias, const OptTensor& labels, float mask_value) {
    Grads d;
    const int rc = run_backward_qkv(d, qkv, d_o, scale, bias, mask, want_dbias, labels, mask_value);
    if (rc != FWA_OK) return py::cast(rc);
    return py::make_tuple(d.q, or_none(d.bias));
}

py::object bias_gather(const at::Tensor& table, int k, std::optional<uintptr_t> stream) {
    if (table.dim() != 2 || table.size(1) != (2LL * k - 1) * (2LL * k - 1)) value_error("table must be [heads, (2k-1)^2]");
    const float* const src = static_cast<const float*>(dense_ptr(table, "table", true));
    const at::Tensor bias = at::empty({table.size(0), (int64_t)k * k, (int64_t)k * k}, table.options());
    float* const dst = bias.data_ptr<float>();
    void* const st = stream_of(stream, table);
    int rc;
    {
        const c10::DeviceGuard guard(table.device());
        const py::gil_scoped_release nogil;
        rc = fwa_bias_gather(src, dst, (int)table.size(0), k, st);
    }
    return rc == FWA_OK ? py::cast(bias) : py::cast(rc);
}

py::object bias_scatter(const at::Tensor& dbias, int k, std::optional<uintptr_t> stream) {
    if (dbias.dim() != 3 || dbias.size(1) != (int64_t)k * k || dbias.size(2) != (int64_t)k * k)
        value_error("dbias must be [heads, k*k, k*k]");
    const float* const src = static_cast<const float*>(dense_ptr(dbias, "dbias", true));
    const at::Tensor dtable = at::empty({dbias.size(0), (2LL * k - 1) * (2LL * k - 1)}, dbias.options());
    float* const dst = dtable.data_ptr<float>();
    void* const st = stream_of(stream, dbias);
    int rc;
    {
        const c10::DeviceGuard guard(dbias.device());
        const py::gil_scoped_release nogil;
        rc = fwa_bias_scatter(src, dst, (int)dbias.size(0), k, st);
    }
    return rc == FWA_OK ? py::cast(dtable) : py::cast(rc);
}

// ------------------------------------------------------------------ autograd
// The two differentiable calls as native nodes.  What they save goes through the engine's saved variables (version counters,
// saved-tensor hooks); an error in the backward reaches Python as the exception that the direct call raises.
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

OptTensor opt(const at::Tensor& t) { return t.defined() ? OptTensor(t) : OptTensor(); }
at::Tensor or_undefined(const OptTensor& t) { return t ? *t : at::Tensor(); }

std::string entry_name(const char* what, const OptTensor& bias, const OptTensor& labels) {
    return std::string(what) + (labels || (bias && bias->scalar_type() == at::kBFloat16) ? "_labels" : "_strided");
}

// `body`, with whatever it raises left as a Python error that may cross the engine's threads
template <class Body>
variable_list with_python_errors(Body body) {
    try {
        return body();
    } catch (py::builtin_exception& e) {
        const py::gil_scoped_acquire gil;
        e.set_error();
        python_error err;
        err.persist();
        throw err;
    }
}
[[noreturn]] void raise_status(int rc, const std::string& entry) {
    const py::gil_scoped_acquire gil;
    const py::object type = py::module_::import("paper_2501_06480_amd.binding").attr("FwaError");
    PyErr_SetObject(type.ptr(), type(rc, entry).ptr());
    python_error err;
    err.persist();
    throw err;
}

// a gradient of the bias that this shape and type do not have is refused in front of the forward
void need_dbias(const at::Tensor& q, int64_t N, int64_t L, int64_t C, int64_t heads, const OptTensor& bias) {
    if (!bias || !bias->requires_grad() || N == 0) return;
    if (fwa_backward_workspace_bytes(N, (int)L, (int)C, (int)heads, dtype_code(q), 1) != 0) return;
    PyErr_SetString(PyExc_NotImplementedError, "the gradient of the bias is not available for this shape and dtype");
    throw py::error_already_set();
}

struct Attention : torch::autograd::Function<Attention> {
    static at::Tensor forward(AutogradContext* ctx, const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, const OptTensor& bias,
                              const OptTensor& mask, const OptTensor& labels, int64_t heads, double scale, double mask_value) {
        ctx->save_for_backward({q, k, v, or_undefined(bias), or_undefined(mask), or_undefined(labels)});
        ctx->saved_data["heads"] = heads;
        ctx->saved_data["scale"] = scale;
        ctx->saved_data["mask_value"] = mask_value;
        at::Tensor o;
        const int rc = run_forward(o, q, k, v, (int)heads, (float)scale, bias, mask, std::nullopt, std::nullopt, labels, (float)mask_value);
        if (rc != FWA_OK) raise_status(rc, entry_name("fwa_forward", bias, labels));
        return o;
    }
    static variable_list backward(AutogradContext* ctx, const variable_list& grads) {
        return with_python_errors([&]() -> variable_list {
            const variable_list s = ctx->get_saved_variables();
            Grads d;
            const int rc = run_backward(d, s[0], s[1], s[2], grads[0].contiguous(), (int)ctx->saved_data["heads"].toInt(),
                                        (float)ctx->saved_data["scale"].toDouble(), opt(s[3]), opt(s[4]), s[3].defined() && ctx->needs_input_grad(3),
                                        std::nullopt, std::nullopt, std::nullopt, std::nullopt, std::nullopt, opt(s[5]),
                                        (float)ctx->saved_data["mask_value"].toDouble());
            if (rc != FWA_OK) raise_status(rc, entry_name("fwa_backward", opt(s[3]), opt(s[5])));
            return {d.q, d.k, d.v, d.bias, at::Tensor(), at::Tensor(), at::Tensor(), at::Tensor(), at::Tensor()};
        });
    }
};
struct AttentionQKV : torch::autograd::Function<AttentionQKV> {
    static at::Tensor forward(AutogradContext* ctx, const at::Tensor& qkv, const OptTensor& bias, const OptTensor& mask,
                              const OptTensor& labels, double scale, double mask_value) {
        ctx->save_for_backward({qkv, or_undefined(bias), or_undefined(mask), or_undefined(labels)});
        ctx->saved_data["scale"] = scale;
        ctx->saved_data["mask_value"] = mask_value;
        at::Tensor o;
        const int rc = run_forward_qkv(o, qkv, (float)scale, bias, mask, labels, (float)mask_value);
        if (rc != FWA_OK) raise_status(rc, entry_name("fwa_forward", bias, labels));
        return o;
    }
    static variable_list backward(AutogradContext* ctx, const variable_list& grads) {
        return with_python_errors([&]() -> variable_list {
            const variable_list s = ctx->get_saved_variables();
            Grads d;
            // a saved-tensor hook may have handed the fused tensor back in another layout
            const int rc = run_backward_qkv(d, s[0].contiguous(), grads[0].contiguous(), (float)ctx->saved_data["scale"].toDouble(), opt(s[1]), opt(s[2]),
                                            s[1].defined() && ctx->needs_input_grad(1), opt(s[3]), (float)ctx->saved_data["mask_value"].toDouble());
            if (rc != FWA_OK) raise_status(rc, entry_name("fwa_backward", opt(s[1]), opt(s[3])));
            return {d.q, d.bias, at::Tensor(), at::Tensor(), at::Tensor(), at::Tensor()};
        });
    }
};

at::Tensor attention(const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, int heads, double scale, const OptTensor& bias,
                     const OptTensor& mask, const OptTensor& labels, double mask_value) {
    need_3d(q);
    need_dbias(q, q.size(0), q.size(1), q.size(2), heads, bias);
    return Attention::apply(q, k, v, bias, mask, labels, (int64_t)heads, scale, mask_value);
}
at::Tensor attention_qkv(const at::Tensor& qkv, double scale, const OptTensor& bias, const OptTensor& mask, const OptTensor& labels, double mask_value) {
    need_qkv(qkv);
    need_dbias(qkv, qkv.size(0), qkv.size(1), qkv.size(3) * qkv.size(4), qkv.size(3), bias);
    return AttentionQKV::apply(qkv, bias, mask, labels, scale, mask_value);
}

}  // namespace

PYBIND11_MODULE(_fwa_torch, m) {
    m.def("forward", &forward);
    m.def("forward_qkv", &forward_qkv);
    m.def("backward", &backward);
    m.def("backward_qkv", &backward_qkv);
    m.def("attention", torch::wrap_pybind_function(&attention));
    m.def("attention_qkv", torch::wrap_pybind_function(&attention_qkv));
    m.def("bias_gather", &bias_gather);
    m.def("bias_scatter", &bias_scatter);
}
