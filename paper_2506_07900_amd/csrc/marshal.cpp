// Python extension behind binding.py: tensors -> pointers and strides -> one call of the library.
//
// A decode step is 20 us on the GPU; marshalling its arguments in Python (seven descriptors, the stream, the parameter
// block, the size query) took 13 us of host time on top of the launches and bounded an eager step.  Here it is under
// 1 us.  Results the caller did not provide are allocated uninitialised; the library clears the rows its kernels leave
// alone in kernels it launches anyway (internal.h), where torch's fills cost a launch and a pass over memory each.
#include <dlfcn.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>

#include <algorithm>
#include <stdexcept>
#include <string>

#include "internal.h"

namespace {

struct MarshalError : std::runtime_error {
    using std::runtime_error::runtime_error;
};

PyObject *g_error = nullptr;                              // binding.InfLLMv2Error

// The library binding.py loaded (libinfllmv2.so, its bench build, or another build named by the caller).
struct Library {
#define INFLLMV2_FN(name) decltype(&infllmv2_##name) name = nullptr
#define INFLLMV2_FNI(name) decltype(&infllmv2i_##name) name = nullptr
    INFLLMV2_FN(status_string);
    INFLLMV2_FN(workspace_bytes);
    INFLLMV2_FN(verify_workspace_bytes);
    INFLLMV2_FN(append_kv);
    INFLLMV2_FN(sparse_attn_decode);
    INFLLMV2_FN(decode_step);
    INFLLMV2_FN(append_kv_verify);
    INFLLMV2_FN(select_blocks_verify);
    INFLLMV2_FN(sparse_attn_verify);
    INFLLMV2_FN(verify_step);
    INFLLMV2_FNI(compress_keys);
    INFLLMV2_FNI(select_blocks);
    INFLLMV2_FNI(sparse_attn_prefill);
    INFLLMV2_FNI(sparse_attn_bwd);
#undef INFLLMV2_FN
#undef INFLLMV2_FNI
} lib;

template <typename F>
void symbol(void *handle, const char *name, F &f) {
    f = reinterpret_cast<F>(dlsym(handle, name));
    if (!f) throw MarshalError(std::string("the library does not export ") + name);
}

const at::Tensor &tensor(PyObject *o, const char *name) {
    if (!THPVariable_Check(o)) throw MarshalError(std::string(name) + " must be a tensor");
    return THPVariable_Unpack(o);
}

const at::Tensor &bf16_4d(PyObject *o, const char *name) {
    if (!THPVariable_Check(o)) throw MarshalError(std::string(name) + " must be a 4-d bf16 device tensor");
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != at::kBFloat16 || t.dim() != 4)
        throw MarshalError(std::string(name) + " must be a 4-d bf16 device tensor");
    if (t.stride(3) != 1) throw MarshalError(std::string(name) + ": head_dim axis must be contiguous");
    return t;
}

// caches, compressed keys, new rows: [B, Hkv, T, d]
infllmv2_tensor cache(const at::Tensor &t) { return {t.data_ptr(), t.stride(0), t.stride(1), t.stride(2)}; }
infllmv2_tensor cache(PyObject *o, const char *name) { return cache(bf16_4d(o, name)); }
// queries, outputs: [B, T, Hq, d]
infllmv2_tensor rows(const at::Tensor &t) { return {t.data_ptr(), t.stride(0), t.stride(2), t.stride(1)}; }
infllmv2_tensor rows(PyObject *o, const char *name) { return rows(bf16_4d(o, name)); }

int32_t *i32(PyObject *o, const char *name) {
    if (THPVariable_Check(o)) {
        const at::Tensor &t = THPVariable_Unpack(o);
        if (t.is_cuda() && t.scalar_type() == at::kInt && t.is_contiguous()) return static_cast<int32_t *>(t.data_ptr());
    }
    throw MarshalError(std::string(name) + " must be a contiguous int32 device tensor");
}

int32_t integer(PyObject *o) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw python_error();
    if (v != static_cast<int32_t>(v)) throw MarshalError("an integer argument does not fit 32 bits");
    return static_cast<int32_t>(v);
}

const infllmv2_params *params(PyObject *o) {
    if (!PyBytes_Check(o) || PyBytes_GET_SIZE(o) != static_cast<Py_ssize_t>(sizeof(infllmv2_params)))
        throw MarshalError("prm must be the packed parameter block");
    return reinterpret_cast<const infllmv2_params *>(PyBytes_AS_STRING(o));
}

void *current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// A result: the caller's tensor, or one made here.
struct Result {
    PyObject *given;
    at::Tensor own;
    explicit Result(PyObject *o) : given(o == Py_None ? nullptr : o) {}
    bool make() const { return given == nullptr; }
    PyObject *release() {
        if (!given) return THPVariable_Wrap(std::move(own));
        Py_INCREF(given);
        return given;
    }
};

// The kernels write every row of a tensor shaped like q (like k): it has no heads or channels beyond the parameters'.
bool q_shaped(const at::Tensor &q, const infllmv2_params *prm) { return q.size(2) == prm->n_q_heads && q.size(3) == prm->head_dim; }
bool k_shaped(const at::Tensor &k, const infllmv2_params *prm) { return k.size(1) == prm->n_kv_heads && k.size(3) == prm->head_dim; }

at::TensorOptions like(const at::Tensor &t, at::ScalarType type) { return at::TensorOptions().dtype(type).device(t.device()); }

// The caller's workspace, or scratch that lives until the call has been enqueued (the allocator reuses it in stream order).
struct Workspace {
    at::Tensor t;
    void *ptr;
    size_t bytes;
    Workspace(PyObject *o, size_t need, const at::Tensor &device_of) {
        t = o == Py_None ? at::empty({static_cast<int64_t>(std::max<size_t>(need, 256))}, like(device_of, at::kByte))
                         : tensor(o, "workspace");
        ptr = t.data_ptr();
        bytes = static_cast<size_t>(t.numel()) * t.element_size();
    }
};

template <typename F>
void run(const char *what, F f) {                         // without the interpreter lock, as any foreign call
    int32_t status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    if (status != INFLLMV2_OK)
        throw MarshalError(std::string(what) + " failed: " + lib.status_string(status) + " (" + std::to_string(status) + ")");
}

PyObject *tuple2(Result &a, Result &b) {
    PyObject *r = PyTuple_New(2);
    PyTuple_SET_ITEM(r, 0, a.release());
    PyTuple_SET_ITEM(r, 1, b.release());
    return r;
}
PyObject *tuple3(Result &a, Result &b, Result &c) {
    PyObject *r = PyTuple_New(3);
    PyTuple_SET_ITEM(r, 0, a.release());
    PyTuple_SET_ITEM(r, 1, b.release());
    PyTuple_SET_ITEM(r, 2, c.release());
    return r;
}

using Args = PyObject *const *;

// (prm, k, seqlens, max_seqlen, ck | None, n_new_tokens)
PyObject *compress_keys(Args a) {
    const infllmv2_params *prm = params(a[0]);
    const at::Tensor &k = bf16_4d(a[1], "k");
    const int32_t T = integer(a[3]), n_new = integer(a[5]);
    Result ck(a[4]);
    int32_t fill = 0;
    if (ck.make()) {
        const bool kernels = prm->kernel_size > 0 && prm->kernel_stride > 0 && T >= prm->kernel_size;   // (the library refuses the rest)
        const int64_t n = kernels ? (T - prm->kernel_size) / prm->kernel_stride + 1 : 0;
        const at::IntArrayRef::value_type shape[4] = {k.size(0), k.size(1), std::max<int64_t>(n, 1), k.size(3)};
        fill = n > 0 && n_new <= 0 && k_shaped(k, prm);   // otherwise the kernel does not visit every row
        ck.own = fill ? at::empty(shape, like(k, at::kBFloat16)) : at::zeros(shape, like(k, at::kBFloat16));
    }
    const infllmv2_tensor kd = cache(k), cd = ck.make() ? cache(ck.own) : cache(ck.given, "ck");
    const int32_t *sl = i32(a[2], "seqlens");
    const int32_t B = static_cast<int32_t>(k.size(0));
    run("infllmv2_compress_keys", [&] { return lib.compress_keys(prm, &kd, sl, B, T, n_new, &cd, current_stream(), fill); });
    return ck.release();
}

// (prm, k_new, v_new, k, v, seqlens, max_seqlen, ck | None)
PyObject *append_kv(Args a) {
    const infllmv2_params *prm = params(a[0]);
    const infllmv2_tensor kn = cache(a[1], "k_new"), vn = cache(a[2], "v_new"), k = cache(a[3], "k"), v = cache(a[4], "v");
    infllmv2_tensor ck{};
    if (a[7] != Py_None) ck = cache(a[7], "ck");
    const int32_t *sl = i32(a[5], "seqlens");
    const int32_t T = integer(a[6]), B = static_cast<int32_t>(tensor(a[3], "k").size(0));
    run("infllmv2_append_kv", [&] {
        return lib.append_kv(prm, &kn, &vn, &k, &v, a[7] != Py_None ? &ck : nullptr, sl, B, T, current_stream());
    });
    Py_RETURN_NONE;
}

// (prm, k_new, v_new, k, v, seqlens, max_seqlen, ck | None)
PyObject *append_kv_verify(Args a) {
    const infllmv2_params *prm = params(a[0]);
    const infllmv2_tensor kn = cache(a[1], "k_new"), vn = cache(a[2], "v_new"), k = cache(a[3], "k"), v = cache(a[4], "v");
    infllmv2_tensor ck{};
    if (a[7] != Py_None) ck = cache(a[7], "ck");
    const int32_t *sl = i32(a[5], "seqlens");
    const int32_t T = integer(a[6]), B = static_cast<int32_t>(tensor(a[3], "k").size(0));
    const int32_t n = static_cast<int32_t>(tensor(a[1], "k_new").size(2));
    run("infllmv2_append_kv_verify", [&] {
        return lib.append_kv_verify(prm, &kn, &vn, &k, &v, a[7] != Py_None ? &ck : nullptr, sl, B, T, n, current_stream());
    });
    Py_RETURN_NONE;
}

// (prm, mode, q, ck, seqlens, max_seqlen, block_idx | None, workspace | None)
PyObject *select_blocks(Args a) {
    const infllmv2_params *prm = params(a[0]);
    const int32_t mode = integer(a[1]), T = integer(a[5]);
    const at::Tensor &q = bf16_4d(a[2], "q");
    const int32_t B = static_cast<int32_t>(q.size(0));
    const bool prefill = mode == INFLLMV2_MODE_PREFILL;
    Result idx(a[6]);
    if (idx.make())                                       // (a decode row is written whole)
        idx.own = at::empty({B, prm->n_kv_heads, prefill ? T : 1, prm->topk}, like(q, at::kInt));
    const int32_t op = prefill ? INFLLMV2_OP_SELECT_PREFILL : INFLLMV2_OP_SELECT_DECODE;
    const Workspace ws(a[7], a[7] == Py_None ? lib.workspace_bytes(op, prm, B, T) : 0, q);
    const infllmv2_tensor qd = rows(q), cd = cache(a[3], "ck");
    const int32_t *sl = i32(a[4], "seqlens");
    int32_t *ip = idx.make() ? static_cast<int32_t *>(idx.own.data_ptr()) : i32(idx.given, "block_idx");
    const int32_t fill = idx.make();
    run("infllmv2_select_blocks",
        [&] { return lib.select_blocks(prm, mode, &qd, &cd, sl, B, T, ip, ws.ptr, ws.bytes, current_stream(), fill); });
    return idx.release();
}

// (prm, q, ck, seqlens, max_seqlen, block_idx | None, workspace | None)
PyObject *select_blocks_verify(Args a) {
    const infllmv2_params *prm = params(a[0]);
    const at::Tensor &q = bf16_4d(a[1], "q");
    const int32_t T = integer(a[4]), B = static_cast<int32_t>(q.size(0)), n = static_cast<int32_t>(q.size(1));
    Result idx(a[5]);
    if (idx.make()) idx.own = at::empty({B, prm->n_kv_heads, n, prm->topk}, like(q, at::kInt));   // every row is written whole
    const Workspace ws(a[6], a[6] == Py_None ? lib.verify_workspace_bytes(INFLLMV2_OP_SELECT_VERIFY, prm, B, T, n) : 0, q);
    const infllmv2_tensor qd = rows(q), cd = cache(a[2], "ck");
    const int32_t *sl = i32(a[3], "seqlens");
    int32_t *ip = idx.make() ? static_cast<int32_t *>(idx.own.data_ptr()) : i32(idx.given, "block_idx");
    run("infllmv2_select_blocks_verify",
        [&] { return lib.select_blocks_verify(prm, &qd, &cd, sl, B, T, n, ip, ws.ptr, ws.bytes, current_stream()); });
    return idx.release();
}

// (prm, q, k, v, seqlens, max_seqlen, block_idx, out | None, lse | None, workspace | None)
PyObject *sparse_attn_prefill(Args a) {
    const infllmv2_params *prm = params(a[0]);
    const at::Tensor &q = bf16_4d(a[1], "q");
    const int32_t T = integer(a[5]), B = static_cast<int32_t>(q.size(0));
    Result out(a[7]), lse(a[8]);
    // the call clears rows up to max_seqlen: only where `out`, shaped like q, has just those.  Rows past max_seqlen of a longer
    // tensor, a tensor shorter than max_seqlen, and a tensor next to one of the caller's (whose other rows stay as they
    // are), are cleared by torch
    const bool fill = out.make() && lse.make() && q.size(1) == T && q_shaped(q, prm);
    if (out.make()) out.own = fill ? at::empty_like(q) : at::zeros_like(q);
    if (lse.make())
        lse.own = fill ? at::empty({B, T, prm->n_q_heads}, like(q, at::kFloat)) : at::zeros({B, T, prm->n_q_heads}, like(q, at::kFloat));
    const Workspace ws(a[9], a[9] == Py_None ? lib.workspace_bytes(INFLLMV2_OP_ATTN_PREFILL, prm, B, T) : 0, q);
    const infllmv2_tensor qd = rows(q), kd = cache(a[2], "k"), vd = cache(a[3], "v"),
                          od = out.make() ? rows(out.own) : rows(out.given, "out");
    const int32_t *sl = i32(a[4], "seqlens"), *ip = i32(a[6], "block_idx");
    float *lp = static_cast<float *>((lse.make() ? lse.own : tensor(lse.given, "lse")).data_ptr());
    run("infllmv2_sparse_attn_prefill", [&] {
        return lib.sparse_attn_prefill(prm, &qd, &kd, &vd, sl, B, T, ip, &od, lp, ws.ptr, ws.bytes, current_stream(), fill);
    });
    return tuple2(out, lse);
}

// (prm, q, k, v, seqlens, max_seqlen, block_idx, out | None, lse | None, workspace | None)
PyObject *sparse_attn_decode(Args a) {
    const infllmv2_params *prm = params(a[0]);
    const at::Tensor &q = bf16_4d(a[1], "q");
    const int32_t T = integer(a[5]), B = static_cast<int32_t>(q.size(0));
    Result out(a[7]), lse(a[8]);
    if (out.make()) out.own = q.size(1) == 1 && q_shaped(q, prm) ? at::empty_like(q) : at::zeros_like(q);           // (every row is written)
    if (lse.make()) lse.own = at::empty({B, prm->n_q_heads}, like(q, at::kFloat));
    const Workspace ws(a[9], a[9] == Py_None ? lib.workspace_bytes(INFLLMV2_OP_ATTN_DECODE, prm, B, T) : 0, q);
    const infllmv2_tensor qd = rows(q), kd = cache(a[2], "k"), vd = cache(a[3], "v"),
                          od = out.make() ? rows(out.own) : rows(out.given, "out");
    const int32_t *sl = i32(a[4], "seqlens"), *ip = i32(a[6], "block_idx");
    float *lp = static_cast<float *>((lse.make() ? lse.own : tensor(lse.given, "lse")).data_ptr());
    run("infllmv2_sparse_attn_decode",
        [&] { return lib.sparse_attn_decode(prm, &qd, &kd, &vd, sl, B, T, ip, &od, lp, ws.ptr, ws.bytes, current_stream()); });
    return tuple2(out, lse);
}

const uint64_t *tree_mask(PyObject *o, int64_t B, int64_t n) {
    if (o == Py_None) return nullptr;
    if (THPVariable_Check(o)) {
        const at::Tensor &t = THPVariable_Unpack(o);
        if (t.is_cuda() && t.scalar_type() == at::kLong && t.is_contiguous() && t.dim() == 2 && t.size(0) == B && t.size(1) == n)
            return static_cast<const uint64_t *>(t.data_ptr());
    }
    throw MarshalError("tree_mask must be a contiguous int64 device tensor [B, n_draft]");
}

// (prm, q, k, v, seqlens, max_seqlen, block_idx, tree_mask | None, out | None, lse | None, workspace | None)
PyObject *sparse_attn_verify(Args a) {
    const infllmv2_params *prm = params(a[0]);
    const at::Tensor &q = bf16_4d(a[1], "q");
    const int32_t T = integer(a[5]), B = static_cast<int32_t>(q.size(0)), n = static_cast<int32_t>(q.size(1));
    Result out(a[8]), lse(a[9]);
    if (out.make()) out.own = q_shaped(q, prm) ? at::empty_like(q) : at::zeros_like(q);
    if (lse.make()) lse.own = at::empty({B, n, prm->n_q_heads}, like(q, at::kFloat));
    const uint64_t *mask = tree_mask(a[7], B, n);
    const Workspace ws(a[10], a[10] == Py_None ? lib.verify_workspace_bytes(INFLLMV2_OP_ATTN_VERIFY, prm, B, T, n) : 0, q);
    const infllmv2_tensor qd = rows(q), kd = cache(a[2], "k"), vd = cache(a[3], "v"),
                          od = out.make() ? rows(out.own) : rows(out.given, "out");
    const int32_t *sl = i32(a[4], "seqlens"), *ip = i32(a[6], "block_idx");
    float *lp = static_cast<float *>((lse.make() ? lse.own : tensor(lse.given, "lse")).data_ptr());
    run("infllmv2_sparse_attn_verify", [&] {
        return lib.sparse_attn_verify(prm, &qd, &kd, &vd, sl, B, T, n, mask, ip, &od, lp, ws.ptr, ws.bytes, current_stream());
    });
    return tuple2(out, lse);
}

// (prm, q, k_new, v_new, k, v, ck, seqlens, max_seqlen, block_idx | None, out | None, lse | None, workspace | None)
PyObject *decode_step(Args a) {
    const infllmv2_params *prm = params(a[0]);
    const at::Tensor &q = bf16_4d(a[1], "q");
    const int32_t T = integer(a[8]), B = static_cast<int32_t>(q.size(0));
    Result idx(a[9]), out(a[10]), lse(a[11]);             // every row of every result is written
    if (idx.make()) idx.own = at::empty({B, prm->n_kv_heads, 1, prm->topk}, like(q, at::kInt));
    if (out.make()) out.own = q.size(1) == 1 && q_shaped(q, prm) ? at::empty_like(q) : at::zeros_like(q);
    if (lse.make()) lse.own = at::empty({B, prm->n_q_heads}, like(q, at::kFloat));
    const Workspace ws(a[12], a[12] == Py_None ? lib.workspace_bytes(INFLLMV2_OP_DECODE_STEP, prm, B, T) : 0, q);
    const infllmv2_tensor qd = rows(q), kn = cache(a[2], "k_new"), vn = cache(a[3], "v_new"), k = cache(a[4], "k"),
                          v = cache(a[5], "v"), ck = cache(a[6], "ck"), od = out.make() ? rows(out.own) : rows(out.given, "out");
    const int32_t *sl = i32(a[7], "seqlens");
    int32_t *ip = idx.make() ? static_cast<int32_t *>(idx.own.data_ptr()) : i32(idx.given, "block_idx");
    float *lp = static_cast<float *>((lse.make() ? lse.own : tensor(lse.given, "lse")).data_ptr());
    run("infllmv2_decode_step", [&] {
        return lib.decode_step(prm, &qd, &kn, &vn, &k, &v, &ck, sl, B, T, ip, &od, lp, ws.ptr, ws.bytes, current_stream());
    });
    return tuple3(idx, out, lse);
}

// (prm, q, k_new, v_new, k, v, ck, seqlens, max_seqlen, tree_mask | None, block_idx | None, out | None, lse | None,
//  workspace | None)
PyObject *verify_step(Args a) {
    const infllmv2_params *prm = params(a[0]);
    const at::Tensor &q = bf16_4d(a[1], "q");
    const int32_t T = integer(a[8]), B = static_cast<int32_t>(q.size(0)), n = static_cast<int32_t>(q.size(1));
    Result idx(a[10]), out(a[11]), lse(a[12]);            // every row of every result is written
    if (idx.make()) idx.own = at::empty({B, prm->n_kv_heads, n, prm->topk}, like(q, at::kInt));
    if (out.make()) out.own = q_shaped(q, prm) ? at::empty_like(q) : at::zeros_like(q);
    if (lse.make()) lse.own = at::empty({B, n, prm->n_q_heads}, like(q, at::kFloat));
    const uint64_t *mask = tree_mask(a[9], B, n);
    const Workspace ws(a[13], a[13] == Py_None ? lib.verify_workspace_bytes(INFLLMV2_OP_VERIFY_STEP, prm, B, T, n) : 0, q);
    const infllmv2_tensor qd = rows(q), kn = cache(a[2], "k_new"), vn = cache(a[3], "v_new"), k = cache(a[4], "k"),
                          v = cache(a[5], "v"), ck = cache(a[6], "ck"), od = out.make() ? rows(out.own) : rows(out.given, "out");
    const int32_t *sl = i32(a[7], "seqlens");
    int32_t *ip = idx.make() ? static_cast<int32_t *>(idx.own.data_ptr()) : i32(idx.given, "block_idx");
    float *lp = static_cast<float *>((lse.make() ? lse.own : tensor(lse.given, "lse")).data_ptr());
    run("infllmv2_verify_step", [&] {
        return lib.verify_step(prm, &qd, &kn, &vn, &k, &v, &ck, sl, B, T, n, mask, ip, &od, lp, ws.ptr, ws.bytes, current_stream());
    });
    return tuple3(idx, out, lse);
}

// (prm, q, k, v, out, dout, lse, seqlens, max_seqlen, block_idx, dq | None, dk | None, dv | None, workspace | None)
PyObject *sparse_attn_bwd(Args a) {
    const infllmv2_params *prm = params(a[0]);
    const at::Tensor &q = bf16_4d(a[1], "q"), &k = bf16_4d(a[2], "k"), &v = bf16_4d(a[3], "v");
    const int32_t T = integer(a[8]), B = static_cast<int32_t>(q.size(0));
    Result dq(a[10]), dk(a[11]), dv(a[12]);
    const bool fill = dq.make() && dk.make() && dv.make() && q.size(1) == T && k.size(2) == T && v.size(2) == T && q_shaped(q, prm) &&
                      k_shaped(k, prm) && k_shaped(v, prm) && k.size(0) == B && v.size(0) == B;   // (as for sparse_attn_prefill)
    if (dq.make()) dq.own = fill ? at::empty_like(q) : at::zeros_like(q);
    if (dk.make()) dk.own = fill ? at::empty_like(k) : at::zeros_like(k);
    if (dv.make()) dv.own = fill ? at::empty_like(v) : at::zeros_like(v);
    const Workspace ws(a[13], a[13] == Py_None ? lib.workspace_bytes(INFLLMV2_OP_ATTN_BWD, prm, B, T) : 0, q);
    const infllmv2_tensor qd = rows(q), kd = cache(k), vd = cache(v), od = rows(a[4], "out"), gd = rows(a[5], "dout"),
                          dqd = dq.make() ? rows(dq.own) : rows(dq.given, "dq"),
                          dkd = dk.make() ? cache(dk.own) : cache(dk.given, "dk"),
                          dvd = dv.make() ? cache(dv.own) : cache(dv.given, "dv");
    const at::Tensor &lse = tensor(a[6], "lse");
    if (!lse.is_cuda() || lse.scalar_type() != at::kFloat || !lse.is_contiguous())
        throw MarshalError("lse must be a contiguous fp32 device tensor");
    const float *lp = static_cast<const float *>(lse.data_ptr());
    const int32_t *sl = i32(a[7], "seqlens"), *ip = i32(a[9], "block_idx");
    run("infllmv2_sparse_attn_bwd", [&] {
        return lib.sparse_attn_bwd(prm, &qd, &kd, &vd, &od, &gd, lp, sl, B, T, ip, &dqd, &dkd, &dvd, ws.ptr, ws.bytes,
                                   current_stream(), fill);
    });
    return tuple3(dq, dk, dv);
}

// (path, error class): the library every later call goes through
PyObject *bind(Args a) {
    const char *path = PyUnicode_AsUTF8(a[0]);
    if (!path) throw python_error();
    Py_INCREF(a[1]);
    Py_XSETREF(g_error, a[1]);
    void *handle = dlopen(path, RTLD_NOW | RTLD_LOCAL);
    if (!handle) throw MarshalError(std::string("cannot load ") + path + ": " + dlerror());
    Library l;
    symbol(handle, "infllmv2_status_string", l.status_string);
    symbol(handle, "infllmv2_workspace_bytes", l.workspace_bytes);
    symbol(handle, "infllmv2_verify_workspace_bytes", l.verify_workspace_bytes);
    symbol(handle, "infllmv2_append_kv", l.append_kv);
    symbol(handle, "infllmv2_sparse_attn_decode", l.sparse_attn_decode);
    symbol(handle, "infllmv2_decode_step", l.decode_step);
    symbol(handle, "infllmv2_append_kv_verify", l.append_kv_verify);
    symbol(handle, "infllmv2_select_blocks_verify", l.select_blocks_verify);
    symbol(handle, "infllmv2_sparse_attn_verify", l.sparse_attn_verify);
    symbol(handle, "infllmv2_verify_step", l.verify_step);
    symbol(handle, "infllmv2i_compress_keys", l.compress_keys);
    symbol(handle, "infllmv2i_select_blocks", l.select_blocks);
    symbol(handle, "infllmv2i_sparse_attn_prefill", l.sparse_attn_prefill);
    symbol(handle, "infllmv2i_sparse_attn_bwd", l.sparse_attn_bwd);
    lib = l;
    Py_RETURN_NONE;
}

template <PyObject *(*F)(Args), int N>
PyObject *entry(PyObject *, Args a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
        return nullptr;
    }
    try {
        return F(a);
    } catch (const MarshalError &e) {
        PyErr_SetString(g_error ? g_error : PyExc_RuntimeError, e.what());
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

#define METHOD(name, n) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<name, n>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    METHOD(bind, 2),
    METHOD(compress_keys, 6),
    METHOD(append_kv, 8),
    METHOD(append_kv_verify, 8),
    METHOD(select_blocks, 8),
    METHOD(select_blocks_verify, 7),
    METHOD(sparse_attn_prefill, 10),
    METHOD(sparse_attn_decode, 10),
    METHOD(sparse_attn_verify, 11),
    METHOD(decode_step, 13),
    METHOD(verify_step, 14),
    METHOD(sparse_attn_bwd, 14),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
