// Native argument marshalling of the torch-facing wrappers (ops.py): checks
// the tensors, allocates the outputs that the caller did not give, and calls
// the C ABI on the current stream, with the GIL released during the call as a
// ctypes call does.  A wrapper in Python spends 9-11 us per call (the stream
// lookup 2.8, argument checks and conversions 2.5, the kernel launch itself
// 3.2), more than most kernels of a small verify step run; here it is the
// launch and less than 1 us.
//
// Every function takes the wrapper's arguments positionally, in the order of
// its Python signature.  Invalid arguments raise ValueError, a failed call the
// SpecError class handed over by init().
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ops/empty.h>
#include <ATen/ops/zeros.h>

#include <algorithm>
#include <cstdarg>
#include <string>

#include "../../include/spec_fp8.h"

namespace {

using at::ScalarType;
using at::Tensor;

PyObject* g_spec_error = nullptr;

[[noreturn]] void value_error(const char* format, ...) {
    va_list v;
    va_start(v, format);
    PyErr_FormatV(PyExc_ValueError, format, v);
    va_end(v);
    throw python_error();
}

std::string dtype_name(ScalarType t) {
    switch (t) {
        case ScalarType::BFloat16: return "torch.bfloat16";
        case ScalarType::Float: return "torch.float32";
        case ScalarType::Half: return "torch.float16";
        case ScalarType::Double: return "torch.float64";
        case ScalarType::Byte: return "torch.uint8";
        case ScalarType::Char: return "torch.int8";
        case ScalarType::Int: return "torch.int32";
        case ScalarType::Long: return "torch.int64";
        default: return c10::toString(t);
    }
}

// A GPU tensor argument of a given dtype.
const Tensor& dev_any(PyObject* o, const char* name) {
    if (!THPVariable_Check(o) || !THPVariable_Unpack(o).is_cuda())
        value_error("%s must be a CUDA (HIP) tensor", name);
    return THPVariable_Unpack(o);
}

const Tensor& dev(PyObject* o, ScalarType dtype, const char* name) {
    const Tensor& t = dev_any(o, name);
    if (t.scalar_type() != dtype)
        value_error("%s must have dtype %s, got %s", name, dtype_name(dtype).c_str(),
                                dtype_name(t.scalar_type()).c_str());
    return t;
}

// A tensor whose memory the caller answers for (a workspace, token outputs:
// also GPU-visible host memory).
const Tensor& any_tensor(PyObject* o, const char* name) {
    if (!THPVariable_Check(o)) value_error("%s must be a tensor", name);
    return THPVariable_Unpack(o);
}

void need(bool ok, const char* message) {
    if (!ok) value_error("%s", message);
}

// Leading dimension of a 2-D row-major view (unit stride in the last dim).
int64_t rowmajor(const Tensor& t, const char* name) {
    if (t.dim() != 2 || (t.size(1) > 1 && t.stride(1) != 1))
        value_error("%s must be a 2-D row-major view", name);
    return t.size(0) > 1 ? t.stride(0) : std::max(t.size(1), t.stride(0));
}

int64_t bytes_of(const Tensor& t) { return t.numel() * t.element_size(); }

Tensor new_empty(at::IntArrayRef sizes, ScalarType dtype, const Tensor& like) {
    return at::empty(sizes, like.options().dtype(dtype));
}

// An output the caller gave (returned as the same object) or a new one.
struct Out {
    Tensor t;
    PyObject* given = nullptr;
    PyObject* release() {
        if (!given) return THPVariable_Wrap(t);
        Py_INCREF(given);
        return given;
    }
};

template <class Make>
Out out_arg(PyObject* o, ScalarType dtype, const char* name, Make make) {
    Out r;
    if (o == Py_None) {
        r.t = make();
    } else {
        r.t = dev(o, dtype, name);
        r.given = o;
    }
    return r;
}

PyObject* pair(Out& a, Out& b) {
    PyObject* x = a.release();
    PyObject* y = b.release();
    if (!x || !y) {
        Py_XDECREF(x);
        Py_XDECREF(y);
        return nullptr;
    }
    PyObject* r = PyTuple_Pack(2, x, y);
    Py_DECREF(x);
    Py_DECREF(y);
    return r;
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// The call itself, without the GIL.
template <class F>
spec_status call(F f) {
    spec_status st;
    Py_BEGIN_ALLOW_THREADS
    st = f();
    Py_END_ALLOW_THREADS
    return st;
}

void check(const char* fn, spec_status st) {
    if (st == SPEC_OK) return;
    PyObject* e = PyObject_CallFunction(g_spec_error, "si", fn, (int)st);
    if (e) {
        PyErr_SetObject(reinterpret_cast<PyObject*>(Py_TYPE(e)), e);
        Py_DECREF(e);
    }
    throw python_error();
}

bool truth(PyObject* o) {
    const int r = PyObject_IsTrue(o);
    if (r < 0) throw python_error();
    return r != 0;
}

// float(o) of Python, to fp32
float number(PyObject* o) {
    PyObject* f = PyNumber_Float(o);
    if (!f) throw python_error();
    const double v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return (float)v;
}

void args(Py_ssize_t given, Py_ssize_t wanted) {
    if (given != wanted) value_error("expected %d arguments, got %d", (int)wanted, (int)given);
}

#define SPEC_PY(NAME) PyObject* NAME(PyObject*, PyObject* const* a, Py_ssize_t n)

// rows, cols and the input kind of quantize's input
struct QIn {
    int64_t rows, cols, ld;
    spec_quant_input kind;
};
QIn quant_input(const Tensor& x, bool silu) {
    QIn q;
    q.ld = rowmajor(x, "x");
    q.rows = x.size(0);
    q.cols = silu ? x.size(1) / 2 : x.size(1);
    q.kind = silu ? SPEC_QIN_SILU_MUL_BF16 : SPEC_QIN_BF16;
    return q;
}

// quantize(x, per_tensor_scale, silu_mul, out, scales)
SPEC_PY(py_quantize) {
    HANDLE_TH_ERRORS
    args(n, 5);
    const Tensor& x = dev(a[0], ScalarType::BFloat16, "x");
    const QIn q = quant_input(x, truth(a[2]));
    Out out = out_arg(a[3], ScalarType::Byte, "out",
                      [&] { return new_empty({q.rows, q.cols}, ScalarType::Byte, x); });
    const int64_t ld_q = rowmajor(out.t, "out");
    const bool fixed = a[1] != Py_None;
    Out sc = fixed ? out_arg(a[1], ScalarType::Float, "per_tensor_scale", [] { return Tensor(); })
                   : out_arg(a[4], ScalarType::Float, "scales",
                             [&] { return new_empty({q.rows}, ScalarType::Float, x); });
    void* const s = stream();
    check("spec_fp8_quantize", call([&] {
              return spec_fp8_quantize(x.data_ptr(), q.rows, q.cols, q.ld, q.kind,
                                       fixed ? SPEC_SCALE_PER_TENSOR : SPEC_SCALE_PER_ROW,
                                       (float*)sc.t.data_ptr(), (uint8_t*)out.t.data_ptr(), ld_q, s);
          }));
    return pair(out, sc);
    END_HANDLE_TH_ERRORS
}

// calibrate(x, running_scale, silu_mul)
SPEC_PY(py_calibrate) {
    HANDLE_TH_ERRORS
    args(n, 3);
    const Tensor& x = dev(a[0], ScalarType::BFloat16, "x");
    const Tensor& r = dev(a[1], ScalarType::Float, "running_scale");
    need(r.numel() == 1, "running_scale must hold one fp32 value");
    const QIn q = quant_input(x, truth(a[2]));
    void* const s = stream();
    check("spec_fp8_quantize", call([&] {
              return spec_fp8_quantize(x.data_ptr(), q.rows, q.cols, q.ld, q.kind, SPEC_SCALE_CALIBRATE,
                                       (float*)r.data_ptr(), nullptr, 0, s);
          }));
    Py_INCREF(a[1]);
    return a[1];
    END_HANDLE_TH_ERRORS
}

// silu_mul(x, out)
SPEC_PY(py_silu_mul) {
    HANDLE_TH_ERRORS
    args(n, 2);
    const Tensor& x = dev(a[0], ScalarType::BFloat16, "x");
    const QIn q = quant_input(x, true);
    Out out = out_arg(a[1], ScalarType::BFloat16, "out",
                      [&] { return new_empty({q.rows, q.cols}, ScalarType::BFloat16, x); });
    const int64_t ld = rowmajor(out.t, "out");
    void* const s = stream();
    check("spec_silu_mul_bf16",
          call([&] { return spec_silu_mul_bf16(x.data_ptr(), q.rows, q.cols, q.ld, out.t.data_ptr(), ld, s); }));
    return out.release();
    END_HANDLE_TH_ERRORS
}

// clip_count(x, scale, count)
SPEC_PY(py_clip_count) {
    HANDLE_TH_ERRORS
    args(n, 3);
    const Tensor& x = dev(a[0], ScalarType::BFloat16, "x");
    const Tensor& sc = dev(a[1], ScalarType::Float, "scale");
    need(sc.numel() == 1, "scale must hold one fp32 value");
    Out count = out_arg(a[2], ScalarType::Long, "count",
                        [&] { return at::zeros({1}, x.options().dtype(ScalarType::Long)); });
    const QIn q = quant_input(x, false);
    void* const s = stream();
    check("spec_fp8_clip_count", call([&] {
              return spec_fp8_clip_count(x.data_ptr(), q.rows, q.cols, q.ld, (const float*)sc.data_ptr(),
                                         (uint64_t*)count.t.data_ptr(), s);
          }));
    return count.release();
    END_HANDLE_TH_ERRORS
}

// kv_cache_write(k, v, slot_mapping, k_cache, v_cache, k_scale, v_scale, per_tensor)
SPEC_PY(py_kv_cache_write) {
    HANDLE_TH_ERRORS
    args(n, 8);
    const Tensor& k = dev(a[0], ScalarType::BFloat16, "k");
    const Tensor& v = dev(a[1], ScalarType::BFloat16, "v");
    const Tensor& slots = dev(a[2], ScalarType::Long, "slot_mapping");
    const Tensor& kc = dev(a[3], ScalarType::Byte, "k_cache");
    const Tensor& vc = dev(a[4], ScalarType::Byte, "v_cache");
    const Tensor& ks = dev(a[5], ScalarType::Float, "k_scale");
    const Tensor& vs = dev(a[6], ScalarType::Float, "v_scale");
    need(k.dim() == 3 && v.sizes() == k.sizes(), "k and v must be [T, H, D] of the same shape");
    const int64_t T = k.size(0), H = k.size(1), D = k.size(2);
    auto packed = [&](const Tensor& t, const char* name) {
        if ((D > 1 && t.stride(2) != 1) || (H > 1 && t.stride(1) != D))
            value_error("%s must have unit stride over D and heads packed side by side", name);
    };
    packed(k, "k");
    packed(v, "v");
    need(kc.dim() == 3 && kc.size(1) == H && kc.size(2) == D && vc.sizes() == kc.sizes() && kc.is_contiguous() &&
             vc.is_contiguous(),
         "k_cache and v_cache must be contiguous [num_slots, H, D]");
    need(slots.dim() == 1 && slots.size(0) == T && slots.is_contiguous(), "slot_mapping must be a contiguous int64 [T]");
    const int64_t num = kc.size(0);
    const bool fixed = truth(a[7]);
    if (fixed) {
        need(ks.numel() == 1 && vs.numel() == 1, "per-tensor scales hold one fp32 value each");
    } else {
        auto rows = [&](const Tensor& t) {
            return t.dim() == 2 && t.size(0) == num && t.size(1) == H && t.is_contiguous();
        };
        need(rows(ks) && rows(vs), "per-row scales must be contiguous fp32 [num_slots, H]");
    }
    const int64_t ld_k = T > 1 ? k.stride(0) : H * D, ld_v = T > 1 ? v.stride(0) : H * D;
    void* const s = stream();
    check("spec_fp8_kv_cache_write", call([&] {
              return spec_fp8_kv_cache_write(k.data_ptr(), ld_k, v.data_ptr(), ld_v, (const int64_t*)slots.data_ptr(), T,
                                             H, D, num, fixed ? SPEC_SCALE_PER_TENSOR : SPEC_SCALE_PER_ROW,
                                             (float*)ks.data_ptr(), (float*)vs.data_ptr(), (uint8_t*)kc.data_ptr(),
                                             (uint8_t*)vc.data_ptr(), s);
          }));
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

// The operands of a GEMM: a [M, K], w [N, K] and their scales.
struct Operands {
    const Tensor &a, &w, &sa, &sw;
    int64_t M, N, K, lda, ldw;
    spec_scale_mode a_mode, w_mode;
};
Operands operands(PyObject* const* o, const char* mismatch, bool even_rows) {
    const Tensor& a = dev(o[0], ScalarType::Byte, "a");
    const Tensor& w = dev(o[2], ScalarType::Byte, "w");
    const Tensor& sa = dev(o[1], ScalarType::Float, "sa");
    const Tensor& sw = dev(o[3], ScalarType::Float, "sw");
    const int64_t lda = rowmajor(a, "a"), ldw = rowmajor(w, "w");
    const int64_t M = a.size(0), N = w.size(0), K = a.size(1);
    need(w.size(1) == K && (!even_rows || N % 2 == 0), mismatch);
    Operands r{a, w, sa, sw, M, N, K, lda, ldw, SPEC_SCALE_PER_ROW, SPEC_SCALE_PER_ROW};
    if (sa.numel() == 1 && M != 1) r.a_mode = SPEC_SCALE_PER_TENSOR;
    if (sw.numel() == 1 && N != 1) r.w_mode = SPEC_SCALE_PER_TENSOR;
    need(r.a_mode == SPEC_SCALE_PER_TENSOR || sa.numel() >= M, "sa must hold M per-row scales or one per-tensor scale");
    need(r.w_mode == SPEC_SCALE_PER_TENSOR || sw.numel() >= N,
         "sw must hold N per-channel scales or one per-tensor scale");
    return r;
}
#define SPEC_OPERANDS(x) \
    (const uint8_t*)(x).a.data_ptr(), (x).lda, (const float*)(x).sa.data_ptr(), (x).a_mode, \
        (const uint8_t*)(x).w.data_ptr(), (x).ldw, (const float*)(x).sw.data_ptr(), (x).w_mode

// A new [M, N] view of rows padded to 8 elements (the ABI's row stride).
Tensor padded_rows(int64_t M, int64_t N, ScalarType dtype, const Tensor& like) {
    const int64_t ld = (N + 7) / 8 * 8;
    Tensor t = new_empty({M, ld}, dtype, like);
    return ld == N ? t : t.narrow(1, 0, N);
}

// gemm(a, sa, w, sw, out_dtype_is_f32 (None: not a dtype the kernel writes), out, workspace)
SPEC_PY(py_gemm) {
    HANDLE_TH_ERRORS
    args(n, 7);
    const Operands x = operands(a, "a and w disagree on K", false);
    Out out;
    if (a[5] == Py_None) {
        need(a[4] != Py_None, "out must be bf16 or fp32");
        out.t = padded_rows(x.M, x.N, truth(a[4]) ? ScalarType::Float : ScalarType::BFloat16, x.a);
    } else {
        out.t = dev_any(a[5], "out");
        out.given = a[5];
        need(out.t.scalar_type() == ScalarType::BFloat16 || out.t.scalar_type() == ScalarType::Float,
             "out must be bf16 or fp32");
    }
    const spec_out_dtype odt = out.t.scalar_type() == ScalarType::Float ? SPEC_OUT_F32 : SPEC_OUT_BF16;
    const int64_t ldy = rowmajor(out.t, "out");
    void* ws = nullptr;
    size_t ws_bytes = 0;
    Tensor own;                       // a workspace made here, kept until the call is enqueued
    if (a[6] != Py_None) {
        const Tensor& w = any_tensor(a[6], "workspace");
        ws = w.data_ptr();
        ws_bytes = (size_t)bytes_of(w);
    }
    void* const s = stream();
    auto run = [&] {
        return call([&] {
            return spec_fp8_gemm(SPEC_OPERANDS(x), x.M, x.N, x.K, out.t.data_ptr(), ldy, odt, ws, ws_bytes, s);
        });
    };
    spec_status st = run();
    if (st == SPEC_ERR_WORKSPACE) {
        // the shape needs a workspace and none large enough was given (tickets start at zero)
        own = at::zeros({(int64_t)spec_fp8_gemm_workspace_bytes(x.M, x.N, x.K)}, x.a.options());
        ws = own.data_ptr();
        ws_bytes = (size_t)own.numel();
        st = run();
    }
    check("spec_fp8_gemm", st);
    return out.release();
    END_HANDLE_TH_ERRORS
}

// gemm_silu_mul(a, sa, w, sw, out)
SPEC_PY(py_gemm_silu_mul) {
    HANDLE_TH_ERRORS
    args(n, 5);
    const Operands x = operands(a, "w must be [2I, K] with the activations' K", true);
    const int64_t I = x.N / 2;
    Out out = out_arg(a[4], ScalarType::BFloat16, "out",
                      [&] { return padded_rows(x.M, I, ScalarType::BFloat16, x.a); });
    const int64_t ld = rowmajor(out.t, "out");
    void* const s = stream();
    check("spec_fp8_gemm_silu_mul", call([&] {
              return spec_fp8_gemm_silu_mul(SPEC_OPERANDS(x), x.M, I, x.K, out.t.data_ptr(), ld, s);
          }));
    return out.release();
    END_HANDLE_TH_ERRORS
}

// gemm_logit_stats(a, sa, w, sw, temperature, out, stats)
SPEC_PY(py_gemm_logit_stats) {
    HANDLE_TH_ERRORS
    args(n, 7);
    const Operands x = operands(a, "a and w disagree on K", false);
    const float temperature = number(a[4]);
    Out out = out_arg(a[5], ScalarType::BFloat16, "out",
                      [&] { return padded_rows(x.M, x.N, ScalarType::BFloat16, x.a); });
    Out st = out_arg(a[6], ScalarType::Float, "stats", [&] {
        return new_empty({x.M, (int64_t)spec_logit_stats_count(x.M, x.N, x.K), 2}, ScalarType::Float, x.a);
    });
    need(st.t.dim() == 3 && st.t.size(0) == x.M && st.t.size(2) == 2 && st.t.stride(2) == 1 && st.t.stride(1) == 2,
         "stats must be [M, >=G, 2] with contiguous pairs");
    const int64_t ld = rowmajor(out.t, "out");
    void* const s = stream();
    check("spec_fp8_gemm_logit_stats", call([&] {
              return spec_fp8_gemm_logit_stats(SPEC_OPERANDS(x), x.M, x.N, x.K, temperature, out.t.data_ptr(), ld,
                                               (float*)st.t.data_ptr(), st.t.stride(0) / 2, s);
          }));
    return pair(out, st);
    END_HANDLE_TH_ERRORS
}

// The inputs of a chain acceptance: target [B, k+1, V], draft [B, k, V] or
// None, tokens [B, k], uniforms [B, k+1] or None.
struct Chain {
    int64_t B, k, V;
    const void *target, *draft;
    const int32_t* tokens;
    const float* uniforms;
    const Tensor& like;
};
bool shape2(const Tensor& t, int64_t r, int64_t c) {
    return t.dim() == 2 && t.size(0) == r && t.size(1) == c && t.is_contiguous();
}
Chain chain(PyObject* const* a) {
    const Tensor& zt = dev(a[0], ScalarType::BFloat16, "target_logits");
    need(zt.dim() == 3 && zt.is_contiguous(), "target_logits must be contiguous");
    const int64_t B = zt.size(0), k = zt.size(1) - 1, V = zt.size(2);
    Chain c{B, k, V, zt.data_ptr(), nullptr, nullptr, nullptr, zt};
    if (a[1] != Py_None) {
        const Tensor& zd = dev(a[1], ScalarType::BFloat16, "draft_logits");
        need(zd.dim() == 3 && zd.size(0) == B && zd.size(1) == k && zd.size(2) == V && zd.is_contiguous(),
             "draft_logits must be contiguous [B,k,V]");
        c.draft = zd.data_ptr();
    }
    const Tensor& x = dev(a[2], ScalarType::Int, "draft_tokens");
    need(shape2(x, B, k), "draft_tokens must be contiguous [B,k]");
    c.tokens = (const int32_t*)x.data_ptr();
    if (a[3] != Py_None) {
        const Tensor& u = dev(a[3], ScalarType::Float, "uniforms");
        need(shape2(u, B, k + 1), "uniforms must be contiguous [B,k+1]");
        c.uniforms = (const float*)u.data_ptr();
    }
    return c;
}

// An int32 output the caller gave, as it is, or a new one.
Out int_out(PyObject* o, at::IntArrayRef sizes, const Tensor& like, const char* name) {
    Out r;
    if (o == Py_None) {
        r.t = new_empty(sizes, ScalarType::Int, like);
    } else {
        r.t = any_tensor(o, name);
        r.given = o;
    }
    return r;
}

// The caller's workspace if it is large enough, else a new one.
Tensor scratch(PyObject* o, size_t bytes, const Tensor& like) {
    if (o != Py_None) {
        const Tensor& w = any_tensor(o, "workspace");
        if ((size_t)bytes_of(w) >= bytes) return w;
    }
    return new_empty({(int64_t)std::max<size_t>(bytes, 1)}, ScalarType::Byte, like);
}

// verify_accept(target_logits, draft_logits, draft_tokens, uniforms, temperature, workspace, out_tokens,
//               num_accepted, target_stats)
SPEC_PY(py_verify_accept) {
    HANDLE_TH_ERRORS
    args(n, 9);
    const Chain c = chain(a);
    const float temperature = number(a[4]);
    Out out = int_out(a[6], {c.B, c.k + 1}, c.like, "out_tokens");
    Out num = int_out(a[7], {c.B}, c.like, "num_accepted");
    const Tensor ws = scratch(a[5], spec_verify_accept_workspace_bytes(c.B, c.k, c.V), c.like);
    int32_t* const po = (int32_t*)out.t.data_ptr();
    int32_t* const pn = (int32_t*)num.t.data_ptr();
    void* const s = stream();
    if (a[8] == Py_None) {
        check("spec_verify_accept", call([&] {
                  return spec_verify_accept(c.target, c.draft, c.tokens, c.uniforms, c.B, c.k, c.V, temperature, po, pn,
                                            ws.data_ptr(), (size_t)bytes_of(ws), s);
              }));
    } else {
        const Tensor& st = dev(a[8], ScalarType::Float, "target_stats");
        need(st.dim() == 3 && st.size(0) == c.B * (c.k + 1) && st.size(2) == 2 && st.stride(2) == 1 && st.stride(1) == 2,
             "target_stats must be [B*(k+1), G, 2] with contiguous pairs");
        check("spec_verify_accept_stats", call([&] {
                  return spec_verify_accept_stats(c.target, (const float*)st.data_ptr(), st.size(1), st.stride(0) / 2,
                                                  c.draft, c.tokens, c.uniforms, c.B, c.k, c.V, temperature, po, pn,
                                                  ws.data_ptr(), (size_t)bytes_of(ws), s);
              }));
    }
    return pair(out, num);
    END_HANDLE_TH_ERRORS
}

// verify_accept_noalloc(target_logits, draft_logits, draft_tokens, uniforms, temperature, out_tokens, num_accepted)
SPEC_PY(py_verify_accept_noalloc) {
    HANDLE_TH_ERRORS
    args(n, 7);
    const Chain c = chain(a);
    const float temperature = number(a[4]);
    const Tensor& out = dev(a[5], ScalarType::Int, "out_tokens");
    const Tensor& num = dev(a[6], ScalarType::Int, "num_accepted");
    need(shape2(out, c.B, c.k + 1), "out_tokens must be contiguous [B,k+1]");
    need(num.dim() == 1 && num.size(0) == c.B && num.is_contiguous(), "num_accepted must be contiguous [B]");
    void* const s = stream();
    check("spec_verify_accept_noalloc", call([&] {
              return spec_verify_accept_noalloc(c.target, c.draft, c.tokens, c.uniforms, c.B, c.k, c.V, temperature,
                                                (int32_t*)out.data_ptr(), (int32_t*)num.data_ptr(), s);
          }));
    return PyTuple_Pack(2, a[5], a[6]);
    END_HANDLE_TH_ERRORS
}

// verify_accept_tree(target_logits, parents, tokens, uniforms, temperature, workspace, out_tokens, accepted_nodes,
//                    num_accepted)
SPEC_PY(py_verify_accept_tree) {
    HANDLE_TH_ERRORS
    args(n, 9);
    const Tensor& zt = dev(a[0], ScalarType::BFloat16, "target_logits");
    need(zt.dim() == 3 && zt.is_contiguous(), "target_logits must be contiguous");
    const int64_t B = zt.size(0), N = zt.size(1) - 1, V = zt.size(2);
    const Tensor& par = dev(a[1], ScalarType::Int, "parents");
    need(shape2(par, B, N), "parents must be contiguous [B,N]");
    const Tensor& tok = dev(a[2], ScalarType::Int, "tokens");
    need(shape2(tok, B, N), "tokens must be contiguous [B,N]");
    const float* uniforms = nullptr;
    if (a[3] != Py_None) {
        const Tensor& u = dev(a[3], ScalarType::Float, "uniforms");
        need(shape2(u, B, N + 1), "uniforms must be contiguous [B,N+1]");
        uniforms = (const float*)u.data_ptr();
    }
    const float temperature = number(a[4]);
    Out out = int_out(a[6], {B, N + 1}, zt, "out_tokens");
    Out nodes = int_out(a[7], {B, N}, zt, "accepted_nodes");
    Out num = int_out(a[8], {B}, zt, "num_accepted");
    const Tensor ws = scratch(a[5], spec_verify_accept_tree_workspace_bytes(B, N, V), zt);
    void* const s = stream();
    check("spec_verify_accept_tree", call([&] {
              return spec_verify_accept_tree(zt.data_ptr(), (const int32_t*)par.data_ptr(),
                                             (const int32_t*)tok.data_ptr(), uniforms, B, N, V, temperature,
                                             (int32_t*)out.t.data_ptr(), (int32_t*)nodes.t.data_ptr(),
                                             (int32_t*)num.t.data_ptr(), ws.data_ptr(), (size_t)bytes_of(ws), s);
          }));
    PyObject* x = out.release();
    PyObject* y = nodes.release();
    PyObject* z = num.release();
    PyObject* r = x && y && z ? PyTuple_Pack(3, x, y, z) : nullptr;
    Py_XDECREF(x);
    Py_XDECREF(y);
    Py_XDECREF(z);
    return r;
    END_HANDLE_TH_ERRORS
}

// tree_attention_mask(parents, mask, depth)
SPEC_PY(py_tree_attention_mask) {
    HANDLE_TH_ERRORS
    args(n, 3);
    const Tensor& par = dev(a[0], ScalarType::Int, "parents");
    need(par.dim() == 2 && par.is_contiguous(), "parents must be a contiguous int32 [B, N]");
    const int64_t B = par.size(0), N = par.size(1);
    Out mask = out_arg(a[1], ScalarType::Long, "mask", [&] { return new_empty({B, N}, ScalarType::Long, par); });
    Out depth = out_arg(a[2], ScalarType::Int, "depth", [&] { return new_empty({B, N}, ScalarType::Int, par); });
    need(shape2(mask.t, B, N) && shape2(depth.t, B, N), "mask and depth must be contiguous [B, N]");
    void* const s = stream();
    check("spec_tree_attention_mask", call([&] {
              return spec_tree_attention_mask((const int32_t*)par.data_ptr(), B, N, (uint64_t*)mask.t.data_ptr(),
                                              (int32_t*)depth.t.data_ptr(), s);
          }));
    return pair(mask, depth);
    END_HANDLE_TH_ERRORS
}

// init(SpecError)
PyObject* py_init(PyObject*, PyObject* cls) {
    Py_INCREF(cls);
    Py_XDECREF(g_spec_error);
    g_spec_error = cls;
    Py_RETURN_NONE;
}

#define SPEC_METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##NAME)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    SPEC_METHOD(quantize),
    SPEC_METHOD(calibrate),
    SPEC_METHOD(silu_mul),
    SPEC_METHOD(clip_count),
    SPEC_METHOD(kv_cache_write),
    SPEC_METHOD(gemm),
    SPEC_METHOD(gemm_silu_mul),
    SPEC_METHOD(gemm_logit_stats),
    SPEC_METHOD(verify_accept),
    SPEC_METHOD(verify_accept_noalloc),
    SPEC_METHOD(verify_accept_tree),
    SPEC_METHOD(tree_attention_mask),
    {"init", py_init, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_torch_bind", nullptr, -1, g_methods,
                        nullptr,               nullptr,       nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_bind() { return PyModule_Create(&g_module); }
