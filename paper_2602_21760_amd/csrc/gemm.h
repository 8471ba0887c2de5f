// Internal GEMM interface of libhyb: out = epilogue(A W^T + bias), A [m, k] and W [n, k] both
// k-contiguous.  Up to kMaxGroup independent problems with the same (n, k) and epilogue kind run
// in ONE launch (the image- and text-stream GEMMs of a joint block have different weights and
// row counts but the same shape otherwise).
#pragma once
#include "common.h"

enum GemmEpi {
    EPI_BIAS = 0,        // out[r, c] = acc + bias[c]
    EPI_GELU_TANH = 1,   // out[r, c] = GELUtanh(acc + bias[c])
    EPI_SILU = 2,        // out[r, c] = SiLU(acc + bias[c])
    EPI_GATE_RES = 3,    // out[r, c] (fp32) = res[r, c] (+ res2[r, c]) + gate[(r / rows_per_gate) * gate_stride + c] * (acc + bias[c])
    EPI_QKV = 4,         // scatter (acc + bias[c]) to head-major q / k / v (n = 1, 2 or 3 times heads * 64)
    EPI_GEGLU = 5        // out[r, c] = (acc_u + bias[c]) * GELUerf(acc_g + bias[n + c]), W rows [u; g] (2n rows)
};

constexpr int kMaxGroup = 2;

struct GemmProblem {
    const void* a;       // [m, k]
    const void* w;       // [n, k]  (EPI_GEGLU: [2n, k])
    const float* bias;   // [n] or nullptr
    void* out;           // [m, n] of out dtype (unused for EPI_QKV)
    int m;
    // EPI_GATE_RES
    const float* res;
    const float* res2;   // optional second residual
    const float* gate;   // nullptr -> 1
    int rows_per_gate;
    size_t gate_stride;
    // EPI_QKV: row r = (b, t) with t < tokens; column c = (which, head, i), n = 3 * heads * 64;
    // element -> {q,k,v}[((b * heads + head) * n_total) + tok_offset + t][i]
    void* q; void* k; void* v;
    int tokens, tok_offset, n_total, heads;
    float q_scale;       // EPI_QKV: the q part is multiplied by this before it is rounded (0 means 1): lets the attention
                         // kernel take queries that already carry softmax scale x log2(e)
};

struct GemmGroup {
    GemmProblem p[kMaxGroup];
    int count;
    int n, k;
    int n2, k2;          // of the second problem where they differ from the first's (bf16 EPI_QKV launches only); 0: the same
    // Scratch for the MFMA path's k split (single problem, few tiles, long k: see gemm_mfma.hip), or nullptr.
    void* splitk_ws;
    size_t splitk_bytes;
};

// Whether the MFMA kernel of the operand type takes a launch; the plain kernel has the others.
bool hyb_gemm_f32_mfma_takes(const GemmGroup& g, int epi);
bool hyb_gemm_mfma_takes(const GemmGroup& g, hyb_dtype out_dtype, int epi);
// The error that hyb_launch_gemm would return for a launch that no kernel takes, without launching anything.
int hyb_check_gemm(const GemmGroup& g, hyb_dtype in_dtype, hyb_dtype out_dtype, int epi);
// Plain tiled FMA kernel: any shape, fp32 or bf16 operands, fp32 accumulation.
int hyb_launch_gemm_simple(const GemmGroup& g, hyb_dtype in_dtype, hyb_dtype out_dtype, int epi, hipStream_t st);
// fp32 MFMA kernel (k % 16 == 0, n % 4 == 0; every epilogue), for what hyb_gemm_f32_mfma_takes.
int hyb_launch_gemm_f32_mfma(const GemmGroup& g, hyb_dtype out_dtype, int epi, hipStream_t st);
// bf16 MFMA kernel (k % 64 == 0, n % 8 == 0), for what hyb_gemm_mfma_takes.
int hyb_launch_gemm_mfma(const GemmGroup& g, hyb_dtype out_dtype, int epi, hipStream_t st);
// 128 x 128 tiles of an m x n product (two of them fit a CU).
int hyb_gemm_mfma_tiles(int m, int n);
// Large-tile bf16 MFMA kernel (256 x 128 or 192 x 128 tiles, one workgroup per CU).  Same accumulation order as the kernel above, hence
// the same bits per token, but for the order in which a second residual is added (from 32 k-slabs on).  -1 when the shape or
// the epilogue has no large-tile form.
int hyb_launch_gemm_mfma_big(const GemmGroup& g, hyb_dtype out_dtype, int epi, int rows, hipStream_t st);
// At most 16 rows, one wave per 16 features (bias, GELU-tanh, SiLU, gate * y + residual).  -1 for anything else and where the tiles are faster (very wide
// launches).  Same bits as the tiles.
int hyb_launch_gemm_mfma_rows(const GemmGroup& g, hyb_dtype out_dtype, int epi, hipStream_t st);
// Tiles of a launch of 256-column tiles: the first tall_rows[i] tile rows of problem i are `tall` tokens high, the others `shrt`
// (256 and 192, or 192 and 128).
struct WidePlan {
    int tall, shrt;
    int tall_rows[kMaxGroup];
};
// 256-column tiles, one workgroup of eight waves per CU; bf16 output with bias, GELU-tanh, QKV scatter or
// GEGLU, fp32 output with gate * y + residual(s); at least three k-slabs of 64.  Same bits as the 64- and 128-row tiles.
int hyb_launch_gemm_mfma_wide(const GemmGroup& g, hyb_dtype out_dtype, int epi, const WidePlan& plan, hipStream_t st);
// Dispatch: the MFMA kernel of the operand type when it takes the shape, else the plain kernel.
int hyb_launch_gemm(const GemmGroup& g, hyb_dtype in_dtype, hyb_dtype out_dtype, int epi, hipStream_t st);

// Scalar epilogue of the plain kernel (v = acc + bias already applied by the caller where the epilogue needs it).
template <typename OT>
__device__ __forceinline__ void gemm_store_scalar(const GemmProblem& p, int epi, int n, int r, int c, float v) {
    if (epi == EPI_QKV) {
        const int hd = p.heads * 64;
        const int which = c / hd, cc = c % hd, head = cc / 64, i = cc % 64;
        const int b = r / p.tokens, t = r % p.tokens;
        if (which == 0 && p.q_scale != 0.f) v *= p.q_scale;
        OT* base = static_cast<OT*>(which == 0 ? p.q : (which == 1 ? p.k : p.v));
        base[(((size_t)b * p.heads + head) * p.n_total + p.tok_offset + t) * 64 + i] = from_f32<OT>(v);
        return;
    }
    const size_t o = (size_t)r * n + c;
    if (epi == EPI_GELU_TANH) v = gelu_tanh_f(v);
    else if (epi == EPI_SILU) v = silu_f(v);
    else if (epi == EPI_GATE_RES) {
        const float g = p.gate ? p.gate[(size_t)(r / p.rows_per_gate) * p.gate_stride + c] : 1.f;
        v = fmaf(g, v, p.res[o]);
        if (p.res2) v += p.res2[o];
    }
    static_cast<OT*>(p.out)[o] = from_f32<OT>(v);
}

template <typename OT>
__device__ __forceinline__ void gemm_write_four(OT* dst, f32x4 v) {
    if constexpr (sizeof(OT) == 4) *reinterpret_cast<f32x4*>(dst) = v;
    else *reinterpret_cast<bf16x4*>(dst) = bf16x4{(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
}

// Four consecutive features c .. c + 3 (c % 4 == 0, n % 4 == 0) of row r; sums without the bias.  The operands are read and written in fours, the gate row too.
template <typename OT>
__device__ __forceinline__ void gemm_store_four(const GemmProblem& p, int epi, int n, int r, int c, f32x4 v) {
    if (p.bias) v += *reinterpret_cast<const f32x4*>(p.bias + c);
    if (epi == EPI_QKV) {       // four features stay inside a head
        const int hd = p.heads * 64;
        const int which = c / hd, cc = c % hd, head = cc / 64, i = cc % 64;
        const int b = r / p.tokens, t = r % p.tokens;
        if (which == 0 && p.q_scale != 0.f) v *= p.q_scale;
        OT* base = static_cast<OT*>(which == 0 ? p.q : (which == 1 ? p.k : p.v));
        gemm_write_four<OT>(base + (((size_t)b * p.heads + head) * p.n_total + p.tok_offset + t) * 64 + i, v);
        return;
    }
    const size_t o = (size_t)r * n + c;
    if (epi == EPI_GELU_TANH) {
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = gelu_tanh_f(v[j]);
    } else if (epi == EPI_SILU) {
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = silu_f(v[j]);
    } else if (epi == EPI_GATE_RES) {
        const f32x4 res = *reinterpret_cast<const f32x4*>(p.res + o);
        f32x4 g = {1.f, 1.f, 1.f, 1.f};
        if (p.gate) g = *reinterpret_cast<const f32x4*>(p.gate + (size_t)(r / p.rows_per_gate) * p.gate_stride + c);
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = fmaf(g[j], v[j], res[j]);
        if (p.res2) v += *reinterpret_cast<const f32x4*>(p.res2 + o);
    }
    gemm_write_four<OT>(static_cast<OT*>(p.out) + o, v);
}
