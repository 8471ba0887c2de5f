// bf16 MFMA GEMM for gfx950 of at most 16 rows: the same contraction as gemm_mfma.hip (out = epilogue(A W^T + bias), fp32 accumulation in
// v_mfma_f32_16x16x32_bf16), the timestep and pooled-text MLPs of a denoiser, one row per sample.
//
// What bounds it is latency: the 64 x 128 tiles of the general kernel give such a launch n / 128 workgroups (12 for a width of 1536)
// that copy one slab after the other through LDS.  Here a wave alone owns 16 features and reads both operands straight into registers, 16
// k-steps of 32 at a time and the next 16 while these are multiplied; the weights are read once, in 64-byte row pieces, by n / 16 CUs.
// The k of a lane and the order of accumulation and of the epilogue's operations are those of gemm_mfma.hip, so a row
// has the same bits from either.  Measured, us, weights from memory (before: 64 x 128 tiles): 1 x 1536, k 1536 10.4 ->
// 4.2; 3 x 1536, k 2048 12.9 -> 5.3; 16 x 6144, k 1536 13.2 -> 8.4; 16 x 1536, k 4096 25.4 -> 12.8.
#include "gemm.h"

namespace {

constexpr int kSteps = 16;     // k-steps of 32 in a register set

template <typename OT, int EPI>
__global__ __launch_bounds__(64, 1) void gemm_rows_kernel(GemmProblem p, int n, int k) {
    const int lane = threadIdx.x, l16 = lane % 16, q4 = lane / 16;
    const int kq = (q4 >> 1) | ((q4 & 1) << 1);
    const int f0 = blockIdx.x * 16;
    const bf16x8* w = reinterpret_cast<const bf16x8*>(static_cast<const bf16_t*>(p.w) + (size_t)min(f0 + l16, n - 1) * k) + kq;
    const bf16x8* a = reinterpret_cast<const bf16x8*>(static_cast<const bf16_t*>(p.a) + (size_t)min(l16, p.m - 1) * k) + kq;
    const int steps = k / 32;
    bf16x8 wv[2][kSteps], av[2][kSteps];
    auto load = [&](int set, int s0) {      // clamped: steps past the end are not multiplied
#pragma unroll
        for (int i = 0; i < kSteps; i++) {
            const int s = min(s0 + i, steps - 1) * 4;
            wv[set][i] = w[s];
            av[set][i] = a[s];
        }
    };
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int set, int s0) {
#pragma unroll
        for (int i = 0; i < kSteps; i++)
            if (s0 + i < steps) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[set][i], av[set][i], acc, 0, 0, 0);
    };
    load(0, 0);
    // this lane's part of the epilogue's operands: row l16, features f .. f + 3
    const int f = f0 + 4 * q4, fc = min(f, n - 4), row = min(l16, p.m - 1);
    f32x4 bias = {0.f, 0.f, 0.f, 0.f}, gate = {1.f, 1.f, 1.f, 1.f}, res = {0.f, 0.f, 0.f, 0.f};
    if (p.bias) bias = *reinterpret_cast<const f32x4*>(p.bias + fc);
    if constexpr (EPI == EPI_GATE_RES) {
        res = *reinterpret_cast<const f32x4*>(p.res + (size_t)row * n + fc);
        if (p.res2) res += *reinterpret_cast<const f32x4*>(p.res2 + (size_t)row * n + fc);
        if (p.gate) gate = *reinterpret_cast<const f32x4*>(p.gate + (size_t)(row / p.rows_per_gate) * p.gate_stride + fc);
    }
    for (int s = 0; s < steps; s += 2 * kSteps) {
        if (s + kSteps < steps) load(1, s + kSteps);
        multiply(0, s);
        if (s + 2 * kSteps < steps) load(0, s + 2 * kSteps);
        if (s + kSteps < steps) multiply(1, s + kSteps);
    }
    f32x4 v = acc + bias;
    if constexpr (EPI == EPI_GELU_TANH) {
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = gelu_tanh_f(v[j]);
    } else if constexpr (EPI == EPI_SILU) {
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = silu_f(v[j]);
    } else if constexpr (EPI == EPI_GATE_RES) {
#pragma clang fp contract(off)
        v = v * gate;            // rounded before the residual is added, as in the other kernels
        v = v + res;
    }
    if (l16 >= p.m || f >= n) return;
    OT* dst = static_cast<OT*>(p.out) + (size_t)l16 * n + f;
    if constexpr (sizeof(OT) == 4) *reinterpret_cast<f32x4*>(dst) = v;
    else *reinterpret_cast<bf16x4*>(dst) = bf16x4{(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
}

template <typename OT, int EPI>
int launch_rows(const GemmGroup& g, hipStream_t st) {
    char name[96] = "";
    if (hyb_trace_on()) snprintf(name, sizeof(name), "gemm_mfma_16x16.epi%d.n%d.k%d", EPI, g.n, g.k);
    HybTraceScope trace(name, "flop", 2.0 * g.p[0].m * g.n * g.k, st);
    hipLaunchKernelGGL((gemm_rows_kernel<OT, EPI>), dim3((g.n + 15) / 16), dim3(64), 0, st, g.p[0], g.n, g.k);
    return hyb_check_launch("gemm_mfma_rows");
}

// Where this kernel is the faster one (11 widths x 10 depths x 1, 4, 8 and 16 rows against the 64 x 128 tiles, weights from memory).  Up to one wave per SIMD
// it always is (0.3-1.0 of the time), but for wide launches of a few steps, whose waves request 16 steps all the same (16 x 12288: k 64 4.8 against
// 4.1 us, k 256 5.0 against 5.6).  With more waves the tiles, whose workgroups follow each other, are (3 x 24576, k 64 7.7 against 4.5, k 1536 20 against 18;
// 16 x 24576, k 1536 26 against 18), until a long k with few rows (1 x 18432, k 2048 21 against 29; 1 x 49152, k 4096 79 against 107; 16 x 18432, k 4096 59 against 50).
bool rows_kernel_is_faster(int m, int n, int k) {
    const int per_simd = 16 * 4 * hyb_cu_count();      // features of one wave on every SIMD
    if (n <= per_simd) return k >= 256 || n <= per_simd / 2;
    return m <= 4 && k >= 2048;
}

}  // namespace

int hyb_launch_gemm_mfma_rows(const GemmGroup& g, hyb_dtype out_dtype, int epi, hipStream_t st) {
    const bool f32 = out_dtype == HYB_F32;
    if (g.count != 1 || g.n2 || g.p[0].m < 1 || g.p[0].m > 16 || !rows_kernel_is_faster(g.p[0].m, g.n, g.k)) return -1;
    switch (epi) {
        case EPI_BIAS: return f32 ? launch_rows<float, EPI_BIAS>(g, st) : launch_rows<bf16_t, EPI_BIAS>(g, st);
        case EPI_GELU_TANH: return f32 ? launch_rows<float, EPI_GELU_TANH>(g, st) : launch_rows<bf16_t, EPI_GELU_TANH>(g, st);
        case EPI_SILU: return f32 ? launch_rows<float, EPI_SILU>(g, st) : launch_rows<bf16_t, EPI_SILU>(g, st);
        case EPI_GATE_RES: return f32 ? launch_rows<float, EPI_GATE_RES>(g, st) : -1;
        default: return -1;
    }
}
