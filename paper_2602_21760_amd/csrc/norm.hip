// Bandwidth-bound pieces of the denoiser forward: LayerNorm + adaLN modulate, the adaLN
// modulation GEMV, GroupNorm, timestep features, patchify / unpatchify, dtype conversion.
// (The denoiser f_theta is a black box in the paper, Sec. 4.1; these are the parts of the
// transformer block around the contractions.)
#include "checks.h"

#include <type_traits>

namespace {

// ------------------------------------------------------------------------------------------
// LayerNorm (+ modulate / affine).  One wave per row; the row lives in registers (hidden <=
// 2048), statistics are two-pass in fp32 with wavefront-shuffle reductions.
//   AFFINE = false: out = xhat * (1 + scale[b]) + shift[b]   (adaLN; shift/scale may be NULL)
//   AFFINE = true : out = xhat * scale + shift               (gamma / beta per feature)
// ------------------------------------------------------------------------------------------
constexpr int kLnMaxVec = 8;   // float4 per lane -> hidden <= 8 * 64 * 4 = 2048

// launch(integral_constant<float4 per lane of a row of `hidden`>)
template <typename F> void with_vectors_per_lane(int hidden, F launch) {
    switch ((hidden / 4 + HYB_WAVE - 1) / HYB_WAVE) {
        case 1: launch(std::integral_constant<int, 1>{}); break;
        case 2: launch(std::integral_constant<int, 2>{}); break;
        case 3: launch(std::integral_constant<int, 3>{}); break;
        case 4: launch(std::integral_constant<int, 4>{}); break;
        case 5: launch(std::integral_constant<int, 5>{}); break;
        case 6: launch(std::integral_constant<int, 6>{}); break;
        case 7: launch(std::integral_constant<int, 7>{}); break;
        default: launch(std::integral_constant<int, kLnMaxVec>{}); break;
    }
}

// Up to two independent row sets (the image and the text stream of a joint block) share one launch:
// workgroups [0, blocks0) serve set 0, the rest set 1.
struct LnSet {
    const float* x;
    const float* shift;
    const float* scale;
    void* out;
    size_t mod_stride;
    int rows, tokens;
};
struct LnArgs {
    LnSet s[2];
    int blocks0;
    int hidden;
    float eps;
};

// What bounds it: up to some thousand rows are resident at once (one wave each: 5120 rows of 1536, five waves per SIMD; more of
// shorter rows), and a launch of that many takes as long as one wave's chain of memory latencies; longer ones go
// through in several such turns.  The row's vectors are therefore requested together (NV = vectors per lane is a template parameter,
// addresses past the row's end are clamped: a load under a condition is waited for inside its branch, one latency per
// vector), and shift and scale before the reductions.  4429 rows of 1536 inside a step 11.1 -> 9.4 us, 2048 rows of 1280
// 6.9 -> 5.3 us (2.0 -> 3.0 TB/s).
template <typename OT, bool AFFINE, int NV>
__global__ __launch_bounds__(256) void layernorm_kernel(LnArgs a) {
    const int wave = threadIdx.x / HYB_WAVE, lane = threadIdx.x % HYB_WAVE;
    const int blk = (int)blockIdx.x;
    const int set = blk >= a.blocks0 ? 1 : 0;
    const LnSet& p = a.s[set];
    const int row = (blk - (set ? a.blocks0 : 0)) * 4 + wave;
    if (row >= p.rows) return;
    const float* __restrict__ x = p.x;
    const float* __restrict__ shift = p.shift;
    const float* __restrict__ scale = p.scale;
    OT* __restrict__ out = static_cast<OT*>(p.out);
    const size_t mod_stride = p.mod_stride;
    const int tokens = p.tokens, hidden = a.hidden;
    const float eps = a.eps;
    const int nvec = hidden / 4;
    const f32x4* xr = reinterpret_cast<const f32x4*>(x + (size_t)row * hidden);
    f32x4 r[NV], sc[NV], sh[NV];
#pragma unroll
    for (int i = 0; i < NV; i++) r[i] = xr[min(lane + i * HYB_WAVE, nvec - 1)];
    const size_t b = AFFINE ? 0 : (size_t)(row / tokens);
    const f32x4* shr = reinterpret_cast<const f32x4*>(shift + b * mod_stride);
    const f32x4* scr = reinterpret_cast<const f32x4*>(scale + b * mod_stride);
    if (scale) {
#pragma unroll
        for (int i = 0; i < NV; i++) sc[i] = scr[min(lane + i * HYB_WAVE, nvec - 1)];
    } else {
#pragma unroll
        for (int i = 0; i < NV; i++) sc[i] = AFFINE ? (f32x4){1.f, 1.f, 1.f, 1.f} : (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    if (shift) {
#pragma unroll
        for (int i = 0; i < NV; i++) sh[i] = shr[min(lane + i * HYB_WAVE, nvec - 1)];
    } else {
#pragma unroll
        for (int i = 0; i < NV; i++) sh[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const float t = (r[i][0] + r[i][1]) + (r[i][2] + r[i][3]);
        if (lane + i * HYB_WAVE < nvec) s += t;
    }
    const float mean = wave_sum(s) / (float)hidden;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NV; i++) {
        float t = q;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const float d = r[i][j] - mean;
            t = fmaf(d, d, t);
        }
        if (lane + i * HYB_WAVE < nvec) q = t;
    }
    const float rstd = rsqrtf(wave_sum(q) / (float)hidden + eps);
    OT* orow = out + (size_t)row * hidden;
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int c = lane + i * HYB_WAVE;
        if (c < nvec) {
            f32x4 y;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const float xh = (r[i][j] - mean) * rstd;
                const float g = AFFINE ? sc[i][j] : 1.f + sc[i][j];
                y[j] = fmaf(xh, g, sh[i][j]);
            }
            if constexpr (sizeof(OT) == 4) {
                *reinterpret_cast<f32x4*>(orow + 4 * c) = y;
            } else {
                bf16x4 o = {(bf16_t)y[0], (bf16_t)y[1], (bf16_t)y[2], (bf16_t)y[3]};
                *reinterpret_cast<bf16x4*>(orow + 4 * c) = o;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// adaLN modulation GEMV: out[b, r] = sum_k w[r, k] SiLU(temb[b, k]) + bias[r].  Weight-read bound:
// a wave streams four rows at a time with 16-byte loads; SiLU(temb) of up to kAdaMaxBatch samples
// sits in LDS.  A wave takes several groups of rows and requests the next 512 columns before it multiplies the current ones, also
// across the end of a group: with one group per wave every workgroup began with the activations and ended with the
// reductions with no load in flight.  150528 x 1536 bf16, two samples: 119 -> 92 us (3.9 -> 5.0 TB/s); 445440 x 1536, one
// sample: 235 -> 215 us (5.8 -> 6.4 TB/s).
// ------------------------------------------------------------------------------------------
constexpr int kAdaMaxBatch = 4;
constexpr int kAdaRowsPerWave = 4;
// Waves of a launch at most, 32 for each of 256 CUs.  As many are resident at once only for one sample in bf16; the others' registers leave room for
// five to seven eighths of them (and 64 KB of activations, four samples of 4096, for two workgroups per CU), and the rest start as those end.
constexpr int kAdaWaves = 256 * 32;

// Eight weights of a row as they come from memory (streamed once per call: non-temporal loads, which do not displace what
// the caches hold), and as fp32.
template <typename WT> struct Raw8;
template <> struct Raw8<float> {
    f32x4 a, b;
    __device__ __forceinline__ void load(const float* p) {
        a = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
        b = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p + 4));
    }
    __device__ __forceinline__ void floats(float* r) const {
        r[0] = a[0]; r[1] = a[1]; r[2] = a[2]; r[3] = a[3]; r[4] = b[0]; r[5] = b[1]; r[6] = b[2]; r[7] = b[3];
    }
};
template <> struct Raw8<bf16_t> {
    u32x4 a;
    __device__ __forceinline__ void load(const bf16_t* p) { a = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)); }
    __device__ __forceinline__ void floats(float* r) const {   // bf16 -> fp32: the bits, shifted up
#pragma unroll
        for (int i = 0; i < 4; i++) {
            r[2 * i] = __uint_as_float(a[i] << 16);
            r[2 * i + 1] = __uint_as_float(a[i] & 0xffff0000u);
        }
    }
};

template <typename WT, int NB>
__global__ __launch_bounds__(256) void adaln_kernel(const WT* __restrict__ w, const float* __restrict__ bias,
                                                    const float* __restrict__ temb, float* __restrict__ out, int rows,
                                                    int hidden, int out_stride) {
    extern __shared__ __attribute__((aligned(16))) float s_act[];   // [NB][hidden]
    constexpr int R = kAdaRowsPerWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / HYB_WAVE), lane = threadIdx.x % HYB_WAVE;
    const int groups = (rows + R - 1) / R, step = gridDim.x * 4;
    const int chunks = (hidden + 8 * HYB_WAVE - 1) / (8 * HYB_WAVE);
    int grp = blockIdx.x * 4 + wave, chunk = 0;
    auto load = [&](Raw8<WT>* v, int g, int c) {
        const int k = min(lane * 8 + c * 8 * HYB_WAVE, hidden - 8);   // clamped: in bounds, not used
#pragma unroll
        for (int r = 0; r < R; r++) v[r].load(w + (size_t)min(g * R + r, rows - 1) * hidden + k);
    };
    Raw8<WT> cur[R], next[R];
    if (grp < groups) load(cur, grp, 0);
    for (int i = threadIdx.x; i < NB * hidden; i += 256) s_act[i] = silu_f(temb[i]);
    __syncthreads();
    if (grp >= groups) return;
    float acc[R][NB];
#pragma unroll
    for (int r = 0; r < R; r++)
#pragma unroll
        for (int b = 0; b < NB; b++) acc[r][b] = 0.f;
    for (;;) {
        int next_grp = grp, next_chunk = chunk + 1;
        if (next_chunk == chunks) {
            next_chunk = 0;
            next_grp += step;
        }
        const bool more = next_grp < groups;
        if (more) load(next, next_grp, next_chunk);
        const int k = lane * 8 + chunk * 8 * HYB_WAVE;
        if (k < hidden) {
            float wv[R][8];
#pragma unroll
            for (int r = 0; r < R; r++) cur[r].floats(wv[r]);
#pragma unroll
            for (int b = 0; b < NB; b++) {
                const float* a = s_act + b * hidden + k;
#pragma unroll
                for (int r = 0; r < R; r++)
#pragma unroll
                    for (int j = 0; j < 8; j++) acc[r][b] = fmaf(wv[r][j], a[j], acc[r][b]);
            }
        }
        if (next_chunk == 0) {
            const int row0 = grp * R;
#pragma unroll
            for (int r = 0; r < R; r++)
#pragma unroll
                for (int b = 0; b < NB; b++) {
                    const float t = wave_sum(acc[r][b]);
                    if (lane == 0 && row0 + r < rows) out[(size_t)b * out_stride + row0 + r] = t + bias[row0 + r];
                    acc[r][b] = 0.f;
                }
        }
        if (!more) break;
#pragma unroll
        for (int r = 0; r < R; r++) cur[r] = next[r];
        grp = next_grp;
        chunk = next_chunk;
    }
}

// ------------------------------------------------------------------------------------------
// GroupNorm on token-major data x[B, T, C], groups of C/G consecutive channels, statistics over
// (T, C/G) per sample.  Three kernels; 1 and 3 use one thread per 4-channel vector (so every load and
// store is a coalesced 16-byte access and a thread stays inside one group) and chunks of a few tokens, so
// that a launch has thousands of workgroups with all their loads in flight at once:
//  1. each workgroup sums x and x^2 over its chunk of tokens (fp32 per thread, then the threads of a
//     group are added in a fixed order in fp64) -> partial[b][chunk][group][2];
//  2. one workgroup per sample and group adds the partials (fp64, in a fixed order) and forms mean and 1/std;
//  3. each workgroup normalises its chunk: y = (x - mean) rstd gamma + beta.
// No atomics: the result is deterministic and independent of the batch index.
// ------------------------------------------------------------------------------------------
constexpr int kGnChunks = 1024;   // at most this many chunks per sample
constexpr int kGnTokens = 4;      // tokens per chunk (more when a sample has more than kGnChunks * kGnTokens tokens)

__global__ void groupnorm_stats_kernel(const float* __restrict__ x, double* __restrict__ partial, int tokens,
                                       int channels, int groups, int tokens_per_chunk) {
    extern __shared__ float gn_red[];   // [nvec][2]
    const int nvec = channels / 4, vec = threadIdx.x;
    const int chunk = blockIdx.x, b = blockIdx.y;
    const int t0 = chunk * tokens_per_chunk, t1 = min(tokens, t0 + tokens_per_chunk);
    const f32x4* xb = reinterpret_cast<const f32x4*>(x + (size_t)b * tokens * channels);
    float s = 0.f, q = 0.f;
    for (int t = t0; t < t1; t += kGnTokens) {
        f32x4 v[kGnTokens];
#pragma unroll
        for (int j = 0; j < kGnTokens; j++) v[j] = xb[(size_t)min(t + j, t1 - 1) * nvec + vec];   // clamped: in bounds
#pragma unroll
        for (int j = 0; j < kGnTokens; j++) {
            if (t + j < t1) {
                s += (v[j][0] + v[j][1]) + (v[j][2] + v[j][3]);
                q = fmaf(v[j][0], v[j][0], q); q = fmaf(v[j][1], v[j][1], q);
                q = fmaf(v[j][2], v[j][2], q); q = fmaf(v[j][3], v[j][3], q);
            }
        }
    }
    gn_red[2 * vec] = s;
    gn_red[2 * vec + 1] = q;
    __syncthreads();
    if (vec < groups) {
        const int vpg = nvec / groups;
        double ds = 0.0, dq = 0.0;
        for (int i = 0; i < vpg; i++) {
            ds += (double)gn_red[2 * (vec * vpg + i)];
            dq += (double)gn_red[2 * (vec * vpg + i) + 1];
        }
        double* o = partial + (((size_t)b * gridDim.x + chunk) * groups + vec) * 2;
        o[0] = ds;
        o[1] = dq;
    }
}

// One workgroup per (group, sample): thread j adds the partials of chunks j, j + 256, ... in that order (fp64), the waves add
// their lanes by halving and thread 0 the four waves in order; it leaves (mean, 1/std) as two floats.  One workgroup per
// sample, which read all 512 KB of a sample's partials by itself, took 7.3 us at 2 x 4096 tokens where this takes 4.6 (4.6 us
// either way at 2 x 1024).
__global__ __launch_bounds__(256) void groupnorm_finalize_kernel(const double* __restrict__ partial, float* __restrict__ stats, int nchunks,
                                                                 int groups, double count, float eps) {
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    constexpr int kLoads = (kGnChunks + 255) / 256;
    __shared__ double red[4][2];
    const int g = blockIdx.x, b = blockIdx.y, j = threadIdx.x;
    const f64x2* p = reinterpret_cast<const f64x2*>(partial) + (size_t)b * nchunks * groups + g;
    f64x2 v[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; u++) v[u] = p[(size_t)min(j + 256 * u, nchunks - 1) * groups];   // clamped: in bounds
    double ds = 0.0, dq = 0.0;
#pragma unroll
    for (int u = 0; u < kLoads; u++)
        if (j + 256 * u < nchunks) { ds += v[u][0]; dq += v[u][1]; }
    ds = wave_sum(ds);
    dq = wave_sum(dq);
    if (j % HYB_WAVE == 0) {
        red[j / HYB_WAVE][0] = ds;
        red[j / HYB_WAVE][1] = dq;
    }
    __syncthreads();
    if (j != 0) return;
    ds = (red[0][0] + red[1][0]) + (red[2][0] + red[3][0]);
    dq = (red[0][1] + red[1][1]) + (red[2][1] + red[3][1]);
    const double mean_d = ds / count;
    const double var_d = fmax(dq / count - mean_d * mean_d, 0.0);
    stats[((size_t)b * groups + g) * 2] = (float)mean_d;
    stats[((size_t)b * groups + g) * 2 + 1] = (float)(1.0 / sqrt(var_d + (double)eps));
}

__global__ void groupnorm_apply_kernel(const float* __restrict__ x, const float* __restrict__ stats,
                                       const float* __restrict__ gamma, const float* __restrict__ beta,
                                       float* __restrict__ out, int tokens, int channels, int groups,
                                       int tokens_per_chunk) {
    const int nvec = channels / 4, vec = threadIdx.x;
    const int chunk = blockIdx.x, b = blockIdx.y;
    const int grp = vec / (nvec / groups);
    const float mean = stats[((size_t)b * groups + grp) * 2], rstd = stats[((size_t)b * groups + grp) * 2 + 1];
    const f32x4 gm = reinterpret_cast<const f32x4*>(gamma)[vec], bt = reinterpret_cast<const f32x4*>(beta)[vec];
    const f32x4* xb = reinterpret_cast<const f32x4*>(x + (size_t)b * tokens * channels);
    f32x4* ob = reinterpret_cast<f32x4*>(out + (size_t)b * tokens * channels);
    const int t0 = chunk * tokens_per_chunk, t1 = min(tokens, t0 + tokens_per_chunk);
    for (int t = t0; t < t1; t += kGnTokens) {
        f32x4 v[kGnTokens];
#pragma unroll
        for (int j = 0; j < kGnTokens; j++) v[j] = xb[(size_t)min(t + j, t1 - 1) * nvec + vec];   // clamped: in bounds
#pragma unroll
        for (int j = 0; j < kGnTokens; j++) {
            if (t + j < t1) {
                f32x4 y;
#pragma unroll
                for (int e = 0; e < 4; e++) y[e] = fmaf((v[j][e] - mean) * rstd, gm[e], bt[e]);
                ob[(size_t)(t + j) * nvec + vec] = y;
            }
        }
    }
}

// The apply pass and the affine LayerNorm that follows it in a transformer stage, in one: a wave owns a row, writes
// g = GroupNorm(x) and, from the registers, LayerNorm(g).  Bound by memory latency like the LayerNorm (all loads requested
// together, addresses past the row's end clamped); against the two passes it saves one read of g and a launch: 2 x 4096 tokens of
// 640 channels 6.7 + 7.1 -> 11.0 us, 2 x 1024 of 1280 5.9 + 5.3 -> 7.1 us.
// Same operations in the same order as the two kernels, so the same bits.
template <typename OT, int NV>
__global__ __launch_bounds__(256) void groupnorm_apply_ln_kernel(const float* __restrict__ x, const float* __restrict__ stats,
                                                                 const float* __restrict__ gamma, const float* __restrict__ beta,
                                                                 const float* __restrict__ ln_g, const float* __restrict__ ln_b,
                                                                 float* __restrict__ out, OT* __restrict__ ln_out, int rows, int tokens,
                                                                 int channels, int groups, float ln_eps) {
    const int wave = threadIdx.x / HYB_WAVE, lane = threadIdx.x % HYB_WAVE;
    const int row = blockIdx.x * 4 + wave;
    if (row >= rows) return;
    const int nvec = channels / 4, vpg = nvec / groups;
    const f32x4* xr = reinterpret_cast<const f32x4*>(x + (size_t)row * channels);
    const float2* st = reinterpret_cast<const float2*>(stats) + (size_t)(row / tokens) * groups;   // (mean, 1/std) per group
    f32x4 r[NV], gm[NV], bt[NV];
    float2 gs[NV];
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int c = min(lane + i * HYB_WAVE, nvec - 1);
        r[i] = xr[c];
        gs[i] = st[c / vpg];
        gm[i] = reinterpret_cast<const f32x4*>(gamma)[c];
        bt[i] = reinterpret_cast<const f32x4*>(beta)[c];
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; i++) {
#pragma unroll
        for (int e = 0; e < 4; e++) r[i][e] = fmaf((r[i][e] - gs[i].x) * gs[i].y, gm[i][e], bt[i][e]);
        const float t = (r[i][0] + r[i][1]) + (r[i][2] + r[i][3]);
        if (lane + i * HYB_WAVE < nvec) s += t;
    }
#pragma unroll
    for (int i = 0; i < NV; i++) {   // the affine LayerNorm's vectors, in flight across the reductions
        const int c = min(lane + i * HYB_WAVE, nvec - 1);
        gm[i] = reinterpret_cast<const f32x4*>(ln_g)[c];
        bt[i] = reinterpret_cast<const f32x4*>(ln_b)[c];
    }
    f32x4* gr = reinterpret_cast<f32x4*>(out + (size_t)row * channels);
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int c = lane + i * HYB_WAVE;
        if (c < nvec) gr[c] = r[i];
    }
    const float mean = wave_sum(s) / (float)channels;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NV; i++) {
        float t = q;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const float d = r[i][j] - mean;
            t = fmaf(d, d, t);
        }
        if (lane + i * HYB_WAVE < nvec) q = t;
    }
    const float rstd = rsqrtf(wave_sum(q) / (float)channels + ln_eps);
    OT* orow = ln_out + (size_t)row * channels;
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int c = lane + i * HYB_WAVE;
        if (c < nvec) {
            f32x4 y;
#pragma unroll
            for (int j = 0; j < 4; j++) y[j] = fmaf((r[i][j] - mean) * rstd, gm[i][j], bt[i][j]);
            if constexpr (sizeof(OT) == 4) {
                *reinterpret_cast<f32x4*>(orow + 4 * c) = y;
            } else {
                bf16x4 o = {(bf16_t)y[0], (bf16_t)y[1], (bf16_t)y[2], (bf16_t)y[3]};
                *reinterpret_cast<bf16x4*>(orow + 4 * c) = o;
            }
        }
    }
}

template <typename OT>
__global__ void timestep_embedding_kernel(const float* t, float t_value, OT* out, int batch, int dim) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= batch * dim) return;
    const int b = i / dim, j = i % dim, half = dim / 2;
    const int f = j < half ? j : j - half;
    const double ang = 1000.0 * (double)(t ? t[b] : t_value) * exp(-9.210340371976184 * (double)f / (double)half);  // ln(10000)
    out[i] = from_f32<OT>((float)(j < half ? cos(ang) : sin(ang)));
}

// tokens[b, py*(ww/p)+px, (dy*p+dx)*c + ch] = latent[b, py*p+dy, px*p+dx, ch]
template <typename TT, typename LT, bool TO_TOKENS>
__global__ void patch_kernel(LT* latent, TT* tokens, int batch, int hh, int ww, int c, int p) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t total = (size_t)batch * hh * ww * c;
    if (i >= total) return;
    const int ch = i % c;
    size_t r = i / c;
    const int xw = r % ww; r /= ww;
    const int yh = r % hh;
    const size_t b = r / hh;
    const int py = yh / p, dy = yh % p, px = xw / p, dx = xw % p;
    const size_t tok = (b * (hh / p) + py) * (ww / p) + px;
    const size_t ti = tok * ((size_t)p * p * c) + (size_t)(dy * p + dx) * c + ch;
    using TV = std::remove_const_t<TT>;
    using LV = std::remove_const_t<LT>;
    if constexpr (TO_TOKENS) tokens[ti] = from_f32<TV>(to_f32<LV>(latent[i]));
    else latent[i] = from_f32<LV>(to_f32<TV>(tokens[ti]));
}

template <typename OT>
__global__ void convert_kernel(const float* in, OT* out, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = from_f32<OT>(in[i]);
}

}  // namespace

namespace {
int launch_layernorm(const LnArgs& a, int blocks, double rows, hyb_dtype out_dtype, bool affine, hipStream_t st) {
    dim3 grid(blocks), block(256);
    HybTraceScope trace("layernorm", "byte", rows * a.hidden * (4 + hyb_dtype_size(out_dtype)), st);
    auto launch = [&](auto nv_tag) {
        constexpr int NV = decltype(nv_tag)::value;
        if (out_dtype == HYB_F32) {
            if (affine) hipLaunchKernelGGL((layernorm_kernel<float, true, NV>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((layernorm_kernel<float, false, NV>), grid, block, 0, st, a);
        } else {
            if (affine) hipLaunchKernelGGL((layernorm_kernel<bf16_t, true, NV>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((layernorm_kernel<bf16_t, false, NV>), grid, block, 0, st, a);
        }
    };
    with_vectors_per_lane(a.hidden, launch);
    return hyb_check_launch("layernorm");
}
}  // namespace

// Internal launcher shared with the block composition (affine = gamma/beta LayerNorm).
int hyb_launch_layernorm(const float* x, const float* shift, const float* scale, size_t mod_stride, void* out,
                         int batch, int tokens, int hidden, float eps, hyb_dtype out_dtype, bool affine,
                         hipStream_t st) {
    const int rows = batch * tokens;
    if (rows == 0) return HYB_OK;
    LnArgs a{};
    a.s[0] = LnSet{x, shift, scale, out, mod_stride, rows, tokens};
    a.blocks0 = (rows + 3) / 4;
    a.hidden = hidden;
    a.eps = eps;
    return launch_layernorm(a, a.blocks0, rows, out_dtype, affine, st);
}

// Two modulated LayerNorms (no affine) of the same width in one launch; either set may be empty.
int hyb_launch_layernorm_pair(const float* const x[2], const float* const shift[2], const float* const scale[2],
                              size_t mod_stride, void* const out[2], int batch, const int tokens[2], int hidden,
                              float eps, hyb_dtype out_dtype, hipStream_t st) {
    LnArgs a{};
    int blocks[2];
    for (int i = 0; i < 2; i++) {
        const int rows = batch * tokens[i];
        a.s[i] = LnSet{x[i], shift[i], scale[i], out[i], mod_stride, rows, tokens[i] > 0 ? tokens[i] : 1};
        blocks[i] = (rows + 3) / 4;
    }
    if (blocks[0] + blocks[1] == 0) return HYB_OK;
    a.blocks0 = blocks[0];
    a.hidden = hidden;
    a.eps = eps;
    return launch_layernorm(a, blocks[0] + blocks[1], (double)batch * (tokens[0] + tokens[1]), out_dtype, false, st);
}

// chunk partials (fp64 sum and sum of squares), then (mean, 1/std) per (sample, group)
static size_t gn_partial_bytes(int batch, int groups) {
    return hyb_align_up((size_t)batch * kGnChunks * groups * 2 * sizeof(double), 256);
}
size_t hyb_groupnorm_scratch_bytes(int batch, int groups) {
    return gn_partial_bytes(batch, groups) + hyb_align_up((size_t)batch * groups * 2 * sizeof(float), 256);
}

// Mean and 1/std of every (sample, group), left in the scratch; channels % (4 * groups) == 0 and channels <= 4096 (one thread
// per 4-channel vector, <= 1024 threads).
static int launch_groupnorm_stats(const float* x, int batch, int tokens, int channels, int groups, float eps, void* scratch, hipStream_t st) {
    HYB_REQUIRE(channels % (4 * groups) == 0 && channels <= 4096 && groups <= channels / 4, HYB_ERR_SHAPE,
                "groupnorm: channels %d must be a multiple of 4 * groups (%d) and at most 4096", channels, groups);
    const int nvec = channels / 4;
    const int want = (tokens + kGnTokens - 1) / kGnTokens;
    const int nchunks = want < kGnChunks ? want : kGnChunks;
    const int tpc = (tokens + nchunks - 1) / nchunks;
    const int used = (tokens + tpc - 1) / tpc;     // chunks that actually hold tokens (<= kGnChunks)
    hipLaunchKernelGGL(groupnorm_stats_kernel, dim3(used, batch), dim3(nvec), nvec * 2 * sizeof(float), st, x, (double*)scratch, tokens, channels, groups, tpc);
    float* stats = reinterpret_cast<float*>(static_cast<char*>(scratch) + gn_partial_bytes(batch, groups));
    hipLaunchKernelGGL(groupnorm_finalize_kernel, dim3(groups, batch), dim3(256), 0, st, (const double*)scratch, stats, used, groups,
                       (double)tokens * (channels / groups), eps);
    return hyb_check_launch("groupnorm");
}

int hyb_launch_groupnorm(const float* x, const float* gamma, const float* beta, float* out, int batch, int tokens,
                         int channels, int groups, float eps, void* scratch, hipStream_t st) {
    if (batch == 0 || tokens == 0) return HYB_OK;
    HybTraceScope trace("groupnorm", "byte", (double)batch * tokens * channels * 12, st);
    const int rc = launch_groupnorm_stats(x, batch, tokens, channels, groups, eps, scratch, st);
    if (rc) return rc;
    const float* stats = reinterpret_cast<const float*>(static_cast<char*>(scratch) + gn_partial_bytes(batch, groups));
    const int chunks = (tokens + kGnTokens - 1) / kGnTokens, used = chunks < kGnChunks ? chunks : kGnChunks;
    const int tpc = (tokens + used - 1) / used;
    hipLaunchKernelGGL(groupnorm_apply_kernel, dim3((tokens + tpc - 1) / tpc, batch), dim3(channels / 4), 0, st, x, stats, gamma, beta, out,
                       tokens, channels, groups, tpc);
    return hyb_check_launch("groupnorm");
}

// out = GroupNorm(x) and ln_out = LayerNorm(out) (gain and bias per channel); channels <= 2048, otherwise as above.
int hyb_launch_groupnorm_layernorm(const float* x, const float* gamma, const float* beta, float* out, const float* ln_g, const float* ln_b,
                                   void* ln_out, int batch, int tokens, int channels, int groups, float eps, float ln_eps, hyb_dtype ln_dtype,
                                   void* scratch, hipStream_t st) {
    if (batch == 0 || tokens == 0) return HYB_OK;
    const int rows = batch * tokens;
    HybTraceScope trace("groupnorm_layernorm", "byte", (double)rows * channels * (12 + hyb_dtype_size(ln_dtype)), st);
    const int rc = launch_groupnorm_stats(x, batch, tokens, channels, groups, eps, scratch, st);
    if (rc) return rc;
    const float* stats = reinterpret_cast<const float*>(static_cast<char*>(scratch) + gn_partial_bytes(batch, groups));
    const dim3 grid((rows + 3) / 4), block(256);
    with_vectors_per_lane(channels, [&](auto nv_tag) {
        constexpr int NV = decltype(nv_tag)::value;
        if (ln_dtype == HYB_F32)
            hipLaunchKernelGGL((groupnorm_apply_ln_kernel<float, NV>), grid, block, 0, st, x, stats, gamma, beta, ln_g, ln_b, out,
                               static_cast<float*>(ln_out), rows, tokens, channels, groups, ln_eps);
        else
            hipLaunchKernelGGL((groupnorm_apply_ln_kernel<bf16_t, NV>), grid, block, 0, st, x, stats, gamma, beta, ln_g, ln_b, out,
                               static_cast<bf16_t*>(ln_out), rows, tokens, channels, groups, ln_eps);
    });
    return hyb_check_launch("groupnorm_layernorm");
}

int hyb_check_layernorm_modulate(const float* x, const float* shift, const float* scale, size_t mod_stride, const void* out, int batch, int tokens,
                                 int hidden, hyb_dtype out_dtype) {
    const char* who = "hyb_layernorm_modulate";
    HYB_ARG_DTYPE(who, out_dtype);
    HYB_REQUIRE(batch >= 0 && tokens >= 0, HYB_ERR_SHAPE, "hyb_layernorm_modulate: negative size");
    HYB_REQUIRE(hidden > 0 && hidden % 4 == 0 && hidden <= kLnMaxVec * 256, HYB_ERR_SHAPE,
                "hyb_layernorm_modulate: hidden %d must be a positive multiple of 4, at most %d", hidden, kLnMaxVec * 256);
    if (batch == 0 || tokens == 0) return HYB_OK;
    HYB_ARG_PTR(who, x); HYB_ARG_PTR(who, out);
    HYB_ARG_ALIGN(who, x); HYB_ARG_ALIGN(who, out); HYB_ARG_ALIGN(who, shift); HYB_ARG_ALIGN(who, scale);
    HYB_REQUIRE((shift == nullptr) == (scale == nullptr), HYB_ERR_NULL, "hyb_layernorm_modulate: shift and scale must both be given or both be NULL");
    HYB_REQUIRE(mod_stride % 4 == 0, HYB_ERR_ALIGN, "hyb_layernorm_modulate: mod_stride must be a multiple of 4");
    return HYB_OK;
}

extern "C" int hyb_layernorm_modulate(const float* x, const float* shift, const float* scale, size_t mod_stride,
                                      void* out, int batch, int tokens, int hidden, float eps,
                                      hyb_dtype out_dtype, void* stream) {
    const int rc = hyb_check_layernorm_modulate(x, shift, scale, mod_stride, out, batch, tokens, hidden, out_dtype);
    if (rc || batch == 0 || tokens == 0) return rc;
    return hyb_launch_layernorm(x, shift, scale, mod_stride, out, batch, tokens, hidden, eps, out_dtype, false, (hipStream_t)stream);
}

int hyb_check_adaln_modulation(const void* w, const float* bias, const float* temb, const float* out, int rows, int hidden, int batch, hyb_dtype dtype) {
    const char* who = "hyb_adaln_modulation";
    HYB_ARG_DTYPE(who, dtype);
    HYB_REQUIRE(rows >= 0 && batch >= 0, HYB_ERR_SHAPE, "hyb_adaln_modulation: negative size");
    HYB_REQUIRE(hidden > 0 && hidden % 8 == 0 && hidden <= 4096, HYB_ERR_SHAPE,
                "hyb_adaln_modulation: hidden %d must be a positive multiple of 8, at most 4096", hidden);
    if (rows == 0 || batch == 0) return HYB_OK;
    HYB_ARG_PTR(who, w); HYB_ARG_PTR(who, bias); HYB_ARG_PTR(who, temb); HYB_ARG_PTR(who, out);
    HYB_ARG_ALIGN(who, w); HYB_ARG_ALIGN(who, bias); HYB_ARG_ALIGN(who, temb); HYB_ARG_ALIGN(who, out);
    return HYB_OK;
}

extern "C" int hyb_adaln_modulation(const void* w, const float* bias, const float* temb, float* out,
                                    int rows, int hidden, int batch, hyb_dtype dtype, void* stream) {
    const int bad = hyb_check_adaln_modulation(w, bias, temb, out, rows, hidden, batch, dtype);
    if (bad || rows == 0 || batch == 0) return bad;
    hipStream_t st = (hipStream_t)stream;
    // as many groups of rows for every wave, as few as keep the waves to kAdaWaves
    const int groups = (rows + kAdaRowsPerWave - 1) / kAdaRowsPerWave, each = (groups + kAdaWaves - 1) / kAdaWaves;
    const dim3 grid(((groups + each - 1) / each + 3) / 4), block(256);
    HybTraceScope trace("adaln_modulation", "byte", (double)rows * hidden * hyb_dtype_size(dtype) * ((batch + kAdaMaxBatch - 1) / kAdaMaxBatch), st);
    for (int b0 = 0; b0 < batch; b0 += kAdaMaxBatch) {
        const int nb = batch - b0 < kAdaMaxBatch ? batch - b0 : kAdaMaxBatch;
        const size_t shmem = (size_t)nb * hidden * sizeof(float);
        const float* tp = temb + (size_t)b0 * hidden;
        float* op = out + (size_t)b0 * rows;
        auto launch = [&](auto nb_tag) {
            constexpr int NB = decltype(nb_tag)::value;
            if (dtype == HYB_BF16) hipLaunchKernelGGL((adaln_kernel<bf16_t, NB>), grid, block, shmem, st, (const bf16_t*)w, bias, tp, op, rows, hidden, rows);
            else hipLaunchKernelGGL((adaln_kernel<float, NB>), grid, block, shmem, st, (const float*)w, bias, tp, op, rows, hidden, rows);
        };
        if (nb == 1) launch(std::integral_constant<int, 1>{});
        else if (nb == 2) launch(std::integral_constant<int, 2>{});
        else if (nb == 3) launch(std::integral_constant<int, 3>{});
        else launch(std::integral_constant<int, kAdaMaxBatch>{});
        int rc = hyb_check_launch("hyb_adaln_modulation");
        if (rc != HYB_OK) return rc;
    }
    return HYB_OK;
}

int hyb_check_timestep_embedding(const void* out, int batch, int dim, hyb_dtype out_dtype) {
    const char* who = "hyb_timestep_embedding";
    HYB_ARG_DTYPE(who, out_dtype);
    HYB_REQUIRE(batch >= 0 && dim > 0 && dim % 2 == 0, HYB_ERR_SHAPE, "hyb_timestep_embedding: batch >= 0 and an even dim > 0 required");
    if (batch > 0) HYB_ARG_PTR(who, out);
    return HYB_OK;
}

// t == nullptr: t_value for all samples.  (The arguments have been checked.)
int hyb_launch_timestep_embedding(const float* t, float t_value, void* out, int batch, int dim, hyb_dtype out_dtype, hipStream_t st) {
    if (batch == 0) return HYB_OK;
    const int n = batch * dim;
    if (out_dtype == HYB_F32) hipLaunchKernelGGL((timestep_embedding_kernel<float>), dim3((n + 255) / 256), dim3(256), 0, st, t, t_value, (float*)out, batch, dim);
    else hipLaunchKernelGGL((timestep_embedding_kernel<bf16_t>), dim3((n + 255) / 256), dim3(256), 0, st, t, t_value, (bf16_t*)out, batch, dim);
    return hyb_check_launch("hyb_timestep_embedding");
}

extern "C" int hyb_timestep_embedding(const float* t, void* out, int batch, int dim, hyb_dtype out_dtype, void* stream) {
    const int rc = hyb_check_timestep_embedding(out, batch, dim, out_dtype);
    if (rc) return rc;
    if (batch > 0) HYB_CHECK_PTR(t);
    return hyb_launch_timestep_embedding(t, 0.f, out, batch, dim, out_dtype, (hipStream_t)stream);
}

static int check_patch(const char* who, int batch, int hh, int ww, int c, int p) {
    HYB_REQUIRE(batch >= 0 && hh >= 0 && ww >= 0 && c > 0 && p > 0, HYB_ERR_SHAPE, "%s: bad sizes", who);
    HYB_REQUIRE(hh % p == 0 && ww % p == 0, HYB_ERR_SHAPE, "%s: latent %dx%d is not a multiple of patch %d", who, hh, ww, p);
    return HYB_OK;
}

int hyb_check_patchify(const float* latent, const void* tokens, int batch, int hh, int ww, int c, int p, hyb_dtype out_dtype) {
    const char* who = "hyb_patchify";
    HYB_ARG_DTYPE(who, out_dtype);
    const int rc = check_patch(who, batch, hh, ww, c, p);
    if (rc || (size_t)batch * hh * ww * c == 0) return rc;
    HYB_ARG_PTR(who, latent); HYB_ARG_PTR(who, tokens);
    return HYB_OK;
}

extern "C" int hyb_patchify(const float* latent, void* tokens, int batch, int hh, int ww, int c, int p,
                            hyb_dtype out_dtype, void* stream) {
    const int rc = hyb_check_patchify(latent, tokens, batch, hh, ww, c, p, out_dtype);
    const size_t n = (size_t)batch * hh * ww * c;
    if (rc || n == 0) return rc;
    dim3 grid((unsigned)((n + 255) / 256)), block(256);
    if (out_dtype == HYB_F32) hipLaunchKernelGGL((patch_kernel<float, const float, true>), grid, block, 0, (hipStream_t)stream, latent, (float*)tokens, batch, hh, ww, c, p);
    else hipLaunchKernelGGL((patch_kernel<bf16_t, const float, true>), grid, block, 0, (hipStream_t)stream, latent, (bf16_t*)tokens, batch, hh, ww, c, p);
    return hyb_check_launch("hyb_patchify");
}

int hyb_check_unpatchify(const void* tokens, const void* latent, int batch, int hh, int ww, int c, int p, hyb_dtype in_dtype, hyb_dtype out_dtype) {
    const char* who = "hyb_unpatchify";
    HYB_ARG_DTYPE(who, in_dtype); HYB_ARG_DTYPE(who, out_dtype);
    const int rc = check_patch(who, batch, hh, ww, c, p);
    if (rc || (size_t)batch * hh * ww * c == 0) return rc;
    HYB_ARG_PTR(who, latent); HYB_ARG_PTR(who, tokens);
    return HYB_OK;
}

extern "C" int hyb_unpatchify(const void* tokens, void* latent, int batch, int hh, int ww, int c, int p,
                              hyb_dtype in_dtype, hyb_dtype out_dtype, void* stream) {
    const int rc = hyb_check_unpatchify(tokens, latent, batch, hh, ww, c, p, in_dtype, out_dtype);
    const size_t n = (size_t)batch * hh * ww * c;
    if (rc || n == 0) return rc;
    dim3 grid((unsigned)((n + 255) / 256)), block(256);
    hipStream_t st = (hipStream_t)stream;
    if (in_dtype == HYB_F32 && out_dtype == HYB_F32) hipLaunchKernelGGL((patch_kernel<const float, float, false>), grid, block, 0, st, (float*)latent, (const float*)tokens, batch, hh, ww, c, p);
    else if (in_dtype == HYB_F32) hipLaunchKernelGGL((patch_kernel<const float, bf16_t, false>), grid, block, 0, st, (bf16_t*)latent, (const float*)tokens, batch, hh, ww, c, p);
    else if (out_dtype == HYB_F32) hipLaunchKernelGGL((patch_kernel<const bf16_t, float, false>), grid, block, 0, st, (float*)latent, (const bf16_t*)tokens, batch, hh, ww, c, p);
    else hipLaunchKernelGGL((patch_kernel<const bf16_t, bf16_t, false>), grid, block, 0, st, (bf16_t*)latent, (const bf16_t*)tokens, batch, hh, ww, c, p);
    return hyb_check_launch("hyb_unpatchify");
}

int hyb_check_convert(const float* in, const void* out, size_t n, hyb_dtype out_dtype) {
    const char* who = "hyb_convert";
    HYB_ARG_DTYPE(who, out_dtype);
    if (n == 0) return HYB_OK;
    HYB_ARG_PTR(who, in); HYB_ARG_PTR(who, out);
    return HYB_OK;
}

extern "C" int hyb_convert(const float* in, void* out, size_t n, hyb_dtype out_dtype, void* stream) {
    const int rc = hyb_check_convert(in, out, n, out_dtype);
    if (rc || n == 0) return rc;
    dim3 grid((unsigned)((n + 255) / 256)), block(256);
    if (out_dtype == HYB_F32) hipLaunchKernelGGL((convert_kernel<float>), grid, block, 0, (hipStream_t)stream, in, (float*)out, n);
    else hipLaunchKernelGGL((convert_kernel<bf16_t>), grid, block, 0, (hipStream_t)stream, in, (bf16_t*)out, n);
    return hyb_check_launch("hyb_convert");
}
