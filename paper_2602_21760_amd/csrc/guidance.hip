// Guidance step: classifier-free-guidance combine (Sec. 3), branch discrepancy (Eq. 1, velocity
// form of Sec. 4.2) and the scheduler update, as one coalesced pass over HBM.
//
// The pass is bandwidth-bound: per element it reads v_c, v_u (2 or 4 B each) and x (4 B) and
// writes x_out (4 B).  Each workgroup owns a fixed contiguous chunk of one sample, every thread
// moves 16-byte vectors, and the four running sums (sum|d|, sum d^2, sum|u|, sum u^2) are
// reduced thread -> wave -> workgroup in a fixed order into one fp64 partial per workgroup.  A
// second, tiny kernel adds the partials of a sample in a fixed order, so results are
// deterministic and independent of the batch index (no atomics anywhere).
// A call on few small latents is all launch latency: there one more workgroup per sample reads v_c and v_u on its own and writes the
// sample's discrepancies in the same launch (see kOneLaunchBytes).
#include "common.h"

#include <mutex>

// Scratch of the allocation-free entry point (hyb_cfg_disc_euler_noalloc): the per-workgroup partial sums live in
// this file-scope device array instead of a caller-provided workspace.  Every GPU the library runs on holds its
// own copy until the process ends.  In host code the name is only a handle for hipGetSymbolAddress; kernels get
// the device address obtained from it.
static __device__ __align__(256) unsigned char scratch[HYB_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kThreads = 256;
constexpr int kVec = 8;                          // elements per thread per iteration
constexpr int kIters = 1;                        // one vector per thread: the smallest workgroups stream fastest (5.8 vs 5.5 TB/s with two)

// 16-byte vector accesses.  The inputs are streamed once, so they are read with non-temporal loads (they are not
// kept in the caches on their way in: 6.0-6.4 TB/s instead of 5.6-5.8 on 256 x 262144 elements); stores are plain
// (non-temporal stores are slower here).
template <typename T, int V> struct Vec;
template <> struct Vec<float, 8> {
    static __device__ __forceinline__ void load(const float* p, float* r) {
        const f32x4 a = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
        const f32x4 b = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p + 4));
        r[0] = a[0]; r[1] = a[1]; r[2] = a[2]; r[3] = a[3]; r[4] = b[0]; r[5] = b[1]; r[6] = b[2]; r[7] = b[3];
    }
    static __device__ __forceinline__ void store(float* p, const float* r) {
        f32x4 a = {r[0], r[1], r[2], r[3]}, b = {r[4], r[5], r[6], r[7]};
        *reinterpret_cast<f32x4*>(p) = a;
        *reinterpret_cast<f32x4*>(p + 4) = b;
    }
};
template <> struct Vec<bf16_t, 8> {
    static __device__ __forceinline__ void load(const bf16_t* p, float* r) {
        const u32x4 a = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));   // bf16 -> fp32: the bits, shifted up
#pragma unroll
        for (int i = 0; i < 4; i++) {
            r[2 * i] = __uint_as_float(a[i] << 16);
            r[2 * i + 1] = __uint_as_float(a[i] & 0xffff0000u);
        }
    }
    static __device__ __forceinline__ void store(bf16_t* p, const float* r) {
        bf16x8 a;
#pragma unroll
        for (int i = 0; i < 8; i++) a[i] = (bf16_t)r[i];
        *reinterpret_cast<bf16x8*>(p) = a;
    }
};
template <typename T> struct Vec<T, 1> {
    static __device__ __forceinline__ void load(const T* p, float* r) { r[0] = to_f32<T>(*p); }
    static __device__ __forceinline__ void store(T* p, const float* r) { *p = from_f32<T>(r[0]); }
};

struct GuidanceArgs {
    const void* v_c;
    const void* v_u;
    const float* x;
    float* x_out;
    bf16_t* x_lowp;
    void* v_out;
    size_t n;        // elements per sample
    float s, a, b;   // v = u + s (c - u);  x_out = a x + b v
    double* partial; // [batch][blocks_per_sample][4] or nullptr
};

// V = 8: vector path (n % 8 == 0, so a vector never straddles the end of a sample); V = 1: scalar.
template <typename VT, int V>
__global__ __launch_bounds__(kThreads) void guidance_kernel(GuidanceArgs g) {
    const size_t sample = blockIdx.y;
    const size_t off = sample * g.n;
    const VT* vc = static_cast<const VT*>(g.v_c) + off;
    const VT* vu = static_cast<const VT*>(g.v_u) + off;
    VT* vo = g.v_out ? static_cast<VT*>(g.v_out) + off : nullptr;
    const float* x = g.x ? g.x + off : nullptr;
    float* xo = g.x_out ? g.x_out + off : nullptr;
    bf16_t* xl = g.x_lowp ? g.x_lowp + off : nullptr;

    float s_d1 = 0.f, s_d2 = 0.f, s_u1 = 0.f, s_u2 = 0.f;
    const size_t chunk0 = (size_t)blockIdx.x * (kThreads * V * kIters);
#pragma unroll
    for (int it = 0; it < kIters; it++) {
        const size_t i = chunk0 + ((size_t)it * kThreads + threadIdx.x) * V;
        if (i < g.n) {
            float c[V], u[V], v[V];
            Vec<VT, V>::load(vc + i, c);
            Vec<VT, V>::load(vu + i, u);
#pragma unroll
            for (int j = 0; j < V; j++) {
                const float d = c[j] - u[j];
                s_d1 += fabsf(d);
                s_d2 = fmaf(d, d, s_d2);
                s_u1 += fabsf(u[j]);
                s_u2 = fmaf(u[j], u[j], s_u2);
                v[j] = fmaf(g.s, d, u[j]);
            }
            if (vo) Vec<VT, V>::store(vo + i, v);
            if (xo) {
                float xv[V];
                Vec<float, V>::load(x + i, xv);
#pragma unroll
                for (int j = 0; j < V; j++) xv[j] = fmaf(g.b, v[j], g.a * xv[j]);
                Vec<float, V>::store(xo + i, xv);
                if (xl) Vec<bf16_t, V>::store(xl + i, xv);
            }
        }
    }
    if (g.partial) {
        __shared__ double red[kThreads / HYB_WAVE][4];
        const double r0 = wave_sum((double)s_d1), r1 = wave_sum((double)s_d2);
        const double r2 = wave_sum((double)s_u1), r3 = wave_sum((double)s_u2);
        const int wave = threadIdx.x / HYB_WAVE, lane = threadIdx.x % HYB_WAVE;
        if (lane == 0) { red[wave][0] = r0; red[wave][1] = r1; red[wave][2] = r2; red[wave][3] = r3; }
        __syncthreads();
        if (threadIdx.x < 4) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < kThreads / HYB_WAVE; w++) t += red[w][threadIdx.x];
            g.partial[((size_t)sample * gridDim.x + blockIdx.x) * 4 + threadIdx.x] = t;
        }
    }
}

__device__ __forceinline__ float ratio(double num, double den) {
    if (num == 0.0) return 0.f;
    if (den == 0.0) return __builtin_inff();
    return (float)(num / den);
}

// One wave per sample: lane l adds partials l, l + 64, ... in order, then a fixed butterfly.
__global__ __launch_bounds__(HYB_WAVE) void discrepancy_finalize_kernel(const double* partial, int blocks_per_sample,
                                                                         float* d1, float* d2) {
    const size_t sample = blockIdx.x;
    const double* p = partial + sample * blocks_per_sample * 4;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = threadIdx.x; i < blocks_per_sample; i += HYB_WAVE)
        for (int j = 0; j < 4; j++) acc[j] += p[(size_t)i * 4 + j];
    for (int j = 0; j < 4; j++) acc[j] = wave_sum(acc[j]);
    if (threadIdx.x == 0) {
        if (d1) d1[sample] = ratio(acc[0], acc[2]);
        if (d2) d2[sample] = ratio(sqrt(acc[1]), sqrt(acc[3]));
    }
}

// The pass and the discrepancies of small samples in one launch: workgroups 1 .. of a sample do what guidance_kernel does without its
// sums, workgroup 0 sums over the whole sample, in the order of guidance_kernel and discrepancy_finalize_kernel: a sample has the same
// discrepancies whichever form a call takes.  A "unit" is what a wave of guidance_kernel sums, 64 vectors; a wave here takes up to eight of them,
// all loads in flight (as raw bits: 64 registers), and adds their lanes in one go (wave_sums).
constexpr int kOneThreads = 1024;
constexpr int kOneWaves = kOneThreads / HYB_WAVE;
constexpr int kUnitsPerChunk = kThreads / HYB_WAVE * kIters;       // of a workgroup of guidance_kernel
constexpr int kOneUnits = 128;                                     // the most a sample has
static_assert(kIters == 1 && kOneUnits / kUnitsPerChunk <= HYB_WAVE, "a lane of the finalisation has one chunk");

// V values, as they were loaded and as floats
template <typename VT, int V> struct Raw {
    static constexpr int N = V * (int)sizeof(VT) / 16;
    u32x4 bits[N];
    __device__ __forceinline__ void load(const VT* p) {
#pragma unroll
        for (int i = 0; i < N; i++) bits[i] = reinterpret_cast<const u32x4*>(p)[i];
    }
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int i = 0; i < N; i++) bits[i] = u32x4{0, 0, 0, 0};
    }
    __device__ __forceinline__ float get(int j) const {
        if constexpr (sizeof(VT) == 4) return __uint_as_float(bits[j / 4][j % 4]);
        else return __uint_as_float(j % 2 ? bits[j / 8][j % 8 / 2] & 0xffff0000u : bits[j / 8][j % 8 / 2] << 16);
    }
};
template <typename VT> struct Raw<VT, 1> {
    VT value;
    __device__ __forceinline__ void load(const VT* p) { value = *p; }
    __device__ __forceinline__ void zero() { value = (VT)0.f; }
    __device__ __forceinline__ float get(int) const { return to_f32<VT>(value); }
};

// a + a of lane ^ O in the lanes without bit O, b + b of lane ^ O in those with it.
template <int O>
__device__ __forceinline__ double exchange_add(double a, double b) {
    if constexpr (O >= 16) {
        const u32x2 x = __builtin_bit_cast(u32x2, a), y = __builtin_bit_cast(u32x2, b);
        auto swap = [](unsigned p, unsigned q) {
            if constexpr (O == 32) return __builtin_amdgcn_permlane32_swap(p, q, false, false);
            else return __builtin_amdgcn_permlane16_swap(p, q, false, false);
        };
        const auto lo = swap(x[0], y[0]), hi = swap(x[1], y[1]);
        return __builtin_bit_cast(double, u32x2{lo[0], hi[0]}) + __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
    } else {
        const bool upper = threadIdx.x & O;
        const double keep = upper ? b : a, give = upper ? a : b;
        return keep + __shfl_xor(give, O, 64);
    }
}

// Sums over the lanes of N values, each with the additions of wave_sum(); lane l returns that of value l / (64 / N).  Two halves of the wave
// go on with half of the values each, so N values cost N - 1 exchanges and those of the last 64 / N lanes, not six per value.
template <int N, int O = 32, int C = N / 2>
__device__ __forceinline__ double wave_sums(double (&v)[N]) {
    if constexpr (O == 0) return v[0];
    else {
        if constexpr (C > 0) {
#pragma unroll
            for (int i = 0; i < C; i++) v[i] = exchange_add<O>(v[i], v[i + C]);
        } else v[0] += __shfl_xor(v[0], O, 64);
        return wave_sums<N, O / 2, C / 2>(v);
    }
}

// Sums of the units wave, wave + 16, ... (ROUNDS of them) into red[unit][quantity].
template <typename VT, int V, int ROUNDS>
__device__ __forceinline__ void unit_sums(const VT* vc, const VT* vu, size_t n, double (*red)[4]) {
    const int wave = threadIdx.x / HYB_WAVE, lane = threadIdx.x % HYB_WAVE;
    Raw<VT, V> c[ROUNDS], u[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        const size_t i = ((size_t)r * kOneThreads + threadIdx.x) * V;
        if (i < n) {
            c[r].load(vc + i);
            u[r].load(vu + i);
        } else {
            c[r].zero();
            u[r].zero();
        }
    }
    double sums[4 * ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        float s_d1 = 0.f, s_d2 = 0.f, s_u1 = 0.f, s_u2 = 0.f;
#pragma unroll
        for (int j = 0; j < V; j++) {
            const float uj = u[r].get(j), d = c[r].get(j) - uj;
            s_d1 += fabsf(d);
            s_d2 = fmaf(d, d, s_d2);
            s_u1 += fabsf(uj);
            s_u2 = fmaf(uj, uj, s_u2);
        }
        sums[4 * r] = (double)s_d1; sums[4 * r + 1] = (double)s_d2; sums[4 * r + 2] = (double)s_u1; sums[4 * r + 3] = (double)s_u2;
    }
    constexpr int LANES = HYB_WAVE / (4 * ROUNDS);       // that hold the same sum
    const double t = wave_sums(sums);
    const int value = lane / LANES;
    if (lane % LANES == 0) red[value / 4 * kOneWaves + wave][value % 4] = t;
}

template <typename VT, int V>
__device__ __forceinline__ void whole_sample_sums(const VT* vc, const VT* vu, size_t n, float* d1, float* d2) {
    constexpr int ROUNDS = (sizeof(VT) == 4 && V > 1 ? kOneUnits / 2 : kOneUnits) / kOneWaves;      // (a sample of fp32 vectors has half as many units)
    __shared__ double red[kOneUnits][4];
    if (n <= (size_t)kOneThreads * V) unit_sums<VT, V, 1>(vc, vu, n, red);
    else unit_sums<VT, V, ROUNDS>(vc, vu, n, red);
    __syncthreads();
    if (threadIdx.x < HYB_WAVE) {
        const int lane = threadIdx.x, chunks = (int)((n + kThreads * V - 1) / (kThreads * V));
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        if (lane < chunks) {
#pragma unroll
            for (int j = 0; j < 4; j++) {
                double t = 0.0;
#pragma unroll
                for (int w = 0; w < kUnitsPerChunk; w++) t += red[lane * kUnitsPerChunk + w][j];
                acc[j] += t;
            }
        }
        const double t = wave_sums(acc);
        const double u1 = __shfl(t, 32, 64), d2sum = __shfl(t, 16, 64), u2 = __shfl(t, 48, 64);
        if (lane == 0) {
            if (d1) *d1 = ratio(t, u1);
            if (d2) *d2 = ratio(sqrt(d2sum), sqrt(u2));
        }
    }
}

template <typename VT, int V>
__global__ __launch_bounds__(kOneThreads) void guidance_one_launch_kernel(GuidanceArgs g, float* d1, float* d2) {
    const size_t sample = blockIdx.y, off = sample * g.n;
    const VT* vc = static_cast<const VT*>(g.v_c) + off;
    const VT* vu = static_cast<const VT*>(g.v_u) + off;
    if (blockIdx.x == 0) {
        whole_sample_sums<VT, V>(vc, vu, g.n, d1 ? d1 + sample : nullptr, d2 ? d2 + sample : nullptr);
        return;
    }
    const size_t i = ((size_t)(blockIdx.x - 1) * kOneThreads + threadIdx.x) * V;
    if (i >= g.n) return;
    float c[V], u[V], xv[V], v[V];
    Vec<VT, V>::load(vc + i, c);
    Vec<VT, V>::load(vu + i, u);
    Vec<float, V>::load(g.x + off + i, xv);
#pragma unroll
    for (int j = 0; j < V; j++) {
        v[j] = fmaf(g.s, c[j] - u[j], u[j]);
        xv[j] = fmaf(g.b, v[j], g.a * xv[j]);
    }
    if (g.v_out) Vec<VT, V>::store(static_cast<VT*>(g.v_out) + off + i, v);
    Vec<float, V>::store(g.x_out + off + i, xv);
    if (g.x_lowp) Vec<bf16_t, V>::store(g.x_lowp + off + i, xv);
}

template <typename XT, typename VT>
__global__ __launch_bounds__(kThreads) void euler_kernel(const XT* x, const VT* v, XT* xo, size_t n, float dt) {
    const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) xo[i] = from_f32<XT>(fmaf(dt, to_f32<VT>(v[i]), to_f32<XT>(x[i])));
}

int blocks_for(size_t n, int vec) {
    const size_t chunk = (size_t)kThreads * vec * kIters;
    return (int)((n + chunk - 1) / chunk);
}

// Largest blocks-per-sample over both code paths, so the workspace query does not depend on it.
size_t partial_bytes(int batch, size_t n) { return (size_t)batch * blocks_for(n, 1) * 4 * sizeof(double); }

// One launch where a sample's v_c and v_u together are at most kOneLaunchBytes and those of all samples kOneLaunchTotal.  Two launches against one,
// us, in a stream of calls: 1 x 1024 fp32 8.6 -> 6.1, 1 x 65536 bf16 8.7 -> 6.6 (a call on its own that the host waits for 20.1 -> 20.4: the
// summing workgroup has a CU's arithmetic), 28 x 65536 8.7 -> 8.2, 80 x 16384 8.5 -> 6.5, 32 x 32768 fp32 8.6 -> 6.1.
// Not where its workgroups (one CU holds two of 1024 threads) are more than the CUs: 32 x 65536 8.5 -> 9.9, 128 x 16384 8.7 -> 9.1; samples with one updating
// workgroup have four per CU: 512 x 4096 8.7 -> 8.4, 512 x 1024 fp32 8.8 -> 6.2, but 1024 x 1024 fp32 8.6 -> 10.2.  Element by element
// the pass itself is the longer part: 256 x 8191 23.4 -> 13.6, 1024 x 1023 fp32 14.1 -> 9.4.
// Element by element (n % 8 != 0) a sample of kOneLaunchScalar elements has as many units as the summing workgroup takes (8191: 8.7 -> 6.1).
constexpr size_t kOneLaunchBytes = 256 * 1024, kOneLaunchTotal = 8 * 1024 * 1024, kOneLaunchScalar = 8192;
static_assert(kOneLaunchBytes / 2 / sizeof(bf16_t) <= (size_t)kOneUnits * HYB_WAVE * kVec && kOneLaunchBytes / 2 / sizeof(float) <= (size_t)kOneUnits / 2 * HYB_WAVE * kVec &&
              kOneLaunchScalar <= (size_t)kOneUnits * HYB_WAVE, "a sample's units");

// The summing workgroup reads v_c and v_u while others write, and writes the discrepancies while others read x and write: no output may overlap
// v_c or v_u, and the discrepancies none of the others (two launches read all of v_c, v_u and x first and write the discrepancies last).
bool overlaps(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return a && b && x < y + b_bytes && y < x + a_bytes;
}

bool one_launch(const GuidanceArgs& g, int batch, size_t vs, const float* d1, const float* d2) {
    if (!g.partial || (!d1 && !d2) || !g.x_out || 2 * g.n * vs > kOneLaunchBytes || (size_t)batch * 2 * g.n * vs > kOneLaunchTotal) return false;
    if (g.n % kVec != 0) {
        if (g.n > kOneLaunchScalar) return false;
    } else {
        const size_t updating = (g.n + kOneThreads * kVec - 1) / (kOneThreads * kVec), cus = (size_t)hyb_cu_count();
        if ((size_t)batch * (1 + updating) > (updating == 1 ? 4 * cus : cus)) return false;
    }
    const size_t n = (size_t)batch * g.n;
    for (const void* v : {g.v_c, g.v_u})
        if (overlaps(v, n * vs, g.x_out, n * 4) || overlaps(v, n * vs, g.x_lowp, n * 2) || overlaps(v, n * vs, g.v_out, n * vs) ||
            overlaps(v, n * vs, d1, (size_t)batch * 4) || overlaps(v, n * vs, d2, (size_t)batch * 4)) return false;
    for (const float* d : {d1, d2}) {
        const size_t bytes = (size_t)batch * 4;
        if (overlaps(d, bytes, g.x, n * 4) || overlaps(d, bytes, g.x_out, n * 4) || overlaps(d, bytes, g.x_lowp, n * 2) || overlaps(d, bytes, g.v_out, n * vs)) return false;
    }
    return true;
}

int launch_guidance(const char* who, GuidanceArgs g, int batch, hyb_dtype vd, float* d1, float* d2, hipStream_t st) {
    if (batch == 0 || g.n == 0) {
        // Nothing to read: an empty sample has num = den = 0, i.e. discrepancy 0.
        if (batch > 0 && (d1 || d2)) {
            hipLaunchKernelGGL(discrepancy_finalize_kernel, dim3(batch), dim3(HYB_WAVE), 0, st, (const double*)nullptr, 0, d1, d2);
            return hyb_check_launch(who);
        }
        return HYB_OK;
    }
    const bool vec = (g.n % kVec) == 0;
    const int nblk = blocks_for(g.n, vec ? kVec : 1);
    HYB_REQUIRE(batch <= 65535, HYB_ERR_SHAPE, "%s: batch %d exceeds 65535", who, batch);
    dim3 grid(nblk, batch), block(kThreads);
    // algorithmic bytes: v_c + v_u read, x read, x_out written, plus the optional outputs
    const double vs = (double)hyb_dtype_size(vd);
    const double per_elem = 2 * vs + (g.x_out ? 8 : 0) + (g.x_lowp ? 2 : 0) + (g.v_out ? vs : 0);
    if (one_launch(g, batch, hyb_dtype_size(vd), d1, d2)) {
        const size_t per_wg = (size_t)kOneThreads * (vec ? kVec : 1);
        dim3 grid1(1 + (unsigned)((g.n + per_wg - 1) / per_wg), batch), block1(kOneThreads);
        HybTraceScope trace("guidance_pass", "byte", per_elem * (double)batch * (double)g.n, st);
        if (vd == HYB_BF16) {
            if (vec) hipLaunchKernelGGL((guidance_one_launch_kernel<bf16_t, 8>), grid1, block1, 0, st, g, d1, d2);
            else hipLaunchKernelGGL((guidance_one_launch_kernel<bf16_t, 1>), grid1, block1, 0, st, g, d1, d2);
        } else {
            if (vec) hipLaunchKernelGGL((guidance_one_launch_kernel<float, 8>), grid1, block1, 0, st, g, d1, d2);
            else hipLaunchKernelGGL((guidance_one_launch_kernel<float, 1>), grid1, block1, 0, st, g, d1, d2);
        }
        return hyb_check_launch(who);
    }
    {   // the pass itself; the tiny finalisation below is a launch of its own
        HybTraceScope trace("guidance_pass", "byte", per_elem * (double)batch * (double)g.n, st);
        if (vd == HYB_BF16) {
            if (vec) hipLaunchKernelGGL((guidance_kernel<bf16_t, 8>), grid, block, 0, st, g);
            else hipLaunchKernelGGL((guidance_kernel<bf16_t, 1>), grid, block, 0, st, g);
        } else {
            if (vec) hipLaunchKernelGGL((guidance_kernel<float, 8>), grid, block, 0, st, g);
            else hipLaunchKernelGGL((guidance_kernel<float, 1>), grid, block, 0, st, g);
        }
    }
    int rc = hyb_check_launch(who);
    if (rc != HYB_OK) return rc;
    if (g.partial && (d1 || d2)) {
        HybTraceScope trace("discrepancy_finalize", "byte", (double)batch * nblk * 32.0, st);
        hipLaunchKernelGGL(discrepancy_finalize_kernel, dim3(batch), dim3(HYB_WAVE), 0, st, g.partial, nblk, d1, d2);
        rc = hyb_check_launch(who);
    }
    return rc;
}

}  // namespace

extern "C" size_t hyb_discrepancy_workspace_bytes(int batch, size_t n_per_sample) {
    if (batch <= 0) return 0;
    return hyb_align_up(partial_bytes(batch, n_per_sample), 256);
}

extern "C" int hyb_cfg_combine(const void* v_c, const void* v_u, void* v_out, size_t n, float scale,
                               hyb_dtype dtype, void* stream) {
    HYB_CHECK_DTYPE(dtype);
    if (n == 0) return HYB_OK;
    HYB_CHECK_PTR(v_c); HYB_CHECK_PTR(v_u); HYB_CHECK_PTR(v_out);
    HYB_CHECK_ALIGN(v_c); HYB_CHECK_ALIGN(v_u); HYB_CHECK_ALIGN(v_out);
    GuidanceArgs g = {v_c, v_u, nullptr, nullptr, nullptr, v_out, n, scale, 1.f, 0.f, nullptr};
    // One "sample" of n elements would need n / chunk workgroups in grid.x: fine up to 2^31 - 1.
    HYB_REQUIRE(n / kThreads < 0x7fffffffu, HYB_ERR_SHAPE, "hyb_cfg_combine: n too large");
    return launch_guidance("hyb_cfg_combine", g, 1, dtype, nullptr, nullptr, (hipStream_t)stream);
}

extern "C" int hyb_branch_discrepancy(const void* v_c, const void* v_u, int batch, size_t n_per_sample,
                                      hyb_norm p, hyb_dtype dtype, float* out,
                                      void* workspace, size_t workspace_bytes, void* stream) {
    HYB_CHECK_DTYPE(dtype);
    HYB_REQUIRE(p == HYB_NORM_L1 || p == HYB_NORM_L2, HYB_ERR_DTYPE, "hyb_branch_discrepancy: p must be HYB_NORM_L1 or HYB_NORM_L2");
    HYB_REQUIRE(batch >= 0, HYB_ERR_SHAPE, "hyb_branch_discrepancy: negative batch");
    if (batch == 0) return HYB_OK;
    HYB_CHECK_PTR(out);
    if (n_per_sample > 0) {
        HYB_CHECK_PTR(v_c); HYB_CHECK_PTR(v_u); HYB_CHECK_PTR(workspace);
        HYB_CHECK_ALIGN(v_c); HYB_CHECK_ALIGN(v_u); HYB_CHECK_ALIGN(workspace);
        HYB_REQUIRE(workspace_bytes >= hyb_discrepancy_workspace_bytes(batch, n_per_sample), HYB_ERR_WORKSPACE,
                    "hyb_branch_discrepancy: workspace of %zu bytes is smaller than the %zu required", workspace_bytes,
                    hyb_discrepancy_workspace_bytes(batch, n_per_sample));
    }
    GuidanceArgs g = {v_c, v_u, nullptr, nullptr, nullptr, nullptr, n_per_sample, 0.f, 1.f, 0.f, (double*)workspace};
    return launch_guidance("hyb_branch_discrepancy", g, batch, dtype, p == HYB_NORM_L1 ? out : nullptr,
                           p == HYB_NORM_L2 ? out : nullptr, (hipStream_t)stream);
}

extern "C" int hyb_euler_step(const void* x, const void* v, void* x_out, size_t n, float t, float t_next,
                              hyb_dtype x_dtype, hyb_dtype v_dtype, void* stream) {
    HYB_CHECK_DTYPE(x_dtype); HYB_CHECK_DTYPE(v_dtype);
    if (n == 0) return HYB_OK;
    HYB_CHECK_PTR(x); HYB_CHECK_PTR(v); HYB_CHECK_PTR(x_out);
    HYB_CHECK_ALIGN(x); HYB_CHECK_ALIGN(v); HYB_CHECK_ALIGN(x_out);
    const size_t nblk = (n + kThreads - 1) / kThreads;
    HYB_REQUIRE(nblk < 0x7fffffffu, HYB_ERR_SHAPE, "hyb_euler_step: n too large");
    const float dt = t_next - t;
    hipStream_t st = (hipStream_t)stream;
    dim3 grid((unsigned)nblk), block(kThreads);
    if (x_dtype == HYB_F32 && v_dtype == HYB_F32)
        hipLaunchKernelGGL((euler_kernel<float, float>), grid, block, 0, st, (const float*)x, (const float*)v, (float*)x_out, n, dt);
    else if (x_dtype == HYB_F32)
        hipLaunchKernelGGL((euler_kernel<float, bf16_t>), grid, block, 0, st, (const float*)x, (const bf16_t*)v, (float*)x_out, n, dt);
    else if (v_dtype == HYB_F32)
        hipLaunchKernelGGL((euler_kernel<bf16_t, float>), grid, block, 0, st, (const bf16_t*)x, (const float*)v, (bf16_t*)x_out, n, dt);
    else
        hipLaunchKernelGGL((euler_kernel<bf16_t, bf16_t>), grid, block, 0, st, (const bf16_t*)x, (const bf16_t*)v, (bf16_t*)x_out, n, dt);
    return hyb_check_launch("hyb_euler_step");
}

extern "C" int hyb_cfg_disc_affine(const void* v_c, const void* v_u, const float* x, float* x_out,
                                   void* x_out_lowp, void* v_out, int batch, size_t n_per_sample,
                                   float scale, float a, float b, float* disc_l1, float* disc_l2,
                                   hyb_dtype v_dtype, void* workspace, size_t workspace_bytes, void* stream) {
    HYB_CHECK_DTYPE(v_dtype);
    HYB_REQUIRE(batch >= 0, HYB_ERR_SHAPE, "hyb_cfg_disc_affine: negative batch");
    if (batch == 0) return HYB_OK;
    const bool sums = disc_l1 || disc_l2;
    if (n_per_sample > 0) {
        HYB_CHECK_PTR(v_c); HYB_CHECK_PTR(v_u); HYB_CHECK_PTR(x); HYB_CHECK_PTR(x_out);
        HYB_CHECK_ALIGN(v_c); HYB_CHECK_ALIGN(v_u); HYB_CHECK_ALIGN(x); HYB_CHECK_ALIGN(x_out);
        HYB_CHECK_ALIGN(x_out_lowp); HYB_CHECK_ALIGN(v_out);
        if (sums) {
            HYB_CHECK_PTR(workspace); HYB_CHECK_ALIGN(workspace);
            HYB_REQUIRE(workspace_bytes >= hyb_discrepancy_workspace_bytes(batch, n_per_sample), HYB_ERR_WORKSPACE,
                        "hyb_cfg_disc_affine: workspace of %zu bytes is smaller than the %zu required", workspace_bytes,
                        hyb_discrepancy_workspace_bytes(batch, n_per_sample));
        }
    }
    GuidanceArgs g = {v_c, v_u, x, x_out, (bf16_t*)x_out_lowp, v_out, n_per_sample, scale, a, b,
                      sums ? (double*)workspace : nullptr};
    return launch_guidance("hyb_cfg_disc_affine", g, batch, v_dtype, disc_l1, disc_l2, (hipStream_t)stream);
}

extern "C" int hyb_cfg_disc_euler(const void* v_c, const void* v_u, const float* x, float* x_out,
                                  void* x_out_lowp, void* v_out, int batch, size_t n_per_sample,
                                  float scale, float t, float t_next, float* disc_l1, float* disc_l2,
                                  hyb_dtype v_dtype, void* workspace, size_t workspace_bytes, void* stream) {
    return hyb_cfg_disc_affine(v_c, v_u, x, x_out, x_out_lowp, v_out, batch, n_per_sample, scale, 1.0f,
                               t_next - t, disc_l1, disc_l2, v_dtype, workspace, workspace_bytes, stream);
}

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mx;
void* g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch` on each device, looked up once per device

// Address of the static scratch array on the current device (nullptr + error set on failure).
void* static_scratch() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        hyb_set_error(HYB_ERR_LAUNCH, "hyb_cfg_disc_euler_noalloc: no current device (or device index >= %d)", kMaxDevices);
        return nullptr;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mx);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            hyb_set_error(HYB_ERR_LAUNCH, "hyb_cfg_disc_euler_noalloc: hipGetSymbolAddress failed: %s", hipGetErrorString(e));
            return nullptr;
        }
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}
}  // namespace

extern "C" int hyb_cfg_disc_euler_noalloc(const void* v_c, const void* v_u, const float* x, float* x_out,
                                          void* x_out_lowp, void* v_out, int batch, size_t n_per_sample,
                                          float scale, float t, float t_next, float* disc_l1, float* disc_l2,
                                          hyb_dtype v_dtype, void* stream) {
    HYB_REQUIRE(batch >= 0, HYB_ERR_SHAPE, "hyb_cfg_disc_euler_noalloc: negative batch");
    void* ws = nullptr;
    size_t need = 0;
    if (batch > 0 && n_per_sample > 0 && (disc_l1 || disc_l2)) {
        // size check in integers first (the workspace query itself would overflow an int for absurd sizes)
        HYB_REQUIRE(n_per_sample / kThreads < (size_t)HYB_STATIC_SCRATCH_BYTES, HYB_ERR_WORKSPACE,
                    "hyb_cfg_disc_euler_noalloc: n_per_sample %zu is beyond the static scratch", n_per_sample);
        need = hyb_discrepancy_workspace_bytes(batch, n_per_sample);
        HYB_REQUIRE(need <= (size_t)HYB_STATIC_SCRATCH_BYTES, HYB_ERR_WORKSPACE,
                    "hyb_cfg_disc_euler_noalloc: batch %d x %zu elements needs %zu bytes of partial sums, the static scratch holds %d "
                    "(use hyb_cfg_disc_euler with a workspace)", batch, n_per_sample, need, HYB_STATIC_SCRATCH_BYTES);
        ws = static_scratch();
        if (!ws) return HYB_ERR_LAUNCH;
    }
    // Every partial the finalisation reads is written by this call's first kernel, so nothing has to be cleared.
    return hyb_cfg_disc_affine(v_c, v_u, x, x_out, x_out_lowp, v_out, batch, n_per_sample, scale, 1.0f, t_next - t,
                               disc_l1, disc_l2, v_dtype, ws, need, stream);
}
