// fp32 softmax attention on the fp32 matrix cores (the reference-precision path): o = softmax(q k^T * scale) v with a
// streaming softmax, every product and sum in v_mfma_f32_16x16x4_f32, exponentials to fp32 accuracy (exp_neg below).
//
// What bounds it: the fp32 matrix rate (256 flop per clock and CU), so operands go straight from global memory (L2) to
// registers, without LDS: a wave needs 16 KB for 4096 clocks of MFMAs.  A workgroup of 4 waves owns 32 query rows of one
// (batch, head) and splits the KEYS: wave w takes the 32-key tiles w, w + 4, ... with a running maximum and normaliser of
// its own, and the four partial results are merged in LDS at the end, in a fixed order.  (Queries split over the waves
// would leave three quarters of the chip idle at the few hundred tokens of these models.)
//
// Both contractions are transposed, as in attention_mfma.hip: S^T = K Q^T, O^T += V^T P^T; lane (l16 = lane % 16,
// q4 = lane / 16) of an accumulator tile holds column (query) l16 and rows 4 q4 .. 4 q4 + 3.  The order of a contraction
// index does not matter as long as both operands agree, so
//   S: a 16-byte load gives the lane 4 features of its key (query) row, which feed 4 MFMAs;
//   PV: register i of the exponentiated S^T is the B operand of the MFMA over keys {4 q4 + i}, and the matching V operand
//       is one 16-byte load of row 4 q4 + i: the lane's features 4 l16 .. 4 l16 + 3 are row l16 of the output tiles 0 .. 3.
// Two waves share a SIMD and start together, so neither covers the other's softmax: a wave runs the first contraction of its next tile beside the
// softmax of this one (vector instructions between the MFMAs, no branches in it).
// Measured: batch 2, 12 heads, 653 tokens 37.7 us by itself (70 TFLOP/s; softmax between the contractions 41.1), 2 x 24 x 1400 264 us (91; 275); one
// wave per query row on the vector ALU took 453 us for the first.
#include "attention.h"

namespace {

constexpr int BQ = 32;    // query rows per workgroup
constexpr int BKV = 32;   // keys per tile
constexpr int WAVES = 4;

// e^x for x <= 0, without the library routine's range handling: e^x = 2^n 2^f with n = x log2(e) rounded to a whole number and f
// the rest, taken with log2(e) in two parts, so that neither the product's rounding nor that of log2(e) counts.  The
// power of two is applied by ldexp, which rounds into the subnormal numbers as a product would (1.5 ulp at most, tested); NaN stays NaN.
__device__ __forceinline__ float exp_neg(float x) {
    x = x < -200.f ? -200.f : x;      // 0 well before; minus infinity would make f NaN
    const float n = rintf(x * 1.44269502162933349609375f);
    const float f = fmaf(x, 1.92596299112661746887e-8f, fmaf(x, 1.44269502162933349609375f, -n));
    return __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}

// 64 MFMAs with the vector instructions of the same block spread between them.
template <int J>
__device__ __forceinline__ void interleave_vector_work() {
    if constexpr (J < 64) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x402, 6, 0);
        interleave_vector_work<J + 1>();
    }
}

__global__ __launch_bounds__(256, 2) void attention_f32_kernel(AttnArgs a, int qblocks, int total, int xcd_run) {
    __shared__ float part_o[WAVES][2][4][4][64];   // [wave][query tile][feature tile][register][lane]
    __shared__ float part_ml[WAVES][2][2][16];     // [wave][query tile][maximum, normaliser][query]
    // XCD x serves consecutive query blocks of consecutive (batch, head) pairs: their K and V stay in its L2
    const unsigned id = blockIdx.y * gridDim.x + blockIdx.x;
    const int blk = (int)(id % 8) * xcd_run + (int)(id / 8);
    if ((int)(id / 8) >= xcd_run || blk >= total) return;
    const int pair = blk / qblocks, qb = blk % qblocks;
    const int h = pair % a.heads, b = pair / a.heads;
    const int lane = threadIdx.x % 64, l16 = lane % 16, q4 = lane / 16;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const float* kp = static_cast<const float*>(a.k) + (size_t)pair * a.n_kv * 64;
    const float* vp = static_cast<const float*>(a.v) + (size_t)pair * a.n_kv * 64;

    f32x4 q[2][4];   // [query tile][16-feature step]
#pragma unroll
    for (int qt = 0; qt < 2; qt++) {
        const int row = min(qb * BQ + qt * 16 + l16, a.n_q - 1);
        const float* qp = static_cast<const float*>(a.q) + ((size_t)pair * (a.q_stride ? a.q_stride : a.n_q) + row) * 64;
#pragma unroll
        for (int s = 0; s < 4; s++) q[qt][s] = *reinterpret_cast<const f32x4*>(qp + 16 * s + 4 * q4);
    }
    f32x4 k[2][4], v[2][4];   // K: [key tile][16-feature step]; V: [key tile][row 4 q4 + i]
    auto load_k = [&](int t) {
#pragma unroll
        for (int kt = 0; kt < 2; kt++) {
            const float* row = kp + (size_t)min(t * BKV + kt * 16 + l16, a.n_kv - 1) * 64 + 4 * q4;
#pragma unroll
            for (int s = 0; s < 4; s++) k[kt][s] = *reinterpret_cast<const f32x4*>(row + 16 * s);
        }
    };
    auto load_v = [&](int t) {
#pragma unroll
        for (int kt = 0; kt < 2; kt++)
#pragma unroll
            for (int i = 0; i < 4; i++)
                v[kt][i] = *reinterpret_cast<const f32x4*>(vp + (size_t)min(t * BKV + kt * 16 + 4 * q4 + i, a.n_kv - 1) * 64 + 4 * l16);
    };
    float m[2] = {-__builtin_inff(), -__builtin_inff()}, l[2] = {0.f, 0.f};   // the lane's queries; l: over the lane's own keys
    f32x4 o[4][2];   // [feature tile][query tile]
#pragma unroll
    for (int i = 0; i < 8; i++) o[i / 2][i % 2] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nt = (a.n_kv + BKV - 1) / BKV;
    auto scores = [&](f32x4 (&s)[2][2]) {    // [key tile][query tile]: keys 16 kt + 4 q4 + i
#pragma unroll
        for (int i = 0; i < 4; i++) s[i / 2][i % 2] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int st = 0; st < 4; st++)
#pragma unroll
            for (int j = 0; j < 4; j++)
#pragma unroll
                for (int kt = 0; kt < 2; kt++)
#pragma unroll
                    for (int qt = 0; qt < 2; qt++)
                        s[kt][qt] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[kt][st][j], q[qt][st][j], s[kt][qt], 0, 0, 0);
    };
    // scores of tile t -> probabilities; running maximum, normaliser and output rescaled.  Without a branch, so that it can stand between
    // the next tile's MFMAs (a factor of 1 changes nothing).
    auto softmax = [&](f32x4 (&s)[2][2], int t) {
        const int left = a.n_kv - t * BKV - 4 * q4;      // keys 16 kt + i >= left are past the end
#pragma unroll
        for (int kt = 0; kt < 2; kt++)
#pragma unroll
            for (int qt = 0; qt < 2; qt++)
#pragma unroll
                for (int i = 0; i < 4; i++) s[kt][qt][i] = kt * 16 + i >= left ? -__builtin_inff() : s[kt][qt][i] * a.scale;
#pragma unroll
        for (int qt = 0; qt < 2; qt++) {
            float mx = fmaxf(fmaxf(fmaxf(s[0][qt][0], s[0][qt][1]), fmaxf(s[0][qt][2], s[0][qt][3])),
                             fmaxf(fmaxf(s[1][qt][0], s[1][qt][1]), fmaxf(s[1][qt][2], s[1][qt][3])));
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float m_new = fmaxf(m[qt], mx);
            const float corr = m[qt] == m_new ? 1.f : exp_neg(m[qt] - m_new);   // first tile: exp(-inf) = 0
            m[qt] = m_new;
            l[qt] *= corr;
#pragma unroll
            for (int dt = 0; dt < 4; dt++) o[dt][qt] *= corr;
            const float ref = m_new == -__builtin_inff() ? 0.f : m_new;          // only masked scores so far: all probabilities 0
#pragma unroll
            for (int kt = 0; kt < 2; kt++)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    s[kt][qt][i] = exp_neg(s[kt][qt][i] - ref);
                    l[qt] += s[kt][qt][i];
                }
        }
    };
    auto output = [&](f32x4 (&s)[2][2], int t) {
        if ((t + 1) * BKV > a.n_kv) {   // (a masked key's probability is 0; its V must not turn that into NaN)
#pragma unroll
            for (int kt = 0; kt < 2; kt++)
#pragma unroll
                for (int i = 0; i < 4; i++)
                    if (t * BKV + kt * 16 + 4 * q4 + i >= a.n_kv) v[kt][i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int kt = 0; kt < 2; kt++)
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int dt = 0; dt < 4; dt++)
#pragma unroll
                    for (int qt = 0; qt < 2; qt++)
                        o[dt][qt] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[kt][i][dt], s[kt][qt][i], o[dt][qt], 0, 0, 0);
    };
    // The first contraction of a wave's next tile runs beside the softmax of this one.  K of the tile after that is requested once it is
    // done, V of the next tile once this tile's output is.
    if (wave < nt) {
        f32x4 cur[2][2], next[2][2];
        load_k(wave);
        load_v(wave);
        scores(cur);
        __builtin_amdgcn_sched_barrier(0);
        int t = wave;
        if (t + WAVES < nt) load_k(t + WAVES);
        for (; t + WAVES < nt; t += WAVES) {
            __builtin_amdgcn_sched_barrier(0);
            scores(next);
            softmax(cur, t);
            interleave_vector_work<0>();
            __builtin_amdgcn_sched_barrier(0);
            load_k(t + 2 * WAVES);           // (past the end: the last row)
            __builtin_amdgcn_sched_barrier(0);
            output(cur, t);
            __builtin_amdgcn_sched_barrier(0);
            load_v(t + WAVES);
#pragma unroll
            for (int i = 0; i < 4; i++) cur[i / 2][i % 2] = next[i / 2][i % 2];
        }
        softmax(cur, t);
        output(cur, t);
    }

    // merge of the waves: row = sum_p o_p e^(m_p - M) / sum_p l_p e^(m_p - M), p in order
#pragma unroll
    for (int qt = 0; qt < 2; qt++) {
        l[qt] += __shfl_xor(l[qt], 16, 64);
        l[qt] += __shfl_xor(l[qt], 32, 64);
        if (q4 == 0) {
            part_ml[wave][qt][0][l16] = m[qt];
            part_ml[wave][qt][1][l16] = l[qt];
        }
#pragma unroll
        for (int dt = 0; dt < 4; dt++)
#pragma unroll
            for (int i = 0; i < 4; i++) part_o[wave][qt][dt][i][lane] = o[dt][qt][i];
    }
    __syncthreads();
    // wave w finishes register w of every tile: features 16 q4 + 4 w .. + 3 of query l16
    const int hd = a.heads * 64;
#pragma unroll
    for (int qt = 0; qt < 2; qt++) {
        const int row = qb * BQ + qt * 16 + l16;
        if (row >= a.n_q) continue;
        float m_all = part_ml[0][qt][0][l16];
#pragma unroll
        for (int p = 1; p < WAVES; p++) m_all = fmaxf(m_all, part_ml[p][qt][0][l16]);
        float l_all = 0.f;
        f32x4 r = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int p = 0; p < WAVES; p++) {
            const float mp = part_ml[p][qt][0][l16];
            const float w = mp == -__builtin_inff() ? 0.f : (mp == m_all ? 1.f : exp_neg(mp - m_all));   // a wave without keys counts nothing
            const float lp = part_ml[p][qt][1][l16];
            l_all = fmaf(lp, w, l_all);
#pragma unroll
            for (int dt = 0; dt < 4; dt++) r[dt] = fmaf(part_o[p][qt][dt][wave][lane], w, r[dt]);
        }
        r = r / l_all;
        float* orow;
        if (row < a.split) orow = static_cast<float*>(a.o) + ((size_t)b * a.split + row) * hd;
        else orow = static_cast<float*>(a.o2) + ((size_t)b * (a.n_q - a.split) + (row - a.split)) * hd;
        *reinterpret_cast<f32x4*>(orow + h * 64 + 16 * q4 + 4 * wave) = r;
    }
}

// A grid dimension holds less than 2^32 threads, and a larger one is cut off without an error: blocks beyond this many
// (a multiple of 8, for the XCD order) go into the second dimension.
constexpr int kMaxGridX = 1 << 23;

int launch_f32(const AttnArgs& a, hipStream_t st) {
    const int qblocks = (a.n_q + BQ - 1) / BQ;
    const size_t total = (size_t)qblocks * a.heads * a.batch;
    HYB_REQUIRE(total < 0x7ffffff0u, HYB_ERR_SHAPE, "attention: too many query blocks (%zu)", total);
    const int xcd_run = ((int)total + 7) / 8;
    const int grid_x = 8 * xcd_run < kMaxGridX ? 8 * xcd_run : kMaxGridX, grid_y = (8 * xcd_run - 1) / grid_x + 1;
    HybTraceScope trace("attention_f32", "flop", 4.0 * a.batch * a.heads * (double)a.n_q * a.n_kv * 64, st);
    hipLaunchKernelGGL(attention_f32_kernel, dim3(grid_x, grid_y), dim3(256), 0, st, a, qblocks, (int)total, xcd_run);
    return hyb_check_launch("attention_f32");
}

}  // namespace

int hyb_launch_attention(const AttnArgs& a, hyb_dtype dtype, hipStream_t st) {
    if (a.batch == 0 || a.n_q == 0 || a.heads == 0) return HYB_OK;
    if (dtype == HYB_BF16) return hyb_launch_attention_mfma(a, st);
    return launch_f32(a, st);
}

namespace {
int joint_attention(const char* who, const void* q, const void* k, const void* v, void* o,
                    int batch, int heads, int n_q, int n_kv, int head_dim, float scale,
                    hyb_dtype dtype, void* workspace, size_t workspace_bytes, bool with_ws, bool prescaled, void* stream) {
    HYB_CHECK_DTYPE(dtype);
    HYB_REQUIRE(batch >= 0 && heads >= 0 && n_q >= 0 && n_kv >= 0, HYB_ERR_SHAPE, "%s: negative size", who);
    HYB_REQUIRE(head_dim == 64, HYB_ERR_SHAPE, "%s: head_dim %d is not supported (only 64)", who, head_dim);
    HYB_REQUIRE(batch <= 65535 && heads <= 65535, HYB_ERR_SHAPE, "%s: batch and heads must be at most 65535", who);
    if (batch == 0 || heads == 0 || n_q == 0) return HYB_OK;
    HYB_REQUIRE(n_kv > 0, HYB_ERR_SHAPE, "%s: n_kv == 0 with n_q > 0 (softmax over an empty set)", who);
    HYB_CHECK_PTR(q); HYB_CHECK_PTR(k); HYB_CHECK_PTR(v); HYB_CHECK_PTR(o);
    HYB_CHECK_ALIGN(q); HYB_CHECK_ALIGN(k); HYB_CHECK_ALIGN(v); HYB_CHECK_ALIGN(o);
    AttnArgs a = {q, k, v, o, nullptr, n_q, batch, heads, n_q, n_kv, scale > 0.f ? scale : 0.125f};
    if (prescaled) {
        // q carries scale x log2(e): the bf16 kernel exponentiates the raw scores in base 2; the fp32 kernel, which
        // exponentiates scale x score in base e, gets scale = ln 2
        a.prescaled = dtype == HYB_BF16;
        a.scale = 0.6931471805599453f;
    }
    if (with_ws) {
        const size_t need = hyb_joint_attention_workspace_bytes(batch, heads, n_q, dtype);
        if (need > 0) {
            HYB_CHECK_PTR(workspace); HYB_CHECK_ALIGN(workspace);
            HYB_REQUIRE(workspace_bytes >= need, HYB_ERR_WORKSPACE, "%s: workspace of %zu bytes is smaller than the %zu required", who, workspace_bytes, need);
            a.part = static_cast<float*>(workspace);
        }
    }
    return hyb_launch_attention(a, dtype, (hipStream_t)stream);
}
}  // namespace

extern "C" int hyb_joint_attention(const void* q, const void* k, const void* v, void* o,
                                   int batch, int heads, int n_q, int n_kv, int head_dim, float scale,
                                   hyb_dtype dtype, void* stream) {
    return joint_attention("hyb_joint_attention", q, k, v, o, batch, heads, n_q, n_kv, head_dim, scale, dtype, nullptr, 0, false, false, stream);
}

extern "C" size_t hyb_joint_attention_workspace_bytes(int batch, int heads, int n_q, hyb_dtype dtype) {
    if (dtype != HYB_BF16 || batch <= 0 || heads <= 0 || n_q <= 0) return 0;
    return hyb_align_up(hyb_attention_split_bytes(batch, heads, n_q), 256);
}

extern "C" int hyb_joint_attention_ws(const void* q, const void* k, const void* v, void* o,
                                      int batch, int heads, int n_q, int n_kv, int head_dim, float scale,
                                      hyb_dtype dtype, void* workspace, size_t workspace_bytes, void* stream) {
    return joint_attention("hyb_joint_attention_ws", q, k, v, o, batch, heads, n_q, n_kv, head_dim, scale, dtype, workspace, workspace_bytes, true, false, stream);
}

extern "C" int hyb_joint_attention_prescaled(const void* q, const void* k, const void* v, void* o,
                                             int batch, int heads, int n_q, int n_kv, int head_dim,
                                             hyb_dtype dtype, void* workspace, size_t workspace_bytes, void* stream) {
    return joint_attention("hyb_joint_attention_prescaled", q, k, v, o, batch, heads, n_q, n_kv, head_dim, 0.f, dtype, workspace, workspace_bytes, true, true, stream);
}
