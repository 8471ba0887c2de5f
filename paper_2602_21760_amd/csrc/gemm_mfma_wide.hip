// bf16 MFMA GEMM with 256-column tiles for gfx950: the same contraction as gemm_mfma.hip (out = epilogue(A W^T + bias), A [m, k] tokens x
// features-in, W [n, k] features-out x features-in, fp32 accumulation in v_mfma_f32_16x16x32_bf16, k in slabs of 64, identical
// order of accumulation and of the epilogue's operations: a token's result has the same bits as from the 64- and 128-row tiles).
//
// What bounds the other two kernels is their operand stream: 128 x 128 tiles, two workgroups per CU, copy 64 bytes L2 -> LDS per MFMA
// clock of a CU, 256 x 128 tiles 48, and the path delivers 41-45.  Here a workgroup of eight waves (2 along the tokens, 4 along the features) owns
// 256, 192 or 128 tokens x 256 features alone on its CU; 256 x 256 tiles copy 32 bytes per MFMA clock.  A wave owns 16 TT x 64
// outputs (TT x 4 MFMA tiles, 128 accumulators for TT = 8), two waves share a SIMD: what one waits for, the other covers, which one wave
// per SIMD (the 256 x 128 kernel) has to do by instruction order alone.  Measured, random data, bias epilogue, TFLOP/s (128 x 128 /
// 256 x 128 / this kernel's best): 16717 x 4608 x 1536 865 / 961 / 1210; 4429 x 4608 x 1536 924 / 874 / 1078; 2714 x 4608 x 1536
// 859 / 855 / 1097; 8192^3 1134 / 1363 / 1516 (the vendor library 1348-1567; forced: the launch rule's estimates are too close there to leave the
// 256 x 128 tiles).
//
// Main loop: direct-to-LDS 16-byte buffer loads with the slab's offset as the scalar operand, XOR-swizzled unpadded 128-byte rows, explicit
// waits, as in gemm_mfma.hip, with two slab buffers (64 KB each for 256 rows).  With a copy requested when a whole buffer is released
// it has three quarters of a slab's time to land, and launches waited for that (128 x 256 tiles 250 us at 16717 x 4608 x
// 1536, 219 us now).  So a slab is taken in four half-steps - first half of the wave's tokens, k-step 0 and 1, then
// the second half - which has read W and the first half of A after the first of them: a barrier there releases these (three quarters of the
// buffer) half a slab earlier, and a second one, before the fourth half-step, the rest.  A copy has one to one and a half slab periods to
// land.  W, first and second half of A of both buffers are six arrays, so that the compiler knows that a copy into one and a fragment read
// from another do not alias (in one array it waits for every copy in flight: 1010 instead of 1210 TFLOP/s).  Fragments are read one half-step
// ahead; the reads are placed between the first three quarters of a half-step's MFMAs, so that the last of them has arrived when
// the next begins (evenly spread: 8192^3 745 us, so 725 us), the copies evenly.
//
// Epilogue: every wave stages 32-token pieces through 8 KB of the W buffers (XOR-swizzled 16-byte pieces, no padding) and writes rows of 128
// or 256 bytes.  GEGLU tiles hold 32 u and the 32 gate features of the same outputs per wave, which multiplies them in registers.  One round
// of 256 x 256 tiles costs about 2.3 us before its first MFMA, 1.3 us per slab and 7 us for a bf16 tile's epilogue, of which 5.5
// are the stores of all CUs at once.
//
// Tile order: XCD x (workgroups x, x + 8, ...) gets one run of consecutive tiles of an order that walks groups of four or eight tile rows column by
// column, so the tiles that an XCD works on at a time share few operand panels (its L2 is 4 MB).
#include "gemm.h"
#include "gemm_lds.h"

#include <type_traits>

namespace {

constexpr int BK = 64;
constexpr int ROWB = BK * 2;            // bytes per LDS row of a slab
constexpr int BN = 256, NW = 8, NT = 64 * NW;

template <int TT> struct WideGeo {
    static constexpr int BM = 32 * TT;
    static constexpr int STAGE_BYTES = (BM + BN) * ROWB;      // 64 KB for 256 rows, 56 KB for 192
    static constexpr int CPW = STAGE_BYTES / 1024 / NW;       // 1 KB chunks per wave per slab
    static constexpr int T0 = TT == 6 ? 4 : TT / 2, T1 = TT - T0;   // token tiles of the first and the second half of a wave
};

// Tile rows per group of the tile order: with a short k the operand panels are small and four rows x eight columns at a time share them best (SDXL-shaped
// stage of 640 channels: 3191 us, eight rows 3274); with longer ones eight rows by four columns read fewer (a guided step at 1024 x 1024 4571 ->
// 4542 us, the others 0-0.3 %).
__device__ __forceinline__ int group_rows(int k) { return k >= 1024 ? 8 : 4; }

// MN MFMAs with R fragment reads between the first three quarters of them and V copies spread evenly.
template <int J, int MN, int R, int V>
__device__ __forceinline__ void interleave() {
    if constexpr (J < MN) {
        constexpr int MR = MN * 3 / 4;
        constexpr int r0 = J < MR ? R * J / MR : R, r1 = J + 1 < MR ? R * (J + 1) / MR : R;
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (r1 != r0) __builtin_amdgcn_sched_group_barrier(0x100, r1 - r0, 0);
        if constexpr ((V * (J + 1)) / MN != (V * J) / MN) __builtin_amdgcn_sched_group_barrier(0x020, (V * (J + 1)) / MN - (V * J) / MN, 0);
        interleave<J + 1, MN, R, V>();
    }
}

// The workgroup's LDS: both slab buffers, each as three arrays, and the bias and gate values of the tile's columns.  (Members, not arrays of
// pointers: an array indexed at run time would be kept in memory, and the compiler could no longer tell the buffers apart.)
struct WideLds {
    unsigned char *a0_s0, *a0_s1, *a1_s0, *a1_s1, *w_s0, *w_s1;
    float* vec;
};

template <typename OT, int EPI, int TT>
__device__ __forceinline__ void wide_tile(const GemmProblem& p, int n, int k, int row0, int col0, const WideLds& lds) {
    using G = WideGeo<TT>;
    constexpr int BM = G::BM, CPW = G::CPW;
    constexpr int T0 = G::T0, T1 = G::T1, TM = T0 > T1 ? T0 : T1, AR0 = 32 * T0, AR1 = 32 * T1;
    constexpr bool GEGLU = EPI == EPI_GEGLU, RES = EPI == EPI_GATE_RES;
    constexpr int OCOLS = GEGLU ? BN / 2 : BN;               // output features of a tile
    float* const vec_lds = lds.vec;
    auto a0_lds = [&](int stage) -> unsigned char* { return stage == 0 ? lds.a0_s0 : lds.a0_s1; };
    auto a1_lds = [&](int stage) -> unsigned char* { return stage == 0 ? lds.a1_s0 : lds.a1_s1; };
    auto w_lds = [&](int stage) -> unsigned char* { return stage == 0 ? lds.w_s0 : lds.w_s1; };
    const int m = p.m;
    [[maybe_unused]] void* const out_q = p.q;
    [[maybe_unused]] void* const out_k = p.k;
    [[maybe_unused]] void* const out_v = p.v;
    const bf16_t* A = static_cast<const bf16_t*>(p.a);
    const bf16_t* W = static_cast<const bf16_t*>(p.w);

    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int wt = wave % 2, wf = wave / 2;
    const int l16 = lane % 16, q4 = lane / 16;

    // Slab copies: chunk c of this wave fills 8 rows of a slab, lane i the 16-byte slot i % 8 of row i / 8 with k-vector (slot ^ swz(row)).  Rows
    // past the end are clamped to the last row (their products are never stored).
    const int nslab = k / BK;
    const size_t row_bytes = (size_t)k * 2;
    const bf16_t* a_tile = A + (size_t)row0 * k;
    const unsigned a_tile_bytes = (unsigned)(min(BM, m - row0) * row_bytes);
    const bf16_t* w_tile = W + (size_t)col0 * k;
    const int w_rows = min(OCOLS, n - col0);
    const unsigned w_tile_bytes = (unsigned)((GEGLU ? (size_t)n + w_rows : (size_t)w_rows) * row_bytes);
    // rows of A in a slab: the first halves of the two wave rows (AR0 rows), then the second ones
    int voff[CPW];
#pragma unroll
    for (int c = 0; c < CPW; c++) {
        const int r = (wave + NW * c) * 8 + lane / 8;
        const int kv = (lane % 8) ^ swz(r);
        int row;
        if (r < BM) {
            const int tr = r < AR0 ? r / (16 * T0) * 16 * TT + r % (16 * T0) : (r - AR0) / (16 * T1) * 16 * TT + 16 * T0 + (r - AR0) % (16 * T1);
            row = min(row0 + tr, m - 1) - row0;
        }
        else if constexpr (GEGLU) {
            const int vr = r - BM, f = min(col0 + vr / 64 * 32 + vr % 32, n - 1) - col0;
            row = vr % 64 < 32 ? f : n + f;
        } else row = min(col0 + r - BM, n - 1) - col0;
        voff[c] = row * (int)row_bytes + kv * 16;
    }
    // copies [c0, c1) of a slab in the order first half of A, W, second half of A
    constexpr int CA0 = T0 / 2, CA1 = T1 / 2, CG0 = CPW - CA1;
    auto issue_chunks = [&](int slab, int stage, auto c0_tag, auto c1_tag) {
        constexpr int C0 = decltype(c0_tag)::value, C1 = decltype(c1_tag)::value;
        const int soff = slab * (BK * 2);
#pragma unroll
        for (int i = C0; i < C1; i++) {
            const int c = i < CA0 ? i : (i < CG0 ? i + CA1 : i - CG0 + CA0);
            if (i < CA0) buffer_load_lds16(a_tile, a_tile_bytes, a0_lds(stage) + (wave + NW * i) * 1024, voff[c], soff);
            else if (i < CG0) buffer_load_lds16(w_tile, w_tile_bytes, w_lds(stage) + (wave + NW * (i - CA0)) * 1024, voff[c], soff);
            else buffer_load_lds16(a_tile, a_tile_bytes, a1_lds(stage) + (wave + NW * (i - CG0)) * 1024, voff[c], soff);
        }
    };
    using std::integral_constant;
    constexpr int FT = 4;
    f32x4 acc[FT][TT];

    // Fragment addresses as in gemm_mfma.hip: with rows 16 t + l16 the slot sits at (lane part) ^ (4 ks ^ 2 (t % 4)), four bases per array; rows
    // that start at an odd multiple of 32 flip bit 2.
    const int kq = (q4 >> 1) | ((q4 & 1) << 1);
    const int lb = (kq ^ (l16 & 7) ^ (l16 >> 3)) & 7;
    int a_base[4], a1_base[4], w_base[4];
#pragma unroll
    for (int c = 0; c < 4; c++) {
        a_base[c] = (wt * 16 * T0 + l16) * ROWB + (((T0 % 4 ? lb ^ (4 * wt) : lb) ^ (2 * c)) * 16);
        a1_base[c] = (wt * 16 * T1 + l16) * ROWB + (((T1 % 4 ? lb ^ (4 * wt) : lb) ^ (2 * c)) * 16);
        w_base[c] = (wf * 64 + l16) * ROWB + ((lb ^ (2 * c)) * 16);
    }
    static_assert(AR0 % 64 == 0 && AR1 % 64 == 0, "a wave copies eight rows at a time");
    bf16x8 af[2][TM], wfr[2][FT];
    // half-steps of a slab: 0: first half, k-step 0; 1: first half, k-step 1; 2: second half, k-step 0; 3: second half, k-step 1
    auto read_half = [&](int stage, int hs) {
        const int ks = hs & 1;
        if (hs < 2) {
#pragma unroll
            for (int t = 0; t < T0; t++) af[hs & 1][t] = *reinterpret_cast<const bf16x8*>(a0_lds(stage) + a_base[((2 * ks) ^ t) & 3] + t * 16 * ROWB);
#pragma unroll
            for (int t = 0; t < FT; t++) wfr[ks][t] = *reinterpret_cast<const bf16x8*>(w_lds(stage) + w_base[((2 * ks) ^ t) & 3] + t * 16 * ROWB);
        } else {
#pragma unroll
            for (int t = 0; t < T1; t++) af[hs & 1][t] = *reinterpret_cast<const bf16x8*>(a1_lds(stage) + a1_base[((2 * ks) ^ t) & 3] + t * 16 * ROWB);
        }
    };
    // Bias and gate of the tile's columns: one value per thread, in a register until the main loop is over.  (The gate row must be the
    // same for all rows of the tile; tiles that straddle samples read it in the epilogue.)
    bool gate_in_lds = true;
    if constexpr (RES) {
        if (p.gate) gate_in_lds = row0 / p.rows_per_gate == min(row0 + BM - 1, m - 1) / p.rows_per_gate;
    }
    integral_constant<int, 0> s0; integral_constant<int, 1> s1;
    const bool odd = nslab % 2;
    // slab s sits in buffer (s + odd) % 2, so that the last two slabs are in buffers 0 and 1 whatever their number
    auto prologue = [&](auto stg) {
        issue_chunks(0, decltype(stg)::value, s0, integral_constant<int, CPW>{});
        issue_chunks(1, 1 - decltype(stg)::value, s0, integral_constant<int, CPW>{});
    };
    if (odd) prologue(s1); else prologue(s0);
    float vec_val = 0.f;       // [0, BN): bias, [BN, 2 BN): gate
    {
        const int t = tid % BN;
        int f = min(col0 + t, n - 1);
        if constexpr (GEGLU) { f = min(col0 + t / 64 * 32 + t % 32, n - 1); if (t % 64 >= 32) f += n; }
        if (tid < BN) {
            if (p.bias) vec_val = p.bias[f];
        } else if constexpr (RES) {
            vec_val = 1.f;
            if (p.gate && gate_in_lds) vec_val = p.gate[(size_t)(row0 / p.rows_per_gate) * p.gate_stride + f];
        }
    }
    // (zeroed while the first slab arrives)
#pragma unroll
    for (int fi = 0; fi < FT; fi++)
#pragma unroll
        for (int t = 0; t < TT; t++) acc[fi][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(CPW + CA1) : "memory");
    __builtin_amdgcn_s_barrier();

    auto mfma_half = [&](auto hs_tag, auto reads_tag, auto copies_tag) {
        constexpr int HS = decltype(hs_tag)::value, TN = HS < 2 ? T0 : T1;
#pragma unroll
        for (int fi = 0; fi < FT; fi++)
#pragma unroll
            for (int t = 0; t < TN; t++) {
                const int ti = (HS < 2 ? 0 : T0) + t;
                acc[fi][ti] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wfr[HS & 1][fi], af[HS & 1][t], acc[fi][ti], 0, 0, 0);
            }
        interleave<0, FT * TN, decltype(reads_tag)::value, decltype(copies_tag)::value>();
    };
    // Copies are requested and counted in the order (W and first half of A, second half of A) of slab after slab, CPW per slab and wave.
    // NEXT: there is a slab s + 1; MORE: there is a slab s + 2.
    constexpr int CH = CG0 / 2;
    auto slab_step = [&](int s, auto stage_tag, auto next_tag, auto more_tag) {
        constexpr int STG = decltype(stage_tag)::value;
        constexpr bool NEXT = decltype(next_tag)::value, MORE = decltype(more_tag)::value;
        read_half(STG, 1);
        mfma_half(s0, integral_constant<int, T0 + FT>{}, s0);
        // the second half of A has landed; the first half and W have been read by all waves
        if constexpr (NEXT) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(CPW) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        read_half(STG, 2);
        if constexpr (MORE) issue_chunks(s + 2, STG, s0, integral_constant<int, CH>{});
        mfma_half(s1, integral_constant<int, T1>{}, integral_constant<int, MORE ? CH : 0>{});
        read_half(STG, 3);
        if constexpr (MORE) issue_chunks(s + 2, STG, integral_constant<int, CH>{}, integral_constant<int, CG0>{});
        mfma_half(integral_constant<int, 2>{}, integral_constant<int, T1>{}, integral_constant<int, MORE ? CG0 - CH : 0>{});
        if constexpr (NEXT) {
            // the first half of A and W of slab s + 1 have landed; the second half of A has been read by all waves
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MORE ? CPW : CA1) : "memory");
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            read_half(STG ^ 1, 0);
            if constexpr (MORE) issue_chunks(s + 2, STG, integral_constant<int, CG0>{}, integral_constant<int, CPW>{});
        }
        mfma_half(integral_constant<int, 3>{}, integral_constant<int, NEXT ? T0 + FT : 0>{}, integral_constant<int, MORE ? CA1 : 0>{});
    };
    std::true_type yes; std::false_type no;
    int s = 0;      // (at least three slabs)
    if (odd) {
        read_half(1, 0);
        slab_step(0, s1, yes, yes);
        s = 1;
    } else read_half(0, 0);
    asm volatile("" : "+v"(vec_val));       // long arrived: no wait for it among the copies in flight
    for (; s + 2 < nslab; s += 2) {
        slab_step(s, s0, yes, yes);
        slab_step(s + 1, s1, yes, yes);
    }
    slab_step(s, s0, yes, no);
    slab_step(s + 1, s1, no, no);
    vec_lds[tid] = vec_val;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();

    // ---- epilogue: per wave, registers -> its own LDS piece -> row-contiguous global stores.  Register i of tile (fi, ti): feature
    // 64 wf + 16 fi + 4 q4 + i, token 16 (TT wt + ti) + l16.
    constexpr int WCOLS = GEGLU ? 32 : 64;                   // output features of a wave
    constexpr int SE = (int)sizeof(OT);
    constexpr int PPR = WCOLS * SE / 16;
    constexpr int ITERS = 32 * PPR / 64;
    constexpr int CE = 16 / SE;
    static_assert(32 * PPR * 16 <= BN * ROWB / 4, "a wave's piece must fit its part of the W buffers");
    unsigned char* stg = w_lds(wave & 1) + (wave >> 1) * (BN * ROWB / 4);
    auto piece = [&](int row, int pc) { return stg + row * (PPR * 16) + ((pc ^ (row / (16 / PPR))) & (PPR - 1)) * 16; };
    const int wrow0 = row0 + wt * 16 * TT, wcol0 = col0 + wf * WCOLS;
    f32x4 bv[FT];
#pragma unroll
    for (int fi = 0; fi < FT; fi++) bv[fi] = *reinterpret_cast<const f32x4*>(vec_lds + wf * 64 + fi * 16 + 4 * q4);
    [[maybe_unused]] OT* qkv_base = nullptr;
    [[maybe_unused]] float scale = 1.f;
    [[maybe_unused]] int qkv_b0 = 0, qkv_t0 = 0;      // sample and token of the tile's first row
    if constexpr (EPI == EPI_QKV) {
        const int hd = p.heads * 64, c = min(wcol0, n - 64), which = c / hd, head = (c - which * hd) / 64;
        qkv_base = static_cast<OT*>(which == 0 ? out_q : (which == 1 ? out_k : out_v)) + ((size_t)head * p.n_total + p.tok_offset) * 64;
        if (which == 0 && p.q_scale != 0.f) scale = p.q_scale;
        qkv_b0 = row0 / p.tokens;
        qkv_t0 = row0 - qkv_b0 * p.tokens;
    }
#pragma unroll
    for (int tm = 0; tm < TT / 2; tm++) {
        [[maybe_unused]] f32x4 resv[RES ? ITERS : 1];
        if constexpr (RES) {
#pragma unroll
            for (int j = 0; j < ITERS; j++) {
                const int idx = lane + 64 * j;
                const int r = min(wrow0 + tm * 32 + idx / PPR, m - 1), f = min(wcol0 + (idx % PPR) * CE, n - 4);
                resv[j] = *reinterpret_cast<const f32x4*>(p.res + (size_t)r * n + f);
                if (p.res2) resv[j] += *reinterpret_cast<const f32x4*>(p.res2 + (size_t)r * n + f);
            }
        }
#pragma unroll
        for (int h2 = 0; h2 < 2; h2++) {
            const int prow = h2 * 16 + l16;
#pragma unroll
            for (int fi = 0; fi < (GEGLU ? 2 : FT); fi++) {
                f32x4 v = acc[fi][2 * tm + h2] + bv[fi];
                if constexpr (GEGLU) {
                    const f32x4 gt = acc[fi + 2][2 * tm + h2] + bv[fi + 2];
#pragma unroll
                    for (int j = 0; j < 4; j++) v[j] *= gelu_erf_f(gt[j]);
                } else if constexpr (EPI == EPI_GELU_TANH) {
#pragma unroll
                    for (int j = 0; j < 4; j++) v[j] = gelu_tanh_f(v[j]);
                } else if constexpr (EPI == EPI_QKV) {
                    v *= scale;
                } else if constexpr (RES) {
                    if (gate_in_lds) v *= *reinterpret_cast<const f32x4*>(vec_lds + BN + wf * 64 + fi * 16 + 4 * q4);
                    else {
                        const int r = wrow0 + tm * 32 + prow;
                        v *= *reinterpret_cast<const f32x4*>(p.gate + (size_t)(min(r, m - 1) / p.rows_per_gate) * p.gate_stride + min(wcol0 + fi * 16 + 4 * q4, n - 4));
                    }
                }
                if constexpr (SE == 4) *reinterpret_cast<f32x4*>(piece(prow, fi * 4 + q4)) = v;
                else {
                    bf16x4 o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
                    *reinterpret_cast<bf16x4*>(piece(prow, fi * 2 + q4 / 2) + q4 % 2 * 8) = o;
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int j = 0; j < ITERS; j++) {
            const int idx = lane + 64 * j, prow = idx / PPR, pc = idx % PPR;
            const int r = wrow0 + tm * 32 + prow, f = wcol0 + pc * CE;
            const u32x4 y = *reinterpret_cast<const u32x4*>(piece(prow, pc));
            if (r >= m || f >= n) continue;
            if constexpr (EPI == EPI_QKV) {
                int b, t;
                if (p.tokens >= BM) {           // at most one step into the next sample
                    b = qkv_b0;
                    t = qkv_t0 + (r - row0);
                    if (t >= p.tokens) { t -= p.tokens; b++; }
                } else {
                    b = r / p.tokens;
                    t = r - b * p.tokens;
                }
                // (non-temporal: the launch's operands stay in the L2s; the attention reads q, k and v from another XCD's workgroups anyway.  A guided step
                // at 1024 x 1024 4542 -> 4496 us.  The other epilogues' consumers pay as much for it as the launch gains.)
                __builtin_nontemporal_store(y, reinterpret_cast<u32x4*>(qkv_base + ((size_t)b * p.heads * p.n_total + t) * 64 + pc * CE));
            } else if constexpr (RES) {
                *reinterpret_cast<f32x4*>(static_cast<float*>(p.out) + (size_t)r * n + f) = *reinterpret_cast<const f32x4*>(&y) + resv[j];
            } else {
                *reinterpret_cast<u32x4*>(static_cast<OT*>(p.out) + (size_t)r * n + f) = y;
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Tiles of a launch: XCD x (workgroups x, x + 8, ...) gets the run [x * tall_run, (x + 1) * tall_run) of the tall tiles, then its run of the short ones.
struct WideGrid {
    int tiles_n;
    int tall_rows[kMaxGroup];      // tall tile rows of each problem: its first rows
    int tall, shrt;                // tiles
    int tall0, short0;             // of these, of the first problem
    int tall_run, short_run;
};

// TA, TB: token tiles per wave of the tall and of the short tiles.
template <typename OT, int EPI, int TA, int TB>
__global__ __launch_bounds__(NT, 2) void gemm_wide_kernel(GemmGroup g, WideGrid t) {
    constexpr int OCOLS = EPI == EPI_GEGLU ? BN / 2 : BN;
    constexpr int AR0 = 32 * (WideGeo<TA>::T0 > WideGeo<TB>::T0 ? WideGeo<TA>::T0 : WideGeo<TB>::T0);
    constexpr int AR1 = 32 * (WideGeo<TA>::T1 > WideGeo<TB>::T1 ? WideGeo<TA>::T1 : WideGeo<TB>::T1);
    __shared__ __attribute__((aligned(16))) unsigned char a0_s0[AR0 * ROWB], a0_s1[AR0 * ROWB], a1_s0[AR1 * ROWB], a1_s1[AR1 * ROWB], w_s0[BN * ROWB], w_s1[BN * ROWB];
    __shared__ __attribute__((aligned(16))) float vec_lds[2 * BN];
    WideLds lds;
    lds.a0_s0 = a0_s0; lds.a0_s1 = a0_s1; lds.a1_s0 = a1_s0; lds.a1_s1 = a1_s1; lds.w_s0 = w_s0; lds.w_s1 = w_s1;
    lds.vec = vec_lds;

    const int xcd = blockIdx.x % 8, pos = blockIdx.x / 8;
    const bool is_tall = pos < t.tall_run;
    int tile = is_tall ? xcd * t.tall_run + pos : xcd * t.short_run + pos - t.tall_run;
    if (tile >= (is_tall ? t.tall : t.shrt)) return;
    const int first = is_tall ? t.tall0 : t.short0;
    const bool second = tile >= first;
    if (second) tile -= first;
    // Problem of this tile, selected field by field (indexing the argument array with a run-time index would make the
    // compiler keep a copy of the whole argument block in scratch memory).
    GemmProblem p;
#define HYB_SEL(f) p.f = second ? g.p[1].f : g.p[0].f
    HYB_SEL(a); HYB_SEL(w); HYB_SEL(bias); HYB_SEL(out); HYB_SEL(m);
    HYB_SEL(res); HYB_SEL(res2); HYB_SEL(gate); HYB_SEL(rows_per_gate); HYB_SEL(gate_stride);
    HYB_SEL(q); HYB_SEL(k); HYB_SEL(v); HYB_SEL(tokens); HYB_SEL(tok_offset); HYB_SEL(n_total); HYB_SEL(heads); HYB_SEL(q_scale);
#undef HYB_SEL
    const int tall_rows = second ? t.tall_rows[1] : t.tall_rows[0];
    const int height = is_tall ? 32 * TA : 32 * TB, base = is_tall ? 0 : tall_rows * 32 * TA;
    const int tile_rows = is_tall ? tall_rows : (p.m - base + height - 1) / height;
    const int group = group_rows(g.k), per_group = group * t.tiles_n;
    const int grp = tile / per_group, in = tile - grp * per_group;
    const int rows_in = min(group, tile_rows - grp * group);
    const int row0 = base + (grp * group + in % rows_in) * height, col0 = in / rows_in * OCOLS;
    if (is_tall) wide_tile<OT, EPI, TA>(p, g.n, g.k, row0, col0, lds);
    else wide_tile<OT, EPI, TB>(p, g.n, g.k, row0, col0, lds);
}

template <typename OT, int EPI, int TA, int TB>
int launch_wide(const GemmGroup& g, const WidePlan& plan, hipStream_t st) {
    GemmGroup gg = g;
    WideGrid t = {};
    constexpr int OCOLS = EPI == EPI_GEGLU ? BN / 2 : BN;
    t.tiles_n = (g.n + OCOLS - 1) / OCOLS;
    int order[kMaxGroup] = {0, 1};
    if (gg.count < 2) gg.p[1] = gg.p[0];         // every field the kernel selects from is defined
    // The smaller problem goes first: its tiles fetch a whole weight matrix for few rows, which is better hidden under the start
    // of the large problem than left for the end of the launch.
    if (gg.count > 1 && gg.p[1].m < gg.p[0].m) {
        const GemmProblem x = gg.p[0];
        gg.p[0] = gg.p[1];
        gg.p[1] = x;
        order[0] = 1; order[1] = 0;
    }
    for (int i = 0; i < gg.count; i++) {
        const int a = plan.tall_rows[order[i]], rest = gg.p[i].m - a * 32 * TA;
        const int b = rest > 0 ? (rest + 32 * TB - 1) / (32 * TB) : 0;
        t.tall_rows[i] = a;
        t.tall += a * t.tiles_n;
        t.shrt += b * t.tiles_n;
        if (i == 0) { t.tall0 = t.tall; t.short0 = t.shrt; }
    }
    if (t.tall + t.shrt <= 0) return HYB_OK;
    t.tall_run = (t.tall + 7) / 8;
    t.short_run = (t.shrt + 7) / 8;
    char name[96] = "";
    if (hyb_trace_on()) {
        if (t.tall && t.shrt) snprintf(name, sizeof(name), "gemm_mfma_%d+%dx%d.epi%d.n%d.k%d", 32 * TA, 32 * TB, BN, EPI, g.n, g.k);
        else snprintf(name, sizeof(name), "gemm_mfma_%dx%d.epi%d.n%d.k%d", t.tall ? 32 * TA : 32 * TB, BN, EPI, g.n, g.k);
    }
    double rows = 0;
    for (int i = 0; i < g.count; i++) rows += g.p[i].m;
    HybTraceScope trace(name, "flop", 2.0 * rows * g.n * g.k, st);
    hipLaunchKernelGGL((gemm_wide_kernel<OT, EPI, TA, TB>), dim3(8 * (t.tall_run + t.short_run)), dim3(NT), 0, st, gg, t);
    return hyb_check_launch("gemm_mfma_wide");
}

template <typename OT, int EPI>
int launch_pair(const GemmGroup& g, const WidePlan& plan, hipStream_t st) {
    if (plan.tall == 256 && plan.shrt == 192) return launch_wide<OT, EPI, 8, 6>(g, plan, st);
    if (plan.tall == 192 && plan.shrt == 128) return launch_wide<OT, EPI, 6, 4>(g, plan, st);
    return hyb_set_error(HYB_ERR_SHAPE, "gemm_mfma_wide: no tiles of %d and %d rows", plan.tall, plan.shrt);
}

}  // namespace

int hyb_launch_gemm_mfma_wide(const GemmGroup& g, hyb_dtype out_dtype, int epi, const WidePlan& plan, hipStream_t st) {
    if (g.k / BK < 3 || g.n2) return hyb_set_error(HYB_ERR_SHAPE, "gemm_mfma_wide: unsupported shape (k %d)", g.k);
    const bool f32 = out_dtype == HYB_F32;
    if (!f32 && epi == EPI_BIAS) return launch_pair<bf16_t, EPI_BIAS>(g, plan, st);
    if (!f32 && epi == EPI_GELU_TANH) return launch_pair<bf16_t, EPI_GELU_TANH>(g, plan, st);
    if (!f32 && epi == EPI_QKV) return launch_pair<bf16_t, EPI_QKV>(g, plan, st);
    if (!f32 && epi == EPI_GEGLU) return launch_pair<bf16_t, EPI_GEGLU>(g, plan, st);
    if (f32 && epi == EPI_GATE_RES) return launch_pair<float, EPI_GATE_RES>(g, plan, st);
    return hyb_set_error(HYB_ERR_SHAPE, "gemm_mfma_wide: no such epilogue (%d)", epi);
}
