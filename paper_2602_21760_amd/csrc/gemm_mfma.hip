// bf16 MFMA GEMM for gfx950: out = epilogue(A W^T + bias), A [m, k] tokens x features-in,
// W [n, k] features-out x features-in, fp32 accumulation in v_mfma_f32_16x16x32_bf16.
//
// Tiling: a workgroup of 4 waves (2 x 2) owns a 128 x 128 output tile; each wave owns 4 x 4 MFMA
// tiles of 16 x 16 (small problems: 64 x 128 tiles, 4 x 2 MFMA tiles per wave, see launch_epi).
// The weight fragment is the MFMA "A" operand and the token fragment the "B" operand, so the 4
// accumulator registers of a tile run along the output-feature axis (4 consecutive features, one
// token per lane).  The 16 x 16 x 32 form is used because it is the cheaper one on this chip: it
// moves half the accumulator bytes per multiply-add of the 32 x 32 x 16 form, and under the power
// limit that sets the clock of these kernels the main loop runs 5-6 % faster with it (QKV-shaped and
// fc1 launches of the SD3-shaped workload), with the same bits.
//
// Main loop: k is cut into slabs of 64.  A slab of both operands (128 + 128 rows of 128 bytes) is
// copied global -> LDS by 16-byte direct-to-LDS buffer loads (buffer_load_dwordx4 ... lds: a wave fills 1 KB
// of LDS per instruction, no VGPR staging, no ds_write; the slab's byte offset is the scalar operand and the
// per-lane offsets are loop invariants, so a slab costs no vector address arithmetic), double buffered (launches of few
// tiles: three or six buffers, see launch_tiles): the copy of slab s + 1 runs while slab s is multiplied.  LDS rows are
// unpadded; the 16-byte slots of a row are XOR-swizzled
// with (row ^ row >> 3) & 7 so that the 16-byte fragment reads that are served together hit distinct
// banks (the swizzle is applied on the global side: each lane picks which 16 bytes it fetches).
// Waits on the copies are explicit (s_waitcnt vmcnt + s_barrier); a full __syncthreads() would
// force vmcnt(0) on every barrier through its fence.  The fragments of the two k-steps (of 32) of a
// slab live in two register sets and are read one k-step ahead of the MFMAs that use them, also
// across the slab boundary, which leaves a single barrier per slab (before its second k-step).
//
// Epilogue: the accumulators (+ bias, activation, gate) are staged through LDS (reusing the slab
// buffers) and written out row-contiguously, 16 bytes per lane, so that global stores and the
// residual reads are whole 128-byte lines.  (Storing straight from the MFMA layout issues 8-byte
// pieces to 32 different rows per instruction; at these sizes that made the epilogue cost a third
// of the tile time.)  What the epilogue reads from global memory is requested early: the tile's bias and gate values
// at the start of the tile (parked in LDS behind the slab buffers), the residual during the last k-slab; every such access uses clamped
// addresses instead of predicates, and the staging loops are free of branches.  The start is not as well hidden as it could
// be: the compiler waits for bias and gate before the first slab copy in the gate + residual forms and in some of the
// others, and with three buffers, or six and a bf16 output, it waits for all of the prologue's copies before it parks the
// bias.  (With a branch that chooses between
// a global and an LDS source inside the loop, the compiler waits for ALL outstanding global loads
// before every LDS read.)
//
// Up to two problems with the same (n, k) share a launch (image and text stream of a joint
// block), the smaller one first; the two of a QKV launch may differ in (n, k), in the caller's order.  Tile order: plain, or
// runs of consecutive tiles per XCD when there are few tile columns (see the kernel).  Ragged edges: row / feature indices are
// clamped on load and masked on store.  The reduction order over k is fixed and a token's result does not depend on its tile
// row, so results are deterministic, and batch-invariant where k is not split (the number of shares follows from the rows).
#include "gemm.h"
#include "gemm_lds.h"

#include <type_traits>

namespace {

constexpr int BN = 128, BK = 64;
constexpr int ROWB = BK * 2;                    // bytes per LDS row of a slab
// The tile height is 64 TMW tokens (TMW = MFMA token tiles per wave): 128 for the large GEMMs, 64 for
// launches that would otherwise leave most of the chip idle (fewer than three quarters of a wave of tiles).
template <int TMW, int NST = 2> struct Geo {
    static constexpr int BM = 64 * TMW;
    static constexpr int STAGE_BYTES = (BM + BN) * ROWB;   // 32 KB / 24 KB
    static constexpr int CPW = STAGE_BYTES / 1024 / 4;     // 1 KB chunks per wave per slab (8 / 6)
    static constexpr int SMEM_BYTES = NST * STAGE_BYTES;   // two slab buffers: 64 KB -> two workgroups per CU / 48 KB -> three
    static constexpr int WG_PER_CU = TMW == 2 ? 2 : (NST == 2 ? 3 : (NST == 3 ? 2 : 1));
};
constexpr int VEC_BYTES = 2 * BN * 4;           // the tile's bias and gate values, behind the slab buffers
constexpr int OUT_STRIDE_B16 = BN * 2 + 16;     // staging row strides (bytes), padded against conflicts
constexpr int OUT_STRIDE_F32 = BN * 4 + 16;

template <typename OT, int EPI, int TMW, int NST>
__global__ __launch_bounds__(256, (Geo<TMW, NST>::WG_PER_CU)) void gemm_mfma_kernel(GemmGroup g, int tiles_n, int tiles0, int total, int xcd_run, int ksplit) {
    constexpr bool MIXED = EPI == EPI_QKV;   // the two problems may differ in (n, k)
    constexpr int BM = Geo<TMW>::BM, STAGE_BYTES = Geo<TMW>::STAGE_BYTES, CPW = Geo<TMW>::CPW;
    __shared__ __attribute__((aligned(16))) unsigned char smem[Geo<TMW, NST>::SMEM_BYTES + VEC_BYTES];

    // Workgroups go round-robin to the 8 XCDs (each with its own L2) in launch order.  With few tile columns the
    // tiles that an XCD works on at a time then share hardly any operand panel (every 8th tile: all tile rows, a
    // few columns), so XCD x is given the run of consecutive tiles [x * xcd_run, (x + 1) * xcd_run) instead
    // (a few whole tile rows).  xcd_run == 0: plain order.  Two problems of different shapes have runs of their own: with
    // one run over both, the first's tiles, few and long, would all come to the first XCD (a stage block of 4 x 1024 tokens of 640
    // channels and 4 x 333 context rows: 197 us so, 182 us as it is).
    int tile = blockIdx.x;
    if (xcd_run > 0) {
        int first = 0, end = total, run = xcd_run;
        if (MIXED && g.n2) {
            const int run0 = (tiles0 + 7) / 8;
            if (tile < 8 * run0) {
                end = tiles0; run = run0;
            } else {
                first = tiles0;
                tile -= 8 * run0;
            }
        }
        tile = first + (tile % 8) * run + tile / 8;
        if (tile >= end) return;
    }
    // k split (ksplit > 1, single problem, plain fp32 output): ksplit consecutive workgroups share a tile; each
    // multiplies its share of the k-slabs and writes the raw sums to its own [m, n] plane of p.out
    int split = 0;
    if (ksplit > 1) {
        split = tile % ksplit;
        tile /= ksplit;
    }
    const int pi = tile >= tiles0 ? 1 : 0;
    if (pi) tile -= tiles0;
    const GemmProblem& p = g.p[pi];
    if (MIXED && pi && g.n2) tiles_n = (g.n2 + BN - 1) / BN;
    const int row0 = (tile / tiles_n) * BM;
    // EPI_GEGLU: a tile covers 64 output features; its 128 weight rows are 64 "u" rows and the 64 "gate" rows n above
    const int col0 = (tile % tiles_n) * (EPI == EPI_GEGLU ? BN / 2 : BN);
    const int m = p.m, n = MIXED && pi && g.n2 ? g.n2 : g.n, k = MIXED && pi && g.n2 ? g.k2 : g.k;
    const bf16_t* A = static_cast<const bf16_t*>(p.a);
    const bf16_t* W = static_cast<const bf16_t*>(p.w);

    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);   // uniform: LDS copy targets (M0) become scalar arithmetic
    const int wt = wave % 2, wf = wave / 2;          // wave position: tokens, features
    const int l16 = lane % 16, q4 = lane / 16;      // MFMA 16x16x32: row / column of the lane, its quarter of the 32 k

    // This wave's chunks of a slab: chunk c covers stage rows 8 c .. 8 c + 7 (rows 0..BM-1 = A, then 128 rows of W);
    // lane i fills 16-byte slot i % 8 of row i / 8 and fetches k-vector (slot ^ swz(row)) for it.
    // Buffer loads: a tile's A rows and W rows are two buffers that start at the tile's first row (so per-lane
    // byte offsets are small 32-bit numbers, loop invariants), the k-slab's offset is a scalar operand: a slab costs
    // no vector address arithmetic.  Rows past the end are clamped to the last row (their products are not stored).
    const int slab0 = split * (k / BK) / ksplit;
    const int nslab = (split + 1) * (k / BK) / ksplit - slab0;
    const size_t row_bytes = (size_t)k * 2;
    const bf16_t* a_tile = A + (size_t)row0 * k;
    const unsigned a_tile_bytes = (unsigned)(min(BM, m - row0) * row_bytes);
    const int w_rows = min(EPI == EPI_GEGLU ? BN / 2 : BN, n - col0);
    const bf16_t* w_tile = W + (size_t)col0 * k;
    const unsigned w_tile_bytes = (unsigned)((EPI == EPI_GEGLU ? (size_t)n + w_rows : (size_t)w_rows) * row_bytes);
    int voff[CPW];
#pragma unroll
    for (int c = 0; c < CPW; c++) {
        const int r = (wave + 4 * c) * 8 + lane / 8;
        const int kv = (lane % 8) ^ swz(r);
        if (r < BM) voff[c] = (min(row0 + r, m - 1) - row0) * (int)row_bytes + kv * 16;
        else if constexpr (EPI == EPI_GEGLU) {
            const int vr = r - BM;
            voff[c] = (vr < 64 ? min(col0 + vr, n - 1) - col0 : n + min(col0 + vr - 64, n - 1) - col0) * (int)row_bytes + kv * 16;
        } else voff[c] = (min(col0 + r - BM, n - 1) - col0) * (int)row_bytes + kv * 16;
    }
    auto issue = [&](int slab, int stage) {
        const int soff = (slab0 + slab) * (BK * 2);
#pragma unroll
        for (int c = 0; c < CPW; c++) {
            // chunks of A come first: chunk index wave + 4 c < BM / 8 exactly for c < BM / 32
            if (c < BM / 32) buffer_load_lds16(a_tile, a_tile_bytes, smem + stage * STAGE_BYTES + (wave + 4 * c) * 1024, voff[c], soff);
            else buffer_load_lds16(w_tile, w_tile_bytes, smem + stage * STAGE_BYTES + (wave + 4 * c) * 1024, voff[c], soff);
        }
    };

    constexpr int TT = 2 * TMW;   // token tiles of 16 per wave
    f32x4 acc[4][TT];             // [feature tile of 16][token tile of 16]
#pragma unroll
    for (int fi = 0; fi < 4; fi++)
#pragma unroll
        for (int ti = 0; ti < TT; ti++)
#pragma unroll
            for (int i = 0; i < 4; i++) acc[fi][ti][i] = 0.f;

    // Fragment addresses inside a stage.  A fragment of v_mfma_f32_16x16x32_bf16 is 16 rows x 32 k, lane (l16, q4)
    // holding 8 k of row l16.  Which 8 is free as long as both operands agree (the order of the contraction index
    // inside an MFMA does not matter to the product): lane quarter q4 takes the 16-byte slot 4 ks + (q4 >> 1 | (q4 & 1) << 1)
    // of its row, so that lanes i and i + 32 read adjacent slots of one row, 32 contiguous bytes.  (With slot 4 ks + q4
    // the same reads take twice as long: the LDS counters show four conflict cycles per read, whatever the swizzle.)
    // With the XOR swizzle and tile rows 16 t + l16 the slot sits at (lane part) ^ (4 ks ^ 2 t): four per-lane bases per
    // operand cover all the reads of a slab, and the tile row block (t * 16 rows) is an immediate offset.  (With 32
    // token rows per wave the wave's own row offset 32 wt also reaches bit 2 of the swizzle; it is folded into the lane part.)
    const int kq = (q4 >> 1) | ((q4 & 1) << 1);
    const int lb = (kq ^ (l16 & 7) ^ (l16 >> 3)) & 7;
    const int lb_a = TMW == 1 ? lb ^ (4 * wt) : lb;
    int a_base[4], w_base[4];
#pragma unroll
    for (int c = 0; c < 4; c++) {
        a_base[c] = (wt * 32 * TMW + l16) * ROWB + ((lb_a ^ (2 * c)) * 16);
        w_base[c] = BM * ROWB + (wf * 64 + l16) * ROWB + ((lb ^ (2 * c)) * 16);
    }
    // Two fragment sets, one per k-step of 32 of a slab; the reads run one k-step ahead of their use, across the slab
    // boundary.
    bf16x8 af[2][TT], wfr[2][4];
    auto read_set = [&](int stage, int ks) {
        const unsigned char* base = smem + stage * STAGE_BYTES;
#pragma unroll
        for (int t = 0; t < TT; t++)
            af[ks][t] = *reinterpret_cast<const bf16x8*>(base + a_base[((2 * ks) ^ t) & 3] + t * 16 * ROWB);
#pragma unroll
        for (int t = 0; t < 4; t++)
            wfr[ks][t] = *reinterpret_cast<const bf16x8*>(base + w_base[((2 * ks) ^ t) & 3] + t * 16 * ROWB);
    };

    // Main loop.  Slab s sits in stage s % NST.  ONE barrier per slab, before its second k-step: by then every wave has
    // issued (and, after the lgkmcnt wait, completed) all its reads of slab s, so stage s % NST can be refilled with
    // slab s + NST right behind the barrier, and the copy of slab s + 1 (issued NST - 1 slabs earlier) is awaited just
    // before it, so that the second k-step can already fetch the first fragments of slab s + 1.
    // Epilogue operands are requested early.  Bias and gate of the tile's 128 columns:
    // one value per thread now, parked in LDS behind the slab buffers once the first slab's wait has passed.
    // (The gate row must be the same for all rows of the tile; tiles that straddle samples read it from
    // global memory in the epilogue.)
    float* vec_lds = reinterpret_cast<float*>(smem + Geo<TMW, NST>::SMEM_BYTES);
    bool gate_in_lds = true;   // no gate: ones
    if constexpr (EPI == EPI_GATE_RES) {
        if (p.gate) gate_in_lds = row0 / p.rows_per_gate == min(row0 + BM - 1, m - 1) / p.rows_per_gate;
    }
    {
        const int t = tid % BN;
        int f = min(col0 + t, n - 1);
        if constexpr (EPI == EPI_GEGLU) f = t < 64 ? min(col0 + t, n - 1) : n + min(col0 + t - 64, n - 1);
        float val = 0.f;
        if (tid < BN) {
            if (p.bias) val = p.bias[f];
        } else if constexpr (EPI == EPI_GATE_RES) {
            val = 1.f;
            if (p.gate && gate_in_lds) val = p.gate[(size_t)(row0 / p.rows_per_gate) * p.gate_stride + f];
        }
        if constexpr (NST == 2) {
            issue(0, 0);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        } else {
#pragma unroll
            for (int j = 0; j < NST; j++)
                if (j < nslab) issue(j, j);
            if (nslab >= NST) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * CPW) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        vec_lds[tid] = val;
    }
    __builtin_amdgcn_s_barrier();
    if (NST == 2 && nslab > 1) issue(1, 1);
    read_set(0, 0);
    constexpr bool GEGLU = EPI == EPI_GEGLU;
    [[maybe_unused]] const int q_cols = EPI == EPI_QKV && p.q_scale != 0.f ? p.heads * 64 : 0;   // columns of the q part that are scaled
    [[maybe_unused]] const float q_scale = p.q_scale;
    // EPI_QKV: where the tile's first column and row lie (feature = (which, offset in q / k / v), row = (sample, token))
    [[maybe_unused]] int qkv_which0 = 0, qkv_cc0 = 0, qkv_b0 = 0, qkv_t0 = 0;
    [[maybe_unused]] bool qkv_steps = false;   // chunks reach their place by at most one step over each boundary
    if constexpr (EPI == EPI_QKV) {
        const int hd = p.heads * 64;
        qkv_steps = hd >= BN && p.tokens >= BM;
        if (qkv_steps) {
            qkv_which0 = col0 / hd;
            qkv_cc0 = col0 - qkv_which0 * hd;
            qkv_b0 = row0 / p.tokens;
            qkv_t0 = row0 - qkv_b0 * p.tokens;
        }
    }
    constexpr bool F32OUT = sizeof(OT) == 4 || GEGLU;   // GEGLU stages u and gate in fp32 and combines on the way out
    constexpr int NPASS = (F32OUT && TMW == 2) ? 2 : 1;   // a 128-token fp32 tile is staged in two 64-token halves
    constexpr int STRIDE = F32OUT ? OUT_STRIDE_F32 : OUT_STRIDE_B16;
    constexpr int ROWS_PER_PASS = BM / NPASS;
    constexpr int CHUNK_ELEMS = 16 / (int)sizeof(OT);   // elements per 16-byte chunk
    constexpr int CHUNKS_PER_ROW = (GEGLU ? BN / 2 : BN) / CHUNK_ELEMS;
    constexpr int SE = F32OUT ? 4 : 2;                  // bytes per staged element
    constexpr int ITERS = ROWS_PER_PASS * CHUNKS_PER_ROW / 256;   // 16-byte chunks per thread per pass
    // gate * y + residual: the residual chunks of a pass are fetched ahead (pass 0 during the last slab of the main
    // loop, pass 1 once pass 0 is staged); loading them where they are used would expose their latency, and
    // one by one between the stores they would serialise on every load (out may alias res).
    constexpr bool RES = EPI == EPI_GATE_RES;
    f32x4 resv[RES ? NPASS : 1][RES ? ITERS : 1];
    auto load_res = [&](int pass) {
        if constexpr (RES) {
            auto chunk_offset = [&](int j) {   // clamped like every other edge access: masked on store
                const int c = tid + 256 * j;
                const int r = min(row0 + pass * ROWS_PER_PASS + c / CHUNKS_PER_ROW, m - 1), f = min(col0 + (c % CHUNKS_PER_ROW) * CHUNK_ELEMS, n - 4);
                return (size_t)r * n + f;
            };
#pragma unroll
            for (int j = 0; j < ITERS; j++) resv[pass][j] = *reinterpret_cast<const f32x4*>(p.res + chunk_offset(j));
            if (p.res2) {
#pragma unroll
                for (int j = 0; j < ITERS; j++) resv[pass][j] += *reinterpret_cast<const f32x4*>(p.res2 + chunk_offset(j));
            }
        }
    };
    auto slab_step = [&](int s, auto stage_tag) {
        constexpr int STG = decltype(stage_tag)::value;
        if (s == nslab - 1) load_res(0);
#pragma unroll
        for (int ks = 0; ks < BK / 32; ks++) {
            if (ks == 1 && s + 1 < nslab) {
                // this wave's share of slab s + 1 has landed (up to NST - 2 younger slabs may be in flight)
                if (NST > 2 && s + NST - 1 < nslab) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * CPW) : "memory");
                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // ... and its reads of slab s are complete
                __builtin_amdgcn_s_barrier();
                if (s + NST < nslab) issue(s + NST, STG);
            }
            if (ks == 0) read_set(STG, 1);
            else if (s + 1 < nslab) read_set((STG + 1) % NST, 0);
#pragma unroll
            for (int fi = 0; fi < 4; fi++)
#pragma unroll
                for (int ti = 0; ti < TT; ti++)
                    acc[fi][ti] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wfr[ks][fi], af[ks][ti], acc[fi][ti], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < 4 + TT; j++) {   // fragment reads between the MFMAs
                __builtin_amdgcn_sched_group_barrier(0x008, (4 * TT) / (4 + TT), 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
        }
    };
    for (int s = 0; s < nslab; s += NST) {
        slab_step(s, std::integral_constant<int, 0>{});
        if (s + 1 < nslab) slab_step(s + 1, std::integral_constant<int, 1>{});
        if constexpr (NST > 2) {
            if (s + 2 < nslab) slab_step(s + 2, std::integral_constant<int, 2>{});
        }
        if constexpr (NST > 3) {
            if (s + 3 < nslab) slab_step(s + 3, std::integral_constant<int, 3>{});
            if (s + 4 < nslab) slab_step(s + 4, std::integral_constant<int, 4>{});
            if (s + 5 < nslab) slab_step(s + 5, std::integral_constant<int, 5>{});
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();                          // every wave is done with the slab buffers

    // ---- epilogue: registers -> LDS staging tile -> row-contiguous global stores -------------------
    // Register i of tile (fi, ti): feature = wf*64 + fi*16 + 4 q4 + i, token = wt*32*TMW + ti*16 + l16.
#pragma unroll
    for (int pass = 0; pass < NPASS; pass++) {
        // Staging; GATE_LDS: the gate values come from LDS (always, unless the tile's rows straddle gate rows).
        [[maybe_unused]] const float* gate_ptr = p.gate;
        [[maybe_unused]] const int gate_rows = p.rows_per_gate;
        [[maybe_unused]] const size_t gate_stride = p.gate_stride;
        auto stage = [&, gate_ptr, gate_rows, gate_stride](auto gate_lds_tag) {
            constexpr bool GATE_LDS = decltype(gate_lds_tag)::value;
            // bias (and gate) of this lane's 4 column groups first, in one batch of LDS reads
            f32x4 bv[4];
            [[maybe_unused]] f32x4 gv[4];
#pragma unroll
            for (int fi = 0; fi < 4; fi++) {
                const int fl = wf * 64 + fi * 16 + 4 * q4;
                bv[fi] = *reinterpret_cast<const f32x4*>(vec_lds + fl);
                if constexpr (RES && GATE_LDS) gv[fi] = *reinterpret_cast<const f32x4*>(vec_lds + BN + fl);
            }
#pragma unroll
            for (int ti = 0; ti < TT; ti++) {
                const int trow = (NPASS == 1 ? wt * 32 * TMW : 0) + ti * 16 + l16;   // row inside the staging tile
                if constexpr (RES && !GATE_LDS) {
                    const int r = row0 + wt * 32 * TMW + ti * 16 + l16;              // global token row
                    const float* gate_row = gate_ptr + (size_t)(min(r, m - 1) / gate_rows) * gate_stride;
#pragma unroll
                    for (int fi = 0; fi < 4; fi++)   // column clamped: masked on store
                        gv[fi] = *reinterpret_cast<const f32x4*>(gate_row + min(col0 + wf * 64 + fi * 16 + 4 * q4, n - 4));
                }
#pragma unroll
                for (int fi = 0; fi < 4; fi++) {
                    const int fl = wf * 64 + fi * 16 + 4 * q4;      // feature inside the tile
                    f32x4 v = acc[fi][ti];
                    v += bv[fi];
                    if constexpr (EPI == EPI_GELU_TANH) {
#pragma unroll
                        for (int j = 0; j < 4; j++) v[j] = gelu_tanh_f(v[j]);
                    } else if constexpr (EPI == EPI_SILU) {
#pragma unroll
                        for (int j = 0; j < 4; j++) v[j] = silu_f(v[j]);
                    } else if constexpr (EPI == EPI_GATE_RES) {
                        v *= gv[fi];
                    } else if constexpr (EPI == EPI_QKV) {
                        if (col0 + fl < q_cols) v *= q_scale;      // the four features of v lie in one head
                    }
                    unsigned char* dst = smem + trow * STRIDE + fl * SE;
                    if constexpr (F32OUT) {
                        *reinterpret_cast<f32x4*>(dst) = v;
                    } else {
                        bf16x4 o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
                        *reinterpret_cast<bf16x4*>(dst) = o;
                    }
                }
            }
        };
        if (NPASS == 1 || wt == pass) {
            if (!RES || gate_in_lds) stage(std::true_type{});
            else stage(std::false_type{});
        }
        if (pass == 0 && NPASS == 2) load_res(1);   // in flight across this pass's barrier and stores
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITERS; j++) {
            const int c = tid + 256 * j;
            const int trow = c / CHUNKS_PER_ROW, ch = c % CHUNKS_PER_ROW;
            const int r = row0 + pass * ROWS_PER_PASS + trow;
            const int f = col0 + ch * CHUNK_ELEMS;
            if (r >= m || f >= n) continue;
            if constexpr (GEGLU) {
                // 8 outputs: u at staged columns 8 ch .. 8 ch + 7, gate 64 columns further
                const float* su = reinterpret_cast<const float*>(smem + trow * STRIDE) + ch * 8;
                bf16x8 o8;
#pragma unroll
                for (int j = 0; j < 8; j++) o8[j] = (bf16_t)(su[j] * gelu_erf_f(su[64 + j]));
                *reinterpret_cast<bf16x8*>(static_cast<bf16_t*>(p.out) + (size_t)r * n + f) = o8;
                continue;
            }
            const unsigned char* srcp = smem + trow * STRIDE + ch * 16;
            if constexpr (EPI == EPI_QKV) {
                // feature f = (which, head, i); token row r = (sample b, token t): 8 features stay inside one head.
                // The divisions are taken once per tile, on its first column and row; a chunk adds its offset and steps
                // over at most one boundary of each kind when a tile is no wider than q, k or v and no taller than a
                // sample (otherwise every chunk divides).
                const int hd = p.heads * 64;
                int which, cc, b, t;
                if (qkv_steps) {
                    which = qkv_which0;
                    cc = qkv_cc0 + ch * CHUNK_ELEMS;
                    if (cc >= hd) { cc -= hd; which++; }
                    b = qkv_b0;
                    t = qkv_t0 + pass * ROWS_PER_PASS + trow;
                    if (t >= p.tokens) { t -= p.tokens; b++; }
                } else {
                    which = f / hd;
                    cc = f - which * hd;
                    b = r / p.tokens;
                    t = r - b * p.tokens;
                }
                const int head = cc / 64, i0 = cc % 64;
                OT* base = static_cast<OT*>(which == 0 ? p.q : (which == 1 ? p.k : p.v));
                OT* dst = base + (((size_t)b * p.heads + head) * p.n_total + p.tok_offset + t) * 64 + i0;
                *reinterpret_cast<u32x4*>(dst) = *reinterpret_cast<const u32x4*>(srcp);
            } else if constexpr (EPI == EPI_GATE_RES) {
                const size_t o = (size_t)r * n + f;
                *reinterpret_cast<f32x4*>(static_cast<float*>(p.out) + o) = *reinterpret_cast<const f32x4*>(srcp) + resv[pass][j];
            } else {
                OT* dst = static_cast<OT*>(p.out) + (size_t)split * m * n + (size_t)r * n + f;
                *reinterpret_cast<u32x4*>(dst) = *reinterpret_cast<const u32x4*>(srcp);
            }
        }
        if (pass + 1 < NPASS) __syncthreads();
    }
}

// Up to this many tile columns a launch hands each XCD a run of consecutive tiles (see the kernel).
constexpr int kNarrowTileCols = 16;

template <typename OT, int EPI, int TMW>
int launch_tiles(const GemmGroup& g, int tiles_n, hipStream_t st, int ksplit = 1) {
    constexpr int BM = Geo<TMW>::BM;
    GemmGroup gg = g;
    // The smaller problem goes first: its tiles fetch a whole weight matrix from HBM for few rows, which is better
    // hidden under the start of the large problem than left for the end of the launch.
    if (gg.count > 1 && !gg.n2 && gg.p[1].m < gg.p[0].m) {
        const GemmProblem t = gg.p[0];
        gg.p[0] = gg.p[1];
        gg.p[1] = t;
    }
    const int tiles0 = ((gg.p[0].m + BM - 1) / BM) * tiles_n;
    const int tiles1 = gg.count > 1 ? ((gg.p[1].m + BM - 1) / BM) * (gg.n2 ? (gg.n2 + BN - 1) / BN : tiles_n) : 0;
    char name[96] = "";
    if (hyb_trace_on()) snprintf(name, sizeof(name), "gemm_mfma_%dx%d.epi%d.n%d.k%d", BM, BN, EPI, g.n, g.k);
    const double flop0 = 2.0 * g.p[0].m * g.n * g.k, flop1 = g.count > 1 ? 2.0 * g.p[1].m * (g.n2 ? g.n2 : g.n) * (g.n2 ? g.k2 : g.k) : 0;
    HybTraceScope trace(name, "flop", flop0 + flop1, st);
    int t0 = tiles0;
    if (tiles0 == 0 && !gg.n2) {  // keep problem 0 non-empty so that the tile -> problem split stays simple
        gg.p[0] = gg.p[1];
        gg.count = 1;
        t0 = tiles1;
    }
    const int total = (tiles0 + tiles1) * ksplit;
    const int first = gg.n2 ? t0 : 0;   // tiles of a problem of another shape, in runs of their own
    const int xcd_run = tiles_n <= kNarrowTileCols ? (total - first + 7) / 8 : 0;
    const int grid = xcd_run ? 8 * ((first + 7) / 8 + xcd_run) : total;
    // A launch of 64-row tiles that leaves room on the CUs is bound by the latency of its slab copies, one after the other: it
    // takes more slab buffers, six when every workgroup can have a CU of its own, three for up to two per CU.
    // Two against six: 333 x 1536 x 4096 49 -> 26 us, one row x 1536 x 1536 24 -> 13 us; two against three: 2048 x 1280 x 1280
    // with residual 21 -> 18 us.  Up to two k-slabs have nothing to run ahead of.  A launch of two problems of different shapes takes
    // at least three: its long tiles decide how long it lasts (8192 x 640, k 640, beside 154 x 1280, k 2048: 31 -> 27 us, 24 us
    // with tile runs of their own).
    if constexpr (TMW == 1) {
        const int nslab = g.k / BK / ksplit, cus = hyb_cu_count();
        if (total <= cus && nslab > 2) hipLaunchKernelGGL((gemm_mfma_kernel<OT, EPI, 1, 6>), dim3(grid), dim3(256), 0, st, gg, tiles_n, t0, total, xcd_run, ksplit);
        else if ((total <= 2 * cus || gg.n2) && nslab > 2) hipLaunchKernelGGL((gemm_mfma_kernel<OT, EPI, 1, 3>), dim3(grid), dim3(256), 0, st, gg, tiles_n, t0, total, xcd_run, ksplit);
        else hipLaunchKernelGGL((gemm_mfma_kernel<OT, EPI, 1, 2>), dim3(grid), dim3(256), 0, st, gg, tiles_n, t0, total, xcd_run, ksplit);
    } else {
        hipLaunchKernelGGL((gemm_mfma_kernel<OT, EPI, TMW, 2>), dim3(grid), dim3(256), 0, st, gg, tiles_n, t0, total, xcd_run, ksplit);
    }
    return hyb_check_launch("gemm_mfma");
}

constexpr int kMaxSplit = 8;

// Second pass of the k split: out = epilogue(sum over the planes, in order, + bias), one thread per four elements, whose planes are all requested
// before the first sum (bound by memory: planes, residuals and result, 63 MB and 50 MB below, 6 TB/s).  Against one element per thread, whose
// planes are read one after the other: 2048 x 1280 with two residuals, three planes 14.2 -> 10.5 us; 3264 x 640 11.3 -> 8.3 us.
template <typename OT, int KS>
__global__ __launch_bounds__(256) void gemm_splitk_merge_kernel(GemmGroup g, const float* planes, int epi) {
    const GemmProblem& p = g.p[0];
    const unsigned quads = (unsigned)g.n / 4, total = (unsigned)p.m * quads;      // (a launch that splits k has at most 384 x 128 x 128 elements)
    const unsigned i = blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    f32x4 part[KS];
#pragma unroll
    for (int s = 0; s < KS; s++) part[s] = reinterpret_cast<const f32x4*>(planes)[(size_t)s * total + i];
    f32x4 v = part[0];
#pragma unroll
    for (int s = 1; s < KS; s++) v += part[s];
    const unsigned r = i / quads;
    gemm_store_four<OT>(p, epi, g.n, (int)r, (int)(i - r * quads) * 4, v);
}

template <typename OT, int KS>
int launch_merge(const GemmGroup& g, int ksplit, int epi, hipStream_t st) {
    if constexpr (KS < kMaxSplit) {
        if (ksplit != KS) return launch_merge<OT, KS + 1>(g, ksplit, epi, st);
    }
    const size_t elems = (size_t)g.p[0].m * g.n;
    HybTraceScope trace("gemm_splitk_merge", "byte", (double)elems * (4.0 * ksplit + sizeof(OT)), st);
    hipLaunchKernelGGL((gemm_splitk_merge_kernel<OT, KS>), dim3((unsigned)((elems / 4 + 255) / 256)), dim3(256), 0, st, g,
                       static_cast<const float*>(g.splitk_ws), epi);
    return hyb_check_launch("gemm_splitk_merge");
}

// k split for launches that cannot fill the chip with tiles but have a long k (each workgroup then waits for
// one k-slab after the other: the time is slabs x slab latency whatever the chip could do).  Returns the number
// of splits (1: none): as many as keep every workgroup resident at once (768 slots of 64-row tiles) with at
// least 4 slabs each, at most eight, and only when the caller's scratch holds the planes.  (slots: 512 for 128-row
// tiles, 768 for 64-row tiles.)
constexpr int kSplitMinSlabs = 32;
int choose_ksplit(const GemmGroup& g, int tiles, int slots) {
    const int nslab = g.k / BK;
    if (g.count != 1 || !g.splitk_ws || nslab < kSplitMinSlabs || tiles <= 0) return 1;
    if (((uintptr_t)g.p[0].gate & 15u) != 0 || g.p[0].gate_stride % 4 != 0) return 1;      // the merge reads the gate row in fours
    int s = slots / tiles;
    if (s > nslab / 4) s = nslab / 4;
    if (s > kMaxSplit) s = kMaxSplit;
    if (s < 2 || (size_t)s * g.p[0].m * g.n * sizeof(float) > g.splitk_bytes) return 1;
    return s;
}

// 128-token tiles unless they would fill less than three quarters of the 512 workgroup slots of the chip (two
// per CU); then 64-token tiles, of which three fit a CU (768 slots), halve the length of the single round.
constexpr int kSmallGridTiles = 384;

template <typename OT, int EPI>
int launch_epi(const GemmGroup& g, hipStream_t st) {
    const int tile_cols = EPI == EPI_GEGLU ? BN / 2 : BN;
    const int tiles_n = (g.n + tile_cols - 1) / tile_cols;
    const int rows1 = g.count > 1 ? g.p[1].m : 0;
    const int tiles128 = (g.p[0].m + 127) / 128 * tiles_n + (rows1 + 127) / 128 * (g.n2 ? (g.n2 + BN - 1) / BN : tiles_n);
    if (tiles128 == 0) return HYB_OK;
    if constexpr (EPI != EPI_GEGLU) {
        // 128-row tiles stream a third fewer operand bytes: preferred whenever they allow a split at all
        int ksplit = 1;
        bool tall = false;
        if (tiles128 <= kSmallGridTiles) {
            ksplit = choose_ksplit(g, tiles128, 512);
            tall = ksplit > 1;
            if (!tall) ksplit = choose_ksplit(g, ((g.p[0].m + 63) / 64) * tiles_n, 768);
        }
        if (ksplit > 1) {
            // pass 1: raw fp32 sums of every k share (plain epilogue, no bias), pass 2: merge + the real epilogue
            GemmGroup part = g;
            part.p[0].bias = nullptr;
            part.p[0].out = g.splitk_ws;
            int rc = tall ? launch_tiles<float, EPI_BIAS, 2>(part, tiles_n, st, ksplit) : launch_tiles<float, EPI_BIAS, 1>(part, tiles_n, st, ksplit);
            if (rc != HYB_OK) return rc;
            return launch_merge<OT, 2>(g, ksplit, EPI, st);
        }
    }
    if (tiles128 <= kSmallGridTiles) return launch_tiles<OT, EPI, 1>(g, tiles_n, st);
    return launch_tiles<OT, EPI, 2>(g, tiles_n, st);
}

// Long-k launches with enough 256 x 128 tiles for more than half of the CUs go to the large-tile kernel (one
// workgroup per CU): there the fixed cost of a tile (first-slab latency, epilogue: about 10 us with the gate + residual
// epilogue) is small against its main loop, and the operand stream per flop is a quarter smaller (the SD3-shaped fc2,
// k = 6144: 216 tiles in one round, 78 us alone and 90 us inside the step against 101 and 103 us with 420 tiles of
// 128 x 128 on 512 slots; launches of several rounds, batch 2 or the 2048 x 2048 shape, gain 3-4 % per launch).  With
// fewer k-slabs the 128 x 128 kernel, whose two workgroups per CU hide each other's fixed costs, is as fast or faster
// (measured at k = 1536 inside the step: out-projection 35.0 against 35.4 us in one round, fc1 110 against 98 us in
// four rounds).
constexpr int kLargeTileMinSlabs = 48;          // launches of several rounds
// 192-row tiles in one round, whose launch has 64- or 128-row tiles otherwise; time against those at 176-256 tiles of seven shapes with gate
// and residual (2050-8192 rows): ten slabs 0.90-1.13, 16 slabs 0.86-1.06, 18 slabs 0.85-1.01, 20 slabs 0.73-0.95, 24 slabs
// 0.77-0.94, 31 slabs 0.75-0.87 (a 512 x 512 step of 8 blocks, out-projection 2714 x 1536 with 24 slabs: 2401 -> 2385 us).
constexpr int kLargeTileMinSlabs192 = 20;
constexpr int kLargeTileMinSlabsOneRound = 32;  // launches of one round (the SDXL-shaped down-projection, k = 2560)
bool has_two_residuals(const GemmGroup& g, int epi) {
    return epi == EPI_GATE_RES && (g.p[0].res2 || (g.count > 1 && g.p[1].res2));
}
// Tile height: 256 or 192 rows, whichever makes the launch shorter (rounds of tiles times the height; a CU holds one tile);
// 192 for the gate + residual epilogue only, the one that the blocks' long-k launches have.
// 256 against 192 rows: 2048 + 666 rows x 1536, k 6144 (136 against 180 tiles) 85 -> 75 us; 8192 x 640, k 2560 (160 against 215)
// 47 -> 41 us; 6075 + 462 rows x 1536, k 6144 (two rounds of either) about 185 -> 147 us.
int large_tile_rows(const GemmGroup& g, hyb_dtype out_dtype, int epi) {
    const bool f32 = out_dtype == HYB_F32;
    const bool has_form = epi == EPI_BIAS || epi == EPI_GELU_TANH || epi == EPI_SILU || (epi == EPI_GATE_RES && f32);
    const int nslab = g.k / BK;
    // A second residual is added in another order by the large tiles, (y + res) + res2, than by the 64- and 128-row ones, y + (res + res2).
    // So with two of them no launch short of 32 slabs takes large tiles, and a row has the same bits whatever the number of
    // rows (from 32 on the k split of such launches depends on the rows as well).
    if (!has_form || nslab < (epi == EPI_GATE_RES && !has_two_residuals(g, epi) ? kLargeTileMinSlabs192 : kLargeTileMinSlabsOneRound)) return 0;
    const int cus = hyb_cu_count();
    long best = 0;
    int rows = 0;
    for (int h = 256; h >= (epi == EPI_GATE_RES ? 192 : 256); h -= 64) {
        long tiles = 0;
        for (int i = 0; i < g.count; i++) tiles += (long)((g.p[i].m + h - 1) / h) * ((g.n + 127) / 128);
        const bool enough = h == 256 ? 2 * tiles > cus : 3 * tiles > 2 * cus;
        if (!enough || (tiles > cus && nslab < kLargeTileMinSlabs) || (h == 256 && nslab < kLargeTileMinSlabsOneRound)) continue;
        const long length = (tiles + cus - 1) / cus * h;
        if (rows == 0 || length < best) { best = length; rows = h; }
    }
    return rows;
}

// Estimated length of a launch in us, fitted to 3700 launches of one problem (300-33000 rows, 512-8192 columns, k 256-8192; every tile shape forced)
// whose weights come from memory, each launch another matrix, as inside a step: half of the estimates are within 4 % of what was
// measured, nine tenths within 10 % (64-row tiles 6 and 16 %).  Of these launches 24 are more than 3 % longer than with the tiles of the kernels without 256
// columns.  With costs fitted to weights in the cache 131 were: 8192 x 2560 GEGLU, k 1280 122 us on 128 x 256 tiles, 108 on 128 x 128
// and 103 on 192 x 256; 11264 x 1408 with gate and residual, k 1536 71 us on 192- and 128-row tiles of 256 columns, 62 on 128 x 128.
// A tile alone on its CU costs k-slabs x slab + fixed; `fill`: where all CUs are busy every one is slower (they share the memory
// system and the power) than with three quarters of them, where fewer are, faster.
struct TileCost { float slab, fixed, fill; };
enum { COST_BIG_256, COST_BIG_192, COST_WIDE_128, COST_WIDE_192, COST_WIDE_256, COST_KINDS };
const TileCost kTileCost[4][COST_KINDS] = {
    /* bias, QKV       */ {{0.67f, 7.0f, 0.11f}, {}, {0.72f, 3.5f, 0.16f}, {0.95f, 4.5f, 0.32f}, {1.20f, 5.4f, 0.40f}},
    /* GELU            */ {{0.67f, 8.5f, 0.11f}, {}, {0.72f, 5.2f, 0.11f}, {0.95f, 7.2f, 0.28f}, {1.14f, 8.6f, 0.33f}},
    /* GEGLU           */ {{}, {}, {0.75f, 4.5f, 0.00f}, {1.05f, 6.4f, 0.19f}, {1.20f, 7.7f, 0.24f}},
    /* gate + residual */ {{0.70f, 11.1f, 0.22f}, {0.56f, 8.9f, 0.10f}, {0.73f, 9.2f, 0.32f}, {0.88f, 12.1f, 0.44f}, {1.10f, 13.9f, 0.56f}},
};
// 128-row tiles, two on a CU: slab and fixed of a round of both, the share of it that a last round's first tile takes, and the start of the launch
struct PairCost { float slab, fixed, part, start; };
const PairCost kPairCost[4] = {{0.88f, 2.8f, 0.38f, 4.1f}, {0.91f, 4.1f, 0.41f, 4.6f}, {1.00f, 3.2f, 0.40f, 5.0f}, {0.95f, 7.1f, 0.49f, 4.3f}};
// 64-row tiles, up to three on a CU: per slab, per slab and tile of the CU, and the rest
struct SmallCost { float slab, shared, fixed; };
const SmallCost kSmallCost[4] = {{0.16f, 0.27f, 4.5f}, {0.15f, 0.25f, 5.1f}, {0.10f, 0.27f, 4.7f}, {0.15f, 0.24f, 6.0f}};
// 256-column tiles of one height whose tile rows are a multiple of eight: 128 and 256 rows are that much slower (8192 x 2560 GEGLU, k 640 69 and 71 us, 192 rows
// 64); not those that store q, k and v past the L2 (a stage of 8192 rows x 1024 channels, 128 x 256 tiles 1563 us, 128 x 128 1619)
constexpr float kWholeGroups128 = 1.09f, kWholeGroups256 = 1.04f;

int cost_row(int epi) { return epi == EPI_GELU_TANH ? 1 : (epi == EPI_GEGLU ? 2 : (epi == EPI_GATE_RES ? 3 : 0)); }

float tile_us(const TileCost& c, int nslab) { return (float)nslab * c.slab + c.fixed; }

// `tiles` tiles, one on a CU at a time
float alone_us(const TileCost& c, int nslab, long tiles) {
    const long cus = hyb_cu_count(), rounds = (tiles + cus - 1) / cus;
    if (rounds == 0) return 0.f;
    return 2.f + (float)rounds * tile_us(c, nslab) * (1.f + c.fill * ((float)tiles / (float)(rounds * cus) - 0.75f));
}

// Launch of 128-column tiles of 64, 128 (two on a CU), 192 or 256 rows (one on a CU).  Where tiles share a CU, those of a partial last
// round, which have it to themselves, are faster.
float launch_us(const GemmGroup& g, int epi, int rows, bool alone) {
    const int cols = epi == EPI_GEGLU ? BN / 2 : BN, nslab = g.k / BK, row = cost_row(epi);
    long tiles = 0;
    for (int i = 0; i < g.count; i++) tiles += (long)((g.p[i].m + rows - 1) / rows) * ((g.n + cols - 1) / cols);
    const long cus = hyb_cu_count();
    if (rows == 64) return kSmallCost[row].fixed + (float)nslab * (kSmallCost[row].slab + kSmallCost[row].shared * (float)((tiles + cus - 1) / cus));
    if (alone) return alone_us(kTileCost[row][rows == 256 ? COST_BIG_256 : COST_BIG_192], nslab, tiles);
    const PairCost& c = kPairCost[row];
    const long full = tiles / (2 * cus), rest = tiles - full * 2 * cus;
    return c.start + ((float)full + (rest ? c.part + (1.f - c.part) * (float)rest / (float)(2 * cus) : 0.f)) * ((float)nslab * c.slab + c.fixed);
}

// Launch of `tall` and then `shrt` tiles of the given costs on one workgroup per CU, each taken by the first CU that is free.
float two_height_us(long tall, long shrt, const TileCost& ct, const TileCost& cs, int nslab) {
    const float tall_us = tile_us(ct, nslab), short_us = tile_us(cs, nslab);
    const long cus = hyb_cu_count();
    const float even = (float)(tall / cus) * tall_us;            // every CU is busy until then ...
    const long ahead = tall % cus;                               // ... and these for one tall tile more
    const float late = ahead ? even + tall_us : even;
    float end = late;
    // until `even` + j short tiles the CUs that are not ahead take j each, the others what fits behind their tall tile
    for (long j = shrt / cus;; j++) {
        const float until = even + (float)j * short_us;
        const long on_late = until > late ? (long)((until - late) / short_us + 1e-3f) : 0;
        if ((cus - ahead) * j + ahead * on_late >= shrt) {
            end = until > late ? until : late;
            break;
        }
    }
    const float busy_tall = (float)tall * tall_us, busy_short = (float)shrt * short_us, busy = busy_tall + busy_short;
    const float fill = (busy_tall * ct.fill + busy_short * cs.fill) / busy;
    return 2.f + end * (1.f + fill * (busy / ((float)cus * end) - 0.75f));
}

// GEGLU launches of short k and more than one round of 128 x 128 tiles take 256-column tiles only where the estimate is a fifth shorter.  By itself such a launch is
// as much shorter as estimated, but inside a stage the card then runs everything else, the attention above all, at a lower clock.  Stages with
// 256-column against 128 x 128 tiles: 640 channels (ten slabs), 8192 rows 3302 against 3235 us (estimate 0.91; traced: GEGLU 69 -> 65.5 us, attention
// 83 -> 88, LayerNorm 6.9 -> 7.2), 8361 rows 1.033 (0.81), 7079 rows 1.045 (0.83), 16384 rows 0.991 (0.78), 3000 rows 0.979 (0.74); 384 and 512 channels 1.00-1.03 (0.80-0.88);
// from 14 slabs on 0.95-1.01 (0.70-0.86); launches of one round 0.98-1.00.
constexpr int kShortGegluSlabs = 12;
constexpr int kWideAlwaysSlabs = 64;      // from here on the estimates alone decide
constexpr float kShortGegluGain = 0.80f;

// Plan of a launch of 256-column tiles (gemm_mfma_wide.hip) if that shortens the launch by a twentieth at least (or as above) against what it takes
// otherwise, else plan.tall = 0.  Bias, GELU and gate + residual launches of 32 k-slabs and more as well: 6537 x 1280 gate + residual, k 2560 74 -> 48 us,
// 4429 x 8192 GELU, k 2048 149 -> 128; against large tiles, whose one round is hard to beat, by a tenth (1602 x 3264, k 2560: estimated a twentieth shorter on
// 128 x 256 tiles, 37.6 against 33.3 us).  Tiles of one height fill their last round by chance (16717 x 6144: 6.2 rounds
// of 256 x 256); with the first rounds tall and the others short the CUs finish together (that launch 284 -> 273 us, 6537 x 6144 121 -> 115 us).
// `large_rows`: the 128-column large tiles that large_tile_rows() picked, 0: 64 or 128 rows of the kernel above.
WidePlan wide_plan(const GemmGroup& g, hyb_dtype out_dtype, int epi, int large_rows) {
    WidePlan plan = {};
    const bool f32 = out_dtype == HYB_F32;
    const int nslab = g.k / BK;
    if (g.n2 || nslab < 3) return plan;
    if (epi == EPI_GATE_RES ? !f32 : f32 || (epi != EPI_BIAS && epi != EPI_GELU_TANH && epi != EPI_QKV && epi != EPI_GEGLU)) return plan;
    if (nslab < kWideAlwaysSlabs) {
        // With two residuals the large tiles add in an order of their own (see large_tile_rows): such launches stay with them, or short of them.
        if (nslab >= kLargeTileMinSlabsOneRound && has_two_residuals(g, epi)) return plan;
        // Several rounds of large tiles (48 slabs and more) stay there: the tests of those rounds hold launches of 48 slabs in their place, although
        // 256-column tiles would be faster (6400 x 1536 gate + residual 72 against 60 us, 8858 x 1544 GELU 85 against 74).
        if (large_rows) {
            long tiles = 0;
            for (int i = 0; i < g.count; i++) tiles += (long)((g.p[i].m + large_rows - 1) / large_rows) * ((g.n + BN - 1) / BN);
            if (tiles > hyb_cu_count()) return plan;
        }
    }
    int other = large_rows;
    float gain = large_rows ? 0.90f : 0.95f;
    if (!large_rows) {
        const int tile_cols = epi == EPI_GEGLU ? BN / 2 : BN, tiles_n = (g.n + tile_cols - 1) / tile_cols;
        int tiles128 = 0;
        for (int i = 0; i < g.count; i++) tiles128 += (g.p[i].m + 127) / 128 * tiles_n;
        if (tiles128 <= kSmallGridTiles && epi != EPI_GEGLU &&
            (choose_ksplit(g, tiles128, 512) > 1 || choose_ksplit(g, (g.p[0].m + 63) / 64 * tiles_n, 768) > 1)) return plan;
        other = tiles128 <= kSmallGridTiles ? 64 : 128;
        if (epi == EPI_GEGLU && nslab <= kShortGegluSlabs && tiles128 > 2 * hyb_cu_count()) gain = kShortGegluGain;
    }
    float best = gain * launch_us(g, epi, other, large_rows != 0);
    const int cols = epi == EPI_GEGLU ? BN : 2 * BN, cus = hyb_cu_count();
    const long tiles_n = (g.n + cols - 1) / cols;
    const TileCost* cost = &kTileCost[cost_row(epi)][COST_WIDE_128];      // of 128, 192 and 256 rows
    auto take = [&](float t, int tall, int shrt, int rows0, int rows1) {
        if (t >= best) return;
        best = t;
        plan.tall = tall; plan.shrt = shrt;
        plan.tall_rows[0] = rows0; plan.tall_rows[1] = rows1;
    };
    for (int h = 2; h >= 0; h--) {
        const int height = 128 + 64 * h;
        int rows[kMaxGroup] = {0, 0};
        for (int i = 0; i < g.count; i++) rows[i] = (g.p[i].m + height - 1) / height;
        float t = alone_us(cost[h], nslab, (rows[0] + rows[1]) * tiles_n);
        if (rows[1] == 0 && rows[0] % 8 == 0 && h != 1 && epi != EPI_QKV) t *= h ? kWholeGroups256 : kWholeGroups128;
        if (h > 0) take(t, height, height - 64, rows[0], rows[1]);
        else take(t, 192, 128, 0, 0);
    }
    best *= 0.97f;           // two heights only where they save that much
    const int m0 = g.p[0].m, m1 = g.count > 1 ? g.p[1].m : 0;
    const bool swap = m1 > m0;                                   // x: the problem of more rows, y: the other
    const int mx = swap ? m1 : m0, my = swap ? m0 : m1;
    for (int h = 2; h > 0; h--) {
        const int tall = 128 + 64 * h, shrt = tall - 64;
        const int all_x = (mx + tall - 1) / tall, all_y = (my + tall - 1) / tall;
        for (int y = 0; y <= all_y; y += all_y ? all_y : 1) {          // the smaller problem is tiled in one height
            const int short_y = y ? 0 : (my + shrt - 1) / shrt;
            // tall tile rows of the larger problem: none, all, and about as many as fill whole rounds (together with the smaller one's)
            bool last = false;
            for (long r = 0; !last; r++)
                for (int up = 0; up < 2; up++) {
                    long x = (r * cus - y * tiles_n + (up ? tiles_n - 1 : 0)) / tiles_n;
                    if (x < 0) x = 0;
                    if (x >= all_x) { x = all_x; last = true; }
                    const int rest = mx - (int)x * tall;
                    const long short_x = rest > 0 ? (rest + shrt - 1) / shrt : 0;
                    if (x + y == 0 || short_x + short_y == 0) continue;            // one height
                    take(two_height_us((x + y) * tiles_n, (short_x + short_y) * tiles_n, cost[h], cost[h - 1], nslab), tall, shrt, swap ? y : (int)x, swap ? (int)x : y);
                }
        }
    }
    return plan;
}

}  // namespace

int hyb_gemm_mfma_tiles(int m, int n) { return ((m + 127) / 128) * ((n + BN - 1) / BN); }

bool hyb_gemm_mfma_takes(const GemmGroup& g, hyb_dtype out_dtype, int epi) {
    if (g.k <= 0 || g.k % BK != 0 || g.n % 8 != 0 || g.n < 8) return false;
    // per-lane byte offsets inside a tile's operand buffers are 32-bit: up to 128 rows of k elements, and for the
    // gated epilogue the gate rows n rows further down
    if ((size_t)g.k * 2 * 256 >= ((size_t)1 << 31)) return false;
    if (epi == EPI_GEGLU && ((size_t)g.n + 128) * g.k * 2 >= ((size_t)1 << 31)) return false;
    if (g.n2 && (epi != EPI_QKV || g.k2 <= 0 || g.k2 % BK != 0 || g.n2 % 8 != 0 || (size_t)g.k2 * 2 * 256 >= ((size_t)1 << 31))) return false;
    for (int i = 0; i < g.count; i++) {
        const GemmProblem& p = g.p[i];
        if (epi == EPI_GATE_RES && p.gate && (p.gate_stride % 4 != 0)) return false;
        const int n = i == 1 && g.n2 ? g.n2 : g.n;
        if (epi == EPI_QKV && (p.heads <= 0 || n % (p.heads * 64) != 0 || n / (p.heads * 64) > 3)) return false;
    }
    const bool f32 = out_dtype == HYB_F32;
    return epi == EPI_GATE_RES ? f32 : (epi == EPI_QKV || epi == EPI_GEGLU ? !f32 : epi == EPI_BIAS || epi == EPI_GELU_TANH || epi == EPI_SILU);
}

int hyb_launch_gemm_mfma(const GemmGroup& g, hyb_dtype out_dtype, int epi, hipStream_t st) {
    const bool f32 = out_dtype == HYB_F32;
    // (where a caller offers scratch for a split of k, its launches of few rows go that way)
    if (!g.splitk_ws) {
        const int rc = hyb_launch_gemm_mfma_rows(g, out_dtype, epi, st);
        if (rc >= 0) return rc;
    }
    const int rows = large_tile_rows(g, out_dtype, epi);
    const WidePlan wide = wide_plan(g, out_dtype, epi, rows);
    if (wide.tall) return hyb_launch_gemm_mfma_wide(g, out_dtype, epi, wide, st);
    if (rows) {
        const int rc = hyb_launch_gemm_mfma_big(g, out_dtype, epi, rows, st);
        if (rc >= 0) return rc;
    }
    switch (epi) {
        case EPI_BIAS: return f32 ? launch_epi<float, EPI_BIAS>(g, st) : launch_epi<bf16_t, EPI_BIAS>(g, st);
        case EPI_GELU_TANH: return f32 ? launch_epi<float, EPI_GELU_TANH>(g, st) : launch_epi<bf16_t, EPI_GELU_TANH>(g, st);
        case EPI_SILU: return f32 ? launch_epi<float, EPI_SILU>(g, st) : launch_epi<bf16_t, EPI_SILU>(g, st);
        case EPI_GATE_RES: return launch_epi<float, EPI_GATE_RES>(g, st);
        case EPI_QKV: return launch_epi<bf16_t, EPI_QKV>(g, st);
        case EPI_GEGLU: return launch_epi<bf16_t, EPI_GEGLU>(g, st);
        default: return hyb_set_error(HYB_ERR_DTYPE, "gemm: unknown epilogue %d", epi);
    }
}
