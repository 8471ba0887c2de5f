// fp32 MFMA GEMM for gfx950: out = epilogue(A W^T + bias), fp32 operands, products and sums in
// v_mfma_f32_16x16x4_f32 (full fp32, no split of the operands).
//
// What bounds it: the fp32 matrix rate (256 flop per clock and CU; a 128-byte row piece feeds eight times as many MFMA
// clocks as in bf16), so plain double buffering is enough; what decides the time of the small launches of the
// reference-precision models is how evenly the tiles fill 256 CUs and how many k-slabs stand in a row.
//
// Two tile shapes, both of 4 waves that own 32 tokens x 32 features each (2 x 2 MFMA tiles):
//   KW = 1: the waves form a 64 x 64 tile and share the slabs of a k panel (32 floats = 128-byte rows in LDS)
//           (a launch with one tile per CU: four slab buffers instead of two, and fragments read a slab ahead);
//   KW = 4: the waves share ONE 32 x 32 tile and split k: wave w takes the slabs w, w + 4, ...  A wave copies and reads
//           only its own slabs, so the main loop has no barrier at all; the four sums meet in LDS at the end.
// Both keep FOUR running sums per output, slab s going to sum s % 4, and add them as (0 + 1) + (2 + 3): a result has the
// same bits from either shape, whatever the number of rows of the launch, and each sum is a quarter as long as one
// running over all of k.
//
// The 16-byte direct-to-LDS copies, the XOR swizzle of the 128-byte rows and the assignment of k to lane quarters are
// those of gemm_mfma.hip; a 16-byte fragment read holds four k of a row and feeds four MFMAs.  The weight fragment is
// the "A" operand, so the 4 accumulator registers of a tile are 4 consecutive features of one token: bias, gate, residual
// and output are 16-byte accesses straight from the MFMA layout.
// Measured (us; before: the plain FMA kernel): 1306 x 3072 x 768 GELU 52 (118 TFLOP/s of 157 nominal), 1306 x 768 x 3072
// 55, 160 x 256 x 1024 9 (was 119), 2 rows x 768 x 768 9 (was 78); 4096 x 4096 x 1024 260 (132 TFLOP/s, the rate that the vendor library
// reaches on a large square fp32 product).  With the next slab's fragments prefetched into a second register set the wide
// launches lose 15 % (three waves per SIMD instead of four).
#include "gemm.h"
#include "gemm_lds.h"

#include <type_traits>

namespace {

constexpr int BK = 32;            // floats per slab
constexpr int ROWB = BK * 4;      // bytes per LDS row of a slab

// All eight fragments of a slab, complete on return (byte addresses in LDS, from `BASE` on).  Written as one asm statement with
// its own wait: for a plain read the compiler would wait for every copy that is still on its way to LDS, the other buffer's
// too, which would leave one slab in flight instead of two.
template <int BASE>
__device__ __forceinline__ void read_slab(const unsigned (&aa)[2][2], const unsigned (&wa)[2][2], f32x4 (&af)[2][2], f32x4 (&wv)[2][2]) {
    asm volatile("ds_read_b128 %0, %8 offset:%16\n\tds_read_b128 %1, %9 offset:%16\n\tds_read_b128 %2, %10 offset:%16\n\tds_read_b128 %3, %11 offset:%16\n\t"
                 "ds_read_b128 %4, %12 offset:%16\n\tds_read_b128 %5, %13 offset:%16\n\tds_read_b128 %6, %14 offset:%16\n\tds_read_b128 %7, %15 offset:%16\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(af[0][0]), "=&v"(af[0][1]), "=&v"(af[1][0]), "=&v"(af[1][1]), "=&v"(wv[0][0]), "=&v"(wv[0][1]), "=&v"(wv[1][0]), "=&v"(wv[1][1])
                 : "v"(aa[0][0]), "v"(aa[0][1]), "v"(aa[1][0]), "v"(aa[1][1]), "v"(wa[0][0]), "v"(wa[0][1]), "v"(wa[1][0]), "v"(wa[1][1]), "i"(BASE)
                 : "memory");
}

// MN MFMAs with R fragment reads between the first half of them.
template <int J, int MN, int R>
__device__ __forceinline__ void interleave_reads() {
    if constexpr (J < MN) {
        constexpr int MR = MN / 2, r0 = J < MR ? R * J / MR : R, r1 = J + 1 < MR ? R * (J + 1) / MR : R;
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (r1 != r0) __builtin_amdgcn_sched_group_barrier(0x100, r1 - r0, 0);
        interleave_reads<J + 1, MN, R>();
    }
}

// GEGLU: every 32 weight rows of a tile are 16 "u" rows and the 16 "gate" rows that belong to them (n rows further), so a
// wave's two feature tiles are u and gate of the same 16 output features.
// NST slab buffers: two, or (KW = 1) four with the fragments of the next slab read while this one is multiplied.
template <typename OT, int KW, bool GEGLU, int NST>
__global__ __launch_bounds__(256, 2) void gemm_f32_mfma_kernel(GemmGroup g, int epi, int tiles_m0, int tiles_m, int total, int xcd_run) {
    constexpr int BM = KW == 1 ? 64 : 32, BN = BM;
    constexpr int GROUP_BYTES = (BM + BN) * ROWB;                  // one slab of the tile: 16 KB / 8 KB
    constexpr int STAGE_BYTES = GROUP_BYTES * KW;                  // every k-splitting wave has a slab of its own
    constexpr int CPW = GROUP_BYTES / 1024 / (KW == 1 ? 4 : 1);    // 1 KB chunks per wave per slab
    constexpr int OUT_COLS = GEGLU ? BN / 2 : BN;
    constexpr bool DEEP = NST > 2;
    __shared__ __attribute__((aligned(128))) unsigned char smem[DEEP ? STAGE_BYTES : 2 * STAGE_BYTES];
    // further slab buffers, one array each: the compiler knows that a copy into one and a read from another do not alias
    __shared__ __attribute__((aligned(128))) unsigned char smem1[DEEP ? STAGE_BYTES : 16], smem2[DEEP ? STAGE_BYTES : 16], smem3[DEEP ? STAGE_BYTES : 16];
    auto buffer = [&](int i) -> unsigned char* { return i == 0 ? smem : (i == 1 ? smem1 : (i == 2 ? smem2 : smem3)); };

    // XCD x gets the tiles [x xcd_run, (x + 1) xcd_run) of an order that walks down the rows first: neighbours share their
    // weight rows, and the activations of these models stay in every L2
    const unsigned id = blockIdx.y * gridDim.x + blockIdx.x;
    const int tile = (int)(id % 8) * xcd_run + (int)(id / 8);
    if ((int)(id / 8) >= xcd_run || tile >= total) return;
    int tm = tile % tiles_m;
    const int col0 = (tile / tiles_m) * OUT_COLS;
    const int pi = tm >= tiles_m0 ? 1 : 0;
    if (pi) tm -= tiles_m0;
    const GemmProblem& p = g.p[pi];
    const int row0 = tm * BM, m = p.m, n = g.n, k = g.k;

    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int wt = KW == 1 ? wave % 2 : 0, wf = KW == 1 ? wave / 2 : 0;   // wave position: tokens, features
    const int l16 = lane % 16, q4 = lane / 16;

    // Slab copies, rows 0 .. BM-1 = A, then BN rows of W; lane i fills slot i % 8 of row i / 8 of a chunk with k-vector
    // (slot ^ swz(row)).  Rows past the end are clamped to the last one (never stored).
    const int row_bytes = k * 4;
    const float* a_tile = static_cast<const float*>(p.a) + (size_t)row0 * k;
    const float* w_tile = static_cast<const float*>(p.w) + (size_t)col0 * k;
    const unsigned a_bytes = (unsigned)(min(BM, m - row0) * row_bytes);
    const unsigned w_bytes = (unsigned)(((GEGLU ? n : 0) + min(OUT_COLS, n - col0)) * row_bytes);
    const int nslab = (k + BK - 1) / BK;   // (k % 32 == 16: of the last slab only the first half counts)
    int voff[CPW];
#pragma unroll
    for (int c = 0; c < CPW; c++) {
        const int r = (KW == 1 ? wave + 4 * c : c) * 8 + lane / 8;
        int src;
        if (r < BM) src = min(r, m - 1 - row0);
        else {
            const int f = r - BM;
            if (GEGLU) src = min(f / 32 * 16 + f % 16, n - 1 - col0) + (f % 32 < 16 ? 0 : n);
            else src = min(f, n - 1 - col0);
        }
        voff[c] = src * row_bytes + ((lane % 8) ^ swz(r)) * 16;
    }
    auto issue = [&](int slab, int stage) {
        unsigned char* dst = (DEEP ? buffer(stage) : smem + stage * STAGE_BYTES) + (KW == 1 ? wave * 1024 : wave * GROUP_BYTES);
#pragma unroll
        for (int c = 0; c < CPW; c++) {
            constexpr int STEP = KW == 1 ? 4096 : 1024;
            // (deep form: slabs past the end are requested from buffers of no size, which keeps the count of the waits the same and copies nothing)
            if (c < CPW / 2) buffer_load_lds16(a_tile, !DEEP || slab < nslab ? a_bytes : 0u, dst + c * STEP, voff[c], slab * ROWB);
            else buffer_load_lds16(w_tile, !DEEP || slab < nslab ? w_bytes : 0u, dst + c * STEP, voff[c], slab * ROWB);
        }
    };

    // LDS addresses of the fragments inside the first stage: row 16 t + l16 of the wave's 32, slot (4 ks + kq) ^ swz(row)
    const int kq = (q4 >> 1) | ((q4 & 1) << 1);
    unsigned a_addr[2][2], w_addr[2][2];   // [k-step of 16][tile]
#pragma unroll
    for (int ks = 0; ks < 2; ks++)
#pragma unroll
        for (int t = 0; t < 2; t++) {
            const int ra = wt * 32 + t * 16 + l16, rw = BM + wf * 32 + t * 16 + l16;
            const unsigned own = (unsigned)(size_t)(lptr_t)&smem[KW == 1 ? 0 : wave * GROUP_BYTES];
            a_addr[ks][t] = own + ra * ROWB + (((4 * ks + kq) ^ swz(ra)) * 16);
            w_addr[ks][t] = own + rw * ROWB + (((4 * ks + kq) ^ swz(rw)) * 16);
        }
    constexpr int CHAINS = KW == 1 ? 4 : 1;
    f32x4 acc[CHAINS][2][2];   // [sum][feature tile][token tile]
#pragma unroll
    for (int c = 0; c < CHAINS; c++)
#pragma unroll
        for (int i = 0; i < 4; i++) acc[c][i / 2][i % 2] = f32x4{0.f, 0.f, 0.f, 0.f};

    // multiplies the slab in a stage (whole: not its first half only); then() runs once its fragments are in registers
    auto multiply = [&](auto stage_tag, f32x4 (&sum)[2][2], bool whole, auto then) {
        f32x4 af[2][2], wv[2][2];
        read_slab<decltype(stage_tag)::value * STAGE_BYTES>(a_addr, w_addr, af, wv);
        then();
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            if (ks == 1 && !whole) break;
#pragma unroll
            for (int j = 0; j < 4; j++)
#pragma unroll
                for (int fi = 0; fi < 2; fi++)
#pragma unroll
                    for (int ti = 0; ti < 2; ti++)
                        sum[fi][ti] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[ks][fi][j], af[ks][ti][j], sum[fi][ti], 0, 0, 0);
        }
    };

    if constexpr (DEEP) {
        static_assert(NST == 4 || !DEEP, "slab s sits in buffer s % 4 and goes to sum s % 4");
        f32x4 af[2][2][2], wv[2][2][2];          // [set][k-step][tile]
        const unsigned a0 = (unsigned)(wt * 32 + l16) * ROWB, w0 = (unsigned)(BM + wf * 32 + l16) * ROWB;
        auto read = [&](auto stage_tag, auto set_tag) {
            constexpr int S = decltype(set_tag)::value;
            const unsigned char* base = buffer(decltype(stage_tag)::value);
#pragma unroll
            for (int ks = 0; ks < 2; ks++)
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    const int ra = wt * 32 + t * 16 + l16, rw = BM + wf * 32 + t * 16 + l16;
                    af[S][ks][t] = *reinterpret_cast<const f32x4*>(base + a0 + t * 16 * ROWB + (((4 * ks + kq) ^ swz(ra)) * 16));
                    wv[S][ks][t] = *reinterpret_cast<const f32x4*>(base + w0 + t * 16 * ROWB + (((4 * ks + kq) ^ swz(rw)) * 16));
                }
        };
        // fragments of slab s are in set s % 2 on entry
        auto step = [&](int s, auto i_tag) {
            constexpr int I = decltype(i_tag)::value;
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * CPW) : "memory");
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            issue(s + NST, I % NST);
            read(std::integral_constant<int, (I + 1) % NST>{}, std::integral_constant<int, (I + 1) % 2>{});
            auto half = [&](auto ks_tag) {
                constexpr int ks = decltype(ks_tag)::value;
#pragma unroll
                for (int j = 0; j < 4; j++)
#pragma unroll
                    for (int fi = 0; fi < 2; fi++)
#pragma unroll
                        for (int ti = 0; ti < 2; ti++)
                            acc[I % 4][fi][ti] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[I % 2][ks][fi][j], af[I % 2][ks][ti][j], acc[I % 4][fi][ti], 0, 0, 0);
            };
            half(std::integral_constant<int, 0>{});
            interleave_reads<0, 16, 8>();
            if ((s + 1) * BK <= k) half(std::integral_constant<int, 1>{});
        };
#pragma unroll
        for (int j = 0; j < NST; j++) issue(j, j);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * CPW) : "memory");
        __builtin_amdgcn_s_barrier();
        read(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
        for (int s = 0;; s += NST) {
            step(s, std::integral_constant<int, 0>{});
            if (s + 1 >= nslab) break;
            step(s + 1, std::integral_constant<int, 1>{});
            if (s + 2 >= nslab) break;
            step(s + 2, std::integral_constant<int, 2>{});
            if (s + 3 >= nslab) break;
            step(s + 3, std::integral_constant<int, 3>{});
            if (s + 4 >= nslab) break;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // no copy is on its way to LDS when the workgroup ends
    } else if constexpr (KW == 1) {
        // one barrier per slab: behind it slab s is there for everyone and the other buffer, whose fragments every wave
        // has taken into registers, can be refilled
        auto step = [&](int s, auto i_tag) {
            constexpr int I = decltype(i_tag)::value;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            if (s + 1 < nslab) issue(s + 1, 1 - I % 2);
            multiply(std::integral_constant<int, I % 2>{}, acc[I], (s + 1) * BK <= k, [] {});
        };
        issue(0, 0);
        for (int s = 0; s < nslab; s += 4) {
            step(s, std::integral_constant<int, 0>{});
            if (s + 1 < nslab) step(s + 1, std::integral_constant<int, 1>{});
            if (s + 2 < nslab) step(s + 2, std::integral_constant<int, 2>{});
            if (s + 3 < nslab) step(s + 3, std::integral_constant<int, 3>{});
        }
    }
    if constexpr (KW == 1) {
#pragma unroll
        for (int ti = 0; ti < 2; ti++) {
            const int r = row0 + wt * 32 + ti * 16 + l16;
            if (r >= m) continue;
            f32x4 v[2];
#pragma unroll
            for (int fi = 0; fi < 2; fi++) v[fi] = (acc[0][fi][ti] + acc[1][fi][ti]) + (acc[2][fi][ti] + acc[3][fi][ti]);
            if constexpr (GEGLU) {
                const int c = col0 + wf * 16 + 4 * q4;
                if (c >= n) continue;
                if (p.bias) {
                    v[0] += *reinterpret_cast<const f32x4*>(p.bias + c);
                    v[1] += *reinterpret_cast<const f32x4*>(p.bias + n + c);
                }
#pragma unroll
                for (int j = 0; j < 4; j++) v[0][j] *= gelu_erf_f(v[1][j]);
                gemm_write_four<OT>(static_cast<OT*>(p.out) + (size_t)r * n + c, v[0]);
            } else {
#pragma unroll
                for (int fi = 0; fi < 2; fi++) {
                    const int c = col0 + wf * 32 + fi * 16 + 4 * q4;
                    if (c < n) gemm_store_four<OT>(p, epi, n, r, c, v[fi]);
                }
            }
        }
    } else {
        // the wave's own slabs wave, wave + 4, ...: two in flight, no barriers; a buffer is refilled once its fragments
        // are in registers
        auto step = [&](int s, auto stage_tag) {
            if (s + 4 < nslab) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(CPW) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            multiply(stage_tag, acc[0], (s + 1) * BK <= k, [&] {
                if (s + 8 < nslab) issue(s + 8, decltype(stage_tag)::value);
            });
        };
        if (wave < nslab) issue(wave, 0);
        if (wave + 4 < nslab) issue(wave + 4, 1);
        for (int s = wave; s < nslab; s += 8) {
            step(s, std::integral_constant<int, 0>{});
            if (s + 4 < nslab) step(s + 4, std::integral_constant<int, 1>{});
        }
        __syncthreads();   // every copy has landed and every wave is done with its buffers
        f32x4* red = reinterpret_cast<f32x4*>(smem);   // [sum][tile][lane]
#pragma unroll
        for (int t = 0; t < 4; t++) red[(wave * 4 + t) * 64 + lane] = acc[0][t / 2][t % 2];
        __syncthreads();
        auto total_of = [&](int t) { return (red[t * 64 + lane] + red[(4 + t) * 64 + lane]) + (red[(8 + t) * 64 + lane] + red[(12 + t) * 64 + lane]); };
        const int ti = wave % 2, fi = wave / 2;          // wave w finishes MFMA tile (w / 2, w % 2)
        const int r = row0 + ti * 16 + l16;
        if (r >= m) return;
        if constexpr (GEGLU) {
            const int c = col0 + 4 * q4;
            if (fi != 0 || c >= n) return;
            f32x4 u = total_of(ti), gt = total_of(2 + ti);
            if (p.bias) {
                u += *reinterpret_cast<const f32x4*>(p.bias + c);
                gt += *reinterpret_cast<const f32x4*>(p.bias + n + c);
            }
#pragma unroll
            for (int j = 0; j < 4; j++) u[j] *= gelu_erf_f(gt[j]);
            gemm_write_four<OT>(static_cast<OT*>(p.out) + (size_t)r * n + c, u);
        } else {
            const int c = col0 + fi * 16 + 4 * q4;
            if (c < n) gemm_store_four<OT>(p, epi, n, r, c, total_of(wave));
        }
    }
}

// A grid dimension holds less than 2^32 threads, and a larger one is cut off without an error: tiles beyond this many
// (a multiple of 8, for the XCD order) go into the second dimension.
constexpr int kMaxGridX = 1 << 23;

template <typename OT, int KW, bool GEGLU, int NST>
int launch(const GemmGroup& g, int epi, hipStream_t st) {
    constexpr int T = KW == 1 ? 64 : 32;
    const int tiles_m0 = (g.p[0].m + T - 1) / T, tiles_m1 = g.count > 1 ? (g.p[1].m + T - 1) / T : 0;
    const int cols = GEGLU ? T / 2 : T;
    const int total = (tiles_m0 + tiles_m1) * ((g.n + cols - 1) / cols);
    char name[96] = "";
    if (hyb_trace_on()) snprintf(name, sizeof(name), "gemm_f32_mfma_%dx%d.epi%d.n%d.k%d", T, T, epi, g.n, g.k);
    const double rows = g.p[0].m + (g.count > 1 ? g.p[1].m : 0);
    HybTraceScope trace(name, "flop", 2.0 * rows * g.n * g.k * (GEGLU ? 2 : 1), st);
    const int xcd_run = (total + 7) / 8;
    const int grid_x = 8 * xcd_run < kMaxGridX ? 8 * xcd_run : kMaxGridX, grid_y = (8 * xcd_run - 1) / grid_x + 1;
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<OT, KW, GEGLU, NST>), dim3(grid_x, grid_y), dim3(256), 0, st, g, epi, tiles_m0, tiles_m0 + tiles_m1, total, xcd_run);
    return hyb_check_launch("gemm_f32_mfma");
}

template <typename OT>
int launch_any(const GemmGroup& g, int epi, bool small, bool deep, hipStream_t st) {
    if (epi == EPI_GEGLU) return small ? launch<OT, 4, true, 2>(g, epi, st) : launch<OT, 1, true, 2>(g, epi, st);
    if (deep) return launch<OT, 1, false, 4>(g, epi, st);
    return small ? launch<OT, 4, false, 2>(g, epi, st) : launch<OT, 1, false, 2>(g, epi, st);
}

}  // namespace

// Tiles of a launch: `rows` x `rows`, half as many output columns for GEGLU.
static double tiles_of(const GemmGroup& g, int epi, int rows) {
    const int cols = epi == EPI_GEGLU ? rows / 2 : rows;
    double tiles = 0;
    for (int i = 0; i < g.count; i++) tiles += ((g.p[i].m + rows - 1) / rows) * (double)((g.n + cols - 1) / cols);
    return tiles;
}

bool hyb_gemm_f32_mfma_takes(const GemmGroup& g, int epi) {
    if (g.k <= 0 || g.k % (BK / 2) != 0 || g.n % 4 != 0 || g.n < 4) return false;
    // per-lane byte offsets inside a tile's operand rows are 32-bit; for GEGLU the gate rows lie n rows further down
    if ((size_t)g.k * 4 * ((epi == EPI_GEGLU ? (size_t)g.n : 0) + 64) >= ((size_t)1 << 31)) return false;
    for (int i = 0; i < g.count; i++) {
        const GemmProblem& p = g.p[i];
        if (epi == EPI_GATE_RES && p.gate && p.gate_stride % 4 != 0) return false;
        if (((uintptr_t)p.gate & 15u) != 0) return false;
    }
    return tiles_of(g, epi, 32) <= 1e9;
}

int hyb_launch_gemm_f32_mfma(const GemmGroup& g, hyb_dtype out_dtype, int epi, hipStream_t st) {
    const double tiles64 = tiles_of(g, epi, 64), tiles32 = tiles_of(g, epi, 32);
    if (tiles32 == 0) return HYB_OK;
    // A 64 x 64 tile takes a CU four times as long as a 32 x 32 one: the small tiles where they take a fifth or more off the
    // work of the busiest CU, the large ones (half the operand traffic) otherwise; small against large tiles of two slab buffers over 124 random shapes:
    // 0.30-1.08 of the time where that work is 0.75 or less, 0.97-1.73 where it is more.  (653 x 768 x 3072: 30 against
    // 61 us; 1306 x 3072 x 768: 65 against 52; 2704 x 1024 x 320: 32 against 22.)
    // A single round of large tiles that leaves CUs idle takes as long as a full one.  With four slab buffers (below) it is faster all the same: small against large
    // tiles, 193-256 of the latter, 1.02-1.22 (k 256-4096; 192 and fewer, which the line above leaves to the small ones, 0.76-0.99, 1.08 at k 320).  With two
    // (GEGLU) a long k gains from small tiles what they lose on operands: 198-210 tiles 1.15-1.22 at k 320, 0.97-0.99 at 768, 0.86-0.91 at 4096;
    // 252-256 tiles 0.98-1.03 from 768 on.
    const int cus = hyb_cu_count();
    const double busy64 = 4.0 * (double)(((long long)tiles64 + cus - 1) / cus), busy32 = (double)(((long long)tiles32 + cus - 1) / cus);
    const bool small = busy32 < 0.8 * busy64 || (epi == EPI_GEGLU && tiles64 < 0.85 * cus && g.k >= 768);
    // One large tile on nearly every CU, one wave per SIMD: nothing covers a wave's waits but its own deeper pipeline.  Two against four buffers:
    // 1306 x 768 (252 tiles) 62 -> 55 us at k 3072, 19.8 -> 18.5 at 768; with two tiles per CU and more they cover each other (504 tiles of k
    // 768: 28.8 against 28.1 us, 1008: 53 against 55).
    const bool deep = !small && epi != EPI_GEGLU && tiles64 <= cus;
    return out_dtype == HYB_F32 ? launch_any<float>(g, epi, small, deep, st) : launch_any<bf16_t>(g, epi, small, deep, st);
}
