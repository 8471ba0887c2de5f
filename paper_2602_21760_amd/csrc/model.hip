// Host-side composition of a whole MMDiT-shaped denoiser evaluation (the f_theta of one guidance branch, Sec. 4.1, or of both
// branches batched): embeddings, modulations, the joint blocks and the final projection, one call from the host's language instead of a call
// per kernel group.  A small model's step is bound by the host: the tiny fp32 guided step (batch 2, 64 + 16 tokens of 256 channels) spent 125 us
// in the host's calls for 86 us of kernels.
#include "checks.h"
#include "gemm.h"

int hyb_launch_timestep_embedding(const float* t, float t_value, void* out, int batch, int dim, hyb_dtype out_dtype, hipStream_t st);

namespace {

int check(const char* who, const hyb_mmdit_desc* d, const hyb_mmdit_weights* w, const hyb_mmdit_buffers* b) {
    HYB_REQUIRE(d && w && b, HYB_ERR_NULL, "%s: a descriptor is NULL", who);
    HYB_ARG_DTYPE(who, d->dtype);
    HYB_REQUIRE(d->batch >= 0 && d->blocks >= 0 && d->n_txt >= 0 && d->hidden > 0 && d->heads > 0 && d->patch > 0 && d->latent_c > 0, HYB_ERR_SHAPE,
                "%s: bad sizes", who);
    HYB_REQUIRE(d->latent_h >= 0 && d->latent_w >= 0 && d->latent_h % d->patch == 0 && d->latent_w % d->patch == 0, HYB_ERR_SHAPE,
                "%s: latent %dx%d is not a multiple of patch %d", who, d->latent_h, d->latent_w, d->patch);
    HYB_REQUIRE(d->blocks == 0 || w->block_weights != nullptr, HYB_ERR_NULL, "%s: no block weights", who);
    return HYB_OK;
}

struct Inputs {
    const float *latent, *ctx, *t, *pooled;
    float t_value;
    int shared_latent, txt_pre_only_last;
};

// The calls of a forward in order.  LAUNCH = false makes their argument checks only, so that an error is found before anything is enqueued, and
// the same lines say what is checked and what is launched (LAUNCH = true leaves out the checks of the frequent calls).
template <bool LAUNCH>
int forward(const hyb_mmdit_desc& d, const hyb_mmdit_weights& w, const hyb_mmdit_buffers& f, const Inputs& in, void* stream) {
    const int B = d.batch, D = d.hidden, pd = d.patch * d.patch * d.latent_c;
    const int n_img = (d.latent_h / d.patch) * (d.latent_w / d.patch);
    const hyb_dtype dt = d.dtype;
    const size_t es = hyb_dtype_size(dt);
    const size_t mod_rows = ((size_t)12 * d.blocks + 2) * D;
    hipStream_t st = (hipStream_t)stream;
    int rc;
    auto linear = [&](const void* a, const void* weight, const float* bias, void* out, int m, int n, int k, hyb_dtype out_dtype, hyb_epilogue epi, const float* residual) {
        if constexpr (LAUNCH) return hyb_run_linear(a, weight, bias, out, m, n, k, dt, out_dtype, epi, residual, nullptr, 1, 0, st);
        else return hyb_check_linear(a, weight, bias, out, m, n, k, dt, out_dtype, epi, residual, nullptr, 1, 0);
    };
    // fp32 models read their inputs where they are (a copy where they are not aligned for 16-byte loads, or share memory with the m results of the
    // layer that reads them)
    auto input = [&](const float* src, void* own, size_t n, const void* out, size_t m, const void** use) {
        *use = own;
        const uintptr_t s0 = (uintptr_t)src, o0 = (uintptr_t)out;
        if (dt == HYB_F32 && src && s0 % 16 == 0 && (s0 + 4 * n <= o0 || o0 + 4 * m <= s0)) {
            *use = src;
            return (int)HYB_OK;
        }
        if constexpr (LAUNCH) return hyb_convert(src, own, n, dt, stream);
        else return hyb_check_convert(src, own, n, dt);
    };
    // timestep (and pooled text) vector, modulations of all blocks and of the final layer
    if constexpr (LAUNCH) rc = hyb_launch_timestep_embedding(in.t, in.t_value, f.t_feat, B, d.temb_dim, dt, st);
    else rc = hyb_check_timestep_embedding(f.t_feat, B, d.temb_dim, dt);
    if (rc) return rc;
    if ((rc = linear(f.t_feat, w.t1_w, w.t1_b, f.t_hid, B, D, d.temb_dim, dt, HYB_EPI_SILU, nullptr))) return rc;
    if ((rc = linear(f.t_hid, w.t2_w, w.t2_b, f.temb, B, D, D, HYB_F32, HYB_EPI_BIAS, nullptr))) return rc;
    if (d.pooled_dim > 0) {          // temb += W_p2 SiLU(W_p1 pooled + b_p1) + b_p2 (the sum is the residual epilogue)
        const void* pooled_act;
        if ((rc = input(in.pooled, f.pooled_act, (size_t)B * d.pooled_dim, f.p_hid, (size_t)B * D, &pooled_act))) return rc;
        if ((rc = linear(pooled_act, w.p1_w, w.p1_b, f.p_hid, B, D, d.pooled_dim, dt, HYB_EPI_SILU, nullptr))) return rc;
        if ((rc = linear(f.p_hid, w.p2_w, w.p2_b, f.temb, B, D, D, HYB_F32, HYB_EPI_GATE_RESIDUAL, f.temb))) return rc;
    }
    HYB_REQUIRE(mod_rows <= 0x7fffffffu, HYB_ERR_SHAPE, "too many blocks");
    if constexpr (LAUNCH) rc = hyb_adaln_modulation(w.ada_w, w.ada_b, f.temb, f.mod, (int)mod_rows, D, B, dt, stream);
    else rc = hyb_check_adaln_modulation(w.ada_w, w.ada_b, f.temb, f.mod, (int)mod_rows, D, B, dt);
    if (rc) return rc;
    // patches -> image tokens; the positional table is the residual of the projection.  Two samples share a launch.
    const int own = in.shared_latent ? 1 : B;          // latents that differ
    if constexpr (LAUNCH) rc = hyb_patchify(in.latent, f.tok, own, d.latent_h, d.latent_w, d.latent_c, d.patch, dt, stream);
    else rc = hyb_check_patchify(in.latent, f.tok, own, d.latent_h, d.latent_w, d.latent_c, d.patch, dt);
    if (rc) return rc;
    if (n_img > 0) {
        if constexpr (!LAUNCH) {
            HYB_ARG_PTR("patch projection", w.pe_w); HYB_ARG_PTR("patch projection", w.pos); HYB_ARG_PTR("patch projection", f.x_img);
            HYB_ARG_ALIGN("patch projection", w.pe_w); HYB_ARG_ALIGN("patch projection", w.pe_b); HYB_ARG_ALIGN("patch projection", w.pos);
        }
        for (int b = 0; b < B; b += kMaxGroup) {
            GemmGroup g = {};
            g.count = B - b < kMaxGroup ? B - b : kMaxGroup;
            g.n = D; g.k = pd;
            for (int i = 0; i < g.count; i++) {
                GemmProblem& p = g.p[i];
                p.a = static_cast<char*>(f.tok) + (in.shared_latent ? 0 : (size_t)(b + i) * n_img * pd * es);
                p.w = w.pe_w; p.bias = w.pe_b; p.out = f.x_img + (size_t)(b + i) * n_img * D; p.m = n_img;
                p.res = w.pos; p.rows_per_gate = 1;
                if constexpr (!LAUNCH) { HYB_ARG_ALIGN("patch projection", p.a); HYB_ARG_ALIGN("patch projection", p.out); }
            }
            if constexpr (LAUNCH) rc = hyb_launch_gemm(g, dt, HYB_F32, EPI_GATE_RES, st);
            else rc = hyb_check_gemm(g, dt, HYB_F32, EPI_GATE_RES);
            if (rc) return rc;
        }
    }
    if (d.n_txt > 0) {
        const void* ctx_act;
        if ((rc = input(in.ctx, f.ctx_act, (size_t)B * d.n_txt * d.ctx_dim, f.x_txt, (size_t)B * d.n_txt * D, &ctx_act))) return rc;
        if ((rc = linear(ctx_act, w.ce_w, w.ce_b, f.x_txt, B * d.n_txt, D, d.ctx_dim, HYB_F32, HYB_EPI_BIAS, nullptr))) return rc;
    }
    hyb_block_desc bd = {B, n_img, d.n_txt, D, d.heads, 64, d.mlp_ratio, dt, d.ln_eps, 0};
    for (int i = 0; i < d.blocks; i++) {
        bd.txt_pre_only = in.txt_pre_only_last && i == d.blocks - 1;      // nothing reads the text output of the last block
        const float* mod = f.mod + (size_t)12 * i * D;
        if constexpr (LAUNCH) rc = hyb_run_block(&bd, &w.block_weights[i], f.x_img, f.x_txt, mod, mod + 6 * D, mod_rows, f.x_img, f.x_txt, f.ws, st);
        else rc = hyb_check_block_forward(&bd, &w.block_weights[i], f.x_img, f.x_txt, mod, mod + 6 * D, mod_rows, f.x_img, f.x_txt, f.ws, f.ws_bytes);
        if (rc) return rc;
    }
    const float* last = f.mod + (size_t)12 * d.blocks * D;
    if constexpr (LAUNCH) rc = hyb_layernorm_modulate(f.x_img, last, last + D, mod_rows, f.y, B, n_img, D, d.ln_eps, dt, stream);
    else rc = hyb_check_layernorm_modulate(f.x_img, last, last + D, mod_rows, f.y, B, n_img, D, dt);
    if (rc) return rc;
    if ((rc = linear(f.y, w.f_w, w.f_b, f.out_tok, B * n_img, pd, D, dt, HYB_EPI_BIAS, nullptr))) return rc;
    if constexpr (LAUNCH) return hyb_unpatchify(f.out_tok, f.v, B, d.latent_h, d.latent_w, d.latent_c, d.patch, dt, dt, stream);
    else return hyb_check_unpatchify(f.out_tok, f.v, B, d.latent_h, d.latent_w, d.latent_c, d.patch, dt, dt);
}

}  // namespace

extern "C" int hyb_mmdit_forward(const hyb_mmdit_desc* desc, const hyb_mmdit_weights* weights, const hyb_mmdit_buffers* buffers,
                                 const float* latent, int shared_latent, const float* ctx, const float* t, float t_value, const float* pooled,
                                 int txt_pre_only_last, void* stream) {
    int rc = check("hyb_mmdit_forward", desc, weights, buffers);
    if (rc || desc->batch == 0) return rc;
    const Inputs in = {latent, ctx, t, pooled, t_value, shared_latent, txt_pre_only_last};
    if ((rc = forward<false>(*desc, *weights, *buffers, in, stream))) {
        char what[400];
        snprintf(what, sizeof(what), "%s", hyb_last_error_string());
        return hyb_set_error(rc, "hyb_mmdit_forward: %s", what);
    }
    return forward<true>(*desc, *weights, *buffers, in, stream);
}
