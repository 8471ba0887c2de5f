// Host-side composition of a whole MMDiT-shaped denoiser evaluation (the f_theta of one guidance branch, Sec. 4.1, or of both
// branches batched): embeddings, modulations, the joint blocks and the final projection, one call from the host's language instead of a call
// per kernel group.  A small model's step is bound by the host: the tiny fp32 guided step (batch 2, 64 + 16 tokens of 256 channels) spent 125 us
// in the host's calls for 86 us of kernels.
#include "gemm.h"

int hyb_launch_timestep_embedding(const float* t, float t_value, void* out, int batch, int dim, hyb_dtype out_dtype, hipStream_t st);

namespace {

int check(const char* who, const hyb_mmdit_desc* d, const hyb_mmdit_weights* w, const hyb_mmdit_buffers* b) {
    HYB_CHECK_PTR(d); HYB_CHECK_PTR(w); HYB_CHECK_PTR(b);
    HYB_CHECK_DTYPE(d->dtype);
    HYB_REQUIRE(d->batch >= 0 && d->blocks >= 0 && d->n_txt >= 0 && d->hidden > 0 && d->heads > 0 && d->patch > 0 && d->latent_c > 0, HYB_ERR_SHAPE,
                "%s: bad sizes", who);
    HYB_REQUIRE(d->latent_h >= 0 && d->latent_w >= 0 && d->latent_h % d->patch == 0 && d->latent_w % d->patch == 0, HYB_ERR_SHAPE,
                "%s: latent %dx%d is not a multiple of patch %d", who, d->latent_h, d->latent_w, d->patch);
    HYB_REQUIRE(d->blocks == 0 || w->block_weights != nullptr, HYB_ERR_NULL, "%s: no block weights", who);
    return HYB_OK;
}

}  // namespace

extern "C" int hyb_mmdit_forward(const hyb_mmdit_desc* desc, const hyb_mmdit_weights* weights, const hyb_mmdit_buffers* buffers,
                                 const float* latent, int shared_latent, const float* ctx, const float* t, float t_value, const float* pooled,
                                 int txt_pre_only_last, void* stream) {
    int rc = check("hyb_mmdit_forward", desc, weights, buffers);
    if (rc) return rc;
    const hyb_mmdit_desc& d = *desc;
    const hyb_mmdit_weights& w = *weights;
    const hyb_mmdit_buffers& f = *buffers;
    const int B = d.batch, D = d.hidden, pd = d.patch * d.patch * d.latent_c;
    const int n_img = (d.latent_h / d.patch) * (d.latent_w / d.patch);
    if (B == 0) return HYB_OK;
    const hyb_dtype dt = d.dtype;
    const size_t es = hyb_dtype_size(dt);
    const size_t mod_rows = ((size_t)12 * d.blocks + 2) * D;
    hipStream_t st = (hipStream_t)stream;
    // fp32 models read their inputs where they are (a copy where they are not aligned for 16-byte loads)
    auto input = [&](const float* src, void* own, size_t n, const void** use) {
        *use = own;
        if (dt == HYB_F32 && src && ((uintptr_t)src & 15u) == 0) {
            *use = src;
            return (int)HYB_OK;
        }
        return hyb_convert(src, own, n, dt, stream);
    };
    // timestep (and pooled text) vector, modulations of all blocks and of the final layer
    HYB_CHECK_PTR(f.t_feat);
    if ((rc = hyb_launch_timestep_embedding(t, t_value, f.t_feat, B, d.temb_dim, dt, st))) return rc;
    if ((rc = hyb_linear(f.t_feat, w.t1_w, w.t1_b, f.t_hid, B, D, d.temb_dim, dt, dt, HYB_EPI_SILU, nullptr, nullptr, 1, 0, stream))) return rc;
    if ((rc = hyb_linear(f.t_hid, w.t2_w, w.t2_b, f.temb, B, D, D, dt, HYB_F32, HYB_EPI_BIAS, nullptr, nullptr, 1, 0, stream))) return rc;
    if (d.pooled_dim > 0) {          // temb += W_p2 SiLU(W_p1 pooled + b_p1) + b_p2 (the sum is the residual epilogue)
        const void* pooled_act;
        HYB_CHECK_PTR(pooled);
        if ((rc = input(pooled, f.pooled_act, (size_t)B * d.pooled_dim, &pooled_act))) return rc;
        if ((rc = hyb_linear(pooled_act, w.p1_w, w.p1_b, f.p_hid, B, D, d.pooled_dim, dt, dt, HYB_EPI_SILU, nullptr, nullptr, 1, 0, stream))) return rc;
        if ((rc = hyb_linear(f.p_hid, w.p2_w, w.p2_b, f.temb, B, D, D, dt, HYB_F32, HYB_EPI_GATE_RESIDUAL, f.temb, nullptr, 1, 0, stream))) return rc;
    }
    HYB_REQUIRE(mod_rows <= 0x7fffffffu, HYB_ERR_SHAPE, "hyb_mmdit_forward: too many blocks");
    if ((rc = hyb_adaln_modulation(w.ada_w, w.ada_b, f.temb, f.mod, (int)mod_rows, D, B, dt, stream))) return rc;
    // patches -> image tokens; the positional table is the residual of the projection.  Two samples share a launch.
    const int own = shared_latent ? 1 : B;          // latents that differ
    if ((rc = hyb_patchify(latent, f.tok, own, d.latent_h, d.latent_w, d.latent_c, d.patch, dt, stream))) return rc;
    if (n_img > 0) {
        HYB_CHECK_PTR(w.pe_w); HYB_CHECK_PTR(w.pos); HYB_CHECK_PTR(f.x_img);
        HYB_CHECK_ALIGN(w.pe_w); HYB_CHECK_ALIGN(w.pe_b); HYB_CHECK_ALIGN(w.pos); HYB_CHECK_ALIGN(f.tok); HYB_CHECK_ALIGN(f.x_img);
        for (int b = 0; b < B; b += kMaxGroup) {
            GemmGroup g = {};
            g.count = B - b < kMaxGroup ? B - b : kMaxGroup;
            g.n = D; g.k = pd;
            for (int i = 0; i < g.count; i++) {
                GemmProblem& p = g.p[i];
                p.a = static_cast<char*>(f.tok) + (shared_latent ? 0 : (size_t)(b + i) * n_img * pd * es);
                p.w = w.pe_w; p.bias = w.pe_b; p.out = f.x_img + (size_t)(b + i) * n_img * D; p.m = n_img;
                p.res = w.pos; p.rows_per_gate = 1;
                HYB_CHECK_ALIGN(p.a); HYB_CHECK_ALIGN(p.out);
            }
            if ((rc = hyb_launch_gemm(g, dt, HYB_F32, EPI_GATE_RES, st))) return rc;
        }
    }
    if (d.n_txt > 0) {
        const void* ctx_act;
        HYB_CHECK_PTR(ctx);
        if ((rc = input(ctx, f.ctx_act, (size_t)B * d.n_txt * d.ctx_dim, &ctx_act))) return rc;
        if ((rc = hyb_linear(ctx_act, w.ce_w, w.ce_b, f.x_txt, B * d.n_txt, D, d.ctx_dim, dt, HYB_F32, HYB_EPI_BIAS, nullptr, nullptr, 1, 0, stream))) return rc;
    }
    hyb_block_desc bd = {B, n_img, d.n_txt, D, d.heads, 64, d.mlp_ratio, dt, d.ln_eps, 0};
    for (int i = 0; i < d.blocks; i++) {
        bd.txt_pre_only = txt_pre_only_last && i == d.blocks - 1;      // nothing reads the text output of the last block
        const float* mod = f.mod + (size_t)12 * i * D;
        if ((rc = hyb_block_forward(&bd, &w.block_weights[i], f.x_img, f.x_txt, mod, mod + 6 * D, mod_rows, f.x_img, f.x_txt, f.ws, f.ws_bytes, stream))) return rc;
    }
    const float* last = f.mod + (size_t)12 * d.blocks * D;
    if ((rc = hyb_layernorm_modulate(f.x_img, last, last + D, mod_rows, f.y, B, n_img, D, d.ln_eps, dt, stream))) return rc;
    if ((rc = hyb_linear(f.y, w.f_w, w.f_b, f.out_tok, B * n_img, pd, D, dt, dt, HYB_EPI_BIAS, nullptr, nullptr, 1, 0, stream))) return rc;
    return hyb_unpatchify(f.out_tok, f.v, B, d.latent_h, d.latent_w, d.latent_c, d.patch, dt, dt, stream);
}
