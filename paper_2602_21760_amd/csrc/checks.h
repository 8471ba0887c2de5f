// Argument checks of the entry points that hyb_mmdit_forward strings together (each entry point makes its own before it launches anything): they
// take the entry point's arguments but the stream, touch no device, and set the same errors.  hyb_run_*: the launches alone, after the checks.
#pragma once
#include "common.h"

int hyb_check_linear(const void* a, const void* w, const float* bias, const void* out, int m, int n, int k, hyb_dtype dtype, hyb_dtype out_dtype,
                     hyb_epilogue epi, const float* residual, const float* gate, int rows_per_gate, size_t gate_stride);
int hyb_run_linear(const void* a, const void* w, const float* bias, void* out, int m, int n, int k, hyb_dtype dtype, hyb_dtype out_dtype,
                   hyb_epilogue epi, const float* residual, const float* gate, int rows_per_gate, size_t gate_stride, hipStream_t st);
int hyb_run_block(const hyb_block_desc* desc, const hyb_block_weights* weights, const float* x_img_in, const float* x_txt_in, const float* mod_img,
                  const float* mod_txt, size_t mod_stride, float* x_img_out, float* x_txt_out, void* workspace, hipStream_t st);
int hyb_check_block_forward(const hyb_block_desc* desc, const hyb_block_weights* weights, const float* x_img_in, const float* x_txt_in,
                            const float* mod_img, const float* mod_txt, size_t mod_stride, const float* x_img_out, const float* x_txt_out,
                            const void* workspace, size_t workspace_bytes);
int hyb_check_timestep_embedding(const void* out, int batch, int dim, hyb_dtype out_dtype);
int hyb_check_adaln_modulation(const void* w, const float* bias, const float* temb, const float* out, int rows, int hidden, int batch, hyb_dtype dtype);
int hyb_check_layernorm_modulate(const float* x, const float* shift, const float* scale, size_t mod_stride, const void* out, int batch, int tokens,
                                 int hidden, hyb_dtype out_dtype);
int hyb_check_patchify(const float* latent, const void* tokens, int batch, int hh, int ww, int c, int p, hyb_dtype out_dtype);
int hyb_check_unpatchify(const void* tokens, const void* latent, int batch, int hh, int ww, int c, int p, hyb_dtype in_dtype, hyb_dtype out_dtype);
int hyb_check_convert(const float* in, const void* out, size_t n, hyb_dtype out_dtype);
