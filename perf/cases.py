"""The work whose speed is followed: whole calls of the framework as a sampling program makes them, on synthetic
inputs and random-init weights of the repository's own configurations (paper_2602_21760_amd/synth.py).

Kinds of a case:
  guidance   one fused CFG + discrepancy + Euler pass (hyb_cfg_disc_euler)
  attention  one attention call of its own (hyb_joint_attention)
  branch     one denoiser forward (model.MMDiT.forward)
  step       one guided sampling step, both branches batched (model.GuidedSampler.step)
  stage      one U-Net transformer stage (model.SDXLStage.forward)"""
import math

import torch

from paper_2602_21760_amd import binding as hb, model, synth

DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def _branch(name, kind, cfg, **extra):
    """A case dict from an MMDiT configuration."""
    fields = ("blocks", "hidden", "heads", "latent_hw", "latent_c", "n_txt", "ctx_dim", "batch", "dtype", "pooled_dim")
    case = {"name": name, "kind": kind, "txt_pre_only_last": False}
    case.update({f: getattr(cfg, f) for f in fields})
    case.update(extra)
    return case


def _stage(name, cfg, **extra):
    case = {"name": name, "kind": "stage"}
    case.update({f: getattr(cfg, f) for f in ("blocks", "tokens", "channels", "heads", "n_ctx", "ctx_dim", "batch", "dtype")})
    case.update(extra)
    return case


def listed():
    cases = [
        # The guidance pass of one 1024 x 1024 latent of 4 channels: the smallest call a sampler makes, all latency.
        {"name": "guidance_one_latent", "kind": "guidance", "batch": 1, "elems": 65536, "dtype": "bf16"},
        # The same pass over a serving batch of 256 latents of 16 channels: bandwidth.
        {"name": "guidance_256_latents", "kind": "guidance", "batch": 256, "elems": 262144, "dtype": "bf16"},
        # The tiny fp32 model, one guided step: about 25 short launches, host time and launch latency.
        _branch("tiny_f32_step", "step", synth.CFG1),
        # A small model at reference precision (fp32 throughout), both branches in one batch.
        _branch("small_f32_branch", "branch", synth.CFG1, blocks=4, hidden=768, heads=12, latent_hw=48, latent_c=16,
                n_txt=77, ctx_dim=2048),
        # A guided step at 512 x 512: previews and small images (1024 + 333 tokens, both branches).
        _branch("sd3_512_step", "step", synth.CFG3, latent_hw=64, blocks=8),
        # The headline workload: one branch at 1024 x 1024, all 24 blocks.
        _branch("sd3_1024_branch", "branch", synth.CFG2),
        # The guided step of the sampling loop at 1024 x 1024: both branches batched, then the guidance pass.
        _branch("sd3_1024_step", "step", synth.CFG3, blocks=6),
        # One branch at 2048 x 2048: attention over 16717 tokens dominates.
        _branch("sd3_2048_branch", "branch", synth.CFG4, blocks=3),
        # A resolution that no tile size divides (720 x 720: 2025 tokens, 154 text tokens), three samples, pooled text
        # conditioning and a last block whose text stream only supplies keys and values.
        _branch("sd3_720_batch3_pooled", "branch", synth.CFG2, latent_hw=90, n_txt=154, batch=3, blocks=4,
                pooled_dim=2048, txt_pre_only_last=True),
        # The two transformer stages of the U-Net at 1024 x 1024, both branches batched.
        _stage("sdxl_stage_a", synth.CFG5A),
        _stage("sdxl_stage_b", synth.CFG5B, blocks=10),
        # Attention on its own, ragged both ways, through the entry point without scratch.
        {"name": "attention_ragged", "kind": "attention", "batch": 2, "heads": 20, "n_q": 1501, "n_kv": 2333, "dtype": "bf16"},
    ]
    return cases


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choice(("guidance", "attention", "branch", "branch", "step", "step", "stage", "f32"))
    if kind == "guidance":
        batch = _log_int(rng, 1, 256)
        elems = _log_int(rng, 4096, 1 << 20)
        if rng.random() < 0.7:
            elems = (elems + 7) // 8 * 8
        return {"kind": "guidance", "batch": batch, "elems": elems, "dtype": rng.choice(("bf16", "bf16", "f32"))}
    if kind == "attention":
        return {"kind": "attention", "batch": rng.randint(1, 4), "heads": rng.choice((5, 8, 10, 16, 20, 24)),
                "n_q": _log_int(rng, 64, 8192), "n_kv": _log_int(rng, 77, 8192), "dtype": "bf16"}
    if kind == "stage":
        cfg = rng.choice((synth.CFG5A, synth.CFG5B))
        return dict(_stage(None, cfg, blocks=rng.randint(2, 6), tokens=_log_int(rng, 200, 16384), batch=rng.randint(1, 3),
                           n_ctx=rng.choice((77, 77, 154))))
    if kind == "f32":
        heads = rng.choice((4, 6, 8, 12))
        return _branch(None, rng.choice(("branch", "step")), synth.CFG1, blocks=rng.randint(1, 4), hidden=64 * heads, heads=heads,
                       latent_hw=2 * _log_int(rng, 4, 28), latent_c=rng.choice((4, 16)), n_txt=rng.randint(1, 154),
                       ctx_dim=rng.choice((256, 2048)))
    heads = rng.choice((12, 18, 24, 24, 24))
    # (a step's branches have to differ by more than the rounding of bf16: with few blocks the text reaches little)
    c = _branch(None, kind, synth.CFG2, blocks=rng.randint(4 if kind == "step" else 1, 6), hidden=64 * heads, heads=heads,
                latent_hw=2 * _log_int(rng, 12, 128), n_txt=rng.choice((77, 154, 333, 333)) + rng.choice((0, 0, 1)),
                batch=2 if kind == "step" else rng.randint(1, 4))
    if kind == "branch" and rng.random() < 0.3:
        c["pooled_dim"] = 2048
    if kind == "branch":
        c["txt_pre_only_last"] = rng.random() < 0.5
    return c


def draw(rng):
    """One more case of the ranges above, no more expensive than the listed ones of its kind."""
    while True:
        c = _draw_once(rng)
        c.pop("name", None)
        w = work(c)
        cap = 2e11 if c["dtype"] == "f32" else 8e12
        if w["flops"] <= cap and w["bytes"] <= 8e8 + 3e9 * (c["kind"] in ("branch", "step", "stage")):
            return c


def _cfg(case):
    if case["kind"] == "stage":
        return synth.SDXLStageConfig("case", blocks=case["blocks"], tokens=case["tokens"], channels=case["channels"],
                                     heads=case["heads"], n_ctx=case["n_ctx"], ctx_dim=case["ctx_dim"],
                                     batch=case["batch"], dtype=case["dtype"])
    return synth.MMDiTConfig("case", blocks=case["blocks"], hidden=case["hidden"], heads=case["heads"],
                             latent_hw=case["latent_hw"], latent_c=case["latent_c"], n_txt=case["n_txt"],
                             ctx_dim=case["ctx_dim"], batch=case["batch"], dtype=case["dtype"],
                             pooled_dim=case["pooled_dim"])


class _Draws:
    """Seeded normal numbers made on the GPU, rounded once to the precision of the workload; handed to the model
    classes as host arrays, which is what their constructors take."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.dtype = DT[dtype]

    def dev(self, shape, std=1.0, mean=0.0):
        t = torch.randn(shape, generator=self.g, device="cuda")
        return t.mul_(std).add_(mean).to(self.dtype).float()

    def tokens(self, shape):
        """Text features [batch, tokens, width]: the tokens of one prompt share half of their variance, as the outputs of
        a text encoder do (with independent tokens attention would average the prompt away, and the two branches of
        a guided step would differ by less than the rounding of bf16)."""
        return (self.dev((shape[0], 1, shape[2]), math.sqrt(0.5)) + self.dev(shape, math.sqrt(0.5))).to(self.dtype).float()

    def host(self, shape, std=0.02, mean=0.0):
        return self.dev(shape, std, mean).cpu().numpy()


def _mmdit(case, d):
    cfg = _cfg(case)
    D = cfg.hidden
    shapes = {"pe_w": (D, cfg.patch_dim), "pe_b": (D,), "ce_w": (D, cfg.ctx_dim), "ce_b": (D,), "t1_w": (D, cfg.temb_dim),
              "t1_b": (D,), "t2_w": (D, D), "t2_b": (D,), "f_ada_w": (2 * D, D), "f_ada_b": (2 * D,),
              "f_w": (cfg.patch_dim, D), "f_b": (cfg.patch_dim,), "pos": (cfg.n_img, D)}
    if cfg.pooled_dim:
        shapes.update({"p1_w": (D, cfg.pooled_dim), "p1_b": (D,), "p2_w": (D, D), "p2_b": (D,)})
    block = {"ada_w": (6 * D, D), "ada_b": (6 * D,), "qkv_w": (3 * D, D), "qkv_b": (3 * D,), "out_w": (D, D), "out_b": (D,),
             "fc1_w": (4 * D, D), "fc1_b": (4 * D,), "fc2_w": (D, 4 * D), "fc2_b": (D,)}
    globals_np = {n: d.host(s) for n, s in shapes.items()}
    # Two different blocks, alternating: every block still has its own copy of its weights on the GPU.
    two = [{s: {n: d.host(sh) for n, sh in block.items()} for s in ("img", "txt")} for _ in range(min(2, cfg.blocks))]
    return cfg, model.MMDiT(cfg, globals_np, (two[i % 2] for i in range(cfg.blocks)),
                            txt_pre_only_last=case["txt_pre_only_last"])


def _sdxl(case, d):
    cfg = _cfg(case)
    C, X = cfg.channels, cfg.ctx_dim
    shapes = {"q1_w": (C, C), "k1_w": (C, C), "v1_w": (C, C), "o1_w": (C, C), "o1_b": (C,), "q2_w": (C, C), "k2_w": (C, X),
              "v2_w": (C, X), "o2_w": (C, C), "o2_b": (C,), "ff1_w": (8 * C, C), "ff1_b": (8 * C,), "ff2_w": (C, 4 * C),
              "ff2_b": (C,)}
    shapes.update({n + s: (C,) for n in ("gn", "ln1", "ln2", "ln3") for s in ("_g", "_b")})
    two = [{n: d.host(sh, mean=1.0 if n.endswith("_g") else 0.0) for n, sh in shapes.items()} for _ in range(min(2, cfg.blocks))]
    return cfg, model.SDXLStage(cfg, (two[i % 2] for i in range(cfg.blocks)))


def prepare(case, seed):
    kind = case["kind"]
    d = _Draws(seed, case["dtype"])
    if kind == "guidance":
        # branch velocities that differ by a tenth, as conditional and unconditional predictions do; fp32 latent
        B, n, dt = case["batch"], case["elems"], DT[case["dtype"]]
        v_u = d.dev((B, n))
        v_c = (v_u + 0.1 * d.dev((B, n))).to(dt)
        x = torch.randn((B, n), generator=d.g, device="cuda")
        return {"kind": kind, "v_c": v_c, "v_u": v_u.to(dt), "x": x, "x_out": torch.empty_like(x),
                "l1": torch.empty(B, device="cuda"), "l2": torch.empty(B, device="cuda"),
                "ws": torch.empty(max(hb.hyb_discrepancy_workspace_bytes(B, n), 256), device="cuda", dtype=torch.uint8)}
    if kind == "attention":
        B, H, dt = case["batch"], case["heads"], DT[case["dtype"]]
        q, k, v = (d.dev((B, H, case[n], 64)).to(dt) for n in ("n_q", "n_kv", "n_kv"))
        return {"kind": kind, "q": q, "k": k, "v": v, "o": torch.empty(B, case["n_q"], H * 64, device="cuda", dtype=dt)}
    if kind == "stage":
        cfg, st = _sdxl(case, d)
        return {"kind": kind, "stage": st, "x": d.dev((cfg.batch, cfg.tokens, cfg.channels)),
                "ctx": d.tokens((cfg.batch, cfg.n_ctx, cfg.ctx_dim))}
    cfg, m = _mmdit(case, d)
    ctx = d.tokens((cfg.batch, cfg.n_txt, cfg.ctx_dim))
    if kind == "step":
        return {"kind": kind, "sampler": model.GuidedSampler(m, cfg.guidance), "ctx": ctx,
                "x": d.dev((cfg.latent_hw, cfg.latent_hw, cfg.latent_c))}
    return {"kind": kind, "model": m, "ctx": ctx, "latent": d.dev((cfg.batch, cfg.latent_hw, cfg.latent_hw, cfg.latent_c)),
            "t": torch.full((cfg.batch,), 0.5, device="cuda"), "pooled": d.dev((cfg.batch, cfg.pooled_dim)) if cfg.pooled_dim else None}


def run(state):
    kind = state["kind"]
    if kind == "guidance":
        hb.hyb_cfg_disc_euler(state["v_c"], state["v_u"], state["x"], state["x_out"], 7.0, 0.5, 0.45, state["l1"], state["l2"],
                              state["ws"])
        return state["x_out"], state["l1"], state["l2"]
    if kind == "attention":
        return hb.hyb_joint_attention(state["q"], state["k"], state["v"], state["o"])
    if kind == "stage":
        return state["stage"].forward(state["x"], state["ctx"])
    if kind == "step":
        s = state["sampler"]
        s.step(state["x"], state["ctx"], 0.5, 0.45)
        return state["x"], s.disc[:, :1]
    return state["model"].forward(state["latent"], state["ctx"], state["t"], state["pooled"])


def work(case):
    kind, es = case["kind"], 4 if case["dtype"] == "f32" else 2
    B = case["batch"]
    if kind == "guidance":
        n = B * case["elems"]
        return {"bytes": n * (2 * es + 8), "flops": 12 * n}
    if kind == "attention":
        H, nq, nk = case["heads"], case["n_q"], case["n_kv"]
        return {"bytes": B * H * 64 * es * (2 * nq + 2 * nk), "flops": 4 * B * H * nq * nk * 64}
    cfg = _cfg(case)
    if kind == "stage":
        C, X = cfg.channels, cfg.ctx_dim
        weights = cfg.blocks * (18 * C * C + 2 * C * X) * es
        return {"bytes": weights + B * (8 * cfg.tokens * C + 4 * cfg.n_ctx * X), "flops": B * cfg.flops_per_sample()}
    D, N = cfg.hidden, cfg.n_img + cfg.n_txt
    streams = 2 if cfg.n_txt else 1
    weights = cfg.blocks * (streams * 12 + 12) * D * D + D * (2 * cfg.patch_dim + cfg.ctx_dim + cfg.temb_dim + 3 * D)
    weights += D * (cfg.pooled_dim + D) if cfg.pooled_dim else 0
    flops = B * cfg.flops_per_sample()
    if case["txt_pre_only_last"]:    # no text queries, output projection and MLP in the last block
        flops -= B * (20 * D * D * cfg.n_txt + 4 * cfg.n_txt * N * D)
    latent = cfg.latent_elems * (4 + es) * B
    return {"bytes": weights * es + 4 * D * cfg.n_img + latent + 4 * B * (cfg.n_txt * cfg.ctx_dim + cfg.pooled_dim), "flops": flops}


def tolerance(case):
    """Measured against the same path in fp32 (bf16 cases), with inputs moved by a part in 1e7 (fp32) and, for the sums
    of the guidance pass, against another order of addition; about four times what was seen."""
    if case["kind"] == "guidance":
        return {"rel": 1e-6}
    if case["dtype"] == "f32":      # 2.7e-7 on velocities; 2.6e-6 on a step's discrepancies, ratios of small differences
        return {"rel": 1e-5 if case["kind"] == "step" else 2e-6}
    if case["kind"] == "stage":     # 1.0e-3 (the residual stream carries most of the result)
        return {"rel": 4e-3}
    return {"rel": 1e-2}            # 3.7e-3 on velocities, 2.3e-3 on attention rows; discrepancies of a step likewise
