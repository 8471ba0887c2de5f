"""CPU-side checks of the boundary: the library builds/loads and exports every entry point that
include/hyb.h declares, and the Python binding names match the C names."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "hyb.h")
LIB = os.path.join(ROOT, "paper_2602_21760_amd", "libhyb.so")


def declared_functions():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(hyb_[a-z0-9_]+)\s*\(", src)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2602_21760_amd import build
        build.build()
    return ctypes.CDLL(LIB)


def test_header_declares_the_named_calls():
    names = declared_functions()
    for required in ("hyb_block_forward", "hyb_joint_attention", "hyb_cfg_combine", "hyb_branch_discrepancy",
                     "hyb_euler_step", "hyb_cfg_disc_euler"):
        assert required in names


def test_library_exports_every_declared_symbol(lib):
    for name in declared_functions():
        assert hasattr(lib, name), "libhyb.so does not export " + name


def test_binding_covers_every_declared_symbol():
    from paper_2602_21760_amd import binding
    for name in declared_functions():
        assert name in binding.SIGNATURES, "binding has no signature for " + name
    assert set(binding.SIGNATURES) == set(declared_functions())


def test_no_compute_calls_needed_for_queries(lib):
    lib.hyb_version.restype = ctypes.c_int
    assert lib.hyb_version() >= 100
    lib.hyb_last_error_string.restype = ctypes.c_char_p
    assert lib.hyb_last_error_string() is not None
    lib.hyb_discrepancy_workspace_bytes.restype = ctypes.c_size_t
    lib.hyb_discrepancy_workspace_bytes.argtypes = [ctypes.c_int, ctypes.c_size_t]
    assert lib.hyb_discrepancy_workspace_bytes(0, 100) == 0
    a = lib.hyb_discrepancy_workspace_bytes(1, 262144)
    b = lib.hyb_discrepancy_workspace_bytes(2, 262144)
    assert a > 0 and a % 256 == 0 and b >= 2 * a - 256


def test_argument_validation_happens_before_any_gpu_work(lib):
    """NULL / shape / dtype errors are reported by the host checks (no device needed)."""
    vp, sz, f, i = ctypes.c_void_p, ctypes.c_size_t, ctypes.c_float, ctypes.c_int
    lib.hyb_cfg_combine.argtypes = [vp, vp, vp, sz, f, i, vp]
    assert lib.hyb_cfg_combine(None, None, None, 0, 1.0, 0, None) == 0          # n == 0: no-op
    assert lib.hyb_cfg_combine(None, None, None, 16, 1.0, 0, None) == 1         # HYB_ERR_NULL
    assert lib.hyb_cfg_combine(None, None, None, 16, 1.0, 7, None) == 3         # HYB_ERR_DTYPE
    assert lib.hyb_cfg_combine(vp(24), vp(32), vp(48), 16, 1.0, 0, None) == 4   # HYB_ERR_ALIGN (not dereferenced)
    lib.hyb_joint_attention.argtypes = [vp, vp, vp, vp, i, i, i, i, i, f, i, vp]
    assert lib.hyb_joint_attention(vp(16), vp(16), vp(16), vp(16), 1, 1, 8, 8, 32, 0.0, 0, None) == 2   # head_dim
    assert lib.hyb_joint_attention(vp(16), vp(16), vp(16), vp(16), 1, 1, 8, 0, 64, 0.0, 0, None) == 2   # n_kv == 0
    assert lib.hyb_joint_attention(None, None, None, None, 1, 1, 0, 0, 64, 0.0, 0, None) == 0           # n_q == 0
    # workspace form: the query is 0 for fp32 and for shapes that are never split; the cfg 2 shape (24 heads,
    # 4429 rows: 105 query blocks per XCD on 32 CUs) wants scratch, and a short one is an error
    lib.hyb_joint_attention_workspace_bytes.restype = sz
    lib.hyb_joint_attention_workspace_bytes.argtypes = [i, i, i, i]
    assert lib.hyb_joint_attention_workspace_bytes(1, 24, 4429, 0) == 0
    assert lib.hyb_joint_attention_workspace_bytes(1, 3, 4429, 1) == 0          # pairs not a multiple of 8
    need = lib.hyb_joint_attention_workspace_bytes(1, 24, 4429, 1)
    assert need > 0 and need % 256 == 0
    lib.hyb_joint_attention_ws.argtypes = [vp, vp, vp, vp, i, i, i, i, i, f, i, vp, sz, vp]
    assert lib.hyb_joint_attention_ws(vp(16), vp(16), vp(16), vp(16), 1, 24, 4429, 4429, 64, 0.0, 1, vp(256), need - 1, None) == 5
    assert lib.hyb_joint_attention_ws(vp(16), vp(16), vp(16), vp(16), 1, 24, 4429, 4429, 64, 0.0, 1, None, 0, None) == 1
    assert lib.hyb_joint_attention_ws(None, None, None, None, 1, 1, 0, 0, 64, 0.0, 0, None, 0, None) == 0
    lib.hyb_branch_discrepancy.argtypes = [vp, vp, i, sz, i, i, vp, vp, sz, vp]
    assert lib.hyb_branch_discrepancy(vp(16), vp(16), 1, 4096, 2, 0, vp(16), vp(256), 8, None) == 5     # workspace
    assert lib.hyb_branch_discrepancy(vp(16), vp(16), 1, 4096, 3, 0, vp(16), vp(256), 1 << 20, None) == 3
    lib.hyb_last_error_string.restype = ctypes.c_char_p
    assert b"p must be" in lib.hyb_last_error_string()
    # hyb_linear: epilogue values are 0..3 and 5 (HYB_EPI_GEGLU); m == 0 is a no-op for every valid one
    lib.hyb_linear.argtypes = [vp, vp, vp, vp, i, i, i, i, i, i, vp, vp, i, sz, vp]
    for epi, want in ((0, 0), (3, 0), (5, 0), (4, 3), (6, 3), (-1, 3)):
        assert lib.hyb_linear(None, None, None, None, 0, 64, 64, 1, 1, epi, None, None, 1, 0, None) == want, epi
    assert lib.hyb_linear(None, vp(16), None, vp(16), 8, 64, 64, 1, 1, 5, None, None, 1, 0, None) == 1    # NULL a


FORWARD_ERRORS = [
    # (what is wrong, error code): a descriptor field, a weight, a buffer, a weight of one block, an argument
    ("desc.temb_dim=255", 2), ("desc.hidden=192", 2), ("desc.hidden=2112", 2), ("desc.heads=3", 2), ("desc.patch=3", 2), ("desc.dtype=7", 3), ("desc.mlp_ratio=0", 2), ("desc.batch=65536", 2),
    ("weights.t1_w=0", 1), ("weights.t2_w=8", 4), ("weights.p1_w=0", 1), ("weights.p2_b=8", 4), ("weights.pe_w=0", 1), ("weights.pe_b=8", 4), ("weights.pos=0", 1),
    ("weights.ce_w=0", 1), ("weights.ada_w=0", 1), ("weights.ada_b=0", 1), ("weights.f_w=0", 1), ("weights.f_b=8", 4), ("weights.block_weights=0", 1),
    ("buffers.t_feat=0", 1), ("buffers.t_hid=8", 4), ("buffers.pooled_act=0", 1), ("buffers.p_hid=0", 1), ("buffers.temb=0", 1), ("buffers.mod=0", 1), ("buffers.tok=0", 1),
    ("buffers.ctx_act=0", 1), ("buffers.x_img=0", 1), ("buffers.x_txt=0", 1), ("buffers.y=0", 1), ("buffers.out_tok=8", 4), ("buffers.v=0", 1), ("buffers.ws=0", 1), ("buffers.ws=8", 4),
    ("buffers.ws_bytes=1024", 5), ("block.img.qkv_w=0", 1), ("block.txt.fc2_b=0", 1), ("block.img.fc1_w=8", 4), ("args.latent=0", 1), ("args.ctx=0", 1), ("args.pooled=0", 1)]


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("wrong,code", FORWARD_ERRORS)
def test_forward_errors_come_before_any_launch(lib, wrong, code, dtype):
    """hyb_mmdit_forward finds every error before it enqueues anything: without a device a launch is an error of its own
    (HYB_ERR_LAUNCH), and the pointers here lead nowhere."""
    from paper_2602_21760_amd import binding
    lib.hyb_mmdit_forward.restype, lib.hyb_mmdit_forward.argtypes = binding.SIGNATURES["hyb_mmdit_forward"]
    some = 4096
    blocks = (binding.BlockWeights * 2)(*[binding.BlockWeights(*[binding.StreamWeights(*[some] * 8) for _ in range(2)]) for _ in range(2)])
    desc = binding.MMDiTDesc(batch=2, blocks=2, hidden=128, heads=2, mlp_ratio=4, latent_h=8, latent_w=8, latent_c=16, patch=2, n_txt=5, ctx_dim=64, temb_dim=256,
                             pooled_dim=64, dtype=dtype, ln_eps=1e-6)
    weights = binding.MMDiTWeights(*[some] * len(binding.MMDIT_WEIGHT_FIELDS), blocks)
    buffers = binding.MMDiTBuffers(*[some] * len(binding.MMDIT_BUFFER_FIELDS), 1 << 30)
    args = {"latent": some, "ctx": some, "pooled": some}
    where, field, value = re.match(r"(\w+)\.(.+)=(\d+)", wrong).groups()
    if field in ("pooled_act", "ctx_act") and dtype == 0:      # fp32 models copy only what is not aligned
        args[field.split("_")[0]] = some + 4
    if where == "args":
        args[field] = int(value) or None
    elif where == "block":
        stream, name = field.split(".")
        part = getattr(blocks[1], stream)
        names = ("qkv_w", "out_w", "fc1_w", "fc2_w", "qkv_b", "out_b", "fc1_b", "fc2_b")
        setattr(part, binding.StreamWeights._fields_[names.index(name)][0], int(value) or None)
    elif field == "block_weights":
        weights.block_weights = None
    else:
        setattr({"desc": desc, "weights": weights, "buffers": buffers}[where], field, int(value) or (None if where != "desc" else 0))
    rc = lib.hyb_mmdit_forward(ctypes.byref(desc), ctypes.byref(weights), ctypes.byref(buffers), args["latent"], 0, args["ctx"], None, 0.5, args["pooled"], 0, None)
    lib.hyb_last_error_string.restype = ctypes.c_char_p
    assert rc == code, (wrong, rc, lib.hyb_last_error_string())
    assert lib.hyb_last_error_string().startswith(b"hyb_mmdit_forward: "), lib.hyb_last_error_string()


def test_struct_layouts_match_the_header(tmp_path):
    """The ctypes structures of the binding against sizeof / offsetof of the C declarations (compiled with gcc:
    the header is plain C)."""
    import shutil
    import subprocess
    from paper_2602_21760_amd import binding
    if shutil.which("gcc") is None:
        pytest.skip("no gcc")
    structs = {"hyb_block_desc": binding.BlockDesc, "hyb_stream_weights": binding.StreamWeights,
               "hyb_block_weights": binding.BlockWeights, "hyb_sdxl_block_desc": binding.SdxlBlockDesc,
               "hyb_sdxl_block_weights": binding.SdxlBlockWeights, "hyb_switch_state": binding.SwitchState,
               "hyb_mmdit_desc": binding.MMDiTDesc, "hyb_mmdit_weights": binding.MMDiTWeights, "hyb_mmdit_buffers": binding.MMDiTBuffers}
    lines = ['#include <stdio.h>', '#include <stddef.h>', '#include "hyb.h"', 'int main(void) {']
    for cname, ct in structs.items():
        lines.append('printf("%s size %%zu\\n", sizeof(%s));' % (cname, cname))
        for fname, _ in ct._fields_:
            lines.append('printf("%s %s %%zu\\n", offsetof(%s, %s));' % (cname, fname, cname, fname))
    lines.append("return 0; }")
    src = tmp_path / "layout.c"
    src.write_text("\n".join(lines))
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-std=c99", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    got = {tuple(l.split()[:2]): int(l.split()[2]) for l in out if l}
    for cname, ct in structs.items():
        assert got[(cname, "size")] == ctypes.sizeof(ct), cname
        for fname, _ in ct._fields_:
            assert got[(cname, fname)] == getattr(ct, fname).offset, (cname, fname)


def test_forward_structs_from_dicts_of_tensors():
    """mmdit_weights / mmdit_buffers: fields by name, missing ones NULL."""
    import torch
    from paper_2602_21760_amd import binding
    blocks = (binding.BlockWeights * 1)()
    t = {n: torch.empty(8) for n in ("t1_w", "pos", "ada_b")}
    w = binding.mmdit_weights(t, blocks)
    assert (w.t1_w, w.pos, w.ada_b) == tuple(t[n].data_ptr() for n in ("t1_w", "pos", "ada_b")) and w.p1_w is None and w.f_b is None
    t = {"v": torch.empty(8), "ws": torch.empty(24, dtype=torch.uint8)}
    b = binding.mmdit_buffers(t)
    assert (b.v, b.ws, b.ws_bytes, b.t_feat) == (t["v"].data_ptr(), t["ws"].data_ptr(), 24, None)


@pytest.mark.parametrize("samples,rows,i", [(2, 2, 0), (2, 2, 5), (2, 2, 6), (2, 2, -1), (2, 2, -6), (3, 2, 1), (2, 3, 1), (1, 2, 1), (0, 2, 1), (2, 1, 1), (2, 0, 1)])
def test_step_addresses_are_those_of_the_views(monkeypatch, samples, rows, i):
    """The guidance pass of a step gets the addresses that slices of the branches and of the table have (NULL where a slice is empty), and an
    index that is not there is an error."""
    import torch
    from paper_2602_21760_amd import binding

    class OnGpu(torch.Tensor):
        is_cuda = True
    calls = []

    class Recorder:
        def hyb_cfg_disc_euler(self, *a):
            calls.append(a)
            return 0
    monkeypatch.setattr(binding, "lib", Recorder)
    monkeypatch.setattr(binding, "_stream", lambda: 0)
    v, x, disc, ws = (torch.zeros(*s).as_subclass(OnGpu) for s in ((samples, 3, 4), (3, 4), (rows, 6), (64,)))
    try:
        binding.hyb_cfg_disc_euler(v[0:1], v[1:2], x.view(1, -1), x.view(1, -1), 5.0, 0.5, 0.4, disc[0, i:i + 1], disc[1, i:i + 1], ws)
    except IndexError:
        with pytest.raises(IndexError):
            binding.cfg_disc_euler_of_branches(v, x, 5.0, 0.5, 0.4, disc, i, ws)
        assert not calls
        return
    binding.cfg_disc_euler_of_branches(v, x, 5.0, 0.5, 0.4, disc, i, ws)
    null = lambda call: [a or None if n in (0, 1, 11, 12) else a for n, a in enumerate(call)]      # noqa: E731
    assert len(calls) == 2 and null(calls[0]) == null(calls[1])


def test_pointers_of_several_tensors_are_those_of_each():
    """None (a layer without a bias) is NULL, wherever it stands; what a single tensor is refused for, several are."""
    import torch
    from paper_2602_21760_amd import binding

    class OnGpu(torch.Tensor):
        is_cuda = True
    a, b, low = (torch.zeros(4, 4).as_subclass(OnGpu) for _ in range(3))
    low = low.bfloat16()
    for tensors in ((a, b), (None, a), (a, None, b), (a[1], None)):
        assert binding._pointers(tensors, torch.float32) == [binding._p(t, torch.float32) for t in tensors]
    for bad, error in ((low, TypeError), (b.t(), ValueError), (torch.zeros(4), ValueError)):
        for tensors in ((a, bad), (a, None, bad), (bad, None)):
            with pytest.raises(error):
                binding._pointers(tensors, torch.float32)


def test_missing_library_is_an_error(monkeypatch, tmp_path):
    """No fallback: without libhyb.so the binding raises."""
    from paper_2602_21760_amd import binding
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "LIB_PATH", str(tmp_path / "absent.so"))
    with pytest.raises(Exception):
        binding.lib()
