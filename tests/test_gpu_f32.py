"""GPU parity of the fp32 MFMA kernels (GEMM with its two tile shapes, attention) against float64 on the CPU."""
import numpy as np
import pytest
import torch

from oracle import hyb_oracle as O
from paper_2602_21760_amd import synth
from gpu_util import dev, host, err

pytestmark = pytest.mark.gpu

# fp32 products summed in fp32: the relative error of a row stays below sqrt(k) 2^-24, 3.3e-6 at k = 3072; attention adds
# its exponentials (1.5 ulp each, test_attention_f32_exponentials; arguments below 2^4: 1e-6).
TOL = 4e-6


@pytest.fixture(scope="module")
def hb():
    from paper_2602_21760_amd import binding
    binding.lib()
    return binding


def _traced(hb, call):
    hb.hyb_trace_enable(True)
    call()
    names = hb.hyb_trace_summary()
    hb.hyb_trace_enable(False)
    return list(names)


# 32 x 32 tiles, and 64 x 64 ones for the two shapes of more than 4000 rows (the 64 x 64 tiles have their own test below): one row, ragged
# rows and columns around the tile sizes, one slab of k, fewer slabs than waves, an odd number of slabs, long k; half a slab;
# n % 4 != 0 and k % 16 != 0 take the plain kernel
@pytest.mark.parametrize("m,n,k", [(1, 4, 32), (2, 256, 96), (31, 36, 160), (33, 28, 64), (65, 100, 1056), (653, 768, 3072),
                                   (4097, 2052, 64), (100, 40, 16), (70, 64, 112), (4100, 2048, 80), (40, 30, 64), (40, 32, 72)])
def test_linear_f32(hb, m, n, k):
    g = torch.Generator().manual_seed(m + n + k)
    a, w, b = (torch.randn(s, generator=g).numpy() for s in ((m, k), (n, k), (n,)))
    res, gate = torch.randn(m, n, generator=g).numpy(), torch.randn(2, n + 4, generator=g).numpy()
    y = O.linear(a.astype(np.float64), w.astype(np.float64), b.astype(np.float64))
    da, dw, db = dev(a), dev(w), dev(b)
    out = torch.empty(m, n, device="cuda")
    hb.hyb_linear(da, dw, db, out)
    assert err(host(out), y) < TOL
    whole = host(out)
    hb.hyb_linear(da[m // 2:m // 2 + 1].clone(), dw, db, out[:1])
    if n % 4 == 0 and k % 16 == 0:      # a row has the same bits whatever the tile shape and the rows beside it
        assert np.array_equal(host(out[:1])[0], whole[m // 2])
    dres, rpg = dev(res), (m + 1) // 2
    if n % 4 == 0:
        hb.hyb_linear(da, dw, db, dres, hb.HYB_EPI_GATE_RESIDUAL, residual=dres, gate=dev(gate), rows_per_gate=rpg, gate_stride=n + 4)
        assert err(host(dres), res + gate[np.arange(m) // rpg, :n].astype(np.float64) * y) < TOL
    if n % 8 == 0:                      # u and gate halves of the same weights
        out = torch.empty(m, n // 2, device="cuda")
        hb.hyb_linear(da, dw, db, out, hb.HYB_EPI_GEGLU)
        u, v = torch.from_numpy(y).chunk(2, 1)
        assert err(host(out), (u * torch.nn.functional.gelu(v)).numpy()) < TOL


# keys: fewer than one tile, exactly one, one more, fewer tiles than waves, ragged; queries around the 32-row blocks
@pytest.mark.parametrize("batch,heads,n_q,n_kv", [(1, 1, 1, 1), (2, 3, 31, 32), (1, 5, 33, 33), (2, 4, 80, 80), (1, 2, 64, 129), (2, 8, 97, 653)])
def test_attention_f32(hb, batch, heads, n_q, n_kv):
    g = torch.Generator().manual_seed(n_q + n_kv)
    q, k, v = (torch.randn(batch, heads, n, 64, generator=g) for n in (n_q, n_kv, n_kv))
    o = torch.empty(batch, n_q, heads * 64, device="cuda")
    hb.hyb_joint_attention(q.cuda(), k.cuda(), v.cuda(), o)
    ref = torch.softmax(q.double() @ k.double().transpose(2, 3) / 8, -1) @ v.double()
    assert err(host(o), ref.transpose(1, 2).reshape(batch, n_q, -1).numpy()) < TOL
    # scores of several hundred, largest in the first key or growing along the keys
    for ramp in (torch.arange(n_kv, 0, -1), torch.arange(1, n_kv + 1)):
        kr = k * (1 + 40 * ramp / n_kv).view(1, 1, -1, 1)
        hb.hyb_joint_attention(q.cuda(), kr.cuda(), v.cuda(), o)
        ref = torch.softmax(q.double() @ kr.double().transpose(2, 3) / 8, -1) @ v.double()
        assert err(host(o), ref.transpose(1, 2).reshape(batch, n_q, -1).numpy()) < 40 * TOL   # the exponents' rounding, 40 times larger


def test_attention_f32_more_blocks_than_one_grid_dimension_holds(hb):
    """65535 samples of 257 heads are more than 2^24 workgroups of 256 threads; with one key the output is its value, exactly."""
    q, k = (torch.zeros(65535, 257, 1, 64, device="cuda") for _ in range(2))
    v = torch.randn(65535, 257, 1, 64, device="cuda")
    o = torch.full((65535, 1, 257 * 64), float("nan"), device="cuda")
    hb.hyb_joint_attention(q, k, v, o)
    assert torch.equal(o.view(-1), v.view(-1))


def test_linear_f32_more_tiles_than_one_grid_dimension_holds(hb):
    """65535 x 257 tiles are more than 2^24 workgroups of 256 threads.  (69 GB of output, the least that this many tiles can have here.)"""
    m, n, k = 65535 * 64, 8196, 16
    a, w = torch.randn(m, k, device="cuda"), torch.randn(2 * n, k, device="cuda")
    out = torch.empty(m, n, device="cuda", dtype=torch.bfloat16)
    hb.hyb_linear(a, w, None, out, hb.HYB_EPI_GEGLU)
    rows = torch.tensor([0, 63, 64, m // 2, m - 65, m - 1], device="cuda")
    u, v = (a[rows].double() @ w.double().t()).chunk(2, 1)
    assert err(host(out[rows]), (u * torch.nn.functional.gelu(v)).cpu().numpy()) < 4e-3


def test_geglu_f32_tile_shape_counts_its_own_columns(hb):
    """A GEGLU tile has half as many output columns as the others: 1000 x 508 is one round of 64 x 64 tiles, 1000 x 380 (192 tiles) leaves a
    quarter of the chip idle that 32 x 32 tiles fill."""
    a, w = torch.randn(1000, 32, device="cuda"), torch.randn(1016, 32, device="cuda")
    for n, shape in ((508, "64x64"), (380, "32x32")):
        out = torch.empty(1000, n, device="cuda")
        names = _traced(hb, lambda: hb.hyb_linear(a, w[:2 * n], None, out, hb.HYB_EPI_GEGLU))
        assert names == ["gemm_f32_mfma_%s.epi5.n%d.k32" % (shape, n)], names


# Shapes whose 64 x 64 tiles fill whole rounds of 256 CUs, so that the dispatch takes them: one slab of k and less, fewer slabs than
# running sums, 4 q + 1 of them, half last slabs, ragged rows and columns, long k.
@pytest.mark.parametrize("m,n,k", [(1000, 1020, 16), (1000, 1020, 32), (961, 1012, 48), (961, 1012, 64), (2040, 508, 80), (2040, 508, 96),
                                   (4090, 252, 160), (1000, 1000, 272), (16370, 60, 288), (1306, 768, 3072)])
def test_linear_f32_64x64_tiles(hb, m, n, k):
    g = torch.Generator().manual_seed(m + n + k)
    nh = n // 8 * 4                                  # GEGLU outputs: u and gate rows of one weight matrix
    a, w, b = (torch.randn(s, generator=g) * f for s, f in (((m, k), 1), ((n, k), k ** -0.5), ((n,), 1)))
    res, gate = torch.randn(m, n, generator=g), torch.randn(2, n, generator=g)
    da, dw, db = a.cuda(), w.cuda(), b.cuda()
    y = torch.from_numpy(O.linear(a.double().numpy(), w.double().numpy(), b.double().numpy()))
    u, v = y[:, :nh], y[:, nh:2 * nh]
    F = torch.nn.functional
    rpg = (m + 1) // 2
    cases = [(hb.HYB_EPI_BIAS, n, {}, y), (hb.HYB_EPI_GELU_TANH, n, {}, F.gelu(y, approximate="tanh")), (hb.HYB_EPI_SILU, n, {}, F.silu(y)),
             (hb.HYB_EPI_GATE_RESIDUAL, n, dict(residual=res.cuda(), gate=gate.cuda(), rows_per_gate=rpg, gate_stride=n),
              res + gate.double()[torch.arange(m) // rpg] * y),
             (hb.HYB_EPI_GEGLU, nh, {}, u * F.gelu(v))]
    for epi, cols, kw, ref in cases:
        out, one = torch.empty(m, cols, device="cuda"), torch.empty(1, cols, device="cuda")
        rows = 2 * nh if epi == hb.HYB_EPI_GEGLU else n
        names = _traced(hb, lambda: hb.hyb_linear(da, dw[:rows], db[:rows], out, epi, **kw))
        assert names == ["gemm_f32_mfma_64x64.epi%d.n%d.k%d" % (epi, cols, k)], names
        assert err(host(out), ref.numpy()) < TOL, epi
        # the 32 x 32 tiles, which a single row takes, give the same bits
        r = m // 2
        if kw:
            kw = dict(kw, residual=kw["residual"][r:r + 1], gate=kw["gate"][r // rpg:])
        names = _traced(hb, lambda: hb.hyb_linear(da[r:r + 1].clone(), dw[:rows], db[:rows], one, epi, **kw))
        assert names == ["gemm_f32_mfma_32x32.epi%d.n%d.k%d" % (epi, cols, k)], names
        assert torch.equal(one[0], out[r]), epi
    low = torch.empty(m, n, device="cuda", dtype=torch.bfloat16)
    hb.hyb_linear(da, dw, db, low)
    assert err(host(low), y.numpy()) < 4e-3          # one rounding to bf16: 2^-8 at most, half of it in the mean square


@pytest.mark.parametrize("k", [16, 32, 48, 96, 128, 144, 160, 240, 256, 1040])
def test_linear_f32_64x64_tiles_four_buffers(hb, k):
    """A launch with one 64 x 64 tile per CU runs with four slab buffers, one of twice the rows with two: the same bits, from less than one slab
    to more than the buffers hold, and the oracle's results."""
    m, n = 1000, 1020
    g = torch.Generator().manual_seed(k)
    a, w, b, res = torch.randn(m, k, generator=g), torch.randn(n, k, generator=g) * k ** -0.5, torch.randn(n, generator=g), torch.randn(m, n, generator=g)
    da, dw, db, dr = a.cuda(), w.cuda(), b.cuda(), res.cuda()
    one, two = torch.empty(m, n, device="cuda"), torch.empty(2 * m, n, device="cuda")
    hb.hyb_linear(da, dw, db, one, hb.HYB_EPI_GATE_RESIDUAL, residual=dr)
    names = _traced(hb, lambda: hb.hyb_linear(da.repeat(2, 1), dw, db, two, hb.HYB_EPI_GATE_RESIDUAL, residual=dr.repeat(2, 1)))
    assert names == ["gemm_f32_mfma_64x64.epi%d.n%d.k%d" % (hb.HYB_EPI_GATE_RESIDUAL, n, k)], names
    assert torch.equal(two.view(2, m, n), one.expand(2, m, n))
    assert err(host(one), res.numpy() + O.linear(a.double().numpy(), w.double().numpy(), b.double().numpy())) < TOL


@pytest.mark.parametrize("m,n,k,geglu,tiles", [(1060, 764, 768, False, "64x64"), (1088, 768, 4096, False, "64x64"), (890, 896, 1024, False, "64x64"), (1088, 384, 1024, True, "32x32"),
                                               (1024, 768, 1024, False, "32x32")])
def test_linear_f32_single_round_that_leaves_cus_idle(hb, m, n, k, geglu, tiles):
    """A round of 193-217 tiles of 64 x 64 with a long k: large tiles where they have four slab buffers, small ones for GEGLU (two buffers) and for
    192 tiles; the oracle's results, and the same rows the same bits in a launch of eight times as many."""
    g = torch.Generator().manual_seed(m + k)
    wide = 2 if geglu else 1
    a, w, b = torch.randn(m, k, generator=g), torch.randn(wide * n, k, generator=g) * k ** -0.5, torch.randn(wide * n, generator=g)
    da, dw, db = a.cuda(), w.cuda(), b.cuda()
    out, many = torch.empty(m, n, device="cuda"), torch.empty(8 * m, n, device="cuda")
    epi = hb.HYB_EPI_GEGLU if geglu else hb.HYB_EPI_BIAS
    names = _traced(hb, lambda: hb.hyb_linear(da, dw, db, out, epi))
    assert names == ["gemm_f32_mfma_%s.epi%d.n%d.k%d" % (tiles, epi, n, k)], names
    y = O.linear(a.double().numpy(), w.double().numpy(), b.double().numpy())
    assert err(host(out), y[:, :n] * O.gelu_erf(y[:, n:]) if geglu else y) < TOL
    hb.hyb_linear(da.repeat(8, 1), dw, db, many, epi)
    assert torch.equal(many.view(8, m, n), out.expand(8, m, n))


def test_qkv_scatter_f32_64x64_tiles(hb):
    """The head-major scatter from the 64 x 64 tiles: an fp32 block of two samples with ragged image and text rows, 252 tiles."""
    from test_gpu_block import _block_case
    cfg = synth.scaled(synth.CFG1, hidden=128, heads=2, latent_hw=72, n_txt=25, ctx_dim=64, batch=2)
    got = []
    names = _traced(hb, lambda: got.append(_block_case(hb, cfg)))
    assert "gemm_f32_mfma_64x64.epi4.n384.k128" in names, names
    g_img, g_txt, r_img, r_txt, (x_img, x_txt) = got[0]
    assert err(g_img - x_img, r_img - x_img) < 1e-4 and err(g_txt - x_txt, r_txt - x_txt) < 1e-4


def test_attention_f32_exponentials(hb):
    """Two keys with scores 0 and -x and values 0 and 1: the output is p / (1 + p), p = e^-x, over the whole range of the exponential, the
    subnormal numbers included.  Bounds: 1.5 ulp (2^-23 each) of the exponential, half an ulp each for sum and quotient; below 2^-126
    the spacing of the subnormal numbers, 2^-149, takes the ulp's place."""
    n = 1 << 16
    x = torch.linspace(0, 104, n, dtype=torch.float64).float()
    q, k, v = torch.zeros(1, 1, n, 64), torch.zeros(1, 1, 2, 64), torch.zeros(1, 1, 2, 64)
    q[0, 0, :, 5], k[0, 0, 1, 5], v[0, 0, 1] = x, -1.0, 1.0
    o = torch.empty(1, n, 64, device="cuda")
    hb.hyb_joint_attention(q.cuda(), k.cuda(), v.cuda(), o, 1.0)
    ref = (1 / (1 + torch.exp(x.double())))[:, None]
    got = o[0].double().cpu()
    assert (got == got[:, :1]).all()
    off = (got[:, :1] - ref).abs()
    print("largest error in units of 2^-23: %.2f; below 2^-126 in units of 2^-149: %.2f" % (
        (off / ref)[x < 87].max() * 2 ** 23, off[x >= 87].max() * 2.0 ** 149))
    assert (off <= 2.5 * 2.0 ** -23 * ref + 1.5 * 2.0 ** -149).all()
