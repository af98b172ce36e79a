"""GPU parity of the decode kernels' shapes (16 x 16 and 32 x 32 products, 4, 8
and 16 waves per tile, per-wave and shared activation rings, 1 to 3 weight
tiles) on either side of the dispatch rules, against the CPU oracle: the plain GEMM, the fused
quantize + GEMM (which must sum in the same order) and the gate epilogue."""

import numpy as np
import pytest
import torch

from oracle import gates as OGT
from oracle import gemm as OG
from oracle import quant as OQ
from paper_2609_04098_amd import linear as L
from paper_2609_04098_amd import synth
from tests.gpu_common import bf16_rne_of, check_gemm, log, to_dev_bf16

pytestmark = pytest.mark.gpu


def _inputs(m, n, k):
    rng = np.random.default_rng(m * 17 + n * 3 + k)
    x = rng.standard_normal((m, k))
    x[:, rng.choice(k, max(1, k // 200), replace=False)] *= 100.0
    return synth.f64_to_bf16_bits(x), synth.f64_to_bf16_bits(rng.standard_normal((n, k)) * 0.02)


def _check(m, n, k, offs):
    xb, wb = _inputs(m, n, k)
    x, pw = to_dev_bf16(xb), L.pack_weight(to_dev_bf16(wb), offs)
    aq = L.quantize_act(x)
    y32 = L.gemm(aq, pw, out_dtype=torch.float32)
    y16 = L.gemm(aq, pw)
    act = L.alloc_act(m, k, x.device)
    f32, _ = L.quantize_gemm(x, pw, out_dtype=torch.float32, act_out=act)
    s32, _ = L.quantize_gemm(x, pw, g=float(aq.g.item()), out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert torch.equal(act.codes, aq.codes) and torch.equal(act.scales, aq.scales) and torch.equal(act.g, aq.g)
    assert torch.equal(f32, y32) and torch.equal(s32, y32), "fused and unfused sums differ"
    xp, xs, gx = OQ.quantize_tensor(xb)
    wp, ws, gw = OQ.quantize_segments(wb, offs)
    check_gemm(y32.cpu().numpy().astype(np.float64), OG.gemm_f64(xp, xs, gx, wp, ws, gw, offs),
               OG.abs_bound(xp, xs, gx, wp, ws, gw, offs), "%dx%dx%d" % (m, n, k))
    np.testing.assert_array_equal(y16.view(torch.int16).cpu().numpy().view(np.uint16), bf16_rne_of(y32))
    log("%dx%dx%d: %s" % (m, n, k, L.gemm_kernels(m, n, k)))


@pytest.mark.parametrize("m,n,k,offs", [
    (1, 200, 64, [0, 200]),                # one chunk for 16 waves
    (3, 290, 5120, [0, 100, 290]),         # one launch (fused quantizer), 80 chunks over 16 waves
    (16, 8192, 1088, [0, 4096, 8192]),     # one tile per CU, 17 chunks over 16 waves, most rows of 16 x 16 products
    (17, 8192, 512, [0, 8192]),            # the fewest rows of 32 x 32 products
    (16, 8193, 512, [0, 8193]),            # one tile past one per CU: two tiles for 8 waves, ragged N
    (2, 14720, 320, [0, 14720]),           # 460 tiles: the most in twos, 5 chunks over 8 waves, one launch
    (9, 14721, 320, [0, 9999, 14721]),     # 461 tiles: the fewest in threes
    (16, 24576, 1088, [0, 24576]),         # 768 tiles: a workgroup of three per CU
    (16, 24577, 1088, [0, 24577]),         # one more: two tiles for 8 waves
    (15, 24609, 1088, [0, 24609]),         # ... and at the one-launch limit (M K = 16320)
    (16, 32769, 1088, [0, 9999, 32769]),   # past four per CU: two tiles for 4 waves
    (15, 32800, 1088, [0, 32800]),         # ... in one launch three tiles for 8 waves
    (2, 49153, 320, [0, 49153]),           # past six per CU: two tiles for 8 waves
    (17, 8193, 512, [0, 8193]),            # one tile past one per CU: two tiles for 8 waves, one launch
    (17, 14720, 1024, [0, 14720]),         # the most in twos
    (32, 14721, 192, [0, 9999, 14721]),    # the fewest in threes, 3 chunks over 8 waves
    (18, 24577, 576, [0, 24577]),          # two tiles for 4 waves, one launch, ragged N
    (32, 24700, 1088, [0, 24700]),
    (18, 32769, 576, [0, 32769]),          # past four tiles per CU: five tiles for 4 waves
    (32, 32900, 320, [0, 30000, 32900]),
    (17, 40961, 128, [0, 40961]),          # past five tiles per CU: two tiles for 4 waves
    (1, 160, 8192, [0, 160]),              # long K, one launch
    (8, 170, 8256, [0, 85, 170]),          # long K: 129 chunks over 16 waves
    (20, 170, 8192, [0, 170]),             # long K, more rows: shared ring of 4 stages
    (32, 140, 17408, [0, 140]),
])
def test_decode_shapes(m, n, k, offs):
    _check(m, n, k, offs)


# Up to M K = 16384 one launch of the plain decode kernel's form; past it the fused
# launch has 4 waves, or 8 from K = 2048 on.
@pytest.mark.parametrize("k", [64, 960, 1088, 1984, 2048, 5120, 8192])
@pytest.mark.parametrize("n", [97, 128])
@pytest.mark.parametrize("m", [1, 16, 17, 32])
def test_decode_shapes_of_up_to_four_column_tiles(m, n, k):
    _check(m, n, k, [0, 40, n])


@pytest.mark.parametrize("n,k,name", [
    (24579, 12224, "gemm_rows16_kernel<8,2,2>"),    # M K = 195584
    (24579, 12352, "gemm_rows16_kernel<4,2,3>"),    # 197632
    (49155, 12224, "gemm_rows16_kernel<8,2,2>"),    # past six tiles per CU
    (49155, 12352, "gemm_splitk_kernel<4,1,2,3>"),  # ... 32-row tiles
])
def test_decode_shapes_wide_output_and_long_k(n, k, name):
    """On either side of the length of X from which the 8-wave forms are left; Y
    at a sample of the columns, the last ones among them."""
    m = 16
    gen = torch.Generator(device="cuda").manual_seed(k)
    w = torch.randn(n, k, generator=gen, device="cuda", dtype=torch.bfloat16) * 0.02
    xb = _inputs(m, 16, k)[0]
    pw = L.pack_weight(w)
    cols = np.unique(np.concatenate([np.random.default_rng(k).choice(n, 90, replace=False), np.arange(n - 6, n)]))
    wb = w[torch.from_numpy(cols).cuda()].view(torch.int16).cpu().numpy().view(np.uint16)
    del w
    y32, y16 = (L.gemm(L.quantize_act(to_dev_bf16(xb)), pw, out_dtype=t) for t in (torch.float32, torch.bfloat16))
    xp, xs, gx = OQ.quantize_tensor(xb)
    gw = pw.g_seg.cpu().numpy()
    wp, ws, _ = OQ.quantize_tensor(wb, g=gw[0])
    args = (xp, xs, gx, wp, ws, gw, [0, len(cols)])
    check_gemm(y32.cpu().numpy().astype(np.float64)[:, cols], OG.gemm_f64(*args), OG.abs_bound(*args), "k=%d" % k)
    np.testing.assert_array_equal(y16.view(torch.int16).cpu().numpy().view(np.uint16), bf16_rne_of(y32))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert L.gemm_kernels(m, n, k)[0].startswith(name)


@pytest.mark.parametrize("m,n,k,offs", [
    (5, 96, 5120, [0, 48, 96]),
    (33, 64, 320, [0, 64]),                # 5 chunks over 8 waves, two row tiles
    (2720, 90, 192, [0, 30, 90]),          # 85 x 3 tiles: one fragment per tile
    (2721, 90, 192, [0, 30, 90]),          # 86 x 3 tiles would not fit the CUs: two fragments
    (4097, 96, 128, [0, 48, 96]),          # three fragments
    (8192, 96, 64, [0, 48, 96]),           # one tile per CU
    (8193, 96, 192, [0, 48, 96]),          # two 32 x 96 tiles of 4 waves per CU
    (8200, 70, 2048, [0, 70]),             # ... long K: 64 x 96 tiles; fused, 32 x 96
    (16384, 90, 64, [0, 90]),
    (16385, 90, 64, [0, 90]),              # 64 x 96 tiles for both
])
def test_narrow_shapes(m, n, k, offs):
    _check(m, n, k, offs)


@pytest.mark.parametrize("m,k", [
    (1, 576), (70, 576), (3000, 576), (6000, 576),
    (8200, 576),                           # two 32 x 96 tiles of 4 waves per CU
    (8200, 8256),                          # ... up to K = 8192
])
def test_gate_epilogue_shapes(m, k):
    h = 48
    xb, wb = _inputs(m, 2 * h, k)
    rng = np.random.default_rng(m)
    a_log, dt = np.log(rng.uniform(1, 16, h)).astype(np.float32), rng.uniform(-4, 2, h).astype(np.float32)
    aq, pw = L.quantize_act(to_dev_bf16(xb)), L.pack_weight(to_dev_bf16(wb), [0, h, 2 * h])
    y = L.gemm_gdn_gates(aq, pw, torch.from_numpy(a_log).cuda(), torch.from_numpy(dt).cuda(), out_dtype=torch.float32)
    v = L.gemm(aq, pw, out_dtype=torch.float32).cpu().numpy().astype(np.float64)
    # The gate of the kernel's own product: alpha = exp(g) has a relative error
    # of |g| times a few ulps of binary32, below 100 * 8 * 2^-24 = 5e-5 while
    # alpha is above 1e-38.
    np.testing.assert_allclose(y.cpu().numpy(), OGT.gdn_gates(v, a_log, dt), rtol=1e-4, atol=1e-30)


@pytest.mark.parametrize("m,k,ldx", [
    (1, 16, None),                          # one block
    (64, 256, None),                        # 1024 blocks: one workgroup, its own blocks are all of X
    (41, 400, 416),                         # 1025 blocks, strided rows: two workgroups
    (600, 32, 40),                          # strided: a step of the walk is whole rows
    (3, 17408, 17424),                      # ... less than a row
    (100, 1040, 1056),                      # ... and rows and a part, seven workgroups
    (32, 4096, None),                       # 8192 blocks: the largest one-launch activation
    (8193, 16, 24),                         # 8193 blocks: two launches
])
def test_one_launch_quantizer_limits(m, k, ldx):
    rng = np.random.default_rng(m + k)
    for where in (0, m - 1):                # the maximum in the first or the last block
        x = rng.standard_normal((m, k))
        x[where, -1 if where else 0] = -300.0
        xb = synth.f64_to_bf16_bits(x)
        buf = np.full((m, ldx or k), 0x7F00, dtype=np.uint16)      # padding far above the maximum
        buf[:, :k] = xb
        xd = to_dev_bf16(buf)[:, :k]
        xp, xs, gx = OQ.quantize_tensor(xb)
        for g in (None, gx):
            aq = L.quantize_act(xd, g=g)
            assert np.float32(aq.g.item()) == gx
            np.testing.assert_array_equal(aq.codes.cpu().numpy(), xp)
            np.testing.assert_array_equal(aq.scales.cpu().numpy(), xs)
