"""GPU parity of the GEMM's small tiles (128 x 128, 64 x 256) and of tiles
split over several K parts, at the edges of the tiles and of the parts, against
the CPU oracle; tolerance as in tests/gpu_common.py (FP32 sums, any order)."""

import numpy as np
import pytest
import torch

from oracle import gemm as OG
from oracle import quant as OQ
from paper_2609_04098_amd import linear as L
from paper_2609_04098_amd import nvfp4 as C
from paper_2609_04098_amd import synth
from tests.gpu_common import bf16_rne_of, check_gemm, log, to_dev_bf16, workload

pytestmark = pytest.mark.gpu


def _case(m, n, k, offs, ldy):
    rng = np.random.default_rng(m * 13 + n * 5 + k)
    x = rng.standard_normal((m, k))
    x[:, rng.choice(k, max(1, k // 200), replace=False)] *= 100.0
    xb = synth.f64_to_bf16_bits(x)
    wb = synth.f64_to_bf16_bits(rng.standard_normal((n, k)) * 0.02)
    aq = L.quantize_act(to_dev_bf16(xb))
    pw = L.pack_weight(to_dev_bf16(wb), offs)
    need = C.nvfp4_gemm_workspace(m, n, k)
    guard = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    out = {}
    for dtype in (torch.float32, torch.bfloat16):
        big = torch.full((m + 1, ldy), -7.0, dtype=dtype, device="cuda")
        y = big[:m, :n]
        L.gemm(aq, pw, out=y, workspace=guard[:need] if need else None)
        torch.cuda.synchronize()
        assert bool((big[:m, n:] == -7.0).all()) and bool((big[m] == -7.0).all())
        out[dtype] = y.contiguous()
    assert bool((guard[need:] == 0x5A).all()), "written past the workspace"
    y_nows = L.gemm_no_workspace(aq, pw, out_dtype=torch.float32)
    xp, xs, gx = OQ.quantize_tensor(xb)
    wp, ws, gw = OQ.quantize_segments(wb, offs)
    y_ref = OG.gemm_f64(xp, xs, gx, wp, ws, gw, offs)
    r_ref = OG.abs_bound(xp, xs, gx, wp, ws, gw, offs)
    check_gemm(out[torch.float32].cpu().numpy().astype(np.float64), y_ref, r_ref, "%dx%dx%d" % (m, n, k))
    check_gemm(y_nows.cpu().numpy().astype(np.float64), y_ref, r_ref, "%dx%dx%d no workspace" % (m, n, k))
    np.testing.assert_array_equal(out[torch.bfloat16].view(torch.int16).cpu().numpy().view(np.uint16),
                                  bf16_rne_of(out[torch.float32]))
    return need, aq, pw


@pytest.mark.parametrize("m,n,k,offs,ldy", [
    (33, 97, 64, [0, 97], 97),                       # one chunk, one partial tile
    (64, 256, 320, [0, 256], 256),                   # one 64 x 256 tile, K % 256 != 0
    (65, 257, 576, [0, 100, 257], 264),              # one past a tile in both directions, 9 chunks
    (128, 128, 1024, [0, 128], 128),                 # one 128 x 128 tile
    (129, 385, 2048, [0, 128, 385], 392),            # ragged tiles, 8 groups of chunks in several K parts
    (200, 515, 4352, [0, 256, 515], 515),            # 17 groups of chunks: parts of different length, odd row stride
    (200, 320, 4416, [0, 320], 320),                 # 69 chunks, K % 256 != 0: parts of single chunks
    (100, 2600, 5120, [0, 1300, 2600], 2600),        # segment boundary inside a tile
    (40, 1000, 17408, [0, 1000], 1000),              # long K, many parts
    (600, 1100, 1280, [0, 1100], 1104),              # more rows than columns of tiles
    (1030, 770, 4352, [0, 770], 776),                # past the split-K tiles' rows: 17 groups of chunks
    (1030, 770, 4416, [0, 385, 770], 771),           #   69 chunks, no super-stages
    (1088, 260, 320, [0, 260], 260),
    (1153, 129, 1024, [0, 129], 129),
    (1100, 1500, 64, [0, 700, 1500], 1504),
    (1, 33, 16, [0, 33], 33),                        # K % 64 != 0 (padded with the workspace, register path without):
    (70, 90, 48, [0, 90], 90),                       #   tall-skinny
    (7, 200, 1040, [0, 200], 200),                   #   decode shape
    (300, 515, 80, [0, 256, 515], 515),
    (257, 1300, 4368, [0, 433, 1300], 1304),         #   273 blocks per row
    (200, 600, 17392, [0, 600], 600),                #   K parts behind the padded copy
])
def test_gemm_tiles_and_k_parts(m, n, k, offs, ldy):
    need, _, _ = _case(m, n, k, offs, ldy)
    log("%dx%dx%d: %s, workspace %d" % (m, n, k, L.gemm_kernels(m, n, k), need))


@pytest.mark.parametrize("m,n,k,offs,ldy,name", [
    (33, 97, 64, [0, 97], 97, "gemm_splitk_kernel<4,1,1,3>"),
    (300, 4104, 64, [0, 1000, 4104], 4104, "gemm_splitk_kernel<4,1,2,3>"),
    (777, 1999, 64, [0, 1999], 1999, "gemm_splitk_kernel<4,2,2,3>"),
    (3000, 1999, 192, [0, 700, 1999], 2000, "gemm_splitk_kernel<4,2,3,2>"),
    (100, 4104, 1280, [0, 4104], 4112, "gemm_splitk_kernel<8,1,3,3>"),
    (3000, 1999, 64, [0, 1999], 1999, "gemm_splitk_kernel<4,1,5,2>"),
    (300, 5064, 64, [0, 2000, 5064], 5064, "gemm_lds_kernel<LdsMid> (128x128 tiles)"),
    (1030, 97, 2112, [0, 97], 97, "gemm_lds_kernel<LdsMid> (128x128 tiles, K parts)"),
    (777, 2600, 256, [0, 1300, 2600], 2601, "gemm_lds_kernel<LdsMidSuper> (128x128 tiles, scale super-stages)"),
    (33, 97, 8704, [0, 97], 97, "gemm_lds_kernel<LdsMidSuper> (128x128 tiles, scale super-stages, K parts)"),
    (900, 4104, 128, [0, 4104], 4104, "gemm_lds_kernel<LdsLow> (64x256 tiles)"),
    (900, 4104, 256, [0, 333, 4104], 4106, "gemm_lds_kernel<LdsLowSuper> (64x256 tiles, scale super-stages)"),
    (33, 1999, 17408, [0, 1999], 1999, "gemm_lds_kernel<LdsLowSuper> (64x256 tiles, scale super-stages, K parts)"),
    (3000, 4104, 192, [0, 4104], 4104, "gemm_lds_kernel<LdsSquare> (256x256 tiles)"),
    (3000, 4104, 256, [0, 1000, 4104], 4108, "gemm_lds_kernel<LdsSquareSuper> (256x256 tiles, scale super-stages)"),
    (3000, 1300, 4352, [0, 1300], 1300,
     "gemm_lds_kernel<LdsSquareSuper> (256x256 tiles, scale super-stages, K parts)"),
])
def test_gemm_every_tile_kind(m, n, k, offs, ldy, name):
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert L.gemm_kernels(m, n, k)[0].startswith(name)
    _case(m, n, k, offs, ldy)


def test_gemm_k_parts_without_their_workspace():
    """A workspace short of the K parts' (or none) gives the nvfp4_gemm result."""
    # Long K on few tiles: the shape stays on K parts whatever the small
    # split-K tiles cost.
    need, aq, pw = _case(256, 2600, 17408, [0, 2600], 2600)
    assert need > 0
    y0 = L.gemm_no_workspace(aq, pw, out_dtype=torch.float32)
    y1 = torch.empty_like(y0)
    L.gemm(aq, pw, out=y1, workspace=torch.empty(need - 16, dtype=torch.uint8, device="cuda"))
    assert torch.equal(y0, y1)
    y2 = torch.empty_like(y0)
    C.nvfp4_gemm_with_workspace(aq.codes, aq.scales, aq.g, pw.packed, pw.n, pw.seg_offsets, pw.g_seg, y2, C.NVFP4_F32,
                                None, None, M=aq.m, K=aq.k)
    assert torch.equal(y0, y2)


def test_gemm_last_round_in_k_parts():
    """7000 x 5120 x 17408: 560 tiles of 256 x 256, on 256 CUs two full rounds
    and 48 tiles in K parts (ragged last tile row); sampled rows of every tile
    row against the oracle, the bf16 output equal to RNE of the FP32 output,
    strided output rows, and the first round's columns bit for bit those of
    nvfp4_gemm."""
    wl = workload("mlp_down")
    cfg, m = wl["cfg"], 7000
    aq = L.quantize_act(to_dev_bf16(wl["x"][:m]), g=float(wl["gx"]))
    pw = L.pack_weight(to_dev_bf16(wl["w"]), cfg.seg_offsets)
    kernels = L.gemm_kernels(m, cfg.n, cfg.k)
    log("%s" % kernels)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert "last round" in kernels[1]
    need = C.nvfp4_gemm_workspace(m, cfg.n, cfg.k)
    guard = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    big = torch.full((m, cfg.n + 4), -7.0, dtype=torch.float32, device="cuda")
    y32 = L.gemm(aq, pw, out=big[:, :cfg.n], workspace=guard[:need])
    y16 = L.gemm(aq, pw)
    y_nows = L.gemm_no_workspace(aq, pw, out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert bool((guard[need:] == 0x5A).all()) and bool((big[:, cfg.n:] == -7.0).all())
    assert torch.equal(y16.view(torch.int16), y32.to(torch.bfloat16).view(torch.int16))
    assert torch.equal(y32[:6144], y_nows[:6144])            # six groups of four tile rows: the full rounds
    rows = np.array(sorted(set([t * 256 + (t * 37) % 256 for t in range(20, 27)] + list(range(m - 4, m)))))
    args = (wl["xp"], wl["xs"], wl["gx"], wl["wp"], wl["ws"], wl["gw"], cfg.seg_offsets)
    y_ref, r_ref = OG.gemm_f64(*args, rows=rows), OG.abs_bound(*args, rows=rows)
    at = torch.from_numpy(rows).cuda()
    check_gemm(y32[at].cpu().numpy().astype(np.float64), y_ref, r_ref, "last round in K parts")
    check_gemm(y_nows[at].cpu().numpy().astype(np.float64), y_ref, r_ref, "no workspace")


@pytest.mark.parametrize("m,n,k,kernel", [
    (200, 2600, 17408, "K parts"),           # the whole output in K parts
    (8192, 2304, 512, "two K halves"),       # the last round in K halves
    (7000, 5120, 17408, "last round"),       #   in K parts
])
def test_gemm_partial_sums_past_the_output_range(m, n, k, kernel):
    """Activations near the top of the bf16 range against weights that are
    positive in the first half of K and the same negated in the second: Y is
    far inside FP32's range, the sum over the first half (or a part of it), in
    Y's units, is not."""
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert any(kernel in name for name in L.gemm_kernels(m, n, k))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m)
    half = 8e38 * (k / 512) ** 0.5            # sum over the first half, on average
    x = (torch.rand((m, k), generator=gen, device="cuda") + 1.0).mul_(1.5e38).to(torch.bfloat16)
    w = torch.rand((n, k // 2), generator=gen, device="cuda").add_(1.0).mul_(half / (0.5 * k * 2.25e38) / 1.5)
    w = torch.cat([w, -w], 1)
    aq, pw = L.quantize_act(x), L.pack_weight(w.to(torch.bfloat16))
    y = L.gemm(aq, pw, out_dtype=torch.float32)
    ref = L.gemm_no_workspace(aq, pw, out_dtype=torch.float32)
    assert bool(torch.isfinite(ref).all()) and float(ref.abs().max()) < 1.7e38
    # FP32 sums in another order: within 1e-4 of the sum of the magnitudes, as
    # everywhere (here in units of 1e30, which keeps it inside FP32's range).
    assert float((y * 1e-30 - ref * 1e-30).abs().max()) <= 1e-4 * 2.0 * half * 1e-30
    assert torch.equal(L.gemm(aq, pw).view(torch.int16), y.to(torch.bfloat16).view(torch.int16))


@pytest.mark.parametrize("m,n,k,offs", [
    (1100, 2301, 2112, [0, 37, 1000, 2301]),     # 128 x 128 tiles: odd rows, segments inside a wave's 64 columns
    (1100, 2304, 2048, [0, 2304]),               #   ragged rows only
    (1153, 2298, 2112, [0, 1150, 2298]),         #   one row past a tile, N % 8 == 2
    (131, 20793, 2816, [0, 9000, 9040, 20793]),  # 64 x 256 tiles
    (4100, 8190, 320, [0, 100, 200, 300, 8190]), # 256 x 256 tiles, four segments in a wave's 128 columns
    (4097, 4360, 320, [0, 4360]),                #   a last tile of one row
])
def test_bf16_tiles_past_the_edges(m, n, k, offs):
    """bf16 blocks that reach past M or N, hold segment boundaries, or lie in
    rows that allow 16-byte, 4-byte or only 2-byte stores: equal to RNE of the
    FP32 output, and nothing around them written."""
    assert "gemm_lds_kernel" in L.gemm_kernels(m, n, k, False)[0]
    rng = np.random.default_rng(m + n)
    xb = synth.f64_to_bf16_bits(rng.standard_normal((m, k)))
    wb = synth.f64_to_bf16_bits(rng.standard_normal((n, k)) * 0.02)
    aq, pw = L.quantize_act(to_dev_bf16(xb)), L.pack_weight(to_dev_bf16(wb), offs)
    want = L.gemm_no_workspace(aq, pw, out_dtype=torch.float32).to(torch.bfloat16).view(torch.int16)
    up8 = (n + 7) // 8 * 8
    for ldy, shift in ((n, 0), (up8, 0), (up8 + 8, 1), (up8 + 2, 0), (up8 + 2, 2), (up8 + 8, 8)):
        buf = torch.full(((m + 1) * ldy + shift + 8,), -7.0, dtype=torch.bfloat16, device="cuda")
        y = buf[shift:shift + (m + 1) * ldy].view(m + 1, ldy)
        L.gemm_no_workspace(aq, pw, out=y[:m, :n])
        assert torch.equal(y[:m, :n].view(torch.int16), want), (ldy, shift)
        assert bool((y[:m, n:] == -7.0).all()) and bool((y[m] == -7.0).all())
        assert bool((buf[:shift] == -7.0).all()) and bool((buf[shift + (m + 1) * ldy:] == -7.0).all())


@pytest.mark.parametrize("m,n,k", [(1024, 5120, 128), (3072, 2048, 128), (768, 8192, 320), (2048, 2048, 64),
                                   (1024, 8192, 1088), (1536, 6144, 1536)])
def test_short_k_keeps_off_many_rounds_of_small_tiles(m, n, k):
    """Five or six rounds of split-K tiles at short K took 1.1 to 1.7 times as
    long as the 256 x 256 tiles (768 x 8192 x 128: 17 and 11.3 us)."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the costs are those of 256 compute units")
    for ws in (True, False):
        assert "gemm_lds_kernel" in L.gemm_kernels(m, n, k, ws)[0]


@pytest.mark.parametrize("m,n,k,kept", [
    (6500, 1300, 208, True),               # half a round of tiles or more
    (6500, 1304, 208, False),
    (2200, 3004, 144, True),               # 0.4 of one, three chunks
    (1500, 4004, 112, True),               # a quarter, two chunks
    (1500, 4004, 144, False),
])
def test_k_remainder_with_a_workspace(m, n, k, kept):
    """K % 64 != 0, short, many tiles: rows that allow no 16-byte stores stay
    on the register path also with a workspace, the others and FP32 outputs run on
    the padded copy (each bf16 output is RNE of its own path's FP32 sums)."""
    rng = np.random.default_rng(n)
    xb = synth.f64_to_bf16_bits(rng.standard_normal((m, k)))
    wb = synth.f64_to_bf16_bits(rng.standard_normal((n, k)) * 0.02)
    aq, pw = L.quantize_act(to_dev_bf16(xb)), L.pack_weight(to_dev_bf16(wb))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert ("gemm_reg" in L.gemm_kernels(m, n, k)[0]) == kept
    y32, n32 = L.gemm(aq, pw, out_dtype=torch.float32), L.gemm_no_workspace(aq, pw, out_dtype=torch.float32)
    # k exact products: sums in two orders differ by at most 2 k 2^-24 of the sum
    # of magnitudes, here below k |x| |w| of the largest.
    bound = 2.0 * k * 2.0 ** -24 * k * 6.0 * 0.12
    assert float((y32 - n32).abs().max()) <= bound
    y16, n16 = L.gemm(aq, pw), L.gemm_no_workspace(aq, pw)
    assert torch.equal(n16.view(torch.int16), n32.to(torch.bfloat16).view(torch.int16))
    want = n32 if kept else y32
    assert torch.equal(y16.view(torch.int16), want.to(torch.bfloat16).view(torch.int16))
