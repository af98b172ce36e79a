"""The quantizer's fast form (one multiplication per element) against the exact
decision: on the CPU the same binary32 arithmetic in numpy, over every bf16
significand, every block-scale significand and the reciprocal's error range; on
the GPU whole tensors against the oracle."""

import numpy as np
import pytest

from oracle import quant as OQ

f32 = np.float32
MU = np.array([m * s for s in range(8, 16) for m in (1, 3, 5, 7)], dtype=np.float64)


def _mode(g, rcp_ulps=0):
    """quant_mode of csrc/quant_device.h: (exact, gf), with a reciprocal that is
    off by rcp_ulps."""
    g = f32(g)
    gm = np.frexp(np.float64(g))[0] * 2.0
    if g == 0:
        return True, g
    rcp = (f32(1.0) / f32(gm)).view(np.int32) + rcp_ulps
    t = (MU.astype(f32) * rcp.astype(np.int32).view(f32)).astype(np.float64)
    p = 2.0 ** (8 - np.frexp(t)[1])
    x = np.rint(t * p)
    e = x * gm - MU * p                       # exact in float64 (33 bits less 15)
    near = np.abs(e) <= (MU * p).astype(f32) * f32(2.0 ** -20)
    up, down, tie = bool((near & (e > 0)).any()), bool((near & (e < 0)).any()), bool((near & (e == 0)).any())
    exact = tie or (up and down) or not (2.0 ** -100 <= g <= 2.0 ** 100)
    d = 2.0 ** -21 if up else -2.0 ** -21 if down else 0.0
    return exact, f32(np.float64(g) * d + np.float64(g))


def _e2m1(v):
    """RNE_E2M1 of float64 magnitudes, saturating."""
    step = np.where(v < 2.0, 0.5, np.where(v < 4.0, 1.0, 2.0))
    return np.minimum(np.rint(v / step) * step, 6.0)


def _scales():
    rng = np.random.default_rng(5)
    dynamic = [f32(2688.0) / f32(a * 2.0 ** e) for a in range(128, 256) for e in (-40, -7, 3)]
    near = []
    for mu in (8.0, 33.0, 42.0, 105.0):
        for x in (128.0, 171.0, 255.0):
            for d in (0.0, 2.0 ** -24, -2.0 ** -24, 2.0 ** -22, -2.0 ** -22, 2.0 ** -20.5, -2.0 ** -20.5, 2.0 ** -19):
                near.append(f32(mu / x * (1.0 + d)))
    anything = (rng.uniform(1.0, 2.0, 300) * 2.0 ** rng.integers(-60, 60, 300)).astype(f32)
    return np.array(dynamic + near + list(anything), dtype=f32)


def test_fast_form_matches_the_exact_decision():
    x = np.arange(128, 256, dtype=np.float64)[:, None]
    s = np.arange(8, 16, dtype=np.float64)[None, :]
    fast = 0
    for g in _scales():
        exact, gf = _mode(g)
        if exact:
            continue
        fast += 1
        gm = np.float64(g)
        # every power of two that brings x G / S near the E2M1 range
        base = np.floor(np.log2(x * gm / s))
        for k in range(-4, 5):
            v = x * gm / s * 2.0 ** (k - base)
            want = _e2m1(v)
            sx = s * 2.0 ** (base - k)                       # the scale that gives v
            for ulp in (-1, 0, 1):                            # reciprocal within one ulp
                r = (1.0 / sx).astype(f32)
                r = (r.view(np.int32) + ulp).view(f32)
                c = (gf * r).astype(f32)
                got = _e2m1(np.abs((x.astype(f32) * c).astype(f32)).astype(np.float64))
                assert np.array_equal(got, want), (float(g), k, ulp)
    assert fast > 600


def test_the_form_does_not_hang_on_the_reciprocal():
    for g in _scales():
        assert _mode(g, -1) == _mode(g) == _mode(g, 1), float(g)


def test_exact_form_is_kept_where_it_is_needed():
    # 2688 / amax without rounding: exact ties exist
    for a in (128, 168, 192, 224):
        assert _mode(f32(2688.0) / f32(a))[0]
    assert _mode(f32(2.0 ** 101))[0] and _mode(f32(2.0 ** -101))[0] and _mode(f32(0.0))[0]
    # the other dynamic scales take the fast form
    assert sum(_mode(f32(2688.0) / f32(a))[0] for a in range(128, 256)) == 4


@pytest.mark.gpu
def test_quantizer_over_every_amax_significand():
    """One tensor per bf16 significand of the maximum, values over 14 binades."""
    from paper_2609_04098_amd import linear as L
    from paper_2609_04098_amd import synth
    from tests.gpu_common import to_dev_bf16
    rng = np.random.default_rng(6)
    for a in range(128, 256):
        v = rng.integers(128, 256, (48, 512)) * 2.0 ** rng.integers(-13, 0, (48, 512)) * rng.choice([-1.0, 1.0], (48, 512))
        v *= a / 256.0
        v = np.clip(v, -a / 1.0, a / 1.0)
        v[7, 31] = -float(a)
        bits = synth.f64_to_bf16_bits(v)
        xp, xs, gx = OQ.quantize_tensor(bits)
        aq = L.quantize_act(to_dev_bf16(bits))
        assert f32(aq.g.item()) == gx
        assert np.array_equal(aq.scales.cpu().numpy(), xs) and np.array_equal(aq.codes.cpu().numpy(), xp), a


@pytest.mark.gpu
def test_quantizer_near_thresholds_and_far_out_of_range():
    """Given scales next to a threshold, and values that saturate by far."""
    from paper_2609_04098_amd import linear as L
    from paper_2609_04098_amd import synth
    from tests.gpu_common import to_dev_bf16
    rng = np.random.default_rng(8)
    v = rng.integers(128, 256, (40, 512)) * 2.0 ** rng.integers(-10, 3, (40, 512)) * rng.choice([-1.0, 1.0], (40, 512))
    v[3, :7] = [3.0e38, -3.0e38, 1e30, -1e30, 0.0, -0.0, 1e-39]
    bits = synth.f64_to_bf16_bits(v)
    x = to_dev_bf16(bits)
    for g in list(_scales()[384:480]) + [f32(2.0 ** 99), f32(1.7 * 2.0 ** 100), f32(2.0 ** -99), f32(1e-37), f32(1e38)]:
        xp, xs, _ = OQ.quantize_tensor(bits, g=g)
        aq = L.quantize_act(x, g=float(g))
        assert np.array_equal(aq.scales.cpu().numpy(), xs) and np.array_equal(aq.codes.cpu().numpy(), xp), float(g)


FORMS = [
    (f32(2688.0) / f32(201.0), False),       # fast
    (f32(4.0), True),                        # exact ties, one multiplication for q
    (f32(1.7 * 2.0 ** 100), True),           # two: q's factor could overflow
    (f32(2.0 ** -101), True),                # ... or lose bits
]


def _form_input(rng, m, k, g):
    """Blocks over the scales' whole range under G = g: saturating, normal,
    subnormal and zero scales, the last with elements of both signs."""
    v = rng.integers(128, 256, (m, k)) * rng.choice([-1.0, 1.0], (m, k)) * 2.0 ** rng.integers(-6, 1, (m, k))
    e = np.floor(-np.log2(np.float64(g)))
    v *= 2.0 ** np.repeat(rng.integers(-17, 7, (m, k // 16)), 16, axis=1) * 2.0 ** np.clip(e, -100, 100)
    v[0, :16] *= 2.0 ** -20                  # S = 0
    return v


@pytest.mark.gpu
@pytest.mark.parametrize("g,exact", FORMS)
@pytest.mark.parametrize("path,m,k", [
    ("small", 20, 512), ("large", 272, 512), ("norm", 33, 512), ("norm", 5, 8208), ("narrow", 40, 512),
    ("narrow", 300, 512), ("decode", 3, 512), ("decode", 20, 512)])
def test_every_form_in_every_kernel(path, m, k, g, exact):
    """Codes and scales of the quantizer's kernels, of the normalizing ones and of
    both fused products, in each form, against the oracle."""
    import torch
    from paper_2609_04098_amd import linear as L
    from paper_2609_04098_amd import synth
    from tests.gpu_common import np_u8, to_dev_bf16
    assert _mode(g)[0] == exact
    rng = np.random.default_rng(m + k)
    bits = synth.f64_to_bf16_bits(_form_input(rng, m, k, g))
    x = to_dev_bf16(bits)
    if path == "norm":
        # gamma spreads the normalized rows (all of about 1) over the scales' range
        gamma = to_dev_bf16(synth.f64_to_bf16_bits(_form_input(rng, 1, k, g))).reshape(-1)
        x = to_dev_bf16(synth.f64_to_bf16_bits(rng.standard_normal((m, k))))
        y = torch.empty_like(x)
        aq = L.rmsnorm_quantize_act(x, gamma, 1e-6, float(g), y=y)
        bits = y.view(torch.int16).cpu().numpy().view(np.uint16)
    elif path in ("narrow", "decode"):
        n = 96 if path == "narrow" else 200
        pw = L.pack_weight(to_dev_bf16(synth.f64_to_bf16_bits(rng.standard_normal((n, k)))))
        aq = L.alloc_act(m, k, x.device)
        L.quantize_gemm(x, pw, g=float(g), act_out=aq)
    else:
        aq = L.quantize_act(x, g=float(g))
    xp, xs, _ = OQ.quantize_tensor(bits, g=g)
    s = np.unique(xs)
    assert s.min() == 0 and (s == 126).any() and ((s > 0) & (s < 8)).any()
    np.testing.assert_array_equal(np_u8(aq.scales), xs)
    np.testing.assert_array_equal(np_u8(aq.codes), xp)
