"""Calls on an explicit stream: which stream their scratch memory and their own
tensor copies belong to (on the CPU, with the library and the stream switch
replaced by recorders), and on the GPU results while the current stream
allocates and writes."""

import contextlib

import numpy as np
import pytest
import torch

from paper_2609_04098_amd import linear as L
from paper_2609_04098_amd import synth


class FakeStream:
    cuda_stream = 0x1000


class Recorder:
    """Replaces torch.cuda.stream, torch.empty and the library's calls."""

    def __init__(self, monkeypatch):
        self.current = None                    # stream made current
        self.allocated = {}                    # data_ptr -> stream at allocation
        self.kept, self.calls = [], {}
        empty = torch.empty

        @contextlib.contextmanager
        def switch(stream):
            before, self.current = self.current, stream
            try:
                yield
            finally:
                self.current = before

        def recorded_empty(*args, **kwargs):
            t = empty(*args, **kwargs)
            self.kept.append(t)                # no address is used twice
            self.allocated[t.data_ptr()] = self.current
            return t

        self.copied = {}                       # data_ptr of the target -> stream of its copy
        copy = torch.Tensor.copy_

        def recorded_copy(t, src, *args):
            self.copied[t.data_ptr()] = self.current
            return copy(t, src, *args)

        monkeypatch.setattr(torch.Tensor, "copy_", recorded_copy)
        monkeypatch.setattr(torch.cuda, "stream", switch)
        monkeypatch.setattr(torch, "empty", recorded_empty)
        for name in ("nvfp4_quantize_act", "nvfp4_rmsnorm_quantize_act", "nvfp4_pack_weight", "nvfp4_harmonize_weight",
                     "nvfp4_gemm_with_workspace", "nvfp4_quantize_gemm"):
            monkeypatch.setattr(L._c, name, lambda *a, _n=name, **k: self.calls.setdefault(_n, a))
        monkeypatch.setattr(L._c, "nvfp4_gemm_workspace", lambda m, n, k: 4096)

    def stream_of(self, t):
        return self.allocated[t.data_ptr()]


def _tensors():
    x, w = torch.ones((40, 64), dtype=torch.bfloat16), torch.ones((160, 64), dtype=torch.bfloat16)
    pw = L.PackedWeight(torch.zeros(8192, dtype=torch.uint8), torch.ones(1), 160, 64, [0, 160])
    return x, w, pw


@pytest.mark.parametrize("stream", [FakeStream(), None])
def test_scratch_belongs_to_the_stream_that_uses_it(monkeypatch, stream):
    """Scratch that a call allocates and drops on return; the outputs stay the
    current stream's."""
    x, w, pw = _tensors()
    rec = Recorder(monkeypatch)
    L.pack_weight(w, stream=stream)
    aq = L.quantize_act(x, stream=stream)
    y = L.gemm(aq, pw, stream=stream)
    yf, _ = L.quantize_gemm(x[:8], pw, stream=stream)
    for name, at in (("nvfp4_pack_weight", 5), ("nvfp4_quantize_act", 5), ("nvfp4_gemm_with_workspace", 9),
                     ("nvfp4_quantize_gemm", 8)):
        ws = rec.calls[name][at]
        assert ws.dtype == torch.uint8 and ws.dim() == 1
        assert rec.stream_of(ws) is stream, name
    for t in (aq.codes, aq.scales, aq.g, y, yf):
        assert rec.stream_of(t) is None


@pytest.mark.parametrize("stream", [FakeStream(), None])
def test_copies_are_in_the_order_of_the_call(monkeypatch, stream):
    """A scale given as a tensor, and the weight that harmonize_weight leaves
    as it was, are copied on the stream whose kernel reads the copy."""
    x, w, pw = _tensors()
    rec = Recorder(monkeypatch)
    aq = L.rmsnorm_quantize_act(x, x[0], 1e-6, torch.tensor([3.0]), stream=stream)
    hw = L.harmonize_weight(pw, stream=stream)
    pg = L.pack_weight(w, g_seg=torch.tensor([3.0], dtype=torch.float64), stream=stream)
    for t in (aq.g, hw.packed, pg.g_seg):
        assert rec.copied[t.data_ptr()] is stream
    assert aq.g.item() == 3.0 and pg.g_seg.dtype == torch.float32 and pg.g_seg.item() == 3.0
    assert torch.equal(hw.packed, pw.packed) and hw.packed.data_ptr() != pw.packed.data_ptr()
    g = torch.tensor([2.0])
    assert L.pack_weight(w, g_seg=g).g_seg is g and L.pack_weight(w, g_seg=[5.0]).g_seg.item() == 5.0


def test_a_learned_scale_leaves_plain_buffers(monkeypatch):
    """A scale tensor that requires a gradient does not make G one that does."""
    x, w, pw = _tensors()
    Recorder(monkeypatch)
    g = torch.nn.Parameter(torch.tensor([3.0]))
    for aq in (L.rmsnorm_quantize_act(x, x[0], 1e-6, g), L.quantize_act(x, g=g)):
        assert not aq.g.requires_grad and aq.g.item() == 3.0
    assert not L.quantize_gemm(x[:8], pw, g=g)[1].requires_grad


@pytest.mark.gpu
def test_a_learned_scale_on_the_device():
    x = torch.ones((40, 64), dtype=torch.bfloat16, device="cuda")
    pw = L.pack_weight(torch.ones((96, 64), dtype=torch.bfloat16, device="cuda"))
    g = torch.nn.Parameter(torch.tensor([3.0], device="cuda"))
    for got in (L.rmsnorm_quantize_act(x, x[0], 1e-6, g).g, L.quantize_act(x, g=g).g, L.quantize_gemm(x, pw, g=g)[1]):
        assert not got.requires_grad and got.item() == 3.0


@pytest.mark.gpu
def test_side_stream_calls_while_the_current_stream_allocates():
    """K parts (whole output; 12 MB of partial sums), the padded activation copy
    (K % 64 != 0), the quantizer's and the fused call's scratch: called on a side
    stream without a workspace, while the current stream allocates blocks of the
    same sizes and writes them."""
    def case(m, n, k):
        rng = np.random.default_rng(m + n)
        up = lambda a: torch.from_numpy(synth.f64_to_bf16_bits(a).view(np.int16)).view(torch.bfloat16).cuda()
        return up(rng.standard_normal((m, k))), L.pack_weight(up(rng.standard_normal((n, k)) * 0.02))

    cases = [case(200, 2560, 17408), case(300, 515, 1040), case(8, 2600, 5120)]
    want = []
    for x, pw in cases:
        aq = L.quantize_act(x)
        want.append((aq, L.gemm(aq, pw), L.quantize_gemm(x, pw)[0] if x.shape[0] <= 32 else None))
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    sizes = [n for n in (L._c.nvfp4_gemm_workspace(x.shape[0], pw.n, pw.k) for x, pw in cases) if n]
    sizes += [L._c.nvfp4_quantize_act_workspace(1, 16), L._c.nvfp4_quantize_gemm_workspace(8, 2600, 5120)]
    assert len(sizes) == 4
    for handle in (side, side.cuda_stream):
        for _ in range(5):
            for (x, pw), (aq0, y0, f0) in zip(cases, want):
                aq, y = L.alloc_act(aq0.m, aq0.k, x.device), torch.empty_like(y0)
                f = None if f0 is None else torch.empty_like(f0)
                side.wait_stream(torch.cuda.current_stream())
                L.quantize_act(x, out=aq, stream=handle)
                L.gemm(aq, pw, out=y, stream=handle)
                if f is not None:
                    L.quantize_gemm(x, pw, out=f, stream=handle)
                junk = [torch.empty(n, dtype=torch.uint8, device="cuda").fill_(0x7F) for n in sizes]
                side.synchronize()
                assert torch.equal(aq.codes, aq0.codes) and torch.equal(aq.scales, aq0.scales)
                assert torch.equal(y, y0) and (f is None or torch.equal(f, f0))
                del junk
