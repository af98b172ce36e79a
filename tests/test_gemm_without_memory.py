"""gemm() where no memory is left for the workspace it would use (on the CPU, with
the library's call and the allocation replaced)."""

import pytest
import torch

from paper_2609_04098_amd import linear as L


@pytest.mark.parametrize("status", [0, L._c.NVFP4_EWORKSPACE, L._c.NVFP4_EHIP])
def test_gemm_without_memory_for_its_workspace(monkeypatch, status):
    """Shapes whose workspace is optional run without; those that need one (the
    library answers NVFP4_EWORKSPACE) report the missing memory."""
    pw = L.PackedWeight(torch.zeros(8192, dtype=torch.uint8), torch.ones(1), 160, 64, [0, 160])
    aq = L.alloc_act(40, 64, "cpu")
    empty, given = torch.empty, []

    def no_room(*args, **kwargs):
        if args and args[0] == 4096:
            raise torch.OutOfMemoryError("no memory for the workspace")
        return empty(*args, **kwargs)

    def call(*args, **kwargs):
        given.append(args[9])
        if status:
            raise L._c.Nvfp4Error(status, "nvfp4_gemm_with_workspace")

    monkeypatch.setattr(torch, "empty", no_room)
    monkeypatch.setattr(L._c, "nvfp4_gemm_workspace", lambda m, n, k: 4096)
    monkeypatch.setattr(L._c, "nvfp4_gemm_with_workspace", call)
    if status == 0:
        assert L.gemm(aq, pw).shape == (40, 160)
    else:
        with pytest.raises(torch.OutOfMemoryError if status == L._c.NVFP4_EWORKSPACE else L._c.Nvfp4Error):
            L.gemm(aq, pw)
    assert given == [None]
