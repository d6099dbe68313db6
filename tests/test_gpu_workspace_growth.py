"""The cached workspace grows without holding the smaller buffer beside the
larger one, as where a process renders in bfloat16 and then in float32."""

import pytest

pytestmark = pytest.mark.gpu


def test_growth_holds_one_buffer(gpu_lib, monkeypatch):
    import torch
    from paper_2111_11215_amd import api
    first, second = 64 << 20, 80 << 20
    monkeypatch.setattr(api, "_WS", {})   # (a stream of the pool may have a workspace already)
    with torch.cuda.stream(torch.cuda.Stream()):
        torch.cuda.synchronize()
        base = torch.cuda.memory_allocated()
        torch.cuda.reset_peak_memory_stats()
        assert api.workspace(first, "cuda:0").numel() == first
        assert api.workspace(second, "cuda:0").numel() == second
        assert torch.cuda.max_memory_allocated() - base < first + second
        assert api.workspace(first, "cuda:0").numel() == second
        torch.cuda.synchronize()
