"""Calls go to torch's current stream: the handle the binding passes on is that of the
default stream, of a side stream inside its block and of the default one after it,
by torch's raw query and by the Stream object; work on a side stream is ordered
with torch's there (exact result of an operator of ones)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")
from paper_2506_20994_amd import _binding as B  # noqa: E402


@pytest.mark.parametrize("raw", [True, False])
def test_current_stream(monkeypatch, raw):
    if not raw:
        monkeypatch.setattr(B, "_raw_stream", None)
    default = torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    assert B._current_stream() == default
    nel, lx = 40, 4
    ctx = P.sem_create()
    with torch.cuda.stream(side):
        assert B._current_stream() == side.cuda_stream
        D = [torch.eye(lx, dtype=torch.float64, device="cuda") for _ in range(6)]
        u = torch.ones(nel, lx, lx, lx, dtype=torch.float64, device="cuda")
        z = torch.zeros_like(u)
        w = torch.full_like(u, 9.0)
        P.sem_ax(ctx, w, u, *D, None, u, u, u, z, z, z, nel, lx)
        w = w * 2.0                            # D = 1, G = 1: w = 3 u
    side.synchronize()
    assert bool((w == 6.0).all())
    assert B._current_stream() == default
    ctx.close()
