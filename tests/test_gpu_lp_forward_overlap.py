"""sem_lp_forward where the outputs lie over the features (a program that reuses one
buffer): equal, bit for bit, to the call with buffers of its own, for row counts with one
and with many workgroups, and untouched where the two only meet at their ends."""
import pytest
import torch

from tests.test_gpu_train_shapes import _network, _rows

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")


@pytest.mark.parametrize("lx,rows,at", [(4, 8, 0), (4, 5000, 0), (8, 600, 0), (8, 600, 7), (6, 8200, 1000), (8, 100, -1)])
def test_outputs_over_the_features(sem_ctx, lx, rows, at):
    """at: first row of the features in the buffer of the outputs (-1: right behind them)"""
    n, _, nip = P.lp_sizes(lx)
    lp, _ = _network(sem_ctx, lx, 64, rows, "mse")
    X, _ = _rows(lx, rows, 65)
    want = torch.empty((rows, n), dtype=torch.float32, device="cuda")
    P.sem_lp_forward(lp, X, want)
    buf = torch.zeros(rows * n * 2 + (rows + 2000) * nip, dtype=torch.bfloat16, device="cuda")
    first = rows * n * 2 if at < 0 else at * nip
    Xo = buf[first:first + rows * nip].view(rows, nip)
    Xo.copy_(X)
    Y = buf[:rows * n * 2].view(torch.float32).view(rows, n)
    P.sem_lp_forward(lp, Xo, Y)
    torch.cuda.synchronize()
    assert torch.equal(Y, want)
    if at < 0:
        assert torch.equal(Xo, X)
    lp.close()
