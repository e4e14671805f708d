"""A forward pass of few rows of a large network is three products, of many rows one kernel:
both add the same products in the same order, so a row's outputs are the same bits in a
call of any length, on either side of that line, for networks on either side of the size
from which it is drawn; and in agreement with the oracle (bound of test_gpu_train_shapes.py)."""
import pytest
import torch

from oracle import mlp
from tests.test_gpu_train_shapes import EW_NET, _network, _rows

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")


@pytest.mark.parametrize("form", ["mse", "linear"])
@pytest.mark.parametrize("lx,hidden", [(8, 384), (8, 352), (10, 256), (12, 1024), (4, 656), (4, 640)])
def test_rows_are_the_same_in_a_call_of_any_length(sem_ctx, lx, hidden, form):
    n = lx ** 3
    most = 1100
    lp, params = _network(sem_ctx, lx, hidden, most, form)
    X, _ = _rows(lx, most, 71)
    want = torch.empty((most, n), dtype=torch.float32, device="cuda")
    P.sem_lp_forward(lp, X, want)
    for rows in (1, 15, 17, 33, 100, 1023, 1024, 1025):
        Y = torch.full((rows + 1, n), -7.0, dtype=torch.float32, device="cuda")
        P.sem_lp_forward(lp, X[:rows].contiguous(), Y[:rows])
        torch.cuda.synchronize()
        assert torch.equal(Y[:rows], want[:rows]), rows
        assert bool((Y[rows] == -7.0).all())
    few = X[:40].float().cpu().double().numpy()[:, :n + 6]
    ref = torch.from_numpy(mlp.forward_bf16(params, few, linear=form == "linear")[2])
    assert float((want[:40].cpu().double() - ref).abs().max()) <= EW_NET * float(ref.abs().max())
    lp.close()
