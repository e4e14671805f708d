"""Captured calls of the network use the weights of their replay: weights set between the
capture and a replay (sem_lp_set, sem_lp_load) and weights that other steps trained give,
bit for bit, what the same call gives without a graph."""
import numpy as np
import pytest
import torch

from tests.test_gpu_train_shapes import _network, _rows

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")

LX, HIDDEN, B = 6, 64, 64


def _slots(lp):
    return [P.sem_lp_get(lp, s).copy() for s in range(18)]


def _put(lp, slots, step):
    for s, v in enumerate(slots):
        P.sem_lp_set(lp, s, v)
    P.sem_lp_set_step(lp, step)


@pytest.mark.parametrize("form", ["mse", "linear"])
def test_replays_use_the_weights_of_their_time(sem_ctx, tmp_path, form):
    lp, _ = _network(sem_ctx, LX, HIDDEN, B, form)
    other, _ = _network(sem_ctx, LX, HIDDEN, B, form)
    X, T = _rows(LX, B, 67)
    rows = torch.arange(B, device="cuda")
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    Y = torch.empty((B, LX ** 3), dtype=torch.float32, device="cuda")
    want = torch.empty_like(Y)
    P.sem_lp_train_step(lp, X, T, rows, 1e-3, loss)          # work buffers exist from here on
    forward, step = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(forward):
        P.sem_lp_forward(lp, X, Y)
    with torch.cuda.graph(step):
        P.sem_lp_train_step(lp, X, T, rows, 1e-3, loss)      # Adam's second step
    r = np.random.default_rng(5)
    base = _slots(lp)
    for turn in range(4):
        fresh = [(v + 0.05 * r.standard_normal(v.shape)).astype(np.float32) if s < 6 else v
                 for s, v in enumerate(base)]
        _put(other, fresh, 1)
        if turn == 2:                                        # through a file
            path = str(tmp_path / "net")
            P.sem_lp_save(other, path)
            P.sem_lp_load(lp, path)
        else:
            _put(lp, fresh, 1)
        P.sem_lp_forward(other, X, want)
        torch.cuda.synchronize()
        forward.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want), turn
        step.replay()
        P.sem_lp_train_step(other, X, T, rows, 1e-3, loss)
        torch.cuda.synchronize()
        for a, b in zip(_slots(lp), _slots(other)):
            assert np.array_equal(a, b), turn
        forward.replay()                                     # the weights that the step trained
        P.sem_lp_forward(other, X, want)
        torch.cuda.synchronize()
        assert torch.equal(Y, want), turn
    lp.close()
    other.close()
