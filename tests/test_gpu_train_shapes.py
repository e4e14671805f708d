"""The network's products at the edges of their tiles: a forward pass of row
counts around the 16- and 32-row workgroups, and in training batches that are
not whole 16- or 32-row tiles (one smaller than an earlier one of the same
network), element and hidden sizes that are not whole tiles, a batch taken
through row indices, and features that do not lie on 16 bytes.

Gradients against the oracle's bfloat16-storage emulation at the bound of
test_gpu_learned.py: 2e-3 of the largest entry, a float32 sum that tips a
bfloat16 rounding moves an output by about 2^-8 / sqrt(fan-in) of that.  A
step through row indices multiplies the same values in the same order as the
gradients of the gathered batch, so its weights are bit-equal."""
import numpy as np
import pytest
import torch

import synth
from oracle import mlp
from oracle.quant import to_bf16

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")

EW_NET = 2e-3


def _network(ctx, lx, hidden, max_rows, form):
    n = lx ** 3
    p = synth.mlp_init(60 + lx, (n + 6, hidden, hidden, n))
    r = synth.rng(61)
    p = [q if q.ndim == 2 else 0.1 * r.standard_normal(q.shape) for q in p]
    p = [q.astype(np.float32) for q in p]
    lp = P.sem_lp_create(ctx, max_rows, lx=lx, hidden=hidden)
    for s, q in enumerate(p):
        P.sem_lp_set(lp, s, q)
    if form == "metric":
        P.sem_lp_set_metric(lp, 1.0)
    if form == "linear":
        P.sem_lp_set_linear(lp, 1)
    return lp, [q.astype(np.float64) for q in p]


def _rows(lx, count, seed):
    n, ni, nip = P.lp_sizes(lx)
    r = synth.rng(seed)
    X = r.standard_normal((count, ni))
    X[:, :n] /= np.linalg.norm(X[:, :n], axis=1, keepdims=True)
    Xpad = np.zeros((count, nip), dtype=np.float32)
    Xpad[:, :ni] = to_bf16(X)
    T = (0.1 * r.standard_normal((count, n))).astype(np.float32)
    return torch.from_numpy(Xpad).to(torch.bfloat16).cuda(), torch.from_numpy(T).cuda()


@pytest.mark.parametrize("form", ["mse", "linear"])
@pytest.mark.parametrize("lx,hidden,rows", [(4, 16, 1), (6, 48, 17), (4, 256, 33), (4, 80, 8192), (6, 16, 8209),
                                            (12, 1024, 5)])
def test_forward_of_ragged_rows(sem_ctx, lx, hidden, rows, form):
    lp, params = _network(sem_ctx, lx, hidden, rows, form)
    X, _ = _rows(lx, rows, 63)
    Y = torch.full((rows + 1, lx ** 3), -7.0, dtype=torch.float32, device="cuda")
    P.sem_lp_forward(lp, X, Y[:rows])
    assert bool((Y[rows] == -7.0).all())          # nothing past the last row
    Xq = X.float().cpu().numpy().astype(np.float64)[:, :lx ** 3 + 6]
    ref = mlp.forward_bf16(params, Xq, linear=form == "linear")[2]
    err = np.max(np.abs(Y[:rows].cpu().numpy() - ref))
    assert err <= EW_NET * np.max(np.abs(ref)), err
    lp.close()


@pytest.mark.parametrize("form", ["mse", "metric", "linear"])
@pytest.mark.parametrize("lx,hidden", [(4, 16), (6, 48), (4, 256)])
def test_gradients_of_ragged_batches(sem_ctx, lx, hidden, form):
    lp, params = _network(sem_ctx, lx, hidden, 136, form)
    K = mlp.reference_metric(lx, 1.0) if form == "metric" else None
    for B in (136, 8, 72, 24):
        X, T = _rows(lx, B, 62 + B)
        loss = P.sem_lp_gradients(lp, X, T)
        Xq = X.float().cpu().numpy().astype(np.float64)[:, :lx ** 3 + 6]
        lq, gq = mlp.backward_bf16(params, Xq, T.cpu().numpy().astype(np.float64), K, linear=form == "linear")
        assert abs(loss - lq) <= 1e-3 * lq, (B, loss, lq)
        for s in range(6):
            g = P.sem_lp_get(lp, 18 + s).astype(np.float64)
            scale = np.max(np.abs(gq[s]))
            err = np.max(np.abs(g - gq[s]))
            assert err <= EW_NET * scale, (B, s, err, scale)
    lp.close()


@pytest.mark.parametrize("form", ["mse", "metric", "linear"])
def test_step_through_row_indices_and_unaligned_features(sem_ctx, form):
    lx, hidden, B, rows = 6, 48, 40, 97
    X, T = _rows(lx, rows, 70)
    pick = torch.from_numpy(synth.permutation(71, rows)[:B].copy()).cuda()
    shifted = torch.empty(X.numel() + 1, dtype=X.dtype, device="cuda")[1:].view_as(X)   # 2 bytes off
    shifted.copy_(X)
    weights = []
    for source in ("gathered", "indexed", "unaligned"):
        lp, _ = _network(sem_ctx, lx, hidden, B, form)
        loss = torch.zeros(2, dtype=torch.float32, device="cuda")
        for step in range(2):
            if source == "gathered":
                loss[step] = P.sem_lp_gradients(lp, X[pick].contiguous(), T[pick].contiguous())
                P.sem_lp_adam(lp, 1e-3)
            else:
                P.sem_lp_train_step(lp, X if source == "indexed" else shifted, T, pick, 1e-3, loss[step:step + 1])
        weights.append([loss.cpu().numpy()] + [P.sem_lp_get(lp, s) for s in range(18)])
        lp.close()
    for other in weights[1:]:
        for a, b in zip(weights[0], other):
            assert np.array_equal(a, b)
