"""SEM_AX_COLUMN is the column mapping at every order and size, also where the built-in
choice takes whole elements: its results are those of the mapping with the other prefetch,
bit for bit, and not those of whole elements, whose sums round differently.  sem_ax_tune
times whole elements beside it and keeps the faster."""
import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")


def _fields(nel, lx):
    g = torch.Generator(device="cuda").manual_seed(31 + lx)
    u, h1, hb, *G = (torch.rand((nel, lx, lx, lx), generator=g, dtype=torch.float64, device="cuda") for _ in range(9))
    _, _, dx, dxt = P.sem_gll(lx)
    return u, h1, hb, G, [torch.from_numpy(d).cuda() for d in (dx, dx, dx, dxt, dxt, dxt)]


@pytest.mark.parametrize("lx,nel", [(12, 1), (12, 67), (6, 24300), (5, 42000)])
@pytest.mark.parametrize("with_h2", [False, True])
def test_column_is_the_column_mapping(sem_ctx, lx, nel, with_h2):
    u, h1, hb, G, D = _fields(nel, lx)

    def run(variant):
        P.sem_ax_set_variant(sem_ctx, lx, variant)
        w = torch.full_like(u, float("nan"))
        if with_h2:
            P.sem_ax_helmholtz(sem_ctx, w, u, *D, h1, *G, hb, nel, lx)
        else:
            P.sem_ax(sem_ctx, w, u, *D, h1, *G, nel, lx)
        return w

    try:
        column, other, builtin = (run(v) for v in (P.SEM_AX_COLUMN, P.SEM_AX_COLUMN_PF, P.SEM_AX_DEFAULT))
        torch.cuda.synchronize()
        assert torch.equal(column, other)
        assert not torch.equal(column, builtin)
        assert float((column - builtin).abs().max()) <= 1e-12 * float(builtin.abs().max())
    finally:
        P.sem_ax_set_variant(sem_ctx, lx, P.SEM_AX_DEFAULT)


def test_the_tuner_keeps_whole_elements_where_they_are_faster(sem_ctx):
    """at lx = 12 they take little more than half the column mapping's time at 256 elements"""
    lx, nel = 12, 256
    u, h1, _, G, D = _fields(nel, lx)
    w = [torch.full_like(u, float("nan")) for _ in range(3)]
    try:
        P.sem_ax_set_variant(sem_ctx, lx, P.SEM_AX_DEFAULT)
        P.sem_ax(sem_ctx, w[0], u, *D, h1, *G, nel, lx)
        best, us = P.sem_ax_tune_on(sem_ctx, w[1], u, *D, h1, *G, nel, lx, reps=20)
        assert best == P.SEM_AX_COLUMN == P.sem_ax_get_variant(sem_ctx, lx) and us[best] == min(t for t in us if t > 0)
        P.sem_ax(sem_ctx, w[1], u, *D, h1, *G, nel, lx)
        P.sem_ax_set_variant(sem_ctx, lx, P.SEM_AX_COLUMN)
        P.sem_ax(sem_ctx, w[2], u, *D, h1, *G, nel, lx)
        torch.cuda.synchronize()
        assert torch.equal(w[1], w[0]) and not torch.equal(w[2], w[0])
    finally:
        P.sem_ax_set_variant(sem_ctx, lx, P.SEM_AX_DEFAULT)
