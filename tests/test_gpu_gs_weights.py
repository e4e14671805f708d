"""Multiplicities and owner weights of plans at their edges: no node, one, Dirichlet nodes
only, none shared, all copies of one id, and random ids with every number of copies from one
to dozens and Dirichlet nodes between them; exact, against the numbering itself."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")


def _ids(kind):
    r = synth.rng(81)
    if kind == "random":
        ids = r.integers(0, 300, size=5000) ** 2 // 300
        ids[r.random(5000) < 0.1] = -1
        return ids
    return {"none": np.zeros(0), "one": np.array([7]), "two": np.array([3, 3]), "masked": np.full(70, -1),
            "distinct": np.arange(1000)[::-1], "all": np.full(300, 5), "sparse": np.array([10 ** 12, 4, 10 ** 12, -1])}[kind]


@pytest.mark.parametrize("kind", ["none", "one", "two", "masked", "distinct", "all", "sparse", "random"])
def test_multiplicity_and_owner(sem_ctx, kind):
    ids = _ids(kind).astype(np.int64)
    gs = P.sem_gs_setup(sem_ctx, ids)
    mult, owner, u = (torch.full((max(ids.size, 1),), -7.0, dtype=torch.float64, device="cuda") for _ in range(3))
    if ids.size:
        P.sem_gs_mult(gs, mult)
        P.sem_gs_owner(gs, owner)
        u.fill_(1.0)
        P.sem_gs(gs, u)
        torch.cuda.synchronize()
        keys, first, inverse, counts = np.unique(ids, return_index=True, return_inverse=True, return_counts=True)
        free = ids >= 0
        want = np.where(free, counts[inverse], 1)
        assert np.array_equal(mult.cpu().numpy(), want)
        assert np.array_equal(owner.cpu().numpy(), (free & (np.arange(ids.size) == first[inverse])).astype(float))
        assert np.array_equal(u.cpu().numpy(), np.where(free, want, 0))
    n_unique, n_shared = P.sem_gs_info(gs)
    assert n_unique == np.unique(ids[ids >= 0]).size
    assert n_shared == int((np.unique(ids[ids >= 0], return_counts=True)[1] > 1).sum())
    gs.close()
