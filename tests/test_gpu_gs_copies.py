"""Sums over the copies of a node (gather-scatter, and the solver's assembly) for
numberings other than a hexahedral box's: every count of copies from one to
beyond two of the plan's four-wide lists, Dirichlet nodes among them, sizes
around a workgroup.  The sums are taken in increasing local index, so they equal
a sequential sum bit for bit, in either type."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n_ids,most", [(1, 1), (3, 13), (255, 4), (512, 9), (1031, 23)])
def test_sums_of_any_number_of_copies(sem_ctx, n_ids, most, dtype):
    r = synth.rng(n_ids + most)
    copies = 1 + np.arange(n_ids) % most
    ids = np.repeat(r.permutation(5 * n_ids)[:n_ids], copies)
    ids = np.concatenate([ids, np.full(7, -1)])
    r.shuffle(ids)
    u = r.standard_normal(ids.size).astype(np.float64 if dtype == torch.float64 else np.float32)
    ref = u.copy()
    for g in np.unique(ids):
        at = np.nonzero(ids == g)[0]
        if g < 0:
            ref[at] = 0
        elif at.size > 1:
            s = u[at[0]]
            for L in at[1:]:
                s = s + u[L]
            ref[at] = s
    gs = P.sem_gs_setup(sem_ctx, ids)
    d = torch.from_numpy(u).cuda()
    P.sem_gs(gs, d)
    assert np.array_equal(d.cpu().numpy(), ref)
    assert P.sem_gs_info(gs) == (n_ids, int(np.sum(copies > 1)))
    gs.close()
