"""Jacobi-PCG on an indefinite operator (A + h2 B with a large negative h2): the loop ends
at the first direction with p^T A p <= 0 as SEM_EBREAKDOWN, with the iterations counted and
x left at the steps taken before it, at both workgroup shapes of the vector kernels.

The loop in numpy on the oracle's operator says where it ends.  A relative change of the
right-hand side by 1e-12 moves that x by 3e-12 and 1e-12 of its largest value, rounding
(1e-16 an operation, sums of a few hundred terms) by less: bound 1e-9."""
import ctypes

import numpy as np
import pytest
import torch

import synth
from oracle.solve import BoxProblem

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")
from paper_2506_20994_amd import _binding as B  # noqa: E402
from paper_2506_20994_amd.box import BoxOperator  # noqa: E402


def _solve(cg, x, b, **opts):
    o, st = B._opts(**opts), B.SemSolveStats()
    cg.ctx.bind()
    rc = B.lib().sem_cg_solve(cg.handle, x.data_ptr(), b.data_ptr(), ctypes.byref(o), ctypes.byref(st))
    return rc, st.as_dict()


def _until_breakdown(ref, b):
    minv = 1.0 / ref.diagonal()
    x, r = np.zeros_like(b), b.copy()
    p = minv * r
    rz = r @ p
    for it in range(100):
        w = ref.apply(p)
        pap = p @ w
        if pap <= 0:
            return x, it
        x += rz / pap * p
        r -= rz / pap * w
        new = r @ (minv * r)
        p = minv * r + new / rz * p
        rz = new
    raise AssertionError("no breakdown")


@pytest.mark.parametrize("n,lx,h2,its", [(3, 6, -200.0, 9), (10, 8, -3000.0, 2), (11, 8, -3000.0, 2)])
def test_breakdown(sem_ctx, n, lx, h2, its):
    op = BoxOperator(sem_ctx, n, lx, 0.1)
    ref = BoxProblem(n, lx, 0.1, h2=h2)
    k, a, ph = synth.fourier_modes(3)
    b = op.fourier_rhs(k, a, ph, project=False)
    xs, count = _until_breakdown(ref, ref.fourier_rhs(k, a, ph))
    assert count == its
    cg = op.solver(P.SEM_SOLVE_F64, h2b=h2 * op.bm)
    first = None
    for check in (1, 16):               # the host looks right behind the breakdown, or later
        x = torch.empty_like(b)
        rc, st = _solve(cg, x, b, tol=1e-10, check_every=check)
        torch.cuda.synchronize()
        assert rc == P.SEM_EBREAKDOWN and st["breakdown"] and not st["converged"], st
        assert st["iterations"] == its
        xg = np.zeros(ref.nu)
        xg[ref.ids.ravel()] = x.cpu().numpy().ravel()
        assert np.max(np.abs(xg - xs)) <= 1e-9 * np.max(np.abs(xs))
        first = x if first is None else first
        assert torch.equal(x, first)
    cg.close()
    cg = op.solver(P.SEM_SOLVE_F32_IR, h2b=h2 * op.bm)
    rc, st = _solve(cg, x, b, tol=1e-10, precision=P.SEM_SOLVE_F32_IR, ir_mode=1)
    assert rc == P.SEM_EBREAKDOWN and st["breakdown"] and bool(torch.isfinite(x).all()), st
    cg.close()
    op.gs.close()
