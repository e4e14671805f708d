"""Krylov solves of the forms that the solver's whole-element operator (lx 6, 10, 12) has
beside the plain Poisson one: the mass term, which enters p^T A p by itself, Dirichlet
nodes, which its wide index loads read as -1, and the mass term beside a coefficient h1,
on 27 elements (a ragged last workgroup wherever one holds several).  And boxes on either
side of the line from which the vector kernels run 1024 threads a workgroup, with their
vectors in the last-level cache.

Against the oracle's operator and solution, bounds as in test_gpu_solve.py."""
import numpy as np
import pytest
import torch

import synth
from oracle.solve import BoxProblem, pcg

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")
from paper_2506_20994_amd.box import BoxOperator  # noqa: E402

CODE = {"f64": P.SEM_SOLVE_F64, "f32": P.SEM_SOLVE_F32_IR, "bf16": P.SEM_SOLVE_BF16_IR}
_REF = {}


def _reference(n, lx, h1u, dirichlet, h2):
    """problem, right-hand side, solution and the oracle's iterations to 1e-10; one held at a time"""
    key = (n, lx, h1u is not None, dirichlet, h2)
    if key not in _REF:
        _REF.clear()
        ref = BoxProblem(n, lx, 0.1, h1u, dirichlet=dirichlet, h2=h2)
        bref = ref.fourier_rhs(*synth.fourier_modes(3))
        minv = 1.0 / ref.diagonal()
        xs, _, hist = pcg(ref.apply, bref, minv, tol=1e-13, project=ref.project)
        _REF[key] = ref, bref, xs, next(k for k, r in enumerate(hist) if r <= 1e-10)
    return _REF[key]


def _check(ctx, n, lx, prec, dirichlet, h2, with_h1, modes):
    nu = (n * (lx - 1) - 1) ** 3 if dirichlet else (n * (lx - 1)) ** 3
    h1u = synth.unique_uniform(nu, 0.5, 2.0, 1) if with_h1 else None
    op = BoxOperator(ctx, n, lx, 0.1, h1_unique=h1u, dirichlet=dirichlet)
    ref, bref, xs, ito = _reference(n, lx, h1u, dirichlet, h2)
    b = op.fourier_rhs(*synth.fourier_modes(3), project=ref.project)
    free = ref.ids >= 0
    cg = op.solver(CODE[prec], h2b=None if h2 is None else h2 * op.bm)
    for mode in modes:
        x = torch.empty_like(b)
        rc, st = P.sem_cg_solve(cg, x, b, tol=1e-10, precision=CODE[prec], ir_mode=mode)
        torch.cuda.synchronize()
        assert rc == P.SEM_OK and st["converged"], st
        xl = x.cpu().numpy()
        assert np.all(xl[~free] == 0.0)
        xg = np.zeros(ref.nu)
        xg[ref.ids[free]] = xl[free]
        assert np.linalg.norm(bref - ref.apply(xg)) / np.linalg.norm(bref) <= 1.2e-10
        assert np.max(np.abs(xg - xs)) <= 1e-6 * np.max(np.abs(xs))
        if prec == "f64":
            assert abs(st["iterations"] - ito) <= 2, (st["iterations"], ito)
    cg.close()
    op.gs.close()


@pytest.mark.parametrize("dirichlet,h2,with_h1", [(False, 20.0, False), (True, None, False), (True, 20.0, False)])
@pytest.mark.parametrize("lx,prec", [(6, "f64"), (6, "f32"), (6, "bf16"), (10, "f32"), (10, "bf16"), (12, "f64"),
                                     (12, "f32")])
def test_whole_element_forms(sem_ctx, lx, prec, dirichlet, h2, with_h1):
    _check(sem_ctx, 3, lx, prec, dirichlet, h2, with_h1, (0,) if prec == "f64" else (1,))


@pytest.mark.parametrize("lx,prec", [(6, "f64"), (6, "f32"), (6, "bf16"), (10, "f32"), (12, "f64")])
def test_whole_element_forms_with_h1(sem_ctx, lx, prec):
    _check(sem_ctx, 3, lx, prec, False, 20.0, True, (0,) if prec == "f64" else (1,))


@pytest.mark.parametrize("n,prec,modes", [(10, "f64", (0,)), (10, "f32", (0, 1)), (10, "bf16", (0, 1)),
                                          (11, "f64", (0,)), (11, "f32", (1,)), (11, "bf16", (0,))])
def test_wide_workgroups_with_cached_vectors(sem_ctx, n, prec, modes):
    """343000 unknowns, 1340 workgroups of 256 threads, and 456533 in 512 of 1024"""
    _check(sem_ctx, n, 8, prec, False, 1e4, False, modes)
