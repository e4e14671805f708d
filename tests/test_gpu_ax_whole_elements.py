"""The whole-element kernel of the operator (matrix-core products of an element's
lines) at its edges: element counts that leave the last workgroup ragged or
make it the only one, the Helmholtz term, no h1, at the orders that run it at
every size (the rows of the short orders at these counts run the column mapping;
test_gpu_ax_whole_elements_large.py has their whole elements); the size from
which short orders take it; arrays that do not lie on
its access width (a view into a buffer
takes the column mapping); non-finite values, which stay in their element; and
the solver's form with its plane layout of the factors.

Bounds as in test_gpu_ax.py: float64 1e-12, the others 1e-5 of the largest value
against the oracle on the stored inputs; the solves as in test_gpu_solve.py."""
import numpy as np
import pytest
import torch

import synth
from oracle.ax import ax_einsum
from oracle.gll import listing_matrices
from oracle.quant import to_bf16, to_f32
from oracle.solve import pcg
from tests.test_gpu_solve import _setup, _unique

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")

TYPES = {"f64": (torch.float64, torch.float64, lambda a: a, 1e-12),
         "f32": (torch.float32, torch.float32, to_f32, 1e-5),
         "bf16": (torch.bfloat16, torch.float32, to_bf16, 1e-5)}


def _device(a, dt, shift=0):
    """a on the GPU, `shift` values into its buffer"""
    t = torch.empty(a.size + shift, dtype=dt, device="cuda")[shift:].view(a.shape)
    t.copy_(torch.from_numpy(np.ascontiguousarray(a)))
    return t


def _case(nel, lx, kind, with_h1, with_h2, shift=0, poison=None):
    """(GPU result as float64, oracle result); the values after w are checked"""
    dt, out, q, _ = TYPES[kind]
    G, h1 = synth.random_spd_factors(nel, lx, 900 + lx)
    u = synth.local_normal(nel, lx, 901 + lx)
    hb = np.abs(synth.local_normal(nel, lx, 902 + lx))
    G, h1, u, hb = [q(g) for g in G], q(h1), q(u), q(hb)
    if poison is not None:
        u[poison] = np.nan
    dd = torch.float64 if kind == "f64" else torch.float32
    _, _, dx, dxt = P.sem_gll(lx)
    D = [torch.from_numpy(d).cuda().to(dd) for d in (dx, dx, dx, dxt, dxt, dxt)]
    buf = torch.full((u.size + shift + 9,), 7.0, dtype=out, device="cuda")
    w = buf[shift:shift + u.size].view(u.shape)
    ctx = P.sem_create()
    args = (ctx, w, _device(u, dt, shift), *D, _device(h1, dt, shift) if with_h1 else None,
            *[_device(g, dt, shift) for g in G])
    if with_h2:
        P.sem_ax_helmholtz(*args, _device(hb, dt, shift), nel, lx)
    else:
        P.sem_ax(*args, nel, lx)
    torch.cuda.synchronize()
    ctx.close()
    assert bool((buf[:shift] == 7.0).all()) and bool((buf[shift + u.size:] == 7.0).all())
    M = listing_matrices(lx) if kind == "f64" else [to_f32(m) for m in listing_matrices(lx)]
    ref = ax_einsum(u, *M, h1 if with_h1 else None, *G)
    return w.double().cpu().numpy(), ref + hb * u if with_h2 else ref


def _close(got, ref, kind):
    assert np.max(np.abs(got - ref)) <= TYPES[kind][3] * np.max(np.abs(ref))


@pytest.mark.parametrize("kind", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("lx", list(range(4, 13)))
def test_ragged_element_counts(lx, kind):
    for nel, h1, h2 in ((1, True, False), (3, False, True), (33, True, True), (67, True, False)):
        got, ref = _case(nel, lx, kind, h1, h2)
        _close(got, ref, kind)


@pytest.mark.parametrize("kind", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("lx", [4, 5, 6, 10, 12])
def test_arrays_off_the_access_width(lx, kind):
    got, ref = _case(35, lx, kind, True, True, shift=1)
    _close(got, ref, kind)


@pytest.mark.parametrize("kind,lx", [("f64", 5), ("f64", 6), ("f32", 4), ("f32", 5), ("f32", 6), ("f32", 7),
                                     ("bf16", 4), ("bf16", 5), ("bf16", 6), ("bf16", 7)])
def test_orders_that_take_it_for_large_arrays(lx, kind):
    """either side of 320 MB of arrays (bfloat16 lx = 6, 7: 40 MB), and there off the access width: 61 elements
    repeated, every copy against the oracle's 61"""
    dt, out, q, tol = TYPES[kind]
    size = {"f64": 8, "f32": 4, "bf16": 2}[kind]
    least = (40 if kind == "bf16" and lx >= 6 else 320) << 20
    edge = -(-least // (lx ** 3 * 10 * size))  # the first element count of that size
    p = 61
    G, h1 = synth.random_spd_factors(p, lx, 910 + lx)
    u, hb = synth.local_normal(p, lx, 911 + lx), np.abs(synth.local_normal(p, lx, 912 + lx))
    G, h1, u, hb = [q(g) for g in G], q(h1), q(u), q(hb)
    M = listing_matrices(lx) if kind == "f64" else [to_f32(m) for m in listing_matrices(lx)]
    ref = torch.from_numpy(ax_einsum(u, *M, h1, *G) + hb * u).cuda()
    dd = torch.float64 if kind == "f64" else torch.float32
    _, _, dx, dxt = P.sem_gll(lx)
    D = [torch.from_numpy(d).cuda().to(dd) for d in (dx, dx, dx, dxt, dxt, dxt)]
    ctx = P.sem_create()
    for nel, shift in ((edge - 1, 0), (edge, 0), (edge + 1, 0), (edge, 1)):
        idx = torch.arange(nel, device="cuda") % p

        def field(a, dtype=dt):
            t = torch.empty(nel * lx ** 3 + shift, dtype=dtype, device="cuda")[shift:].view(nel, lx, lx, lx)
            return t.copy_(torch.from_numpy(np.ascontiguousarray(a)).cuda().reshape(p, lx, lx, lx)[idx])

        w = field(u, out).fill_(7.0)
        P.sem_ax_helmholtz(ctx, w, field(u), *D, field(h1), *[field(g) for g in G], field(hb), nel, lx)
        torch.cuda.synchronize()
        worst = max(float((w[k:k + 4096].double() - ref.reshape(p, lx, lx, lx)[idx[k:k + 4096]]).abs().max())
                    for k in range(0, nel, 4096))
        assert worst <= tol * float(ref.abs().max()), (nel, shift)
    ctx.close()


@pytest.mark.parametrize("kind,lx", [("f64", 5), ("f64", 12), ("f32", 4), ("f32", 7), ("bf16", 8), ("bf16", 11)])
def test_nan_stays_in_its_element(lx, kind):
    clean, _ = _case(37, lx, kind, True, True)
    got, _ = _case(37, lx, kind, True, True, poison=(20, 1, 2, 1))
    assert np.isnan(got[20]).any()
    keep = np.arange(37) != 20
    assert np.array_equal(got[keep], clean[keep])


@pytest.mark.parametrize("lx,prec,h1", [(5, "f64", True), (6, "f64", False), (4, "f32", True), (5, "f32", False),
                                        (6, "f32", True), (10, "f32", False), (4, "bf16", False), (5, "bf16", True),
                                        (6, "bf16", False), (10, "bf16", True)])
def test_solver_form(sem_ctx, lx, prec, h1):
    op, b, ref, bref = _setup(sem_ctx, 3, lx, 0.1, with_h1=h1)
    code = {"f64": P.SEM_SOLVE_F64, "f32": P.SEM_SOLVE_F32_IR, "bf16": P.SEM_SOLVE_BF16_IR}[prec]
    cg = op.solver(code)
    x = torch.empty_like(b)
    rc, st = P.sem_cg_solve(cg, x, b, tol=1e-10, precision=code, ir_mode=0 if prec == "f64" else 1)
    torch.cuda.synchronize()
    assert rc == P.SEM_OK and st["converged"], st
    xg = _unique(ref, x.cpu().numpy())
    assert np.linalg.norm(bref - ref.apply(xg)) / np.linalg.norm(bref) <= 1.2e-10
    xs, _, _ = pcg(ref.apply, bref, 1.0 / ref.diagonal(), tol=1e-13)
    assert np.max(np.abs(xg - xs)) <= 1e-6 * np.max(np.abs(xs))
    cg.close()
