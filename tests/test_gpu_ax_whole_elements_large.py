"""The whole-element kernel at the orders that take it for large arrays only: every form
(h1, none, the mass term without h1; test_gpu_ax_whole_elements.py has both) on either side
of the size from which it runs, with a ragged last workgroup, and non-finite values, which
stay in their element.  The kernel sums each direction by itself and the column mapping all
three in one chain, so the same elements' results differ in their last bits across that
size: that says which kernel ran.

61 elements repeated, every copy against the oracle's 61, bounds as in test_gpu_ax.py."""
import numpy as np
import pytest
import torch

import synth
from oracle.ax import ax_einsum
from oracle.gll import listing_matrices
from oracle.quant import to_f32
from tests.test_gpu_ax_whole_elements import TYPES

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")

ORDERS = [("f64", 5), ("f64", 6), ("f32", 4), ("f32", 5), ("f32", 6), ("f32", 7),
          ("bf16", 4), ("bf16", 5), ("bf16", 6), ("bf16", 7)]
PERIOD = 61


def _first_count(kind, lx, with_h2):
    """the first element count whose arrays (u, w, h1, six factors, h2 B) reach the size"""
    least = (40 if kind == "bf16" and lx >= 6 else 320) << 20
    return -(-least // (lx ** 3 * (10 if with_h2 else 9) * {"f64": 8, "f32": 4, "bf16": 2}[kind]))


class _Fields:
    def __init__(self, kind, lx):
        self.kind, self.lx = kind, lx
        self.dt, self.out, q, self.tol = TYPES[kind]
        G, h1 = synth.random_spd_factors(PERIOD, lx, 920 + lx)
        u, hb = synth.local_normal(PERIOD, lx, 921 + lx), np.abs(synth.local_normal(PERIOD, lx, 922 + lx))
        self.G, self.h1, self.u, self.hb = [q(g) for g in G], q(h1), q(u), q(hb)
        self.M = listing_matrices(lx) if kind == "f64" else [to_f32(m) for m in listing_matrices(lx)]
        dd = torch.float64 if kind == "f64" else torch.float32
        _, _, dx, dxt = P.sem_gll(lx)
        self.D = [torch.from_numpy(d).cuda().to(dd) for d in (dx, dx, dx, dxt, dxt, dxt)]

    def repeated(self, a, nel):
        t = torch.from_numpy(np.ascontiguousarray(a)).cuda().to(self.dt)
        return t[torch.arange(nel, device="cuda") % PERIOD].contiguous()

    def run(self, ctx, nel, with_h1, with_h2, poison=()):
        u = self.repeated(self.u, nel)
        for e in poison:
            u[e, 1, 2, 1] = float("nan")
        buf = torch.full((u.numel() + 9,), 7.0, dtype=self.out, device="cuda")
        w = buf[:u.numel()].view(u.shape)
        args = (ctx, w, u, *self.D, self.repeated(self.h1, nel) if with_h1 else None,
                *[self.repeated(g, nel) for g in self.G])
        if with_h2:
            P.sem_ax_helmholtz(*args, self.repeated(self.hb, nel), nel, self.lx)
        else:
            P.sem_ax(*args, nel, self.lx)
        torch.cuda.synchronize()
        assert bool((buf[u.numel():] == 7.0).all())
        return w


@pytest.mark.parametrize("with_h1,with_h2", [(True, False), (False, False), (False, True)])
@pytest.mark.parametrize("kind,lx", ORDERS)
def test_forms_on_either_side(sem_ctx, kind, lx, with_h1, with_h2):
    f = _Fields(kind, lx)
    ref = ax_einsum(f.u, *f.M, f.h1 if with_h1 else None, *f.G)
    ref = torch.from_numpy(ref + f.hb * f.u if with_h2 else ref).cuda()
    edge = _first_count(kind, lx, with_h2)
    got = {nel: f.run(sem_ctx, nel, with_h1, with_h2) for nel in (edge - 1, edge, edge + 1)}
    for nel, w in got.items():
        worst = max(float((w[k:k + 61 * 64].double() - ref[torch.arange(k, min(k + 61 * 64, nel), device="cuda") % PERIOD])
                          .abs().max()) for k in range(0, nel, 61 * 64))
        assert worst <= f.tol * float(ref.abs().max()), nel
    assert torch.equal(got[edge][:PERIOD], got[edge + 1][:PERIOD])
    assert not torch.equal(got[edge][:PERIOD], got[edge - 1][:PERIOD])


@pytest.mark.parametrize("kind,lx", ORDERS)
def test_nan_stays_in_its_element(sem_ctx, kind, lx):
    f = _Fields(kind, lx)
    nel = _first_count(kind, lx, True) + 1
    nel += 1 - nel % 2                  # odd: the last workgroup of four elements or more is ragged
    clean = f.run(sem_ctx, nel, True, True)
    bad = (0, 20, nel // 2, nel - 1)
    got = f.run(sem_ctx, nel, True, True, bad)
    keep = torch.ones(nel, dtype=torch.bool, device="cuda")
    keep[list(bad)] = False
    assert torch.equal(got[keep], clean[keep])
    assert all(bool(got[e].isnan().any()) for e in bad)
