"""The mesh's last workgroup of the whole-element kernel reads vectors that end with the last
node, and moves their values into place where elements are no whole vectors: every count of
elements that it can hold, alone and behind whole ones, all arrays inside buffers of NaN, so
that a value from past an end would show.  Oracle and bounds as in test_gpu_ax.py."""
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


def _inside(a, dt):
    """a on the GPU, between 64 values of NaN"""
    t = torch.full((a.size + 128,), float("nan"), dtype=dt, device="cuda")
    t[64:-64] = torch.from_numpy(np.ascontiguousarray(a)).reshape(-1).to(dt)
    return t[64:-64].view(a.shape)


@pytest.mark.parametrize("with_h1,with_h2", [(True, True), (False, False)])
@pytest.mark.parametrize("kind,lx", [("f64", 12), ("f32", 10), ("f32", 12), ("bf16", 8), ("bf16", 9), ("bf16", 10),
                                     ("bf16", 11), ("bf16", 12)])
def test_every_count_of_the_last_workgroup(sem_ctx, kind, lx, with_h1, with_h2):
    dt, out, q, tol = TYPES[kind]
    most = 9
    G, h1 = synth.random_spd_factors(most, lx, 930 + lx)
    u, hb = synth.local_normal(most, lx, 931 + lx), np.abs(synth.local_normal(most, lx, 932 + lx))
    G, h1, u, hb = [q(g) for g in G], q(h1), q(u), q(hb)
    M = listing_matrices(lx) if kind == "f64" else [to_f32(m) for m in listing_matrices(lx)]
    ref = ax_einsum(u, *M, h1 if with_h1 else None, *G)
    ref = ref + hb * u if with_h2 else ref
    _, _, dx, dxt = P.sem_gll(lx)
    D = [torch.from_numpy(d).cuda().to(torch.float64 if kind == "f64" else torch.float32)
         for d in (dx, dx, dx, dxt, dxt, dxt)]
    for nel in range(1, most + 1):
        w = _inside(np.zeros((nel, lx, lx, lx)), out)
        args = (sem_ctx, w, _inside(u[:nel], dt), *D, _inside(h1[:nel], dt) if with_h1 else None,
                *[_inside(g[:nel], dt) for g in G])
        if with_h2:
            P.sem_ax_helmholtz(*args, _inside(hb[:nel], dt), nel, lx)
        else:
            P.sem_ax(*args, nel, lx)
        torch.cuda.synchronize()
        got = w.double().cpu().numpy()
        assert np.max(np.abs(got - ref[:nel])) <= tol * np.max(np.abs(ref[:nel])), nel
        assert bool(w._base[:64].isnan().all()) and bool(w._base[-64:].isnan().all())
