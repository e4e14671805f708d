"""sem_operator_t promises no more for h1 and h2 B than the alignment of a float64 (a view
into a buffer): solves with both one value into theirs equal, bit for bit, those with arrays
of their own, at the orders whose float64 operator reads them in wide vectors (lx = 6, 12;
the refinements through their float64 residual) and at one of the others."""
import pytest
import torch

import synth
from paper_2506_20994_amd import _binding as B

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2506_20994_amd")
from paper_2506_20994_amd.box import BoxOperator  # noqa: E402


def _moved(t):
    return torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)[1:].view(t.shape).copy_(t)


@pytest.mark.parametrize("lx,prec", [(6, "f64"), (12, "f64"), (8, "f64"), (6, "f32"), (12, "bf16")])
def test_coefficients_off_16_bytes(sem_ctx, lx, prec):
    n, h2 = 3, 20.0                     # 27 elements: a ragged last workgroup at lx = 6
    op = BoxOperator(sem_ctx, n, lx, 0.1, h1_unique=synth.unique_uniform((n * (lx - 1)) ** 3, 0.5, 2.0, 1))
    k, a, ph = synth.fourier_modes(3)
    b = op.fourier_rhs(k, a, ph, project=False)
    code = {"f64": P.SEM_SOLVE_F64, "f32": P.SEM_SOLVE_F32_IR, "bf16": P.SEM_SOLVE_BF16_IR}[prec]
    hb, out = h2 * op.bm, []
    for h1, h2b in ((op.h1, hb), (_moved(op.h1), _moved(hb))):
        assert (h1.data_ptr() | h2b.data_ptr()) % 16 == (8 if out else 0)
        cg = B.sem_cg_setup(sem_ctx, op.gs, op.D, h1, op.G, op.nel, lx, h2b=h2b, precision=code)
        x = torch.empty_like(b)
        rc, st = P.sem_cg_solve(cg, x, b, tol=1e-10, precision=code, ir_mode=0 if prec == "f64" else 1)
        torch.cuda.synchronize()
        assert rc == P.SEM_OK and st["converged"], st
        out.append((x, st["iterations"]))
        cg.close()
    assert out[0][1] == out[1][1] and torch.equal(out[0][0], out[1][0])
    op.gs.close()
