"""The workloads this library is timed on, each one pass through its public entry points.

Five kinds, over the sizes that bench.py, sweep.py and the tests use:
  ax       the element-local operator (sem_ax, sem_ax_helmholtz) on random symmetric positive definite factors:
           the paper's grid of 128 to 32768 elements, lx 2 to 12, float64, float32 and bfloat16 storage
  apply    the assembled operator of a deformed box, BoxOperator.apply: sem_ax, then sem_gs
  solve    sem_cg_solve to a relative residual of 1e-11 (bench.py solves to 1e-10, the training's reference
           solutions to 1e-12): float64 Jacobi-PCG, float32 and bfloat16 refinement, the multigrid V-cycle;
           periodic, Dirichlet and Helmholtz boxes
  train    minibatch steps of the learned preconditioner's network, then its weights read back
  precond  the trained network applied to a residual on the unique nodes, as flexible CG calls it

`exact` is the same mathematics in plain float64 torch: its own GLL points, box geometry, operator and network.
"""
import math

import numpy as np
import torch

import paper_2506_20994_amd as P
from paper_2506_20994_amd.box import BoxOperator

DTYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
PRECISIONS = {"f64": P.SEM_SOLVE_F64, "f32": P.SEM_SOLVE_F32_IR, "bf16": P.SEM_SOLVE_BF16_IR}
MG_OPTS = dict(degree=3, lo=0.1, fine_bf16=1, galerkin=1)      # the settings bench.py solves with
NODES_MAX = 32768 * 12 ** 3


def listed():
    return [
        # the smallest point of the paper's grid: a call that is all launch and host latency
        dict(name="ax_f64_128el_lx4", kind="ax", nel=128, lx=4, dtype="f64", h1=True, h2=False),
        # the headline mesh, 32^3 elements at lx = 8, as a solver applies it: the operator, then the gather-scatter
        dict(name="apply_f64_32c_lx8", kind="apply", n=32, lx=8, amp=0.1, h1=True, dirichlet=False),
        # the highest order at the largest element count
        dict(name="ax_f64_32768el_lx12", kind="ax", nel=32768, lx=12, dtype="f64", h1=True, h2=False),
        # the Helmholtz form of a velocity solve at the paper's middle order
        dict(name="helm_f64_21952el_lx6", kind="ax", nel=21952, lx=6, dtype="f64", h1=True, h2=True),
        # float32 fields at the order of the full-stack runs
        dict(name="ax_f32_10648el_lx10", kind="ax", nel=10648, lx=10, dtype="f32", h1=False, h2=False),
        # bfloat16 factors, the storage of the mixed-precision path, on the headline mesh
        dict(name="ax_bf16_32768el_lx8", kind="ax", nel=32768, lx=8, dtype="bf16", h1=True, h2=False),
        # an odd box with u = 0 on its boundary: ragged blocks, a masked plan
        dict(name="apply_f64_19c_lx7_dir", kind="apply", n=19, lx=7, amp=0.1, h1=False, dirichlet=True),
        # a small solve, where every launch of the iteration counts
        dict(name="solve_f64_6c_lx6", kind="solve", n=6, lx=6, amp=0.1, precision="f64", ir_mode=0, mg=False,
             dirichlet=False, h2=0.0),
        # mixed precision: float32 Krylov iteration with its residual replaced in float64
        dict(name="solve_f32_16c_lx8", kind="solve", n=16, lx=8, amp=0.1, precision="f32", ir_mode=1, mg=False,
             dirichlet=False, h2=0.0),
        # the production solve: multigrid inside residual replacement on the headline mesh
        dict(name="solve_mg_32c_lx8", kind="solve", n=32, lx=8, amp=0.1, precision="f32", ir_mode=1, mg=True,
             n_coarse=8, dirichlet=False, h2=0.0),
        # training the preconditioner that solves with: the linear form, energy-norm loss, batches of 1024
        dict(name="train_lx8_b1024", kind="train", lx=8, hidden=256, batch=1024, steps=8, linear=True),
        # one application of the network with its hidden layers (ReLU) to a float32 residual
        dict(name="precond_20c_lx8", kind="precond", n=20, lx=8, amp=0.1, linear=False, dtype="f32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ax", "ax", "ax", "ax", "apply", "apply", "solve", "solve", "train", "precond"])
    if kind == "ax":
        return dict(kind=kind, nel=_log_int(rng, 64, 32768), lx=rng.randint(2, 12),
                    dtype=rng.choice(["f64", "f64", "f64", "f32", "bf16"]), h1=rng.random() < 0.5,
                    h2=rng.random() < 0.3)
    if kind == "apply":
        lx = rng.randint(2, 12)
        return dict(kind=kind, n=_log_int(rng, 3, max(4, 224 // lx)), lx=lx, amp=round(rng.uniform(0.02, 0.08), 3),
                    h1=rng.random() < 0.5, dirichlet=rng.random() < 0.4)
    if kind == "solve":
        lx = rng.randint(4, 10)
        mg = rng.random() < 0.4
        n = rng.choice([4, 6, 8, 10, 12, 16]) if mg else _log_int(rng, 3, max(4, 84 // (lx - 1)))
        case = dict(kind=kind, n=n, lx=lx, amp=round(rng.uniform(0.02, 0.08), 3),
                    precision=rng.choice(["f64", "f32"]) if mg else rng.choice(["f64", "f64", "f32", "bf16"]),
                    ir_mode=1 if mg else rng.choice([0, 1]), mg=mg, dirichlet=rng.random() < 0.4,
                    h2=rng.choice([0.0, 0.0, 20.0]))
        if mg:
            case["n_coarse"] = 2
        return case
    if kind == "train":
        return dict(kind=kind, lx=rng.choice([4, 6, 8, 10]), hidden=rng.choice([128, 256]),
                    batch=8 * _log_int(rng, 8, 128), steps=rng.randint(2, 8), linear=rng.random() < 0.5)
    lx = rng.choice([4, 6, 8, 10])
    return dict(kind="precond", n=_log_int(rng, 3, 192 // lx), lx=lx, amp=round(rng.uniform(0.02, 0.08), 3),
                linear=rng.random() < 0.5, dtype=rng.choice(["f64", "f32"]))


# ------------------------------------------------------------------ inputs, from the seed alone
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 62))


def _randn(g, *shape, dtype=torch.float64):
    return torch.randn(*shape, generator=g, dtype=dtype, device="cuda")


def _rand(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, dtype=torch.float64, device="cuda")


def _ax_fields(case, seed):
    """u ~ N(0, 1); per node G = L L^T + 0.1 I, L lower triangular N(0, 1); h1 ~ U[0.5, 2]; h2 B ~ U[0.1, 1];
    in the storage type."""
    g, dt = _gen(seed), DTYPES[case["dtype"]]
    shp = (case["nel"],) + (case["lx"],) * 3
    f = {"u": _randn(g, *shp).to(dt)}
    l11, l21, l22, l31, l32, l33 = (_randn(g, *shp) for _ in range(6))
    f["G"] = tuple(t.to(dt) for t in (l11 * l11 + 0.1, l21 * l21 + l22 * l22 + 0.1,
                                      l31 * l31 + l32 * l32 + l33 * l33 + 0.1,
                                      l11 * l21, l11 * l31, l21 * l31 + l22 * l32))
    f["h1"] = _rand(g, 0.5, 2.0, *shp).to(dt) if case["h1"] else None
    f["h2b"] = _rand(g, 0.1, 1.0, *shp).to(dt) if case["h2"] else None
    return f


def _unique_count(case):
    m = case["n"] * (case["lx"] - 1)
    return (m - 1) ** 3 if case.get("dirichlet") else m ** 3


def _box_fields(case, seed):
    """u ~ N(0, 1) and h1 ~ U[0.5, 2] on the lattice of unique nodes."""
    g, nu = _gen(seed), _unique_count(case)
    return _randn(g, nu), (_rand(g, 0.5, 2.0, nu) if case["h1"] else None)


def _solution(case, seed):
    """The solution a solve has to find, on the lattice of unique nodes: 32 Fourier modes of the undeformed
    position (|k| <= 8), times the sines that vanish on the boundary of a Dirichlet box, or less its mean where the
    periodic operator leaves it open."""
    n, lx, dirichlet = case["n"], case["lx"], case["dirichlet"]
    r = np.random.Generator(np.random.PCG64(int(seed)))
    k = r.integers(-8, 9, size=(32, 3))
    k[np.all(k == 0, axis=1)] = 1
    amp, phase = r.standard_normal(32), r.uniform(0.0, 2.0 * np.pi, 32)
    xi = _gll(lx)[0]
    X = ((np.arange(n)[:, None] + 0.5 * (1.0 + xi[None, :-1])) / n).ravel()
    X = torch.from_numpy(X[1:] if dirichlet else X).cuda()
    out = torch.zeros((X.numel(),) * 3, dtype=torch.float64, device="cuda")
    for (a, b, c), am, ph in zip(k, amp, phase):
        wave = [torch.exp(2j * math.pi * float(q) * X) for q in (a, b, c)]
        plane = (wave[1][:, None] * wave[0][None, :]) * (am * np.exp(1j * ph))
        out += wave[2].real[:, None, None] * plane.real - wave[2].imag[:, None, None] * plane.imag
    if dirichlet:
        s = torch.sin(math.pi * X)
        out *= s[:, None, None] * s[None, :, None] * s[None, None, :]
    elif not case["h2"]:
        out -= out.mean()
    return out.reshape(-1)


def _train_data(case, seed):
    """Feature rows (unit residual, the six geometric means or zeros, padding) and targets of 4 batches, He weights."""
    g = _gen(seed)
    n, h = case["lx"] ** 3, case["hidden"]
    rows = 4 * case["batch"]
    X = torch.zeros(rows, (n + 6 + 15) // 16 * 16, dtype=torch.float64, device="cuda")
    r = _randn(g, rows, n)
    X[:, :n] = r / r.norm(dim=1, keepdim=True)
    if not case["linear"]:
        X[:, n:n + 3] = _rand(g, 0.7, 1.4, rows, 3)
        X[:, n + 3:n + 6] = 0.1 * _randn(g, rows, 3)
    T = 0.5 * X[:, :n].roll(1, 1) + 0.3 * X[:, :n] + 0.01 * _randn(g, rows, n)
    order = torch.cat([torch.randperm(rows, generator=g, device="cuda")
                       for _ in range((case["steps"] + 3) // 4)])[:case["steps"] * case["batch"]]
    return X.to(torch.bfloat16), T.to(torch.float32), order, _weights(g, n, h)


def _weights(g, n, h):
    """He-initialised float32 weights and small biases of the (n + 6)-h-h-n network."""
    sizes = (n + 6, h, h, n)
    out = []
    for a, b in zip(sizes[:-1], sizes[1:]):
        out.append((_randn(g, b, a) * math.sqrt(2.0 / a)).float())
        out.append((0.01 * _randn(g, b)).float())
    return out


def _precond_data(case, seed):
    """A residual ~ N(0, 1) per unique node, the network's weights; the linear form gets W = M M^T / n, the symmetric
    positive definite element block that training ends at, through sem_lp_set_block."""
    g = _gen(seed)
    n = case["lx"] ** 3
    r = _randn(g, _unique_count(case)).to(DTYPES[case["dtype"]])
    if case["linear"]:
        M = _randn(g, n, n)
        return r, ((M @ M.T) / n).float()
    return r, _weights(g, n, 256)


def prepare(case, seed):
    torch.cuda.set_device(0)
    ctx = P.sem_create()
    kind, lx = case["kind"], case["lx"]
    if kind == "ax":
        f = _ax_fields(case, seed)
        dt = torch.float64 if case["dtype"] == "f64" else torch.float32
        _, _, dx, dxt = P.sem_gll(lx)
        D = [torch.from_numpy(d).to("cuda", dt) for d in (dx, dx, dx, dxt, dxt, dxt)]
        w = torch.empty(f["u"].shape, dtype=dt, device="cuda")
        return dict(f, case=case, ctx=ctx, D=D, w=w)
    if kind == "train":
        X, T, order, weights = _train_data(case, seed)
        lp = P.sem_lp_create(ctx, case["batch"], lx, case["hidden"])
        if case["linear"]:
            P.sem_lp_set_linear(lp, True)
            P.sem_lp_set_metric(lp, 1.0)
        for s, v in enumerate(weights):
            P.sem_lp_set(lp, s, v.cpu().numpy())
        loss = torch.zeros(case["steps"], dtype=torch.float32, device="cuda")
        rows = [order[q * case["batch"]:(q + 1) * case["batch"]].contiguous() for q in range(case["steps"])]
        return dict(case=case, ctx=ctx, lp=lp, X=X, T=T, rows=rows, loss=loss)
    op = BoxOperator(ctx, case["n"], lx, case["amp"], keep_coords=False, dirichlet=case.get("dirichlet", False))

    def scatter(v):
        out = torch.empty(op.ids.shape, dtype=v.dtype, device="cuda")
        P.sem_scatter(ctx, out, v, op.ids)
        return out

    if kind == "apply":
        u, h1 = _box_fields(case, seed)
        u = scatter(u)
        op.h1 = None if h1 is None else scatter(h1)
        return dict(case=case, op=op, u=u, w=torch.empty_like(u))
    if kind == "solve":
        xs = scatter(_solution(case, seed))
        b = torch.empty_like(xs)
        h2b = case["h2"] * op.bm if case["h2"] else None
        if h2b is None:
            op.apply(b, xs)
        else:
            P.sem_ax_helmholtz(ctx, b, xs, *op.D, None, *op.G, h2b, op.nel, lx)
            P.sem_gs(op.gs, b)
        code = PRECISIONS[case["precision"]]
        mg = op.multigrid(h2=case["h2"], n_coarse=case["n_coarse"], **MG_OPTS) if case["mg"] else None
        cg = op.solver(code, h2b=h2b, mg=mg)
        return dict(case=case, op=op, b=b, x=torch.empty_like(b), cg=cg, mg=mg, h2b=h2b,
                    opts=dict(tol=1e-11, precision=code, ir_mode=case["ir_mode"], mg=mg))
    r, net = _precond_data(case, seed)
    lp = P.sem_lp_create(ctx, op.nel, lx)
    if case["linear"]:
        P.sem_lp_set_jacobi_base(lp, True)
        P.sem_lp_set_block(lp, net.cpu().numpy())
    else:
        for s, v in enumerate(net):
            P.sem_lp_set(lp, s, v.cpu().numpy())
    op.bind(lp)
    # the layout that solvers iterate in: unique nodes in the order of their first local copy
    r = r[_first_seen(op.ids)[0]].contiguous()
    return dict(case=case, op=op, lp=lp, r=r, z=torch.empty_like(r))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "ax":
        args = (state["ctx"], state["w"], state["u"], *state["D"], state["h1"], *state["G"])
        if state["h2b"] is None:
            P.sem_ax(*args, case["nel"], case["lx"])
        else:
            P.sem_ax_helmholtz(*args, state["h2b"], case["nel"], case["lx"])
        return state["w"]
    if kind == "apply":
        state["op"].apply(state["w"], state["u"])
        return state["w"]
    if kind == "solve":
        P.sem_cg_solve(state["cg"], state["x"], state["b"], **state["opts"])
        return state["x"]
    if kind == "train":
        lp, loss = state["lp"], state["loss"]
        for q, rows in enumerate(state["rows"]):
            P.sem_lp_train_step(lp, state["X"], state["T"], rows, 3e-4, loss[q:q + 1])
        return {"loss": loss, "weights": [P.sem_lp_get(lp, s) for s in range(6)]}
    P.sem_lp_apply_unique(state["lp"], state["z"], state["r"])
    return state["z"]


def work(case):
    lx = case["lx"]
    if case["kind"] == "train":
        n, h = lx ** 3, case["hidden"]
        params = (n + 6) * h + h * h + h * n
        # forward, both backward products (+ the metric's); per step: rows in, the weights and both Adam moments
        # read and written
        flops = case["steps"] * case["batch"] * (6 * params + (2 * n * n if case["linear"] else 0))
        return {"bytes": float(case["steps"] * (case["batch"] * (2 * (n + 6) + 4 * n) + 24 * params)),
                "flops": float(flops)}
    nel = case["nel"] if case["kind"] == "ax" else case["n"] ** 3
    nodes = nel * lx ** 3
    if case["kind"] == "ax":
        size = {"f64": 8, "f32": 4, "bf16": 2}[case["dtype"]]
        per = size * (7 + bool(case["h1"]) + bool(case["h2"])) + (8 if size == 8 else 4)
        return {"bytes": float(per * nodes), "flops": float((12 * lx + 18) * nodes)}
    nu = _unique_count(case)
    if case["kind"] == "apply":
        return {"bytes": float((64 + 8 * bool(case["h1"])) * nodes), "flops": float((12 * lx + 18) * nodes)}
    if case["kind"] == "precond":
        n, size = lx ** 3, DTYPES[case["dtype"]].itemsize
        flops = 2 * nel * (n * n if case["linear"] else (n + 6) * 256 + 256 * 256 + 256 * n)
        # the residual in, z out, the node numbering
        return {"bytes": float(2 * size * nu + 4 * nodes), "flops": float(flops)}
    # solve: iterations of this tolerance times one operator application (factors, node numbering) and the vectors'
    # reads and writes (x, r, p both ways, Minv)
    m = case["n"] * (lx - 1)
    its = 29 if case["mg"] else max(20, 11.5 * m / (1.0 + case["h2"] / 40.0) ** 0.5)
    size, factor = (8, 48) if case["precision"] == "f64" else (4, 24 if case["precision"] == "f32" else 12)
    per = nodes * (factor + 4) + nu * 7 * size
    flops = (12 * lx + 18) * nodes
    if case["mg"]:      # six operator applications of the V-cycle on its finest level in bfloat16
        per += 6 * (nodes * 16 + nu * 16)
        flops *= 7
    return {"bytes": float(its * per), "flops": float(its * flops)}


# ------------------------------------------------------------------ the same mathematics in float64 torch
def _gll(lx):
    """Nodes, weights and D[i, l] = l_l'(x_i) of the Gauss-Lobatto-Legendre points."""
    N = lx - 1
    leg = np.polynomial.legendre.Legendre.basis(N)
    x = np.concatenate([[-1.0], np.sort(leg.deriv().roots().real), [1.0]])
    for _ in range(3):      # Newton on P_N' for the inner nodes
        x[1:-1] -= leg.deriv()(x[1:-1]) / leg.deriv(2)(x[1:-1]) if lx > 2 else 0.0
    p = leg(x)
    w = 2.0 / (N * (N + 1) * p * p)
    D = np.zeros((lx, lx))
    for i in range(lx):
        for j in range(lx):
            if i != j:
                D[i, j] = p[i] / (p[j] * (x[i] - x[j]))
    D[0, 0], D[-1, -1] = -N * (N + 1) / 4.0, N * (N + 1) / 4.0
    return x, w, D


def _grad(D, f):
    lx = D.shape[0]
    r = f @ D.T
    s = torch.matmul(D, f)
    t = torch.matmul(D, f.reshape(-1, lx, lx * lx)).reshape(f.shape)
    return r, s, t


def _operator(D, u, G, h1=None, h2b=None):
    """w = D^T (h1 G D u) + h2b u, in slabs of elements."""
    out = torch.empty_like(u)
    step = max(1, (1 << 24) // u[0].numel())
    for a in range(0, u.shape[0], step):
        s = slice(a, a + step)
        r = _grad(D, u[s])
        g = [t[s] for t in G]
        h = 1.0 if h1 is None else h1[s]
        v = [h * (g[0] * r[0] + g[3] * r[1] + g[4] * r[2]), h * (g[3] * r[0] + g[1] * r[1] + g[5] * r[2]),
             h * (g[4] * r[0] + g[5] * r[1] + g[2] * r[2])]
        out[s] = _grad(D.T, v[0])[0] + _grad(D.T, v[1])[1] + _grad(D.T, v[2])[2]
        if h2b is not None:
            out[s] += h2b[s] * u[s]
    return out


def _ids(n, lx, dirichlet):
    """Global ids (e, k, j, i); -1 on the boundary of the Dirichlet box."""
    N, M = lx - 1, n * (lx - 1)
    g = torch.arange(n, device="cuda")[:, None] * N + torch.arange(lx, device="cuda")      # (element, node) of a line
    K, J, I = (g[:, None, None, :, None, None], g[None, :, None, None, :, None], g[None, None, :, None, None, :])
    if dirichlet:
        inside = [(q > 0) & (q < M) for q in (K, J, I)]
        ids = ((K - 1) * (M - 1) + (J - 1)) * (M - 1) + (I - 1)
        ids = torch.where(inside[0] & inside[1] & inside[2], ids, -torch.ones_like(ids))
    else:
        ids = ((K % M) * M + J % M) * M + I % M
    return ids.reshape(n ** 3, lx, lx, lx)


def _box(n, lx, amp):
    """Factors of the deformed box: x = X + amp sin(2 pi Y) sin(2 pi Z), cyclically."""
    xi, w, D = _gll(lx)
    p = torch.from_numpy((np.arange(n)[:, None] + 0.5 * (1.0 + xi)) / n).cuda()
    shape = (n, n, n, lx, lx, lx)
    X, Y, Z = (q.expand(shape).reshape(-1, lx, lx, lx) for q in (
        p[None, None, :, None, None, :], p[None, :, None, None, :, None], p[:, None, None, :, None, None]))
    s = [torch.sin(2.0 * math.pi * q) for q in (X, Y, Z)]
    Dt, w = torch.from_numpy(D).cuda(), torch.from_numpy(w).cuda()
    J = [_grad(Dt, c) for c in (X + amp * s[1] * s[2], Y + amp * s[2] * s[0], Z + amp * s[0] * s[1])]   # dx_c / dr_a
    det = (J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) - J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0])
           + J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]))

    def cof(a, c):      # det * dr_a / dx_c
        a1, a2, c1, c2 = (a + 1) % 3, (a + 2) % 3, (c + 1) % 3, (c + 2) % 3
        return J[c1][a1] * J[c2][a2] - J[c1][a2] * J[c2][a1]

    scale = w[:, None, None] * w[None, :, None] * w / det
    return tuple(scale * sum(cof(a, c) * cof(b, c) for c in range(3))
                 for a, b in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)))


def _sum_copies(v, ids, nu):
    """Sum over the local copies of each unique node."""
    i = ids.reshape(-1)
    ok = i >= 0
    return torch.zeros(nu, dtype=v.dtype, device="cuda").index_add_(0, i[ok], v.reshape(-1)[ok])


def _to_local(v, ids):
    return torch.where(ids >= 0, v[ids.clamp(min=0)], torch.zeros((), dtype=v.dtype, device="cuda"))


def _first_seen(ids):
    """Unique ids in the order of their first local copy, and the position of each id in that order."""
    flat = ids.reshape(-1)
    nu = int(flat.max()) + 1
    first = torch.full((nu,), flat.numel(), dtype=torch.int64, device="cuda")
    first.scatter_reduce_(0, flat, torch.arange(flat.numel(), device="cuda"), "amin")
    order = torch.argsort(first)
    place = torch.empty_like(order)
    place[order] = torch.arange(nu, device="cuda")
    return order, place


def _net(weights, X, linear):
    W1, b1, W2, b2, W3, b3 = weights
    if linear:
        y1 = X @ W1.T
        y2 = y1 @ W2.T
        return y1, y2, y2 @ W3.T
    y1 = torch.relu(X @ W1.T + b1)
    y2 = torch.relu(y1 @ W2.T + b2)
    return y1, y2, y2 @ W3.T + b3


def _metric(lx):
    """K = the reference element's stiffness + mass, over the mean of w_i w_j w_k."""
    _, w, D = _gll(lx)
    w, D = torch.from_numpy(w).cuda(), torch.from_numpy(D).cuda()
    K1, B1 = D.T @ (w[:, None] * D), torch.diag(w)
    K = (torch.kron(B1, torch.kron(B1, K1)) + torch.kron(B1, torch.kron(K1, B1)) + torch.kron(K1, torch.kron(B1, B1))
         + torch.kron(B1, torch.kron(B1, B1)))
    return K / w.mean() ** 3


def _train_exact(case, seed):
    X, T, order, weights = _train_data(case, seed)
    n, lin, B = case["lx"] ** 3, case["linear"], case["batch"]
    p = [v.double() for v in weights]
    m, v = [torch.zeros_like(q) for q in p], [torch.zeros_like(q) for q in p]
    K, losses = _metric(case["lx"]) if lin else None, []
    for q in range(case["steps"]):
        rows = order[q * B:(q + 1) * B]
        x, t = X[rows][:, :n + 6].double(), T[rows].double()
        y1, y2, y3 = _net(p, x, lin)
        d = y3 - t
        if lin:
            kd = d @ K
            losses.append((d * kd).sum(1).mean())
            d3 = 2.0 * kd / B
        else:
            losses.append((d * d).mean())
            d3 = 2.0 * d / d.numel()
        d2 = d3 @ p[4] if lin else (d3 @ p[4]) * (y2 > 0)
        d1 = d2 @ p[2] if lin else (d2 @ p[2]) * (y1 > 0)
        g = [d1.T @ x, d1.sum(0), d2.T @ y1, d2.sum(0), d3.T @ y2, d3.sum(0)]
        if lin:
            g[1], g[3], g[5] = 0 * g[1], 0 * g[3], 0 * g[5]
        for a in range(6):
            m[a] = 0.9 * m[a] + 0.1 * g[a]
            v[a] = 0.999 * v[a] + 0.001 * g[a] * g[a]
            p[a] = p[a] - 3e-4 * (m[a] / (1 - 0.9 ** (q + 1))) / ((v[a] / (1 - 0.999 ** (q + 1))).sqrt() + 1e-8)
    return {"loss": torch.stack(losses), "weights": p}


def _precond_exact(case, seed):
    n, lx = case["n"], case["lx"]
    ids, nu, nl = _ids(n, lx, False), _unique_count(case), lx ** 3
    order, _ = _first_seen(ids)
    r, net = _precond_data(case, seed)
    G = _box(n, lx, case["amp"])
    ru = r.double()
    mult = _sum_copies(torch.ones(ids.shape, dtype=torch.float64, device="cuda"), ids, nu)
    kappa = ((G[0] + G[1] + G[2]).reshape(-1, nl).mean(1) / 3.0)[:, None]
    v = ru[ids].reshape(-1, nl)
    if not case["linear"]:
        s = v.norm(dim=1, keepdim=True)
        geo = torch.stack([g.reshape(-1, nl).mean(1) for g in G], 1) / kappa
        y = _net([q.double() for q in net], torch.cat([v / s, geo], 1), False)[2]
        return (_sum_copies(y * (s / kappa), ids, nu) / mult)[order]
    S = mult.rsqrt()
    z = (S[ids].reshape(-1, nl) * v) @ net.double() / kappa
    _, _, D = _gll(lx)
    D2 = torch.from_numpy(D).cuda()
    dd, sq = torch.diagonal(D2), (D2 * D2).T      # sq[i, l] = D[l, i]^2
    diag = _grad(sq, G[0])[0] + _grad(sq, G[1])[1] + _grad(sq, G[2])[2]
    di, dj, dk = dd[None, None, :], dd[None, :, None], dd[:, None, None]
    diag = diag + 2.0 * (di * dj * G[3] + di * dk * G[4] + dj * dk * G[5])
    return (S * _sum_copies(z, ids, nu) + ru / _sum_copies(diag, ids, nu))[order]


def exact(case, seed):
    kind, lx = case["kind"], case["lx"]
    if kind == "train":
        return _train_exact(case, seed)
    if kind == "precond":
        return _precond_exact(case, seed)
    D = torch.from_numpy(_gll(lx)[2]).cuda()
    if kind == "ax":
        f = _ax_fields(case, seed)
        dbl = lambda t: None if t is None else t.double()      # noqa: E731
        return _operator(D, f["u"].double(), [t.double() for t in f["G"]], dbl(f["h1"]), dbl(f["h2b"]))
    ids = _ids(case["n"], lx, case["dirichlet"])
    if kind == "solve":
        return _to_local(_solution(case, seed), ids)
    u, h1 = _box_fields(case, seed)
    w = _operator(D, _to_local(u, ids), _box(case["n"], lx, case["amp"]), None if h1 is None else _to_local(h1, ids))
    return _to_local(_sum_copies(w, ids, _unique_count(case)), ids)
