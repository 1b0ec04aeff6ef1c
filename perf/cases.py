"""Performance cases: the work a user of the library has it do, through the
public entry points, over the range of sizes and options it is used at.

listed() names the cases, draw() gives further ones of the same ranges,
prepare() builds what a program holds before the call (systems in GPU memory,
a context, options, network weights), run() makes one pass, work() counts what
a pass cannot do without and exact() computes the same outputs with plain
torch in 64 bits.

Kinds
  solve        one Jacobi-PCG solve (apcg_ksp_solve) to a tolerance, or the
               stencil benchmark's fixed number of iterations
  tfqmr        a fixed number of TFQMR iterations on a convection-diffusion
               operator (apcg_ksp_solve_tfqmr)
  composed     CG written with the asynchronous vector and matrix calls
  batch        a batch of uneven systems in one apcg_ksp_solve_batched call
  learned      one system through the learned polynomial preconditioner
  learned_batch  a mixed 2D / 3D batch through it in one call
  train        one training step of the preconditioner's network
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2306_17801_amd as apcg
from paper_2306_17801_amd import composed, problems
from paper_2306_17801_amd.device import DeviceCSR, DeviceVec
from paper_2306_17801_amd.learned import pack_params

DEV = "cuda:0"
MAXIT = 20000
NPARAM, NFEAT, NCOEF = 5833, 16, 9


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # the smallest solve: 4,096 rows, bound by latency; parity tolerance
        dict(name="solve_poisson2d_64", kind="solve", problem="poisson", ny=64, nx=64, nz=0, points=5, rtol=1e-10,
             its=0, mode="auto", layout="default"),
        # a small ragged 2D log-normal system as a user solves it untuned
        dict(name="solve_2d_ragged_30k", kind="solve", problem="lognormal", ny=173, nx=173, nz=0, points=5, rtol=1e-10,
             its=0, mode="graph", layout="default", sigma=1.0, aniso=3.0),
        # an ordinary 3D system, untuned, at the benchmark's tolerance
        dict(name="solve_3d_64", kind="solve", problem="smoothed", ny=64, nx=64, nz=64, points=7, rtol=1e-8, its=0,
             mode="graph", layout="default"),
        # the benchmark's headline solve at the layout its autotuner picks
        dict(name="solve_3d_128_tuned", kind="solve", problem="smoothed", ny=128, nx=128, nz=128, points=7, rtol=1e-8,
             its=0, mode="graph", layout="march8"),
        # the paper's protocol on the widest stencil: exactly 20 iterations
        dict(name="solve20_27point_96", kind="solve", problem="laplace", ny=96, nx=96, nz=96, points=27, rtol=0.0,
             its=20, mode="graph", layout="default"),
        # the paper's second method, same protocol, a ragged 3D grid
        dict(name="tfqmr20_3d_ragged", kind="tfqmr", problem="convection", ny=61, nx=83, nz=70, points=7, its=20,
             layout="default"),
        # CG out of single asynchronous calls: launch-bound and bandwidth-bound
        dict(name="composed20_2d_64", kind="composed", problem="laplace", ny=64, nx=64, nz=0, points=5, its=20),
        dict(name="composed20_3d_128", kind="composed", problem="laplace", ny=128, nx=128, nz=128, points=7, its=20),
        # hundreds of uneven systems in one call
        dict(name="batch2d_256", kind="batch", dim="2", count=256, n_lo=1024, n_hi=65536, sigma=1.0, aniso=1.0,
             rtol=1e-8, layout="default"),
        # the learned preconditioner on one held-out-sized 3D system
        dict(name="learned_3d_64", kind="learned", problem="lognormal", ny=64, nx=64, nz=64, points=7, sigma=1.2,
             aniso=10.0, rtol=1e-8, layout="sdia"),
        # and on a mixed 2D / 3D batch
        dict(name="learned_mixed_48", kind="learned_batch", dim="mixed", count=48, n_lo=1000, n_hi=100000, sigma=1.2,
             aniso=30.0, rtol=1e-8, layout="sdia"),
        # one Adam step of the network on a minibatch
        dict(name="train_step_128", kind="train", batch=128),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _grid(rng, dim, n):
    """A ragged grid of about n cells."""
    side = n ** (1.0 / dim)
    f = rng.uniform(0.75, 1.3)
    ny = max(3, round(side * f))
    if dim == 2:
        return dict(ny=ny, nx=max(3, round(n / ny)), nz=0)
    nx = max(3, round(side))
    return dict(ny=ny, nx=nx, nz=max(3, round(n / (nx * ny))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve20", "tfqmr", "composed", "batch", "learned", "learned_batch",
                       "train"])
    dim = rng.choice([2, 3])
    star = 5 if dim == 2 else 7
    if kind == "solve":
        n = _log_uniform(rng, 1e3, 2.6e5 if dim == 2 else 2.0e6)
        return dict(kind="solve", problem="lognormal", points=star, rtol=rng.choice([1e-8, 1e-10]), its=0,
                    mode=rng.choice(["auto", "graph"]), layout=rng.choice(["default", "sdia"]),
                    sigma=rng.uniform(0.5, 1.5), aniso=_log_uniform(rng, 1.0, 10.0), **_grid(rng, dim, n))
    if kind == "solve20":
        n = _log_uniform(rng, 1e3, 2.0e6)
        return dict(kind="solve", problem="laplace", points=rng.choice([5, 9] if dim == 2 else [7, 27]), rtol=0.0,
                    its=20, mode="graph", layout=rng.choice(["default", "sdia"]), **_grid(rng, dim, n))
    if kind == "tfqmr":
        n = _log_uniform(rng, 1e3, 1.5e6)
        return dict(kind="tfqmr", problem="convection", points=star, its=20, layout="default", **_grid(rng, dim, n))
    if kind == "composed":
        n = _log_uniform(rng, 1e3, 2.0e6)
        return dict(kind="composed", problem="laplace", points=star, its=20, **_grid(rng, dim, n))
    if kind == "batch":
        return dict(kind="batch", dim=rng.choice(["2", "mixed"]), count=round(_log_uniform(rng, 8, 160)), n_lo=1000,
                    n_hi=round(_log_uniform(rng, 4e3, 6e4)), sigma=rng.uniform(0.5, 1.5),
                    aniso=_log_uniform(rng, 1.0, 10.0), rtol=1e-8, layout=rng.choice(["default", "sdia"]))
    if kind == "learned":
        n = _log_uniform(rng, 4e3, 8e5 if dim == 3 else 1e5)
        return dict(kind="learned", problem="lognormal", points=star, sigma=rng.uniform(0.5, 1.5),
                    aniso=_log_uniform(rng, 1.0, 30.0), rtol=1e-8, layout=rng.choice(["default", "sdia"]),
                    **_grid(rng, dim, n))
    if kind == "learned_batch":
        return dict(kind="learned_batch", dim=rng.choice(["2", "mixed"]), count=round(_log_uniform(rng, 6, 48)),
                    n_lo=1000, n_hi=round(_log_uniform(rng, 4e3, 1e5)), sigma=rng.uniform(0.5, 1.5),
                    aniso=_log_uniform(rng, 1.0, 30.0), rtol=1e-8, layout=rng.choice(["default", "sdia"]))
    return dict(kind="train", batch=round(_log_uniform(rng, 16, 2000)))


# --------------------------------------------------------------- the systems

def _shape(case):
    return (case["nz"], case["ny"], case["nx"]) if case["nz"] else (case["ny"], case["nx"])


def _generator(seed, device):
    return torch.Generator(device=device).manual_seed(int(seed) & 0x7FFFFFFF)


def _lognormal(shape, sigma, aniso, gen, device):
    """CSR arrays and right-hand side of a log-normal diffusion system."""
    k = torch.exp(sigma * torch.randn(shape, generator=gen, dtype=torch.float64, device=device))
    A = problems.diffusion_csr_torch(k, aniso)
    b = 2.0 * torch.rand(math.prod(shape), generator=gen, dtype=torch.float64, device=device) - 1.0
    return A, b


def _arrays(case, seed, device):
    """((rowptr, col, val), b) on `device`, drawn from the seed alone."""
    gen = _generator(seed, device)
    shape = _shape(case)
    n = math.prod(shape)
    if case["problem"] == "lognormal":
        return _lognormal(shape, case["sigma"], case["aniso"], gen, device)
    if case["problem"] == "smoothed":  # k = exp of a 3^d box mean of N(0,1)
        g = torch.randn([s + 2 for s in shape], generator=gen, dtype=torch.float64, device=device)
        for axis in range(len(shape)):
            g = g.unfold(axis, 3, 1).mean(-1)
        A = problems.diffusion_csr_torch(torch.exp(g).contiguous())
    else:
        if case["problem"] == "convection":
            M = problems.convection_diffusion(shape, (0.3, -0.2, 0.5)[: len(shape)])
        else:
            M = problems.stencil_laplacian(shape, case["points"])
        A = tuple(torch.from_numpy(np.ascontiguousarray(a)).to(device) for a in (M.rowptr, M.col, M.val))
    b = 2.0 * torch.rand(n, generator=gen, dtype=torch.float64, device=device) - 1.0
    if case["problem"] == "poisson":  # manufactured: b = A x*, x* uniform
        b = _matrix(A, n) @ b
    return A, b


def _batch_arrays(case, seed, device):
    """The systems of a batch: sizes log-uniform in [n_lo, n_hi] (2D sides
    uniform), dimension 2 or mixed, sigma and anisotropy around the case's --
    all drawn from the case -- and fields and right-hand sides drawn from the
    seed."""
    rng = np.random.default_rng([case["count"], case["n_lo"], case["n_hi"]])
    gen = _generator(seed, device)
    out = []
    for _ in range(case["count"]):
        dim = 2 if case["dim"] == "2" else int(rng.integers(2, 4))
        if case["dim"] == "2":
            lo, hi = math.sqrt(case["n_lo"]), math.sqrt(case["n_hi"])
            side = int(rng.integers(round(lo), round(hi) + 1))
        else:
            n = math.exp(rng.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))
            side = max(2, round(n ** (1.0 / dim)))
        sigma = case["sigma"] * rng.uniform(0.8, 1.2)
        aniso = max(1.0, case["aniso"] ** rng.uniform(0.0, 1.0))
        out.append(_lognormal((side,) * dim, sigma, aniso, gen, device))
    return out


def _network(seed):
    """Weights of a trained network as the library keeps them: the output
    bias carries the degree-8 Chebyshev semi-iterative polynomial on
    [lmax / 100, lmax] of a diagonally scaled diffusion matrix (lmax = 2),
    the hidden layers shift it a little from system to system."""
    lmax, a = 2.0, 0.02
    T9 = np.polynomial.chebyshev.Chebyshev.basis(NCOEF)
    s0 = (lmax + a) / (lmax - a)

    def p(y):
        t = 0.5 * (y + 1.0) * lmax
        return (1.0 - T9((lmax + a - 2.0 * t) / (lmax - a)) / T9(s0)) / t

    params = problems.mlp_initial_params(7)
    params["W3"] = 1e-3 * params["W3"]
    params["b3"] = np.polynomial.chebyshev.chebinterpolate(p, NCOEF - 1)
    f32 = lambda v: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).to(DEV)  # noqa: E731
    mean = np.array([4.5, 6.0, 0.0, 2.0, 1.0, 0.7, 1.0, .01, .05, .1, .8, .85, .9, 2.0, -1.0, -2.0])
    return f32(pack_params(params)), f32(mean), f32(np.full(NFEAT, 0.5))


# ----------------------------------------------------------------- the state

class _State:
    """A program's context and result records, and what the case adds;
    released with the state."""

    def __init__(self, case, records):
        self.case = case
        self.ctx = apcg.apcg_ctx_create(0)
        self.info = apcg.apcg_info_create(0, records)
        self.opts = apcg.apcg_solve_opts_default(x0_is_zero=1)

    def __del__(self):
        try:
            apcg.apcg_info_destroy(self.info)
            apcg.apcg_ctx_destroy(self.ctx)
        except Exception:
            pass


def _layout(A, layout):
    """The product schedule a program has chosen; a pattern that does not
    allow it stays on the default."""
    lanes = {"sdia": 1, "march8": 8}.get(layout)
    if lanes is None:
        return
    try:
        apcg.apcg_mat_set_spmv_config(A.h, lanes, 256, 0, apcg.APCG_SPMV_SDIA)
    except apcg.ApcgError:
        pass


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        s = _State(case, 1)
        for name, t in _train_arrays(case, seed, DEV).items():
            setattr(s, name, t.to(torch.float32).contiguous())
        s.loss = torch.zeros(1, dtype=torch.float32, device=DEV)
    elif kind in ("batch", "learned_batch"):
        arrays = _batch_arrays(case, seed, DEV)
        s = _State(case, len(arrays))
        s.A = [DeviceCSR.from_tensors(*A) for A, _ in arrays]
        s.b = [DeviceVec(b) for _, b in arrays]
        # the solutions lie in one tensor, each from a multiple of 64 entries on
        off = _offsets([a.n for a in s.A])
        s.solution = torch.zeros(off[-1], dtype=torch.float64, device=DEV)
        s.x = [DeviceVec(s.solution[o:o + a.n]) for a, o in zip(s.A, off)]
        for a in s.A:
            _layout(a, case["layout"])
        s.hA, s.hb, s.hx = ([v.h for v in vs] for vs in (s.A, s.b, s.x))
    else:
        A, b = _arrays(case, seed, DEV)
        s = _State(case, 1)
        s.A, s.b = DeviceCSR.from_tensors(*A), DeviceVec(b)
        s.x = DeviceVec.zeros(s.A.n)
        _layout(s.A, case.get("layout"))
        if kind == "solve":
            s.opts.mode = apcg.APCG_MODE_AUTO if case["mode"] == "auto" else apcg.APCG_MODE_GRAPH
        if kind == "composed":
            s.cg = composed.ComposedCG(s.ctx, s.A.n)
            s.diag = float(2 * len(_shape(case)))
    if kind in ("learned", "learned_batch"):
        s.params, s.mean, s.std = _network(seed)
    torch.cuda.synchronize()
    return s


def run(s):
    case = s.case
    kind = case["kind"]
    if kind == "solve":
        apcg.apcg_ksp_solve(s.ctx, s.A.h, s.b.h, s.x.h, case["rtol"], case["its"] or MAXIT, s.opts, s.info, 0)
        return s.x.t
    if kind == "tfqmr":
        apcg.apcg_ksp_solve_tfqmr(s.ctx, s.A.h, s.b.h, s.x.h, 0.0, case["its"], s.opts, s.info, 0)
        return s.x.t
    if kind == "composed":
        apcg.apcg_vec_set_async(s.x.h, 0.0, s.ctx)
        res = s.cg.solve(s.A.h, s.b.h, s.x.h, s.diag, case["its"])
        return [s.x.t, res]
    if kind == "batch":
        apcg.apcg_ksp_solve_batched(s.ctx, s.hA, s.hb, s.hx, case["rtol"], MAXIT, s.opts, s.info)
        return s.solution
    if kind == "learned":
        apcg.apcg_ksp_solve_learned(s.ctx, s.A.h, s.b.h, s.x.h, case["rtol"], MAXIT, s.params, s.mean, s.std, s.opts,
                                    None, s.info, 0)
        return s.x.t
    if kind == "learned_batch":
        apcg.apcg_ksp_solve_batched_learned(s.ctx, s.hA, s.hb, s.hx, case["rtol"], MAXIT, s.params, s.mean, s.std,
                                            s.opts, None, s.info)
        return s.solution
    apcg.apcg_mlp_train_step(s.ctx, s.params, s.m, s.v, 100, 3e-3, s.X, s.G, s.h, s.loss)
    return [s.params, s.m, s.v, s.loss]


def _offsets(sizes):
    """Where each of the vectors of these sizes begins in one tensor (a
    multiple of 64 entries), and the tensor's length."""
    return [0] + [int(o) for o in np.cumsum([(n + 63) // 64 * 64 for n in sizes])]


# -------------------------------------------------------- work and exactness

def _sizes(case):
    """(rows, nonzeros) of a single system."""
    shape = _shape(case)
    n = math.prod(shape)
    if case["points"] in (5, 7):
        return n, n + 2 * sum(n // s * (s - 1) for s in shape)
    return n, math.prod(3 * s - 2 for s in shape)


def work(case):
    """Each input read once and each output written once; operations of the
    iterations a fixed-count pass makes, or of as many as the grid is long
    (a lower bound of what reaching the tolerance takes)."""
    kind = case["kind"]
    if kind == "train":
        B = case["batch"]
        weights = 16 * 64 + 64 * 64 + 64 * 9
        return {"bytes": 4.0 * (B * (NFEAT + NCOEF * NCOEF + NCOEF) + 6 * NPARAM),
                "flops": 6.0 * B * weights + B * (4.0 * 81 + 4.0 * 64 * 9) + 12.0 * NPARAM}
    if kind in ("batch", "learned_batch"):
        if case["dim"] == "2":  # sides uniform
            lo, hi = math.sqrt(case["n_lo"]), math.sqrt(case["n_hi"])
            mean = (hi ** 3 - lo ** 3) / (3.0 * (hi - lo))
        else:
            mean = (case["n_hi"] - case["n_lo"]) / math.log(case["n_hi"] / case["n_lo"])
        n = case["count"] * mean
        nnz = n * (5.0 if case["dim"] == "2" else 6.0)
        its = mean ** (0.5 if case["dim"] == "2" else 0.4)
    else:
        n, nnz = _sizes(case)
        its = case.get("its") or max(_shape(case))
    per_iteration = 2.0 * nnz + 12.0 * n
    if kind == "tfqmr":
        per_iteration *= 2.0
    if kind in ("learned", "learned_batch"):  # one product more per polynomial degree, far fewer iterations
        its, per_iteration = max(10.0, its / 4.0), 18.0 * nnz + 40.0 * n
    return {"bytes": 12.0 * nnz + 4.0 * n + 16.0 * n, "flops": its * per_iteration}


def _matrix(A, n):
    return torch.sparse_csr_tensor(A[0].to(torch.int64), A[1].to(torch.int64), A[2], size=(n, n))


def _diagonal(A, n):
    rows = torch.repeat_interleave(torch.arange(n, device=A[0].device), (A[0][1:] - A[0][:-1]).to(torch.int64))
    d = torch.zeros(n, dtype=torch.float64, device=A[0].device)
    on = A[1].to(torch.int64) == rows
    d[rows[on]] = A[2][on]
    return d


def _reference_cg(A, b, its=0, limit=30000):
    """Jacobi-PCG from x = 0: exactly `its` iterations, or until the
    residual stands at the rounding of the right-hand side."""
    n = b.numel()
    M, dinv = _matrix(A, n), 1.0 / _diagonal(A, n)
    x, r = torch.zeros_like(b), b.clone()
    z = dinv * r
    p, rho = z.clone(), torch.dot(r, z)
    stop = 1e-14 * float(torch.linalg.norm(b))
    for k in range(1, (its or limit) + 1):
        w = M @ p
        alpha = rho / torch.dot(p, w)
        x += alpha * p
        r -= alpha * w
        z = dinv * r
        if not its and k % 50 == 0 and float(torch.linalg.norm(r)) <= stop:
            break
        rho, old = torch.dot(r, z), rho
        p = z + (rho / old) * p
    return x, float(torch.linalg.norm(r))


def _reference_tfqmr(A, b, its):
    """Freund's TFQMR from x = 0, left Jacobi preconditioning, two products
    per iteration."""
    n = b.numel()
    M, dinv = _matrix(A, n), 1.0 / _diagonal(A, n)
    r0 = dinv * b
    x, w, y1, d = torch.zeros_like(b), r0.clone(), r0.clone(), torch.zeros_like(b)
    u1 = dinv * (M @ y1)
    v = u1.clone()
    tau, theta, eta, rho = torch.linalg.norm(r0), 0.0, 0.0, torch.dot(r0, r0)
    for _ in range(its):
        alpha = rho / torch.dot(r0, v)
        y2 = y1 - alpha * v
        u2 = dinv * (M @ y2)
        for y, u in ((y1, u1), (y2, u2)):
            d = y + (theta * theta * eta / alpha) * d
            w = w - alpha * u
            theta = torch.linalg.norm(w) / tau
            c2 = 1.0 / (1.0 + theta * theta)
            tau, eta = tau * theta * torch.sqrt(c2), c2 * alpha
            x = x + eta * d
        rho, old = torch.dot(r0, w), rho
        beta = rho / old
        y1 = w + beta * y2
        u1 = dinv * (M @ y1)
        v = u1 + beta * (u2 + beta * v)
    return x


def _train_arrays(case, seed, device):
    """A minibatch of standardised features and loss forms, and a network
    with Adam moments some way into training (all rounded to float32)."""
    gen = _generator(seed, "cpu")
    B = case["batch"]
    normal = lambda *s: torch.randn(s, generator=gen, dtype=torch.float64)  # noqa: E731
    params = torch.from_numpy(pack_params(problems.mlp_initial_params(int(seed) % 1000)).astype(np.float64))
    Q = normal(B, NCOEF, NCOEF)
    G = Q @ Q.transpose(1, 2) / NCOEF + 0.05 * torch.eye(NCOEF, dtype=torch.float64)
    out = dict(params=params + 0.01 * normal(NPARAM), m=1e-3 * normal(NPARAM), v=1e-4 * (0.5 + normal(NPARAM) ** 2),
               X=normal(B, NFEAT), G=G.reshape(B, NCOEF * NCOEF), h=0.3 * normal(B, NCOEF))
    return {k: t.to(torch.float32).to(torch.float64).to(device) for k, t in out.items()}


def _reference_train(case, seed, device, t=100, lr=3e-3, mu=1.0, eps=0.05):
    a = _train_arrays(case, seed, device)
    flat = a["params"].clone().requires_grad_(True)
    cut = torch.split(flat, [64 * 16, 64, 64 * 64, 64, 9 * 64, 9])
    h1 = torch.tanh(a["X"] @ cut[0].view(64, 16).T + cut[1])
    h2 = torch.tanh(h1 @ cut[2].view(64, 64).T + cut[3])
    C = h2 @ cut[4].view(9, 64).T + cut[5]
    y = torch.linspace(-1.0, 1.0, 64, dtype=torch.float64, device=device)
    T = [torch.ones_like(y), y]
    for _ in range(NCOEF - 2):
        T.append(2.0 * y * T[-1] - T[-2])
    low = torch.clamp(eps - C @ torch.stack(T), min=0.0)
    G = a["G"].view(-1, NCOEF, NCOEF)
    loss = ((C[:, None, :] @ G @ C[:, :, None]).reshape(-1) - 2.0 * (a["h"] * C).sum(1) + 1.0
            + mu / 64.0 * (low * low).sum(1)).mean()
    g, = torch.autograd.grad(loss, flat)
    m = 0.9 * a["m"] + 0.1 * g
    v = 0.999 * a["v"] + 0.001 * g * g
    p = a["params"] - lr * (m / (1.0 - 0.9 ** t)) / (torch.sqrt(v / (1.0 - 0.999 ** t)) + 1e-8)
    return [p, m, v, loss.detach().reshape(1)]


def exact(case, seed):
    device = DEV if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    if kind == "train":
        return _reference_train(case, seed, device)
    if kind in ("batch", "learned_batch"):
        systems = _batch_arrays(case, seed, device)
        # one block-diagonal system
        n = [b.numel() for _, b in systems]
        row0 = np.concatenate([[0], np.cumsum(n)])
        nnz0 = np.concatenate([[0], np.cumsum([A[1].numel() for A, _ in systems])])
        rp = torch.cat([A[0][:-1].to(torch.int64) + int(o) for (A, _), o in zip(systems, nnz0)]
                       + [torch.tensor([int(nnz0[-1])], device=device)])
        cl = torch.cat([A[1].to(torch.int64) + int(o) for (A, _), o in zip(systems, row0)])
        x, _ = _reference_cg((rp, cl, torch.cat([A[2] for A, _ in systems])), torch.cat([b for _, b in systems]))
        off = _offsets(n)
        out = torch.zeros(off[-1], dtype=torch.float64, device=device)
        for o, part in zip(off, torch.split(x, n)):
            out[o:o + part.numel()] = part
        return out
    A, b = _arrays(case, seed, device)
    if kind == "tfqmr":
        return _reference_tfqmr(A, b, case["its"])
    x, res = _reference_cg(A, b, case.get("its", 0))
    return [x, res] if kind == "composed" else x
