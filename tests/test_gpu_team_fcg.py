"""Flexible CG with a system's own polynomial by teams of workgroups
(csrc/team_fcg.hip): sizes at the edges of a member (2048 rows) and of the
64-row slices, one member and several, rows of five and of seven entries.

The states, operations and orders of the sums are those of the tile kernels,
so a batch gives the same bits as with the tiles' sizes set; against the
oracle the repository's bar holds (iterations +-1, relative difference 1e-9
at rtol 1e-10)."""
import numpy as np
import pytest

import oracle
from oracle import learned as OL
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


def case(shape, seed, factor=100, coef=None):
    """(system, nine coefficients, lambda_max)."""
    rng = np.random.default_rng(seed)
    A = P.diffusion_csr(np.exp(rng.standard_normal(shape)), aniso=2.0)
    lm = oracle.gershgorin(A)[1]
    c = OL.chebyshev_iteration_coeffs(lm / factor, lm) if coef is None else np.array(coef)
    return P.System(A=A, b=rng.uniform(-1, 1, A.n)), c.astype(np.float32), lm


def solve(apcg, ctx, cases, rtol, maxit, tiles=False, x0s=None, **fo):
    import torch
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    As, bs = [DeviceCSR(s.A) for s, _, _ in cases], [DeviceVec(s.b) for s, _, _ in cases]
    xs = [DeviceVec(np.zeros(s.A.n) if x0s is None else x0s[i]) for i, (s, _, _) in enumerate(cases)]
    C = torch.from_numpy(np.concatenate([c for _, c, _ in cases])).cuda()
    lm = torch.tensor([v for _, _, v in cases], dtype=torch.float64).cuda()
    torch.cuda.synchronize()
    info = apcg.apcg_info_create(0, len(cases))
    opts = apcg.apcg_solve_opts_default(x0_is_zero=int(x0s is None), batch_tile_rows=1024 if tiles else 0)
    apcg.apcg_counters_reset()
    apcg.apcg_ksp_solve_batched_fcg_poly(ctx, [a.h for a in As], [b.h for b in bs], [x.h for x in xs], rtol, maxit, C,
                                         lm, opts, apcg.apcg_fcg_opts_default(**fo) if fo else None, info)
    graphs = apcg.apcg_counters_get()["graph_launches"]
    assert (graphs > 0) == tiles
    out = [apcg.apcg_info_get(info, i) for i in range(len(cases))], [x.numpy() for x in xs]
    apcg.apcg_info_destroy(info)
    return out


def assert_same(a, b):
    assert repr(a[0]) == repr(b[0])  # (a NaN is not equal to itself)
    assert all(np.array_equal(p, q, equal_nan=True) for p, q in zip(a[1], b[1]))


SETS = {
    "5": [(1, 1), (1, 65), (32, 64), (3, 683), (61, 67), (64, 64), (17, 241), (128, 130), (2, 9000)],
    "7": [(12, 13, 14), (2, 32, 32), (13, 14, 15), (3, 41, 53), (64, 66), (2, 1024, 3)],
}


@pytest.mark.parametrize("which", sorted(SETS))
def test_team_fcg_bitwise_equals_tiles(apcg, ctx, which):
    cases = [case(s, i) for i, s in enumerate(SETS[which])]
    print(f"case team fcg entries={which}", flush=True)
    x0s = [np.random.default_rng(9).uniform(-1, 1, s.A.n) for s, _, _ in cases]
    for args, kw in (((1e-8, 20000), {}), ((0.0, 7), {}), ((1e-8, 20000), {"x0s": x0s})):
        assert_same(*(solve(apcg, ctx, cases, *args, tiles=t, **kw) for t in (False, True)))


def test_team_fcg_states(apcg, ctx):
    """A polynomial with a negative value (solved without it), the identity, a
    poor one, a zero and a NaN right-hand side, a bad diagonal, an indefinite
    operator, and the stall rule with and without the way out."""
    cases = [case((70, 70), 0, coef=[0.2, -0.5] + [0] * 7), case((70, 71), 1, coef=[1] + [0] * 8),
             case((90, 90), 2, factor=3), case((60, 50), 3), case((60, 51), 4), case((60, 52), 5), case((60, 53), 6)]
    cases[3][0].b[:] = 0.0
    cases[4][0].b[2500] = np.nan
    d = cases[5][0].A
    d.val[[e for e in range(d.rowptr[2100], d.rowptr[2101]) if d.col[e] == 2100][0]] = -1.0
    d = cases[6][0].A
    off = d.col != np.repeat(np.arange(d.n), np.diff(d.rowptr))
    d.val[off] *= 1.5
    print("case team fcg states", flush=True)
    for fo in ({}, {"fallback": 0}, {"stall_min": 3, "stall_frac": 0.0},
               {"stall_min": 3, "stall_frac": 0.0, "fallback": 0}):
        assert_same(*(solve(apcg, ctx, cases, 1e-8, 500, tiles=t, **fo) for t in (False, True)))


def solve_single(apcg, ctx, c, mode, rtol, maxit):
    import torch
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    s, coef, lm = c
    dA, db, dx = DeviceCSR(s.A), DeviceVec(s.b), DeviceVec.zeros(s.A.n)
    C, L = torch.from_numpy(coef).cuda(), torch.tensor([lm], dtype=torch.float64).cuda()
    torch.cuda.synchronize()
    info = apcg.apcg_info_create(0, 1)
    apcg.apcg_counters_reset()
    apcg.apcg_ksp_solve_fcg_poly(ctx, dA.h, db.h, dx.h, rtol, maxit, C, L,
                                 apcg.apcg_solve_opts_default(x0_is_zero=1, mode=mode), None, info, 0)
    graphs = apcg.apcg_counters_get()["graph_launches"]
    r, x = apcg.apcg_info_get(info, 0), dx.numpy()
    apcg.apcg_info_destroy(info)
    return r, x, graphs


@pytest.mark.parametrize("shape", [(1, 8193), (12, 1000), (23, 21, 25), (6, 41, 53)])
def test_team_fcg_single_matches_oracle(apcg, ctx, shape):
    s, c, lm = case(shape, 11)
    print(f"case team fcg single {shape}", flush=True)
    ref = oracle.fcg_poly(s.A, s.b, c.astype(np.float64), lm, rtol=1e-10, maxit=20000)
    r, x, graphs = solve_single(apcg, ctx, (s, c, lm), apcg.APCG_MODE_GRAPH, 1e-10, 20000)
    assert graphs == 0 and abs(r["iterations"] - ref.its) <= 1
    assert np.linalg.norm(x - ref.x) <= 1e-9 * np.linalg.norm(ref.x)


def test_team_fcg_one_sided_pattern_uses_kernels(apcg, ctx):
    """Row 2048 names row 2047 of the member before it, which names nothing
    back: the members refuse, and the kernels solve the system."""
    s, c, lm = case((1, 10000), 12)
    A = s.A
    keep = np.ones(A.col.size, bool)
    keep[[e for e in range(A.rowptr[2047], A.rowptr[2048]) if A.col[e] == 2048]] = False
    rp = np.concatenate([[0], np.cumsum(np.add.reduceat(keep, A.rowptr[:-1]))]).astype(np.int32)
    one = P.System(A=P.CSR(n=A.n, rowptr=rp, col=A.col[keep], val=A.val[keep]), b=s.b)
    print("case team fcg one-sided pattern", flush=True)
    a = solve_single(apcg, ctx, (one, c, lm), apcg.APCG_MODE_GRAPH, 0.0, 6)
    b = solve_single(apcg, ctx, (one, c, lm), apcg.APCG_MODE_STREAM, 0.0, 6)
    assert a[2] > 0 and a[0] == b[0] and np.array_equal(a[1], b[1])
