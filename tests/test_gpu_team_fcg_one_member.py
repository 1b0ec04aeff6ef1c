"""Flexible CG of systems that one workgroup holds (at most 2048 rows), solved
by Jacobi-PCG after their polynomial was rejected, after a stall or because
r.z fails at the start: the meetings of one member follow each other without
the barriers of the polynomial's steps.  The same bits as with the tiles'
sizes set, every time."""
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


def case(shape, seed, coef=None):
    rng = np.random.default_rng(seed)
    A = P.diffusion_csr(np.exp(rng.standard_normal(shape)), aniso=2.0)
    lm = oracle.gershgorin(A)[1]
    c = OL.chebyshev_iteration_coeffs(lm / 100, lm) if coef is None else np.array(coef)
    return P.System(A=A, b=rng.uniform(-1, 1, A.n)), c.astype(np.float32), lm


def solver(apcg, ctx, cases):
    import torch
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    As, bs = [DeviceCSR(s.A) for s, _, _ in cases], [DeviceVec(s.b) for s, _, _ in cases]
    xs = [DeviceVec.zeros(s.A.n) for s, _, _ in cases]
    C = torch.from_numpy(np.concatenate([c for _, c, _ in cases])).cuda()
    lm = torch.tensor([v for _, _, v in cases], dtype=torch.float64).cuda()
    torch.cuda.synchronize()
    info = apcg.apcg_info_create(0, len(cases))

    def solve(tiles, **fo):
        opts = apcg.apcg_solve_opts_default(x0_is_zero=1, batch_tile_rows=1024 if tiles else 0)
        apcg.apcg_ksp_solve_batched_fcg_poly(ctx, [a.h for a in As], [b.h for b in bs], [x.h for x in xs], 1e-9, 400,
                                             C, lm, opts, apcg.apcg_fcg_opts_default(**fo), info)
        return [apcg.apcg_info_get(info, i) for i in range(len(cases))], [x.numpy() for x in xs]

    return solve


@pytest.mark.parametrize("fo", [{}, {"stall_min": 2, "stall_frac": 0.0}], ids=["default", "stall"])
def test_one_member_fallback_bitwise_equals_tiles(apcg, fo):
    bad = [0.2, -0.5] + [0] * 7  # negative somewhere: rejected
    cases = [case(s, i, bad if i % 2 else None)
             for i, s in enumerate([(1, 2), (1, 64), (9, 9), (32, 64), (45, 45), (12, 13, 13), (31, 66), (40, 51)] * 4)]
    d = cases[4][0].A  # r.z <= 0 after the hand-over: indefinite
    d.val[d.col != np.repeat(np.arange(d.n), np.diff(d.rowptr))] *= 1.6
    print(f"case one member fallback {fo}", flush=True)
    ctx = apcg.apcg_ctx_create(0)
    solve = solver(apcg, ctx, cases)
    want = solve(True, **fo)
    for _ in range(5):
        got = solve(False, **fo)
        assert repr(got[0]) == repr(want[0])
        assert all(np.array_equal(p, q, equal_nan=True) for p, q in zip(got[1], want[1]))
    assert any(r["status"] & apcg.APCG_SOLVE_FALLBACK for r in want[0])
    apcg.apcg_ctx_destroy(ctx)
