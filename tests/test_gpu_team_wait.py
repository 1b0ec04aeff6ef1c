"""Waits of a team that run out (csrc/team.h).  The limit is set so low that
members leave all the time, in the middle of a solve, at its end and before
their team is complete: every kernel ends by itself, a system's x is either
solved or as it was, and the result is that of a solve from the given x0 in
any case."""
import ctypes

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


# (ticks of 10 ns, looks between two readings of the clock less one): at the
# first unsuccessful look; after 5 us; after 30 us
WAITS = [(-1, 0), (500, 0), (3000, 3)]


def impatient(apcg, wait):
    """A context of its own: after a wait has run out, a context leaves its
    next solves to the kernels."""
    c = apcg.apcg_ctx_create(0)
    f = apcg.load().apcg_internal_set_team_wait
    f.argtypes, f.restype = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32], None
    f(c, *wait)
    return c


def grid(shape, seed=0):
    rng = np.random.default_rng(seed)
    A = P.diffusion_csr(np.exp(rng.standard_normal(shape)), aniso=2.0)
    return P.System(A=A, b=rng.uniform(-1, 1, A.n))


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


SHAPES = [(64, 64), (1, 8193), (90, 100), (64, 300), (200, 180), (9, 1000)]


@pytest.mark.parametrize("wait", WAITS, ids=str)
@pytest.mark.parametrize("copies", [1, 8])
def test_pcg_batch_solves_from_x0_whoever_leaves(apcg, wait, copies):
    """copies = 8: more members than compute units, tickets wait for others.
    To a tolerance, the host waits for the launch and the segmented schedule
    solves what is left, to the same bits; 12 iterations are queued with what
    solves the rest, one workgroup per system."""
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print(f"case team wait pcg {wait} copies={copies}", flush=True)
    base = [grid(s, i) for i, s in enumerate(SHAPES)]
    rng = np.random.default_rng(1)
    x0 = [rng.uniform(-1, 1, s.A.n) for s in base]
    As = [DeviceCSR(s.A) for s in base] * copies
    bs = [DeviceVec(s.b) for s in base] * copies
    info = apcg.apcg_info_create(0, len(As))

    def solve(sched, rtol, maxit):
        xs = [DeviceVec(v) for v in x0 * copies]
        c = impatient(apcg, wait)
        apcg.apcg_counters_reset()
        apcg.apcg_ksp_solve_batched(c, [a.h for a in As], [b.h for b in bs], [x.h for x in xs], rtol, maxit,
                                    apcg.apcg_solve_opts_default(batch_schedule=sched), info)
        n = apcg.apcg_counters_get()
        out = [apcg.apcg_info_get(info, k) for k in range(len(xs))], [x.numpy() for x in xs]
        apcg.apcg_ctx_destroy(c)
        return out, n["graph_launches"] > 0

    want, left = solve(2, 1e-8, 20000)[0], 0
    for _ in range(4):
        got, graphs = solve(0, 1e-8, 20000)
        left += graphs
        assert got[0] == want[0] and all(np.array_equal(p, q) for p, q in zip(got[1], want[1]))
    assert left > 0 or wait[0] > 0
    want = [oracle.pcg(s.A, s.b, x0=v, rtol=0.0, maxit=12).x for s, v in zip(base, x0)]
    for _ in range(4):
        got, graphs = solve(0, 0.0, 12)
        assert not graphs
        for k, (r, x) in enumerate(zip(*got)):
            assert (r["status"], r["iterations"]) == (apcg.APCG_SOLVE_MAXIT, 12), k
            assert rel(x, want[k % len(want)]) <= 1e-12, k
    apcg.apcg_info_destroy(info)


@pytest.mark.parametrize("wait", WAITS, ids=str)
def test_features_whoever_leaves(apcg, wait):
    """The feature run's alpha and beta, from whichever kernel."""
    import torch
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print(f"case team wait features {wait}", flush=True)
    s = grid((150, 150), 6)
    dA, db = DeviceCSR(s.A), DeviceVec(s.b)
    calm = apcg.apcg_ctx_create(0)

    def features(c):
        F, L = torch.zeros(16, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        apcg.apcg_pc_features(c, dA.h, db.h, F, L)
        apcg.apcg_ctx_synchronize(c)
        return F.cpu().numpy(), float(L)

    want = features(calm)
    for _ in range(6):
        c = impatient(apcg, wait)
        for _ in range(3):
            got = features(c)
            assert got[1] == want[1]
            np.testing.assert_allclose(got[0], want[0], rtol=2e-6, atol=2e-6)  # FP32 of values equal to about 1e-10
        apcg.apcg_ctx_destroy(c)
    apcg.apcg_ctx_destroy(calm)


@pytest.mark.parametrize("wait", WAITS, ids=str)
def test_single_solves_from_x0_whoever_leaves(apcg, wait):
    import torch
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print(f"case team wait single {wait}", flush=True)
    s = grid((230, 240), 3)
    x0 = np.random.default_rng(2).uniform(-1, 1, s.A.n)
    lm = oracle.gershgorin(s.A)[1]
    coef = OL.chebyshev_iteration_coeffs(lm / 100, lm).astype(np.float32)
    dA, db = DeviceCSR(s.A), DeviceVec(s.b)
    C, L = torch.from_numpy(coef).cuda(), torch.tensor([lm], dtype=torch.float64).cuda()
    torch.cuda.synchronize()
    info = apcg.apcg_info_create(0, 1)

    def solve(c, kind, mode):
        o = apcg.apcg_solve_opts_default(mode=mode)
        x = DeviceVec(x0)
        if kind == "pcg":
            apcg.apcg_ksp_solve(c, dA.h, db.h, x.h, 0.0, 40, o, info, 0)
        elif kind == "fcg":
            apcg.apcg_ksp_solve_fcg_poly(c, dA.h, db.h, x.h, 0.0, 18, C, L, o, None, info, 0)
        else:
            apcg.apcg_ksp_solve_tfqmr(c, dA.h, db.h, x.h, 0.0, 18, o, info, 0)
        r = apcg.apcg_info_get(info, 0)
        return x.numpy(), (r["status"], r["iterations"])

    for kind in ("pcg", "fcg", "tfqmr"):
        calm = apcg.apcg_ctx_create(0)
        want, state = solve(calm, kind, apcg.APCG_MODE_STREAM)
        apcg.apcg_ctx_destroy(calm)
        for _ in range(6):
            c = impatient(apcg, wait)
            got = solve(c, kind, apcg.APCG_MODE_GRAPH)
            assert got[1] == state, kind
            assert rel(got[0], want) <= 1e-10, kind
            apcg.apcg_ctx_destroy(c)
    apcg.apcg_info_destroy(info)


def test_waiting_for_whole_solves_is_no_time_out(apcg):
    """More members than compute units, and solves of 10,000 iterations (about
    60 ms): the members of a system that lacks others wait for whole solves,
    far longer than the limit (15 ms), while those go on."""
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print("case team wait whole solves", flush=True)
    n = 24000  # a chain: as many iterations as rows
    i = np.repeat(np.arange(n), 3)
    j = i + np.tile([-1, 0, 1], n)
    ok = (j >= 0) & (j < n)
    A = P.CSR(n=n, rowptr=np.concatenate([[0], np.cumsum(np.add.reduceat(ok, np.arange(0, 3 * n, 3)))]).astype(np.int32),
              col=j[ok].astype(np.int32), val=np.where(i == j, 2.0, -1.0)[ok])
    rng = np.random.default_rng(4)
    As = [DeviceCSR(A) for _ in range(60)]
    bs = [DeviceVec(rng.uniform(-1, 1, n)) for _ in As]
    xs = [DeviceVec.zeros(n) for _ in As]
    info = apcg.apcg_info_create(0, len(As))
    c = impatient(apcg, (1_500_000, 255))
    for maxit in (10, 10000):
        apcg.apcg_counters_reset()
        apcg.apcg_ksp_solve_batched(c, [a.h for a in As], [b.h for b in bs], [x.h for x in xs], 1e-14, maxit,
                                    apcg.apcg_solve_opts_default(x0_is_zero=1), info)
        k = apcg.apcg_counters_get()
        assert k["graph_launches"] == 0 and k["kernel_launches"] <= 4
        assert [apcg.apcg_info_get(info, q)["iterations"] for q in range(len(As))] == [maxit] * len(As)
    apcg.apcg_info_destroy(info)
    apcg.apcg_ctx_destroy(c)
