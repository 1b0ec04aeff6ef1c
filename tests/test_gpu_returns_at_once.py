"""Calls that return once their work is queued: while the context still waits on
the device for another context's long solve, the call comes back, and the
result is right when that has ended.  These are the calls whose kernels need no
look at the device (a few periods of iterations, one workgroup per system),
whether teams solve them or not."""
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
def busy(apcg):
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    class Busy:
        """A context on which solves of a fixed count are under way."""

        def __init__(self):
            A = P.laplace_2d(1500)
            self.ctx = apcg.apcg_ctx_create(0)
            self.A, self.b, self.x = DeviceCSR(A), DeviceVec(np.ones(A.n)), DeviceVec.zeros(A.n)
            self.info = apcg.apcg_info_create(0, 1)
            self.opts = apcg.apcg_solve_opts_default(x0_is_zero=1, iters_per_graph=64, lookahead=8)
            self.block(None)
            apcg.apcg_ctx_synchronize(self.ctx)

        def block(self, ctx):
            for _ in range(2):
                apcg.apcg_ksp_solve(self.ctx, self.A.h, self.b.h, self.x.h, 0.0, 448, self.opts, self.info, 0)
            if ctx is not None:
                apcg.apcg_ctx_wait_for(ctx, self.ctx)

        def running(self):
            return not apcg.apcg_ctx_query_idle(self.ctx)

    b = Busy()
    yield b
    apcg.apcg_ctx_synchronize(b.ctx)
    apcg.apcg_info_destroy(b.info)
    apcg.apcg_ctx_destroy(b.ctx)


@pytest.fixture()
def ctx(apcg):
    c = apcg.apcg_ctx_create(0)
    yield c
    apcg.apcg_ctx_synchronize(c)
    apcg.apcg_ctx_destroy(c)


def grid(shape, seed=0):
    rng = np.random.default_rng(seed)
    A = P.diffusion_csr(np.exp(rng.standard_normal(shape)), aniso=2.0)
    return P.System(A=A, b=rng.uniform(-1, 1, A.n))


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def at_once(busy, ctx, call, times=2, first=0):
    """The first calls may wait: for a new graph to be captured nothing waits,
    but new descriptors of a batch are uploaded and waited for."""
    for k in range(first + times):
        busy.block(ctx)
        assert busy.running()
        call()
        assert k < first or busy.running(), f"call {k} waited for the device"


@pytest.mark.parametrize("shape,maxit,opts", [
    ((110, 110), 12, {}), ((24, 25, 26), 16, {}), ((110, 110), 0, {}),
    ((400, 400), 14, {"iters_per_graph": 7, "lookahead": 3}),
    ((110, 110), 100, {"iters_per_graph": 64, "lookahead": 8}), ((500, 500), 300, {"iters_per_graph": 64, "lookahead": 8}),
], ids=str)
def test_single_solve(apcg, busy, ctx, shape, maxit, opts):
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print(f"case returns at once pcg {shape} {maxit}", flush=True)
    s = grid(shape, 1)
    x0 = np.random.default_rng(2).uniform(-1, 1, s.A.n)
    dA, db, info = DeviceCSR(s.A), DeviceVec(s.b), apcg.apcg_info_create(0, 1)
    o = apcg.apcg_solve_opts_default(**opts)
    xs = [DeviceVec(x0) for _ in range(3)]
    it = iter(xs)
    at_once(busy, ctx, lambda: apcg.apcg_ksp_solve(ctx, dA.h, db.h, next(it).h, 0.0, maxit, o, info, 0), times=3)
    ref = oracle.pcg(s.A, s.b, x0=x0, rtol=0.0, maxit=maxit)
    # (100 and more iterations on these operators depend on the order of the sums at 1e-9)
    assert all(rel(x.numpy(), ref.x) <= (1e-12 if maxit <= 20 else 1e-7) for x in xs)
    assert apcg.apcg_info_get(info, 0)["iterations"] == maxit
    apcg.apcg_info_destroy(info)


@pytest.mark.parametrize("kind", ["fcg", "tfqmr", "features"])
def test_other_single_calls(apcg, busy, ctx, kind):
    import torch
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print(f"case returns at once {kind}", flush=True)
    s = grid((100, 120), 3)
    lm = oracle.gershgorin(s.A)[1]
    coef = OL.chebyshev_iteration_coeffs(lm / 100, lm).astype(np.float32)
    dA, db, dx = DeviceCSR(s.A), DeviceVec(s.b), DeviceVec.zeros(s.A.n)
    C, L = torch.from_numpy(coef).cuda(), torch.tensor([lm], dtype=torch.float64).cuda()
    F, M = torch.zeros(16, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    info = apcg.apcg_info_create(0, 1)
    o = apcg.apcg_solve_opts_default(x0_is_zero=1)
    calls = {
        # (the fallback, queued behind the flexible phase whether it is needed
        # or not, is paced by polls from its second period on)
        "fcg": lambda: apcg.apcg_ksp_solve_fcg_poly(ctx, dA.h, db.h, dx.h, 0.0, 12, C, L, o,
                                                    apcg.apcg_fcg_opts_default(fallback=0), info, 0),
        "tfqmr": lambda: apcg.apcg_ksp_solve_tfqmr(ctx, dA.h, db.h, dx.h, 0.0, 12, o, info, 0),
        "features": lambda: apcg.apcg_pc_features(ctx, dA.h, db.h, F, M),
    }
    # the first flexible or TFQMR solve of a matrix analyses its pattern on the host
    at_once(busy, ctx, calls[kind], times=3, first=0 if kind == "features" else 1)
    if kind == "fcg":
        ref = oracle.fcg_poly(s.A, s.b, coef.astype(np.float64), lm, rtol=0.0, maxit=12)
    elif kind == "tfqmr":
        ref = oracle.tfqmr(s.A, s.b, rtol=0.0, maxit=12)
    if kind != "features":
        assert rel(dx.numpy(), ref.x) <= 1e-9
    apcg.apcg_info_destroy(info)


@pytest.mark.parametrize("shapes,args", [([(31, 31)] * 300, (1e-8, 20000)), ([(40, 41), (90, 90), (300, 310)], (0.0, 12)),
                                         ([(60, 60)] * 40 + [(12, 30, 30)], (0.0, 16))], ids=["persistent", "12", "16"])
def test_batch(apcg, busy, ctx, shapes, args):
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print(f"case returns at once batch {len(shapes)} {args}", flush=True)
    S = [grid(s, i % 5) for i, s in enumerate(shapes)]
    As, bs, xs = [DeviceCSR(s.A) for s in S], [DeviceVec(s.b) for s in S], [DeviceVec.zeros(s.A.n) for s in S]
    info = apcg.apcg_info_create(0, len(S))
    o = apcg.apcg_solve_opts_default(x0_is_zero=1)
    at_once(busy, ctx, lambda: apcg.apcg_ksp_solve_batched(ctx, [a.h for a in As], [v.h for v in bs], [v.h for v in xs],
                                                           *args, o, info), first=1)
    for k in (0, len(S) // 2, len(S) - 1):
        ref = oracle.pcg(S[k].A, S[k].b, rtol=args[0], maxit=args[1])
        assert abs(apcg.apcg_info_get(info, k)["iterations"] - ref.its) <= 1
        assert rel(xs[k].numpy(), ref.x) <= (1e-12 if args[0] == 0 else 1e-7)
    apcg.apcg_info_destroy(info)


def test_flexible_batch(apcg, busy, ctx):
    import torch
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print("case returns at once flexible batch", flush=True)
    S = [grid(s, i) for i, s in enumerate([(40, 41), (90, 90), (10, 12, 11)])]
    lms = [oracle.gershgorin(s.A)[1] for s in S]
    coefs = [OL.chebyshev_iteration_coeffs(l / 100, l).astype(np.float32) for l in lms]
    C, L = torch.from_numpy(np.concatenate(coefs)).cuda(), torch.tensor(lms, dtype=torch.float64).cuda()
    torch.cuda.synchronize()
    As, bs, xs = [DeviceCSR(s.A) for s in S], [DeviceVec(s.b) for s in S], [DeviceVec.zeros(s.A.n) for s in S]
    info = apcg.apcg_info_create(0, len(S))
    o = apcg.apcg_solve_opts_default(x0_is_zero=1)
    at_once(busy, ctx, lambda: apcg.apcg_ksp_solve_batched_fcg_poly(
        ctx, [a.h for a in As], [v.h for v in bs], [v.h for v in xs], 0.0, 12, C, L, o, None, info), first=1)
    for k, s in enumerate(S):
        ref = oracle.fcg_poly(s.A, s.b, coefs[k].astype(np.float64), lms[k], rtol=0.0, maxit=12)
        assert rel(xs[k].numpy(), ref.x) <= 1e-9
    apcg.apcg_info_destroy(info)


def test_many_queued_launches_and_a_pattern_changed_under_them(apcg, ctx):
    """Nobody waits between the calls; what the members find about a pattern
    that was rewritten in place arrives later, and the result is right at once."""
    import torch
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print("case returns at once pattern changed", flush=True)
    n = 80000
    i = np.arange(n)

    def csr(j):
        c = np.sort(np.stack([i, j], 1), axis=1).astype(np.int32)
        return P.CSR(n=n, rowptr=np.arange(0, 2 * n + 1, 2, dtype=np.int32), col=c.reshape(-1),
                     val=np.where(c == i[:, None], 2.0, -1.0).reshape(-1))

    near, far = csr(i ^ 1), csr((i + n // 2) % n)
    b, x0 = (np.random.default_rng(k).uniform(-1, 1, n) for k in (5, 6))
    dA, db, info = DeviceCSR(near), DeviceVec(b), apcg.apcg_info_create(0, 1)
    o = apcg.apcg_solve_opts_default()
    for A, calls, teams in ((near, 3, None), (near, 3, True), (far, 40, None), (far, 3, False), (near, 3, False)):
        dA.col.copy_(torch.from_numpy(A.col))
        dA.val.copy_(torch.from_numpy(A.val))
        torch.cuda.synchronize()
        ref = oracle.pcg(A, b, x0=x0, rtol=0.0, maxit=1).x
        xs = [DeviceVec(x0) for _ in range(calls)]
        apcg.apcg_counters_reset()
        for x in xs:
            apcg.apcg_ksp_solve_batched(ctx, [dA.h], [db.h], [x.h], 0.0, 1, o, info)
        kernels = apcg.apcg_counters_get()["kernel_launches"]
        apcg.apcg_ctx_synchronize(ctx)
        assert all(rel(x.numpy(), ref) <= 1e-12 for x in xs)
        # teams: the words' clearing, the team and what it leaves
        print(A is near, calls, kernels, flush=True)
        assert teams is None or (kernels == 3 * calls) == teams
    apcg.apcg_info_destroy(info)
