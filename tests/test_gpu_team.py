"""Team solves (csrc/team.hip): one launch in which a team of workgroups holds
a system's matrix and vectors in registers.  Sizes lie at the edges of what a
member holds (2048 rows; 4096 when a batch of five-entry rows queues for the
compute units), of the 64-row slices and of the 2048-row groups the sums are
formed in.

The sums run in the segmented schedule's order, so a batch gives the same bits
on both; against the oracle the repository's bar holds (iterations +-1,
relative difference 1e-9 at rtol 1e-10, 1e-12 at matched counts)."""
import threading

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


def grid(shape, seed=0, sigma=1.0, aniso=2.0):
    rng = np.random.default_rng(seed)
    A = P.diffusion_csr(np.exp(sigma * rng.standard_normal(shape)), aniso=aniso)
    return P.System(A=A, b=rng.uniform(-1, 1, A.n))


def rel(a, b):
    nb = np.linalg.norm(b)
    return np.linalg.norm(a - b) / (nb if nb > 0 else 1.0)


def solve_one(apcg, ctx, A, b, rtol, maxit, x0=None, **o):
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    dA, db, dx = DeviceCSR(A), DeviceVec(b), DeviceVec(np.zeros(A.n) if x0 is None else x0)
    info = apcg.apcg_info_create(0, 1)
    opts = apcg.apcg_solve_opts_default(x0_is_zero=int(x0 is None), **o)
    apcg.apcg_counters_reset()
    apcg.apcg_ksp_solve(ctx, dA.h, db.h, dx.h, rtol, maxit, opts, info, 0)
    graphs = apcg.apcg_counters_get()["graph_launches"]
    r, x = apcg.apcg_info_get(info, 0), dx.numpy()
    apcg.apcg_info_destroy(info)
    return r, x, graphs


def solve_batch(apcg, ctx, systems, rtol, maxit, sched, x0s=None, **o):
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    As, bs = [DeviceCSR(s.A) for s in systems], [DeviceVec(s.b) for s in systems]
    xs = [DeviceVec(np.zeros(s.A.n) if x0s is None else x0) for s, x0 in zip(systems, x0s or [None] * len(systems))]
    info = apcg.apcg_info_create(0, len(systems))
    opts = apcg.apcg_solve_opts_default(x0_is_zero=int(x0s is None), batch_schedule=sched, **o)
    apcg.apcg_ksp_solve_batched(ctx, [a.h for a in As], [b.h for b in bs], [x.h for x in xs], rtol, maxit, opts, info)
    out = [apcg.apcg_info_get(info, i) for i in range(len(systems))], [x.numpy() for x in xs]
    apcg.apcg_info_destroy(info)
    return out


# 8193 rows (one over five members), 10,240 = 5 x 2048, one row more and one
# less, borders longer than what is fetched during a meeting (1024), 7-entry
# rows whose planes are no multiple of 64, a plane longer than a member, and
# more than 256 groups (two to a thread of the tree)
SHAPES = [(1, 8193), (64, 160), (7, 1463), (9, 1000), (12, 1000), (23, 21, 25), (6, 41, 53), (730, 740)]


@pytest.mark.parametrize("shape", SHAPES)
def test_team_single_matches_oracle(apcg, ctx, shape):
    s = grid(shape, seed=sum(shape))
    print(f"case team single {shape} n={s.A.n}", flush=True)
    ref20 = oracle.pcg(s.A, s.b, rtol=0.0, maxit=20)
    r, x, graphs = solve_one(apcg, ctx, s.A, s.b, 0.0, 20)
    assert graphs == 0 and r["status"] == apcg.APCG_SOLVE_MAXIT and r["iterations"] == 20
    assert rel(x, ref20.x) <= 1e-12
    if s.A.n > 100_000:
        return
    x0 = np.random.default_rng(1).uniform(-1, 1, s.A.n)
    for kw in ({}, {"norm_type": 1}):
        ref = oracle.pcg(s.A, s.b, x0=x0, rtol=1e-10, maxit=20000, **kw)
        r, x, _ = solve_one(apcg, ctx, s.A, s.b, 1e-10, 20000, x0=x0, **kw)
        assert r["status"] == apcg.APCG_SOLVE_CONVERGED and abs(r["iterations"] - ref.its) <= 1
        assert rel(x, ref.x) <= 1e-9


def edge_batch():
    return [grid(s, seed=i) for i, s in enumerate([(1, 1), (1, 64), (1, 65), (5, 409), (32, 64), (3, 683), (61, 67),
                                                   (64, 64), (17, 241), (13, 14, 15), (128, 130), (2, 9000)])]


@pytest.mark.parametrize("queue", [False, True])
def test_team_batch_bitwise_equals_segmented(apcg, ctx, queue):
    """queue: so many systems that their members outnumber the compute units,
    which takes members of 4096 rows and hands tickets out as members finish
    (five-entry rows only: the 3D system stays out)."""
    systems = edge_batch()
    if queue:
        systems = [s for s in systems if len(s.A.shape) == 2]
        systems += [grid((90 + i % 7, 120), seed=100 + i) for i in range(60)]
    print(f"case team batch queue={queue}", flush=True)
    rng = np.random.default_rng(3)
    x0s = [rng.uniform(-1, 1, s.A.n) for s in systems]
    for args in ((1e-8, 20000), (0.0, 7)):
        a, b = (solve_batch(apcg, ctx, systems, *args, sched) for sched in (0, 2))
        assert a[0] == b[0] and all(np.array_equal(p, q) for p, q in zip(a[1], b[1]))
    # (without a preconditioner 20 iterations on these operators already depend
    # on the order of the sums at 1e-9: held to the segmented bits, not to the oracle)
    a, b = (solve_batch(apcg, ctx, systems, 1e-8, 200, sched, pc=0) for sched in (0, 2))
    assert a[0] == b[0] and all(np.array_equal(p, q) for p, q in zip(a[1], b[1]))
    a, b = (solve_batch(apcg, ctx, systems, 1e-8, 20000, sched, x0s=x0s, norm_type=1) for sched in (0, 2))
    assert a[0] == b[0] and all(np.array_equal(p, q) for p, q in zip(a[1], b[1]))


def test_team_terminal_states(apcg, ctx):
    """A zero right-hand side, a NaN, a bad diagonal and an indefinite operator
    stop alone, in a batch and singly, as in the segmented schedule."""
    S = [grid((60, 150), seed=i) for i in range(5)]
    S[0].b[:] = 0.0
    S[1].b[7000] = np.nan
    d = S[2].A
    d.val[[e for e in range(d.rowptr[4500], d.rowptr[4501]) if d.col[e] == 4500][0]] = -1.0
    S[3].A.val[:] = -S[3].A.val
    print("case team terminal states", flush=True)
    for pc in (1, 0):
        a, b = (solve_batch(apcg, ctx, S, 1e-8, 2000, sched, pc=pc) for sched in (0, 2))
        assert [r["status"] for r in a[0]] == [r["status"] for r in b[0]]
        assert [r["iterations"] for r in a[0]] == [r["iterations"] for r in b[0]]
        assert all(np.array_equal(p, q, equal_nan=True) for p, q in zip(a[1], b[1]))
    for s, want in zip(S, (apcg.APCG_SOLVE_CONVERGED, apcg.APCG_SOLVE_NAN, apcg.APCG_SOLVE_SETUP_ERROR)):
        assert solve_one(apcg, ctx, s.A, s.b, 1e-8, 2000)[0]["status"] == want


def test_team_pattern_changed_in_place(apcg, ctx):
    """Columns rewritten in place (same row lengths) to a coupling wider than
    a window: the launch finds it, gives up with x untouched, and the kernels
    solve the system; the next solve does not try teams."""
    import torch
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    n = 80000
    i = np.arange(n)
    near, far = i ^ 1, (i + n // 2) % n
    cols = {k: np.sort(np.stack([i, j], 1), axis=1) for k, j in (("near", near), ("far", far))}
    b = np.random.default_rng(5).uniform(-1, 1, n)

    def csr(k):
        c = cols[k].astype(np.int32)
        return P.CSR(n=n, rowptr=np.arange(0, 2 * n + 1, 2, dtype=np.int32), col=c.reshape(-1),
                     val=np.where(c == i[:, None], 2.0, -1.0).reshape(-1))

    print("case team pattern changed in place", flush=True)
    dA, db, dx = DeviceCSR(csr("near")), DeviceVec(b), DeviceVec.zeros(n)
    info = apcg.apcg_info_create(0, 1)
    opts = apcg.apcg_solve_opts_default(x0_is_zero=1)
    for k, teams in (("near", True), ("far", False), ("far", False)):
        A = csr(k)
        dA.col.copy_(torch.from_numpy(A.col))
        dA.val.copy_(torch.from_numpy(A.val))
        torch.cuda.synchronize()
        apcg.apcg_counters_reset()
        apcg.apcg_ksp_solve(ctx, dA.h, db.h, dx.h, 1e-10, 100, opts, info, 0)
        assert (apcg.apcg_counters_get()["graph_launches"] == 0) == teams
        ref = oracle.pcg(A, b, rtol=1e-10, maxit=100)
        r = apcg.apcg_info_get(info, 0)
        assert r["status"] == apcg.APCG_SOLVE_CONVERGED and abs(r["iterations"] - ref.its) <= 1
        assert rel(dx.numpy(), ref.x) <= 1e-9
    apcg.apcg_info_destroy(info)


def test_team_concurrent_contexts(apcg):
    """Threads on contexts of their own, each team as large as the chip's half
    and more: the launches queue behind each other, and every solve gives the
    bits it gives alone."""
    S = [grid((500, 520), seed=7), grid((600, 610), seed=8), grid((300, 310), seed=9)]
    print("case team concurrent contexts", flush=True)
    c = apcg.apcg_ctx_create(0)
    alone = [solve_one(apcg, c, s.A, s.b, 0.0, 60)[1] for s in S]
    apcg.apcg_ctx_destroy(c)
    got = [None] * len(S)

    def work(i):
        k = apcg.apcg_ctx_create(0)
        got[i] = [solve_one(apcg, k, S[i].A, S[i].b, 0.0, 60)[1] for _ in range(4)]
        apcg.apcg_ctx_destroy(k)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(S))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for i, xs in enumerate(got):
        assert all(np.array_equal(x, alone[i]) for x in xs)
