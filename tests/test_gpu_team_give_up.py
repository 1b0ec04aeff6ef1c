"""Team launches that are given up (csrc/team.h): a system whose pattern is no
longer the one its schedule was chosen for is found and solved all the same,
whatever else is in the batch."""
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


def pairs(n, partner):
    """Rows i coupled to partner(i), an involution without fixed points."""
    i = np.arange(n)
    c = np.sort(np.stack([i, partner], 1), axis=1).astype(np.int32)
    return P.CSR(n=n, rowptr=np.arange(0, 2 * n + 1, 2, dtype=np.int32), col=c.reshape(-1),
                 val=np.where(c == i[:, None], 2.0, -1.0).reshape(-1))


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def test_border_grown_in_place_beside_a_wider_system(apcg, ctx):
    """The second system's border grows in place from none to 2048 columns,
    which is no more than the first one's: more than travels during a meeting
    (1792), less than the launch has room for."""
    import torch
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    n = 8000
    i = np.arange(n)
    near, far = pairs(n, i ^ 1), pairs(n, (i + n // 2) % n)
    wide, b = grid((2, 9000), 3), np.random.default_rng(5).uniform(-1, 1, n)
    As, bs = [DeviceCSR(wide.A), DeviceCSR(near)], [DeviceVec(wide.b), DeviceVec(b)]
    xs = [DeviceVec.zeros(wide.A.n), DeviceVec.zeros(n)]
    info = apcg.apcg_info_create(0, 2)
    opts = apcg.apcg_solve_opts_default(x0_is_zero=1)
    print("case border grown in place in a batch", flush=True)
    for A in (near, far, far, near):
        As[1].col.copy_(torch.from_numpy(A.col))
        As[1].val.copy_(torch.from_numpy(A.val))
        torch.cuda.synchronize()
        apcg.apcg_ksp_solve_batched(ctx, [a.h for a in As], [v.h for v in bs], [v.h for v in xs], 1e-10, 20000, opts,
                                    info)
        for k, (M, rhs) in enumerate(((wide.A, wide.b), (A, b))):
            ref = oracle.pcg(M, rhs, rtol=1e-10, maxit=20000)
            r = apcg.apcg_info_get(info, k)
            assert r["status"] == apcg.APCG_SOLVE_CONVERGED and abs(r["iterations"] - ref.its) <= 1, k
            assert rel(xs[k].numpy(), ref.x) <= 1e-9, k
    apcg.apcg_info_destroy(info)


def test_threads_share_a_matrix(apcg):
    """Contexts of several threads solve with one matrix whose border none of
    them has read yet."""
    import threading

    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print("case threads share a matrix", flush=True)
    for rep in range(4):
        s = grid((110 + rep, 120), rep)
        dA, got, start = DeviceCSR(s.A), [None] * 4, threading.Barrier(4)

        def work(k):
            c = apcg.apcg_ctx_create(0)
            b, x, info = DeviceVec(s.b), DeviceVec.zeros(s.A.n), apcg.apcg_info_create(0, 1)
            start.wait()
            for _ in range(3):
                apcg.apcg_ksp_solve(c, dA.h, b.h, x.h, 0.0, 20, apcg.apcg_solve_opts_default(x0_is_zero=1), info, 0)
            got[k] = x.numpy()
            apcg.apcg_info_destroy(info)
            apcg.apcg_ctx_destroy(c)

        ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert all(np.array_equal(g, got[0]) for g in got)
        assert rel(got[0], oracle.pcg(s.A, s.b, rtol=0.0, maxit=20).x) <= 1e-12


def test_refusing_system_leaves_the_others_and_is_remembered(apcg, ctx):
    """A batch in which one matrix is read one way only (row 2048 names row 2047
    of the member before it, which names nothing back): the members of that
    system refuse the flexible solve, the others finish, the tiles solve the
    rest to the same bits; the next call goes to the tiles at once."""
    import torch
    from oracle import learned as OL
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    S = [grid((70, 71), 1), grid((1, 10000), 2), grid((1, 900), 3), grid((90, 50), 4)]
    A = S[1].A
    keep = np.ones(A.col.size, bool)
    keep[[e for e in range(A.rowptr[2047], A.rowptr[2048]) if A.col[e] == 2048]] = False
    rp = np.concatenate([[0], np.cumsum(np.add.reduceat(keep, A.rowptr[:-1]))]).astype(np.int32)
    S[1] = P.System(A=P.CSR(n=A.n, rowptr=rp, col=A.col[keep], val=A.val[keep]), b=S[1].b)
    lms = [oracle.gershgorin(s.A)[1] for s in S]
    C = torch.from_numpy(np.concatenate([OL.chebyshev_iteration_coeffs(l / 100, l) for l in lms]).astype(
        np.float32)).cuda()
    L = torch.tensor(lms, dtype=torch.float64).cuda()
    torch.cuda.synchronize()
    As, bs = [DeviceCSR(s.A) for s in S], [DeviceVec(s.b) for s in S]
    info = apcg.apcg_info_create(0, len(S))
    print("case one-sided matrix in a batch", flush=True)

    def solve(tiles):
        xs = [DeviceVec.zeros(s.A.n) for s in S]
        apcg.apcg_counters_reset()
        apcg.apcg_ksp_solve_batched_fcg_poly(
            ctx, [a.h for a in As], [b.h for b in bs], [x.h for x in xs], 0.0, 6, C, L,
            apcg.apcg_solve_opts_default(x0_is_zero=1, iters_per_graph=2, batch_tile_rows=256 if tiles else 0), None,
            info)
        n = apcg.apcg_counters_get()
        return [apcg.apcg_info_get(info, k) for k in range(len(S))], [x.numpy() for x in xs], n

    want = solve(True)
    first, second = solve(False), solve(False)
    for got in (first, second):
        assert got[0] == want[0] and all(np.array_equal(p, q) for p, q in zip(got[1], want[1]))
        assert got[2]["graph_launches"] > 0  # (the tiles, not one system after the other)
    assert second[2]["kernel_launches"] <= want[2]["kernel_launches"] < first[2]["kernel_launches"]
    apcg.apcg_info_destroy(info)


def test_rows_grown_in_place_are_given_up_twice_at_most(apcg, ctx):
    """Row lengths rewritten in place past what a member holds (9 entries): the
    launch finds it, reads the border again, finds it again and leaves the
    matrix to the other schedules from then on."""
    import torch
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    n = 9000
    i = np.arange(n)
    thin = pairs(n, i ^ 1)
    # no more entries than before: of every 100 rows the first nine couple to each other, the others to none
    rows, cols = [], []
    for r0 in range(0, n, 100):
        for r in range(100):
            c = range(9) if r < 9 else [r]
            rows += [r0 + r] * len(c)
            cols += [r0 + q for q in c]
    rows, cols = np.array(rows), np.array(cols)
    short = 2 * n - rows.size
    assert short >= 0
    thick_val = np.where(rows == cols, 12.0, -1.0)
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    thick = P.CSR(n=n, rowptr=rp, col=cols.astype(np.int32), val=thick_val)
    assert np.diff(rp).max() == 9
    b = np.random.default_rng(8).uniform(-1, 1, n)
    other = grid((60, 61), 5)
    As, bs = [DeviceCSR(thin), DeviceCSR(other.A)], [DeviceVec(b), DeviceVec(other.b)]
    xs = [DeviceVec.zeros(n), DeviceVec.zeros(other.A.n)]
    info = apcg.apcg_info_create(0, 2)
    print("case rows grown in place", flush=True)

    def solve(sched):
        apcg.apcg_counters_reset()
        apcg.apcg_ksp_solve_batched(ctx, [a.h for a in As], [v.h for v in bs], [v.h for v in xs], 1e-10, 20000,
                                    apcg.apcg_solve_opts_default(x0_is_zero=1, batch_schedule=sched), info)
        return apcg.apcg_counters_get()["kernel_launches"], [x.numpy() for x in xs]

    assert solve(0)[0] <= 4  # teams
    pad = np.zeros(short, np.int32)
    As[0].rowptr.copy_(torch.from_numpy(thick.rowptr))
    As[0].col.copy_(torch.from_numpy(np.concatenate([thick.col, pad])))
    As[0].val.copy_(torch.from_numpy(np.concatenate([thick.val, np.zeros(short)])))
    torch.cuda.synchronize()
    kernels, want = solve(2)
    ref = oracle.pcg(thick, b, rtol=1e-10, maxit=20000)
    assert rel(want[0], ref.x) <= 1e-9
    tries = [solve(0) for _ in range(4)]
    assert all(np.array_equal(p, q) for _, got in tries for p, q in zip(got, want))
    assert [k > kernels for k, _ in tries] == [True, True, False, False]
    apcg.apcg_info_destroy(info)
