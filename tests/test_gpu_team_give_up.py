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
