"""The one-workgroup solve (csrc/persist.hip) with the direction in LDS: every
rows-per-thread and entries-per-row variant at its edges, against the oracle
(iterations +-1, relative difference 1e-9 at rtol 1e-10); the no-allocation
calls of two contexts share nothing."""
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


def system(shape, seed=0):
    rng = np.random.default_rng(seed)
    return P.System(A=P.diffusion_csr(np.exp(rng.standard_normal(shape)), aniso=2.0), b=rng.uniform(-1, 1, int(np.prod(shape))))


# 512, 1024, 2048 and 4096 rows and one more or less; rows of 5 and 7 entries
SHAPES = [(1, 1), (1, 512), (1, 513), (32, 32), (25, 41), (32, 64), (3, 683), (64, 64), (63, 65),
          (8, 8, 8), (3, 9, 19), (8, 8, 16), (5, 5, 41), (8, 16, 16), (3, 683, 1), (2, 25, 41), (16, 16, 16), (15, 21, 13)]


@pytest.mark.parametrize("shape", SHAPES)
def test_persistent_matches_oracle(apcg, shape):
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    s = system(shape, seed=len(shape))
    print(f"case persistent lds {shape}", flush=True)
    ctx = apcg.apcg_ctx_create(0)
    dA, db = DeviceCSR(s.A), DeviceVec(s.b)
    info = apcg.apcg_info_create(0, 1)
    x0 = np.random.default_rng(1).uniform(-1, 1, s.A.n)
    for guess in (None, x0):
        dx = DeviceVec(np.zeros(s.A.n) if guess is None else guess)
        opts = apcg.apcg_solve_opts_default(mode=apcg.APCG_MODE_PERSISTENT, x0_is_zero=int(guess is None))
        apcg.apcg_ksp_solve(ctx, dA.h, db.h, dx.h, 1e-10, 20000, opts, info, 0)
        r = apcg.apcg_info_get(info, 0)
        ref = oracle.pcg(s.A, s.b, x0=guess, rtol=1e-10, maxit=20000)
        assert r["status"] == apcg.APCG_SOLVE_CONVERGED and abs(r["iterations"] - ref.its) <= 1
        assert np.linalg.norm(dx.numpy() - ref.x) <= 1e-9 * np.linalg.norm(ref.x)
    apcg.apcg_info_destroy(info)
    apcg.apcg_ctx_synchronize(ctx)
    apcg.apcg_ctx_destroy(ctx)


def test_noalloc_calls_of_two_contexts_overlap(apcg):
    import torch

    S = [system((64, 64), 1), system((60, 61), 2)]
    print("case noalloc overlap", flush=True)
    got = [[] for _ in S]

    def work(i, times):
        A, ctx = S[i].A, apcg.apcg_ctx_create(0)
        t = [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (A.rowptr, A.col, A.val, S[i].b)]
        info = torch.zeros(64, dtype=torch.uint8, device="cuda")
        opts = apcg.apcg_solve_opts_default(x0_is_zero=1)
        xs = [torch.zeros(A.n, dtype=torch.float64, device="cuda") for _ in range(times)]
        torch.cuda.synchronize()
        for x in xs:
            apcg.apcg_ksp_solve_small_noalloc(ctx, A.n, *(v.data_ptr() for v in t), x.data_ptr(), 0.0, 100, opts,
                                              info.data_ptr())
        apcg.apcg_ctx_synchronize(ctx)
        got[i] += [x.cpu().numpy() for x in xs]
        apcg.apcg_ctx_destroy(ctx)

    for i in range(len(S)):
        work(i, 1)  # alone
    threads = [threading.Thread(target=work, args=(i, 6)) for i in range(len(S))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for xs in got:
        assert len(xs) == 7 and all(np.array_equal(x, xs[0]) for x in xs[1:])
