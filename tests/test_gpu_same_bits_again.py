"""The same call gives the same bits whenever it is made: on a matrix that has
not been solved before, on one whose pattern the library knows by then, on a
context that is idle and on one that still waits."""
from hashlib import md5

import numpy as np
import pytest

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


def system(shape):
    rng = np.random.default_rng(len(shape))
    A = P.diffusion_csr(np.exp(rng.standard_normal(shape)), aniso=2.0)
    return A, rng.uniform(-1, 1, A.n), rng.uniform(-1, 1, A.n)


# few iterations are queued without a look at the device, many are polled
@pytest.mark.parametrize("maxit", [1, 5, 16, 17, 40])
@pytest.mark.parametrize("shape", [(64, 64), (110, 110), (300, 310), (24, 25, 26), (64, 64, 64)], ids=str)
@pytest.mark.parametrize("before", ["nothing", "polled solve"])
def test_single_solve(apcg, shape, maxit, before):
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print(f"case same bits {shape} {maxit} {before}", flush=True)
    A, b, x0 = system(shape)
    ctx, info, o = apcg.apcg_ctx_create(0), apcg.apcg_info_create(0, 1), apcg.apcg_solve_opts_default()
    seen = set()
    for fresh in range(2):
        dA, db = DeviceCSR(A), DeviceVec(b)
        if before != "nothing" and fresh:
            first = DeviceVec(x0)
            apcg.apcg_ksp_solve(ctx, dA.h, db.h, first.h, 1e-6, 1000, o, info, 0)
        xs = [DeviceVec(x0) for _ in range(5)]
        for k, x in enumerate(xs):
            apcg.apcg_ksp_solve(ctx, dA.h, db.h, x.h, 0.0, maxit, o, info, 0)
            if k >= 2:
                apcg.apcg_ctx_synchronize(ctx)
        seen |= {md5(x.numpy().tobytes()).hexdigest() for x in xs}
    assert len(seen) == 1
    apcg.apcg_info_destroy(info)
    apcg.apcg_ctx_destroy(ctx)


@pytest.mark.parametrize("shape", [(120, 110), (30, 31, 32)], ids=str)
def test_learned_solve(apcg, shape):
    """Its features come from five steps of the single solve."""
    import torch
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec
    from paper_2306_17801_amd.learned import pack_params

    print(f"case same bits learned {shape}", flush=True)
    A, b, _ = system(shape)
    p = torch.from_numpy(pack_params(P.mlp_initial_params(7))).float().cuda()
    mean, std = torch.zeros(16, device="cuda"), torch.ones(16, device="cuda")
    torch.cuda.synchronize()
    ctx, info = apcg.apcg_ctx_create(0), apcg.apcg_info_create(0, 1)
    o = apcg.apcg_solve_opts_default(x0_is_zero=1)
    dA, db, xs = DeviceCSR(A), DeviceVec(b), [DeviceVec.zeros(A.n) for _ in range(4)]
    for x in xs:
        apcg.apcg_ksp_solve_learned(ctx, dA.h, db.h, x.h, 0.0, 40, p, mean, std, o, None, info, 0)
        apcg.apcg_ctx_synchronize(ctx)
    assert len({md5(x.numpy().tobytes()).hexdigest() for x in xs}) == 1
    apcg.apcg_info_destroy(info)
    apcg.apcg_ctx_destroy(ctx)
