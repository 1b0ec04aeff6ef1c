"""A solve without iterations above the line from which teams solve."""
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


def test_no_iterations_above_the_teams_line(apcg):
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print("case no iterations", flush=True)
    rng = np.random.default_rng(9)
    A = P.diffusion_csr(np.exp(rng.standard_normal((24, 25, 26))), aniso=2.0)
    b, x0 = rng.uniform(-1, 1, A.n), rng.uniform(-1, 1, A.n)
    ctx, info, dA, db = apcg.apcg_ctx_create(0), apcg.apcg_info_create(0, 1), DeviceCSR(A), DeviceVec(b)
    for rtol, status in ((0.0, apcg.APCG_SOLVE_MAXIT), (1e6, apcg.APCG_SOLVE_CONVERGED)):
        dx = DeviceVec(x0)
        apcg.apcg_ksp_solve(ctx, dA.h, db.h, dx.h, rtol, 0, apcg.apcg_solve_opts_default(), info, 0)
        r = apcg.apcg_info_get(info, 0)
        assert (r["status"], r["iterations"]) == (status, 0) and np.array_equal(dx.numpy(), x0)
        ref = oracle.pcg(A, b, x0=x0, rtol=rtol, maxit=0)
        assert abs(r["res_norm"] - ref.res) <= 1e-12 * ref.res
    apcg.apcg_info_destroy(info)
    apcg.apcg_ctx_destroy(ctx)
