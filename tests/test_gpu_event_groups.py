"""Brief operations share one event per group (csrc/runtime.hip): another
context, a host read, a destroyed object and a destroyed context all see what
was queued before, whatever the group's state; a solve ends the group."""
import numpy as np
import pytest

from paper_2306_17801_amd import problems as P

pytestmark = pytest.mark.gpu
N = 1 << 20


@pytest.fixture(scope="module")
def apcg():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_17801_amd as m

    m.load()
    return m


@pytest.mark.parametrize("ops", [1, 7, 8, 9, 20])
def test_other_context_and_host_see_a_group(apcg, ops):
    """x doubled `ops` times on one context, then read by another, then
    written by the first again: the second's copy is in between."""
    from paper_2306_17801_amd.device import DeviceVec

    print(f"case event group ops={ops}", flush=True)
    a, b = apcg.apcg_ctx_create(0), apcg.apcg_ctx_create(0)
    two = apcg.apcg_scalar_create(a)
    apcg.apcg_scalar_set(two, 2.0, a)
    for rep in range(10):
        x, y = DeviceVec(np.ones(N)), DeviceVec.zeros(N)
        for _ in range(ops):
            apcg.apcg_vec_scale_async(x.h, two, a)
        apcg.apcg_vec_copy_async(y.h, x.h, b)
        apcg.apcg_vec_set_async(x.h, -1.0, a)  # waits for b's read
        got = np.empty(N)
        t = apcg.apcg_scalar_create(b)
        apcg.apcg_vec_norm2_async(y.h, t, b)
        assert apcg.apcg_scalar_get(t) == 2.0**ops * np.sqrt(N)
        got = y.numpy()
        assert np.all(got == 2.0**ops) and np.all(x.numpy() == -1.0)
        apcg.apcg_scalar_destroy(t)
        x.close()
        y.close()
    for c in (a, b):
        apcg.apcg_ctx_destroy(c)
    apcg.apcg_scalar_destroy(two)


def test_solve_ends_the_group_and_destroyed_context_is_waited_for(apcg):
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print("case event group solve and destroy", flush=True)
    A = P.laplace_2d(60)
    a, b = apcg.apcg_ctx_create(0), apcg.apcg_ctx_create(0)
    dA, rhs, x, y = DeviceCSR(A), DeviceVec.zeros(A.n), DeviceVec.zeros(A.n), DeviceVec.zeros(A.n)
    apcg.apcg_vec_set_async(rhs.h, 1.0, a)
    info = apcg.apcg_info_create(0, 1)
    apcg.apcg_ksp_solve(b, dA.h, rhs.h, x.h, 1e-10, 1000, apcg.apcg_solve_opts_default(x0_is_zero=1), info, 0)
    apcg.apcg_vec_copy_async(y.h, x.h, a)
    apcg.apcg_ctx_destroy(a)  # with an open group
    apcg.apcg_mat_mult_async(dA.h, y.h, rhs.h, b)
    assert apcg.apcg_info_get(info, 0)["status"] == apcg.APCG_SOLVE_CONVERGED
    assert np.max(np.abs(rhs.numpy() - 1.0)) < 1e-6
    apcg.apcg_ctx_destroy(b)
    apcg.apcg_info_destroy(info)
