"""The event of a group of brief operations (csrc/runtime.hip) lies before
whatever the context is made to wait for, or runs without marks, after them:
who needs a brief operation's result does not wait for that."""
import time

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


class Busy:
    """A context on which a solve of a fixed count is under way (the call
    returns once its iterations are queued)."""

    def __init__(self, apcg):
        from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

        A = P.laplace_2d(1500)
        self.apcg, self.ctx = apcg, apcg.apcg_ctx_create(0)
        self.A, self.b, self.x = DeviceCSR(A), DeviceVec(np.ones(A.n)), DeviceVec.zeros(A.n)
        self.y = DeviceVec.zeros(A.n)
        self.info = apcg.apcg_info_create(0, 1)
        self.opts = apcg.apcg_solve_opts_default(x0_is_zero=1, iters_per_graph=64, lookahead=8)
        self.start()
        apcg.apcg_ctx_synchronize(self.ctx)

    def start(self):
        for _ in range(2):
            self.apcg.apcg_ksp_solve(self.ctx, self.A.h, self.b.h, self.x.h, 0.0, 448, self.opts, self.info, 0)

    def running(self):
        return not self.apcg.apcg_ctx_query_idle(self.ctx)

    def close(self):
        self.apcg.apcg_ctx_synchronize(self.ctx)
        self.apcg.apcg_info_destroy(self.info)
        for v in (self.b, self.x, self.y, self.A):
            v.close()
        self.apcg.apcg_ctx_destroy(self.ctx)


@pytest.mark.parametrize("how", ["read", "wait_for"])
def test_group_is_recorded_before_a_stream_wait(apcg, how):
    print(f"case event order {how}", flush=True)
    busy, a = Busy(apcg), apcg.apcg_ctx_create(0)
    t = apcg.apcg_scalar_create(a)
    apcg.apcg_ctx_synchronize(a)
    busy.start()
    apcg.apcg_scalar_set(t, 3.0, a)
    if how == "read":
        apcg.apcg_vec_copy_async(busy.y.h, busy.x.h, a)  # waits on the device for the solve's x
    else:
        apcg.apcg_ctx_wait_for(a, busy.ctx)
        apcg.apcg_vec_set_async(busy.y.h, 1.0, a)
    assert busy.running()
    assert apcg.apcg_scalar_get(t) == 3.0
    assert busy.running(), "the read of a scalar waited for another context's solve"
    apcg.apcg_ctx_synchronize(a)
    assert not busy.running()
    apcg.apcg_scalar_destroy(t)
    apcg.apcg_ctx_destroy(a)
    busy.close()


def test_group_is_recorded_before_unmarked_work(apcg):
    """Training steps take no part in the marks."""
    import torch
    from paper_2306_17801_amd.learned import NPARAM, pack_params
    from paper_2306_17801_amd.problems import mlp_initial_params

    print("case event order unmarked work", flush=True)
    a = apcg.apcg_ctx_create(0)
    g = torch.Generator(device="cuda").manual_seed(1)
    B = 2000
    params = torch.from_numpy(pack_params(mlp_initial_params(7))).cuda()
    m, v, loss = torch.zeros(NPARAM, device="cuda"), torch.zeros(NPARAM, device="cuda"), torch.zeros(1, device="cuda")
    X, h = torch.randn(B, 16, device="cuda", generator=g), torch.randn(B, 9, device="cuda", generator=g)
    G = torch.eye(9, device="cuda").reshape(1, 81).repeat(B, 1)
    torch.cuda.synchronize()

    def steps(k):
        for i in range(k):
            apcg.apcg_mlp_train_step(a, params, m, v, i + 1, 1e-3, X, G, h, loss, 1.0, 0.05)

    t = apcg.apcg_scalar_create(a)
    steps(10)
    apcg.apcg_ctx_synchronize(a)
    t0 = time.perf_counter()
    steps(200)
    apcg.apcg_ctx_synchronize(a)
    whole = time.perf_counter() - t0
    apcg.apcg_scalar_set(t, 5.0, a)
    steps(200)
    if apcg.apcg_ctx_query_idle(a):
        pytest.skip(f"the steps are queued no faster than they run ({whole * 5:.3f} ms each)")
    assert apcg.apcg_scalar_get(t) == 5.0
    assert not apcg.apcg_ctx_query_idle(a), "the read of a scalar waited for the training steps behind it"
    apcg.apcg_ctx_synchronize(a)
    apcg.apcg_scalar_destroy(t)
    apcg.apcg_ctx_destroy(a)
