"""Events outlive the context they were recorded on (csrc/runtime.hip): objects
that a destroyed context wrote or read last are queried, waited for and
released after its stream would be gone, as are the team launches it had in
flight."""
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


def test_objects_outlive_the_context_that_wrote_them(apcg):
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print("case objects outlive their context", flush=True)
    rng = np.random.default_rng(2)
    n = 5000
    keep = [DeviceVec(rng.uniform(-1, 1, n)) for _ in range(40)]
    want = [v.numpy() for v in keep]
    mats = [DeviceCSR(P.laplace_2d(20 + k)) for k in range(8)]
    scalars, outs = [], []
    for rep in range(6):
        c = apcg.apcg_ctx_create(0)
        two = apcg.apcg_scalar_create(c)
        apcg.apcg_scalar_set(two, 2.0, c)
        scalars.append(two)
        for i, v in enumerate(keep):
            if i % 6 == rep:
                apcg.apcg_vec_scale_async(v.h, two, c)
                want[i] = 2.0 * want[i]
        for A in mats:
            y, z = DeviceVec.zeros(A.n), DeviceVec.zeros(A.n)
            apcg.apcg_mat_mult_async(A.h, y.h, z.h, c)
            y.close()  # (read last by the context; z is written last by it)
            outs.append(z)
        apcg.apcg_ctx_destroy(c)
        # new contexts may get the memory, and the stream, of the old one
        d = apcg.apcg_ctx_create(0)
        apcg.apcg_ctx_synchronize(d)  # releases what has finished
        t = apcg.apcg_scalar_create(d)
        i = rep
        apcg.apcg_vec_norm2_async(keep[i].h, t, d)  # waits on the device for the destroyed context's write
        assert np.isclose(apcg.apcg_scalar_get(t), np.linalg.norm(want[i]), rtol=1e-12)
        assert apcg.apcg_scalar_get(two) == 2.0
        apcg.apcg_scalar_destroy(t)
        apcg.apcg_ctx_destroy(d)
    for v, w in zip(keep, want):
        assert np.array_equal(v.numpy(), w)
        v.close()
    for v in outs:
        v.close()
    for A in mats:
        A.close()
    for s in scalars:
        apcg.apcg_scalar_destroy(s)


def test_team_launches_of_destroyed_contexts(apcg):
    """The next launch asks whether those in flight have ended."""
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print("case team launches of destroyed contexts", flush=True)
    A = P.laplace_2d(110)
    dA, b = DeviceCSR(A), DeviceVec(np.ones(A.n))
    info = apcg.apcg_info_create(0, 1)
    opts = apcg.apcg_solve_opts_default(x0_is_zero=1)
    xs = []
    for _ in range(12):
        c = apcg.apcg_ctx_create(0)
        x = DeviceVec.zeros(A.n)
        apcg.apcg_ksp_solve(c, dA.h, b.h, x.h, 0.0, 30, opts, info, 0)
        apcg.apcg_ctx_destroy(c)
        xs.append(x)
    got = [x.numpy() for x in xs]
    assert all(np.array_equal(g, got[0]) for g in got) and np.all(np.isfinite(got[0]))
    assert apcg.apcg_info_get(info, 0)["iterations"] == 30
    for x in xs:
        x.close()
    apcg.apcg_info_destroy(info)
    b.close()
    dA.close()
