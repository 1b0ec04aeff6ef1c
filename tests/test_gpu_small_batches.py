"""Batches in the AUTO schedule on both sides of where teams take over from one
persistent workgroup per system (rows, rows times iterations, no iterations):
against the oracle, and the bits of the schedule that solves them."""
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


@pytest.mark.parametrize("shape,args,teams", [((16, 20), (1e-10, 2000), False), ((17, 19), (1e-10, 2000), True),
                                              ((25, 40), (0.0, 10), False), ((25, 41), (0.0, 10), True),
                                              ((40, 41), (0.0, 0), False)], ids=str)
def test_batch_of_small_systems(apcg, shape, args, teams):
    from paper_2306_17801_amd.device import DeviceCSR, DeviceVec

    print(f"case small batch {shape} {args}", flush=True)
    S = []
    for i in range(4):
        rng = np.random.default_rng(i)
        A = P.diffusion_csr(np.exp(rng.standard_normal(shape)), aniso=2.0)
        S.append((DeviceCSR(A), A, rng.uniform(-1, 1, A.n), rng.uniform(-1, 1, A.n)))
    count = 300
    ctx, info = apcg.apcg_ctx_create(0), apcg.apcg_info_create(0, count)
    bs = [DeviceVec(S[i % 4][2]) for i in range(count)]

    def solve(sched):
        xs = [DeviceVec(S[i % 4][3]) for i in range(count)]
        apcg.apcg_ksp_solve_batched(ctx, [S[i % 4][0].h for i in range(count)], [b.h for b in bs], [x.h for x in xs],
                                    *args, apcg.apcg_solve_opts_default(batch_schedule=sched), info)
        return [apcg.apcg_info_get(info, k) for k in range(count)], [x.numpy() for x in xs]

    got, same = solve(0), solve(2 if teams else 1)
    assert got[0] == same[0] and all(np.array_equal(p, q) for p, q in zip(got[1], same[1]))
    for k in range(4):
        ref = oracle.pcg(S[k][1], S[k][2], x0=S[k][3], rtol=args[0], maxit=args[1])
        assert abs(got[0][k]["iterations"] - ref.its) <= 1
        assert np.linalg.norm(got[1][k] - ref.x) <= (1e-9 if args[0] else 1e-12) * np.linalg.norm(ref.x)
    apcg.apcg_info_destroy(info)
    apcg.apcg_ctx_destroy(ctx)
