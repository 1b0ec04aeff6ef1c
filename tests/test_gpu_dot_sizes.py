"""Inner products at the edges of the one-launch kernel (8192 entries) and of
its threads, against extended precision: |error| <= n 2^-53 sum |x_i y_i|."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 1023, 1024, 1025, 8191, 8192, 8193, 300001])
def test_dot_and_norm(n):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_17801_amd as apcg
    from paper_2306_17801_amd.device import DeviceVec

    print(f"case dot n={n}", flush=True)
    rng = np.random.default_rng(n)
    x, y = rng.uniform(-1, 1, n), rng.uniform(-1, 1, n)
    ctx = apcg.apcg_ctx_create(0)
    dx, dy, s = DeviceVec(x), DeviceVec(y), apcg.apcg_scalar_create(ctx)
    apcg.apcg_vec_dot_async(dx.h, dy.h, s, ctx)
    assert abs(apcg.apcg_scalar_get(s) - math.fsum(x * y)) <= (n + 1) * 2.0**-53 * math.fsum(np.abs(x * y))
    apcg.apcg_vec_norm2_async(dx.h, s, ctx)
    assert apcg.apcg_scalar_get(s) == pytest.approx(math.sqrt(math.fsum(x * x)), rel=(n + 2) * 2.0**-53)
    apcg.apcg_scalar_destroy(s)
    apcg.apcg_ctx_destroy(ctx)
