"""The two kernels of a training step (csrc/learn.hip) at the edges of what a
workgroup takes: 4 samples in the first, 128 at a time in the second.  Loss
and gradients hold the repository's bar against the FP64 oracle; the step
moves the first moment by 0.1 of the same gradients."""
import numpy as np
import pytest

from oracle import learned as OL
from test_gpu_learned import _mlp_inputs, _params, apcg, ctx, dev, host, pack, unpack  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [2, 3, 4, 5, 127, 128, 129, 257, 2049])
def test_step_kernels_at_batch_edges(apcg, ctx, B):  # noqa: F811
    import torch

    print(f"case mlp step B={B}", flush=True)
    pv = pack(_params())
    X, Gs, hs = _mlp_inputs(B, 20 + B)
    loss, loss2 = (torch.zeros(1, dtype=torch.float32, device="cuda:0") for _ in range(2))
    grad, m, v = (torch.zeros(5833, dtype=torch.float32, device="cuda:0") for _ in range(3))
    dP, dX, dG, dh = dev(pv), dev(X), dev(Gs), dev(hs)
    torch.cuda.synchronize()
    apcg.apcg_mlp_loss_grad(ctx, dP, dX, dG, dh, loss, grad, mu=1.0, eps=0.05)
    apcg.apcg_mlp_train_step(ctx, dP, m, v, 1, 1e-3, dX, dG, dh, loss2)
    g, got = host(apcg, ctx, grad), host(apcg, ctx, m)
    L_ref, g_ref = OL.batch_loss(unpack(pv), X.astype(np.float64), Gs.astype(np.float64), hs.astype(np.float64),
                                 OL.positivity_grid(), 1.0, 0.05)
    assert host(apcg, ctx, loss)[0] == pytest.approx(L_ref, rel=2e-5)
    assert host(apcg, ctx, loss2)[0] == host(apcg, ctx, loss)[0]
    o = 0
    for k, shape in OL.SHAPES:
        n = int(np.prod(shape))
        r = g_ref[k].reshape(-1)
        assert np.max(np.abs(g[o:o + n] - r)) <= 1e-4 * np.max(np.abs(r)) + 1e-9, k
        o += n
    # 1 - 0.9f rounds to 0.1 within 3e-7, and one rounding of the product
    assert np.all(np.abs(got - np.float32(0.1) * g) <= 1e-6 * np.abs(got) + 1e-37)
