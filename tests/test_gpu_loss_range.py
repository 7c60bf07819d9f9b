"""The loss and its gradient of pixel values far from [0, 1], up to where the squares
in SSIM overflow, against the oracle: where the denominator alone overflows S is
0 and the gradient that of the absolute difference, where the numerators do too
the loss is undefined."""
import numpy as np
import pytest
import torch

from oracle import loss as Lm
from tests.gpu_util import rel_max_err, require_gpu, say, sg, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [255.0, 3e3, 1e5, 1e8, 3e9, 5e9, 1e10, 1e15, 2e19])
def test_loss_and_gradient_of_large_values(scale):
    require_gpu()
    m = sg()
    say(f"loss of values up to {scale}")
    w, h = 200, 100
    rng = np.random.default_rng(int(np.log10(scale)))
    x = rng.uniform(0, scale, (3, h, w)).astype(np.float32)
    y = rng.uniform(0, min(scale, 255.0), x.shape).astype(np.float32)
    ws = m.alloc_bytes(m.loss_workspace_size(w, h))
    loss, dl = torch.zeros(1, device="cuda"), torch.full((3 * h * w,), float("nan"), device="cuda")
    dx, dy = to_dev(x.reshape(-1)), to_dev(y.reshape(-1))
    m.photometric_loss(dx, dy, w, h, 0.2, ws, loss)
    m.photometric_loss_backward(dx, dy, w, h, 0.2, ws, None, dl)
    L_ref, g_ref = Lm.photometric_loss_and_grad(x.astype(np.float64), y.astype(np.float64))
    if scale > 1e19:   # inf / inf
        assert bool(torch.isnan(loss).all())
        return
    assert abs(loss.item() - L_ref) <= 1e-5 * abs(L_ref)
    assert rel_max_err(dl.cpu().numpy(), g_ref.numpy().reshape(-1)) < 1e-4


def test_infinite_and_undefined_pixels_stay_in_their_window():
    """What is further than the window from such a pixel is as without it."""
    require_gpu()
    m = sg()
    w, h = 120, 90
    gen = torch.Generator().manual_seed(4)
    x, y = (torch.rand(3, h, w, generator=gen) for _ in range(2))
    grads = []
    for bad in (None, float("inf"), float("nan")):
        xx = x.clone()
        if bad is not None:
            xx[:, 40, 60] = bad
        dx, dy = xx.reshape(-1).cuda(), y.reshape(-1).cuda()
        ws = m.alloc_bytes(m.loss_workspace_size(w, h))
        loss, dl = torch.zeros(1, device="cuda"), torch.zeros_like(dx)
        m.photometric_loss(dx, dy, w, h, 0.2, ws, loss)
        m.photometric_loss_backward(dx, dy, w, h, 0.2, ws, None, dl)
        assert bool(torch.isfinite(loss).all()) == (bad is None)
        grads.append(dl.cpu().reshape(3, h, w))
    far = torch.ones(h, w, dtype=torch.bool)
    far[40 - 10:40 + 11, 60 - 10:60 + 11] = False
    assert bool(torch.isfinite(grads[0]).all())
    for g in grads[1:]:
        assert torch.equal(g[:, far], grads[0][:, far])
