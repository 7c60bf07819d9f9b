"""The loss and its gradient on images around the strip edges of the filter (54
columns, 4 rows and more, one strip of rows and several), against the oracle."""
import numpy as np
import pytest
import torch

from oracle import loss as Lm
from tests.gpu_util import rel_max_err, rel_norm_err, require_gpu, say, sg, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h", [(1, 1), (53, 4), (54, 5), (55, 3), (107, 10), (108, 11), (109, 8),
                                 (2, 300), (700, 2), (541, 409)])
def test_loss_and_gradient_around_strip_edges(w, h):
    require_gpu()
    m = sg()
    say(f"loss strips {w}x{h}")
    rng = np.random.default_rng(h * 1000 + w)
    x = rng.uniform(0, 1, (3, h, w)).astype(np.float32)
    y = np.clip(x + rng.normal(0, 0.15, x.shape), 0, 1).astype(np.float32)
    ws = m.alloc_bytes(m.loss_workspace_size(w, h))
    ws.fill_(0xFF)   # nothing read before it is written
    loss, static = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
    dx, dy = to_dev(x), to_dev(y)
    dl = torch.full_like(dx, float("nan"))
    m.photometric_loss(dx, dy, w, h, 0.2, ws, loss)
    m.photometric_loss_backward(dx, dy, w, h, 0.2, ws, None, dl)
    m.photometric_loss_static(dx, dy, w, h, 0.2, static)
    torch.cuda.synchronize()
    assert loss.item() == static.item()
    L_ref, g_ref = Lm.photometric_loss_and_grad(x.astype(np.float64), y.astype(np.float64))
    assert abs(loss.item() - L_ref) <= 1e-5 * abs(L_ref)
    # float32 moments over C2 = 9e-4: relative rounding 1e-7 becomes 1e-4 at most
    g, g_ref = dl.cpu().numpy(), g_ref.numpy()
    assert rel_norm_err(g, g_ref) < 1e-4
    assert rel_max_err(g, g_ref) < 1e-4
