"""Sums of the loss over images whose strips have many rows, where a sum in FP32
drifts: flat pictures, whose exact loss has a closed form."""
import numpy as np
import pytest
import torch

from tests.gpu_util import require_gpu, say, sg

pytestmark = pytest.mark.gpu

HALF_ULP = 2.0 ** -24   # relative rounding of one FP32 operation


def _loss(m, rgb, target, w, h, lam):
    x = torch.full((3 * w * h,), rgb, device="cuda")
    y = torch.full((3 * w * h,), target, device="cuda")
    lws, loss = m.alloc_bytes(m.loss_workspace_size(w, h)), torch.zeros(1, device="cuda")
    m.photometric_loss(x, y, w, h, lam, lws, loss)
    return loss.item()


@pytest.mark.parametrize("w,h", [(1600, 1060), (3840, 2160), (54, 32768), (8192, 8192)])
@pytest.mark.parametrize("d", [0.1, 0.013, 0.37])
def test_l1_of_a_flat_difference(w, h, d):
    require_gpu()
    m = sg()
    say(f"flat difference {d} at {w}x{h}")
    y = np.float32(0.25)
    x = np.float32(y + np.float32(d))
    want = float(x) - float(y)   # exact in FP32
    got = _loss(m, float(x), float(y), w, h, 0.0)
    # eight equal values added in FP32: the 2nd to 8th partial sums round, 35/8 half
    # ulps of the whole, and the loss itself
    assert abs(got - want) <= (35 / 8 + 1) * HALF_ULP * want


@pytest.mark.parametrize("w,h", [(1600, 1060), (8192, 8192)])
@pytest.mark.parametrize("c", [0.005, 0.0071, 0.013])
def test_ssim_of_black_against_flat(w, h, c):
    require_gpu()
    m = sg()
    say(f"black against {c} at {w}x{h}")
    c = float(np.float32(c))
    g = np.exp(-((np.arange(11) - 5.0) ** 2) / (2 * 1.5 ** 2))
    g /= g.sum()

    def profile(n):   # weight of the window inside the image, at the edges and within
        edge = [g[5 - k:].sum() for k in range(5)]
        return np.array(edge + [1.0]), np.array([2.0] * 5 + [n - 10.0]) / n

    (px, fx), (py, fy) = profile(w), profile(h)
    inside, part = np.outer(py, px), np.outer(fy, fx)
    mu, var = c * inside, c * c * inside - (c * inside) ** 2
    c1, c2 = 0.01 ** 2, 0.03 ** 2
    want = float((part * (c1 / (mu * mu + c1)) * (c2 / (var + c2))).sum())
    got = 1.0 - _loss(m, 0.0, c, w, h, 1.0)
    # mu: two filters of 11 rounded weights and sums, 24 half ulps; S moves by twice
    # the relative error of mu at most, and the variance, below c^2 and 50 half ulps
    # of it off, against c2; 10 for the quotient, the sums over rows and constants
    assert abs(got - want) <= (2 * 24 + 50 * c * c / c2 + 10) * HALF_ULP * want + HALF_ULP
