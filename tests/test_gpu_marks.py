"""The byte an entry that tells the projection backward what a view sees: the
gradients of a batch equal the sums of its single views, at SH degrees and set
sizes on both sides of the launch rule of a batch's projection, with Gaussians
that no view, one view and every view sees and colours clamped at 0."""
import pytest
import torch

from paper_2603_08997_amd import scenes as S
from tests.gpu_util import GpuRender, require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,deg,views", [(700, 0, 2), (700, 3, 16), (2001, 2, 5), (66000, 1, 3)])
def test_batch_gradients_are_the_sums_of_the_views(n, deg, views):
    require_gpu()
    sc = S.mixture_scene(11, n, sh_degree=deg, log_scale_mean=-2.5 if n < 5000 else -4.0)
    sc.means[::7] *= 3.0            # many leave some of the views
    sc.sh[::3, 0, :] -= 2.5         # clamped channels
    cams = S.hemisphere_cameras(6, views, 120, 75)
    batch = GpuRender(sc, cams)
    batch.forward()
    dl = torch.randn(batch.rgb.numel(), generator=torch.Generator().manual_seed(1)).cuda()
    got = batch.backward(dl)
    want, at = torch.zeros_like(got, dtype=torch.float64), 0
    for cam in cams:
        one = GpuRender(sc, [cam])
        one.forward()
        px = 3 * cam.width * cam.height
        want += one.backward(dl[at:at + px].contiguous()).double()
        at += px
    scale = want.abs().amax(1, keepdim=True).clamp_min(1e-30)
    err = ((got.double() - want).abs() / scale).max().item()
    say(f"marks n={n} deg={deg} views={views}: {err:.1e}, unseen {int((want == 0).all(0).sum())}")
    # float32 sums of a few hundred terms by atomics in any order, then over the views
    assert err <= 1e-4
    assert torch.equal((got == 0).all(0), (want == 0).all(0))
