"""A set of SH degree 3 rendered at a lower degree, as while the degree is raised in
training: the planes the degree does not read have a gradient of exactly zero,
whatever the allocator's memory held."""
import pytest
import torch

from paper_2603_08997_amd import autograd as AG
from paper_2603_08997_amd import scenes as S
from tests.gpu_util import require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("recompute", [False, True])
@pytest.mark.parametrize("views", [1, 2])
@pytest.mark.parametrize("deg", [0, 1, 2, 3])
def test_planes_past_the_degree_have_zero_gradient(deg, views, recompute):
    require_gpu()
    n, used = 1000, S.n_planes(deg)
    cams = S.hemisphere_cameras(5, views, 120, 75)
    full = to_dev(S.mixture_scene(7, n, sh_degree=3, log_scale_mean=-2.0).to_planes())
    grads = []
    for planes in (full, full[:used].contiguous()):
        planes = planes.clone().requires_grad_(True)
        img = AG.render(planes, n, deg, cams, recompute=recompute)
        poison = [torch.full_like(planes, float("nan")) for _ in range(4)]
        del poison
        (img * img).sum().backward()
        grads.append(planes.grad)
    assert grads[0].shape == full.shape
    assert bool((grads[0][used:] == 0).all())
    # the others are those of the set with these planes alone, up to the order of
    # the float atomics
    scale = grads[1].abs().amax(1, keepdim=True).clamp_min(1e-30)
    assert ((grads[0][:used] - grads[1]).abs() / scale).max().item() <= 1e-4
