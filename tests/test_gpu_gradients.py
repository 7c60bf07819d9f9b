"""The written gradients against the added ones, at sizes around a workgroup
and with padding, and the scaled loss gradient against the product."""
import pytest
import torch

from paper_2603_08997_amd import autograd as AG
from paper_2603_08997_amd import scenes as S
from tests.gpu_util import GpuRender, require_gpu, sg, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("deg", [0, 1, 2, 3])
@pytest.mark.parametrize("n,views", [(1, 1), (255, 2), (257, 1), (3001, 2)])
def test_written_gradients_equal_the_added_ones(n, views, deg):
    require_gpu()
    m = sg()
    sc = S.mixture_scene(7, n, sh_degree=deg, log_scale_mean=-2.0)
    gr = GpuRender(sc, S.hemisphere_cameras(5, views, 120, 75))
    gr.forward()
    dl = torch.randn(gr.rgb.numel(), generator=torch.Generator().manual_seed(1)).cuda()
    m.rasterize_backward(gr.cams, n, gr.rp, gr.ws, gr.capacity, dl)
    added = torch.zeros_like(gr.planes)
    m.project_backward(gr.planes, n, deg, gr.cams, gr.rp, gr.ws, gr.capacity, None, added)
    written = torch.full_like(gr.planes, float("nan"))
    m.render_gradients(gr.planes, n, deg, gr.cams, gr.rp, gr.ws, gr.capacity, dl, written)
    assert bool((written[:, n:] == 0).all())
    # the two ran the compositing backward, whose float atomics come in any order
    scale = added.abs().amax(1, keepdim=True).clamp_min(1e-30)
    assert ((written - added).abs() / scale).max().item() <= 1e-4
    # what no view sees: exactly zero in both
    unseen = (added == 0).all(0)
    assert torch.equal(unseen, (written == 0).all(0))


@pytest.mark.parametrize("w,h", [(1, 1), (54, 40), (131, 77)])
@pytest.mark.parametrize("scale", [1.0, 0.0, -2.7, float("inf")])
def test_scaled_loss_gradient_is_the_product(w, h, scale):
    require_gpu()
    m = sg()
    gen = torch.Generator().manual_seed(w)
    rgb, target = (torch.rand(3 * w * h, generator=gen).cuda() for _ in range(2))
    lws, loss = m.alloc_bytes(m.loss_workspace_size(w, h)), torch.zeros(1, device="cuda")
    m.photometric_loss(rgb, target, w, h, 0.2, lws, loss)
    plain, scaled = torch.zeros_like(rgb), torch.zeros_like(rgb)
    m.photometric_loss_backward(rgb, target, w, h, 0.2, lws, None, plain)
    g = torch.tensor(scale, device="cuda")
    m.photometric_loss_gradient(rgb, target, w, h, 0.2, lws, g, scaled)
    want = plain * g
    assert torch.equal(torch.nan_to_num(want), torch.nan_to_num(scaled))
    x = rgb.clone().requires_grad_(True)
    (AG.photometric_loss(x, target, w, h) * g).backward()
    assert torch.equal(torch.nan_to_num(want), torch.nan_to_num(x.grad))


def test_render_keeps_the_cameras_of_its_forward():
    require_gpu()
    sc, cams = S.tiny_scene(3, 300), S.tetra_cameras()[:2]
    grads = []
    for change in (False, True):
        planes, mine = to_dev(sc.to_planes()).requires_grad_(True), list(cams)
        img = AG.render(planes, 300, 0, mine, recompute=True)
        if change:
            mine.clear()
        (img * img).sum().backward()
        grads.append(planes.grad)
    scale = grads[0].abs().amax(1, keepdim=True).clamp_min(1e-30)
    assert ((grads[0] - grads[1]).abs() / scale).max().item() <= 1e-4


def test_the_loss_scale_stays_in_a_graph_of_the_backward():
    require_gpu()
    gen = torch.Generator().manual_seed(2)
    rgb, target = (torch.rand(3 * 20 * 12, generator=gen).cuda() for _ in range(2))
    rgb.requires_grad_(True)
    scale = torch.tensor(-1.5, device="cuda", requires_grad=True)
    loss = AG.photometric_loss(rgb, target, 20, 12) * scale
    (g,) = torch.autograd.grad(loss, rgb, create_graph=True)
    g.sum().backward()
    # d/d scale of sum(scale dL/d rgb)
    want = (g.detach().double() / -1.5).sum()
    assert abs(scale.grad.item() - want.item()) <= 1e-5 * g.detach().abs().sum().item()
