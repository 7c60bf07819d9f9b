"""The visible-only Adam step on both sides of the set size from which waves
stream whole lines: Gaussians that no view sees keep every bit, also those in a
wave with seen ones, and the others take the dense step, with most, a few and
none of a wave's Gaussians seen."""
import pytest
import torch

from paper_2603_08997_amd import scenes as S
from tests.gpu_util import require_gpu, say, sg, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("views", [1, 2])
@pytest.mark.parametrize("n", [5000, 131071, 131072, 140001])
def test_visible_only_is_the_dense_step_on_the_seen(n, views):
    require_gpu()
    m = sg()
    sc = S.mixture_scene(13, n, sh_degree=1, log_scale_mean=-5.0)
    k = n // 3
    sc.means[k:2 * k] += 50.0        # whole waves seen by no view
    sc.means[2 * k:][torch.rand(n - 2 * k, generator=torch.Generator().manual_seed(3)).numpy() > 0.03] += 50.0
    cams, rp, cap = S.hemisphere_cameras(5, views, 96, 80), m.RasterParams(), 1 << 22
    ws = m.alloc_bytes(m.forward_workspace_size(rp, n, cams, cap)).zero_()
    rgb = torch.zeros(views * 3 * 96 * 80, device="cuda")
    planes = to_dev(sc.to_planes())
    m.render_forward(planes, n, 1, cams, rp, ws, cap, rgb)
    L = m.get_workspace_layout(rp, n, cams, cap)
    tiles = ws[L.tiles:L.tiles + 4 * n * views].view(torch.int32).view(views, n)
    seen = (tiles > 0).any(0)
    m.rasterize_backward(cams, n, rp, ws, cap, torch.ones_like(rgb))
    gen = torch.Generator().manual_seed(4)
    m0, v0 = (1e-3 * torch.rand(planes.shape, generator=gen).cuda() for _ in range(2))
    out = []
    for visible_only in (False, True):
        p, mm, vv = planes.clone(), m0.clone(), v0.clone()
        step = torch.full((1,), 3, dtype=torch.int32, device="cuda")
        m.project_backward_adam(p, n, 1, cams, rp, ws, cap,
                                m.AdamParams(lr=m.default_lrs(1), visible_only=visible_only), mm, vv, step)
        assert step.item() == 4
        out.append((p, mm, vv))
    say(f"visible Adam n={n} views={views}: seen {int(seen.sum())}")
    assert 0 < int(seen.sum()) < n // 2
    for before, dense, visible in zip((planes, m0, v0), *out):
        assert torch.equal(visible[:, :n][:, seen], dense[:, :n][:, seen])
        assert torch.equal(visible[:, :n][:, ~seen], before[:, :n][:, ~seen])
        assert torch.equal(visible[:, n:], before[:, n:])
