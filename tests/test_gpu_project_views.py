"""Projection of a batch of views by one thread a Gaussian: the records, super-
tile counts and depths equal those of one view at a time bit for bit, on both
sides of the launch rule's Gaussian count."""
import numpy as np
import pytest
import torch

from paper_2603_08997_amd import scenes as S
from tests.gpu_util import region, require_gpu, sg, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("deg", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [65535, 65536, 65601])
def test_batched_projection_matches_single_views(n, deg):
    require_gpu()
    m = sg()
    sc = S.mixture_scene(5, n, sh_degree=deg)
    # some Gaussians behind the cameras and some degenerate
    sc.means[::97] *= 4.0
    sc.quats[5] = 0.0
    sc.log_scales[7] = np.inf
    planes, rp, cap = to_dev(sc.to_planes()), m.RasterParams(), 4096
    cams = S.hemisphere_cameras(3, 1, 320, 201) + S.hemisphere_cameras(4, 2, 64, 77)

    def records(cs):
        ws = m.alloc_bytes(m.forward_workspace_size(rp, n, cs, cap)).zero_()
        L = m.get_workspace_layout(rp, n, cs, cap)
        m.project(planes, n, deg, cs, rp, ws, cap)
        torch.cuda.synchronize()
        k = n * len(cs)
        return [region(ws, o, c * k, np.uint32).reshape(len(cs), -1)
                for o, c in ((L.records, 12), (L.tiles, 1), (L.depth, 1))]

    batch = records(cams)
    for v, cam in enumerate(cams):
        for b, one in zip(batch, records([cam])):
            assert np.array_equal(b[v], one[0]), v
