"""Tiles composited by several waves: the image, the per-pixel state and the
work counters of every strip count equal those of 8x8 tiles (one wave each,
no strips) bit for bit, and the record gradients up to the order of the float
atomic additions."""
import numpy as np
import pytest

from paper_2603_08997_amd import scenes as S
from tests.gpu_util import rel_max_err, require_gpu, say, sg
from tests.test_gpu_stages import Stage, _records

pytestmark = pytest.mark.gpu


# image sizes on both sides of the launch rule's tile counts (1536 and 5120
# tiles of 256 pixels), with partly and wholly empty strips at the lower edge
@pytest.mark.parametrize("tile", [(16, 16), (32, 8)])
@pytest.mark.parametrize("w,h", [(5, 3), (33, 18), (637, 479), (640, 624), (1296, 1003),
                                 (1312, 1009)])
def test_strips_match_unsplit_tiles(tile, w, h):
    require_gpu()
    m = sg()
    cams = [S.look_at_camera((3.0, 1.0, 1.0), w, h)]
    n = min(20000, 50 + w * h // 16)
    recs, cat = _records(n, cams, 77, max_radius=24)
    say(f"strips {tile} {w}x{h} n={n}")
    # the smallest prefix of the list split, so that some tiles are resumed
    out = []
    for tw, th in ((8, 8), tile):
        rp = m.RasterParams(tile_w=tw, tile_h=th, bg=(0.2, 0.4, 0.6), split_prefix=512)
        st = Stage(n, cams, rp, cat, 4_000_000)
        rgb, tf, nl = st.rasterize()
        assert st.flags == 0
        dl = np.random.default_rng(3).normal(0, 1, len(rgb)).astype(np.float32)
        out.append((rgb, tf, m.read_counters(st.ws)["blended"], nl > 0, st.backward(dl)))
    (r0, t0, b0, n0, g0), (r1, t1, b1, n1, g1) = out
    assert np.array_equal(r0, r1)
    assert np.array_equal(t0, t1)
    assert b0 == b1
    assert np.array_equal(n0, n1)
    # sums of the same float terms in another order: a few hundred terms of
    # relative rounding 6e-8 each, against the largest gradient
    assert rel_max_err(g1, g0) < 2e-5, rel_max_err(g1, g0)
