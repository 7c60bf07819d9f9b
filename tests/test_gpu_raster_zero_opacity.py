"""Entries of opacity 0 with alpha_min = 0: they take part in the pixels of their box
(with alpha' = 0) whether one wave takes a tile or several, so the last positions
and the work counters of tiles in parts equal those of 8x8 tiles, one wave each."""
import numpy as np
import pytest

from paper_2603_08997_amd import scenes as S
from tests.gpu_util import require_gpu, say, sg
from tests.test_gpu_stages import Stage, _records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [(16, 16), (32, 8)])
@pytest.mark.parametrize("w,h", [(33, 18), (637, 479), (1312, 1009)])
def test_zero_opacity_takes_part(tile, w, h):
    require_gpu()
    m = sg()
    cams = [S.look_at_camera((3.0, 1.0, 1.0), w, h)]
    n = 50 + w * h // 64
    recs, cat = _records(n, cams, 88, max_radius=24)
    cat["opacity"][::3] = 0.0
    say(f"zero opacity {tile} {w}x{h} n={n}")
    out = []
    for tw, th in ((8, 8), tile):
        rp = m.RasterParams(tile_w=tw, tile_h=th, alpha_min=0.0, t_min=0.0, split_prefix=0)
        st = Stage(n, cams, rp, cat, 4_000_000)
        rgb, tf, nl = st.rasterize()
        assert st.flags == 0
        c = m.read_counters(st.ws)
        out.append((rgb, tf, nl > 0, c["blended"]))
    (r0, t0, n0, b0), (r1, t1, n1, b1) = out
    assert np.array_equal(r0, r1) and np.array_equal(t0, t1)
    assert np.array_equal(n0, n1)
    assert b0 == b1
