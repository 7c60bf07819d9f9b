"""The split of super-tile lists into tile lists at every segment length its
rule picks (64, 128 and 256 pairs): the tile lists are the entries of the
super-tile lists whose rectangles hold the tile, in their order, and lists cut
and completed composite the same image."""
import numpy as np
import pytest

from paper_2603_08997_amd import scenes as S
from tests.gpu_util import require_gpu, say, sg, tile_lists
from tests.test_gpu_stages import Stage, _records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 64, 65, 1025, 65536, 65537, 524289])
def test_tile_lists_are_the_super_lists_split(n):
    require_gpu()
    m = sg()
    cams = [S.look_at_camera((3.0, 1.0, 1.0), 250, 139)]
    recs, cat = _records(n, cams, 810, max_radius=6 if n > 100_000 else 14)
    base = dict(tile_w=16, tile_h=16, super_tile=5)
    st = Stage(n, cams, m.RasterParams(alpha_min=0.0, split_prefix=0, **base), cat, 4_000_000)
    assert st.flags == 0
    say(f"split n={n} pairs {st.kept} items {st.items}")
    keys, ents, ranges = st.lists()
    lists = tile_lists(st.ws, st.L)
    tx_n, ty_n, sx_n, empty = 16, 9, 4, np.zeros(0, np.int64)
    total = 0
    for t in range(tx_n * ty_n):
        tx, ty = t % tx_n, t // tx_n
        a, b = ranges[(ty // 5) * sx_n + tx // 5]
        r, lx, ly = st.rect[a:b], tx % 5, ty % 5
        inside = (r[:, 0] <= lx) & (lx <= r[:, 1]) & (r[:, 2] <= ly) & (ly <= r[:, 3])
        want = ents[a:b][inside].astype(np.int64)
        assert np.array_equal(lists.get(t, empty), want), t
        total += len(want)
    assert st.items == total
    # default thresholds: whole lists against cut and completed ones, twice over
    whole = Stage(n, cams, m.RasterParams(split_prefix=0, **base), cat, 4_000_000)
    cut = Stage(n, cams, m.RasterParams(split_prefix=512, **base), cat, 4_000_000)
    want = whole.rasterize()
    for _ in range(2):
        got = cut.rasterize()
        assert cut.flags == 0
        assert all(np.array_equal(x, y) for x, y in zip(got, want))
