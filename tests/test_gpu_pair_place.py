"""Super-tile lists placed without a sort (few super-tiles) on both sides of the
super-tile bound, against the oracle's box lists: bit for bit without the reach
test, and with it an ordered subsequence whose tile lists keep every entry that
contributes; entries with more candidate super-tiles than are tested, more
pairs than are expanded at a time, and every remainder of the entries a block
takes."""
import numpy as np
import pytest

from paper_2603_08997_amd import scenes as S
from tests.gpu_util import require_gpu, say, sg
from tests.test_gpu_stages import (Stage, _check_tile_lists, _oracle_rects, _oracle_super_lists,
                                   _records, _views)

pytestmark = pytest.mark.gpu


def _check(cams, n, tile, super_tile, max_radius, alpha_min, seed):
    m = sg()
    tw, th = tile
    recs, cat = _records(n, cams, seed, max_radius=max_radius, tie_fraction=0.2)
    rp = m.RasterParams(tile_w=tw, tile_h=th, super_tile=super_tile, split_prefix=0,
                        alpha_min=alpha_min)
    st = Stage(n, cams, rp, cat, 1_000_000)
    assert st.flags == 0
    sups, vals, ranges = _oracle_super_lists(recs, cams, n, tw, th, super_tile)
    keys, ents, granges = st.lists()
    say(f"  n={n} supers={st.L.total_supers} pairs {len(vals)} kept {len(ents)}")
    assert st.needed == len(vals) and st.kept == len(ents)
    assert np.array_equal(keys, np.repeat(np.arange(len(granges)), granges[:, 1] - granges[:, 0]))
    if alpha_min == 0.0:
        assert np.array_equal(ents.astype(np.int64), vals)
        assert np.array_equal(granges.astype(np.int64), ranges)
        assert np.array_equal(st.rect, _oracle_rects(recs, cams, n, tw, th, super_tile, sups, vals))
    else:
        for (lo, hi), (a, b) in zip(ranges, granges):
            o, g = vals[lo:hi], ents[a:b].astype(np.int64)
            assert np.array_equal(o[np.isin(o, g)], g)   # ordered subsequence
    return st, recs


@pytest.mark.parametrize("alpha_min", [0.0, 1.0 / 255.0])
@pytest.mark.parametrize("n", [1, 767, 768, 769, 1537])
def test_pairs_of_large_rectangles(n, alpha_min):
    """8x8 tiles as super-tiles: up to 88 candidates an entry."""
    require_gpu()
    cams = _views()
    st, recs = _check(cams, n, (8, 8), 1, 60, alpha_min, 500 + n)
    _check_tile_lists(st, recs, cams, n, 8, 8, alpha_min)


@pytest.mark.parametrize("w,supers", [(32 * 16, 512), (32 * 16 + 1, 528)])
def test_super_tile_bound(w, supers):
    """512 super-tiles are placed directly, more are sorted: the same lists."""
    require_gpu()
    cams = [S.look_at_camera((3.0, 1.0, 1.0), w, 256)]
    for alpha_min in (0.0, 1.0 / 255.0):
        st, _ = _check(cams, 3000, (16, 16), 1, 24, alpha_min, 600)
        assert st.L.total_supers == supers


def test_pair_overflow_reports_the_need():
    require_gpu()
    m = sg()
    cams = _views()
    n = 2000
    recs, cat = _records(n, cams, 700, max_radius=40)
    rp = m.RasterParams(tile_w=8, tile_h=8, super_tile=2, split_prefix=0, alpha_min=0.0)
    need = Stage(n, cams, rp, cat, 1_000_000).needed
    st = Stage(n, cams, rp, cat, need - 1)
    assert st.flags & m.STATUS_PAIR_OVERFLOW and st.needed == need
    _, _, ranges = st.lists()
    assert ranges.max() == need - 1
