"""The depth sort of sets one workgroup holds and of those sorted in runs and
merged, at the edges of its launch rule (1024, 2048 and 65536 entries): every super-tile's list is in order of depth,
equal depths in entry order, the culled entries are left out, and the lists
equal those of the general sort, which the same records take as the first of
two views."""
import numpy as np
import pytest

from paper_2603_08997_amd import scenes as S
from tests.gpu_util import region, require_gpu, say, sg
from tests.test_gpu_stages import Stage, _records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", [True, False])
@pytest.mark.parametrize("n", [1, 63, 1023, 1024, 1025, 2048, 2049, 4097, 20000, 65535, 65536, 65537])
def test_lists_in_depth_order(n, ties):
    require_gpu()
    m = sg()
    cam = S.look_at_camera((3.0, 1.0, 1.0), 250, 139)
    recs, cat = _records(n, [cam], 77)
    rng = np.random.default_rng(n)
    if ties:   # and values that differ in one digit of the key only
        cat["depth"] = rng.choice(np.array([0.5, 1.0, 1.0000001, 2.0, 3.7, 300.0], np.float32), n)
    cat["extent"][rng.random(n) < 0.3] = -1   # culled
    rp = m.RasterParams(split_prefix=0, alpha_min=0.0)
    st = Stage(n, [cam], rp, cat, 2_000_000)
    keys, ents, ranges = st.lists()
    depth = region(st.ws, st.L.depth, n, np.uint32).astype(np.int64)
    tiles = region(st.ws, st.L.tiles, n, np.uint32)
    say(f"small sort n={n} visible {st.vis} pairs {st.kept}")
    assert st.flags == 0 and st.vis == int((tiles > 0).sum()) and st.needed == int(tiles.sum())
    for a, b in ranges:
        order = (depth[ents[a:b]] << 32) + ents[a:b].astype(np.int64)
        assert (np.diff(order) > 0).all()
    assert np.array_equal(np.bincount(ents, minlength=n), tiles)
    # the first of two views, the other one with enough entries for the general sort
    big = max(n, 32769)
    pad = {k: np.concatenate([v, np.repeat(v[-1:], big - n, 0)]) for k, v in cat.items()}
    pad["extent"][n:] = -1
    two = {k: np.concatenate([v, v]) for k, v in pad.items()}
    two["extent"][big:] = -1
    general = Stage(big, [cam, cam], rp, two, 2_000_000)
    gk, ge, gr = general.lists()
    assert general.vis == st.vis and np.array_equal(ge, ents)
    assert np.array_equal(gr[:len(ranges)], ranges)
