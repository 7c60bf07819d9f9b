"""The waves that share a tile, and the tuner timing what launches the same once."""
import json

import pytest

from paper_2603_08997_amd import scenes as S
from paper_2603_08997_amd import skipgs as sk
from paper_2603_08997_amd import tune as T


def _cams(*sizes):
    return [S.look_at_camera((3.0, 0.5, 1.0), w, h) for w, h in sizes]


@pytest.mark.parametrize("tile,sizes,want", [
    ((16, 16), [(64, 64)], (4, 4)),
    ((16, 16), [(16 * 48, 16 * 32)], (4, 4)),              # 1536 tiles
    ((16, 16), [(16 * 48 + 1, 16 * 32)], (4, 2)),
    ((32, 8), [(32 * 64, 8 * 80)], (4, 2)),                # 5120
    ((32, 8), [(32 * 64, 8 * 79), (64, 16)], (4, 2)),      # 5060
    ((16, 16), [(1600, 1060)], (2, 1)),                    # 6700
    ((8, 8), [(64, 64)], (1, 1)),
    ((8, 8), [(1600, 1060)], (1, 1)),
])
def test_waves_by_tile_shape_and_number(tile, sizes, want):
    rp = sk.RasterParams(tile_w=tile[0], tile_h=tile[1])
    assert sk.tile_waves(rp, _cams(*sizes)) == want


def test_waves_reject_bad_arguments():
    with pytest.raises(sk.SkipGSError):
        sk.tile_waves(sk.RasterParams(tile_w=24, tile_h=16), _cams((64, 64)))
    with pytest.raises(sk.SkipGSError):
        sk.tile_waves(sk.RasterParams(), [])


@pytest.mark.parametrize("size,programs", [((320, 240), 8 + 2 + 2), ((1600, 1060), 8 + 8 + 8)])
def test_programs_that_launch_the_same_are_timed_once(monkeypatch, tmp_path, size, programs):
    timed = []

    def candidate(planes, n, sh_degree, cams, dl, rp, reps=3):
        timed.append((rp.tile_w, rp.lds_batch, rp.super_tile))
        return 1.0 + 0.001 * len(timed) - (0.5 if (rp.tile_w, rp.super_tile) == (16, 8) else 0.0)

    monkeypatch.setattr(T, "time_candidate", candidate)
    monkeypatch.setattr(T, "workload_key", lambda *a: "w")
    monkeypatch.setattr(T.torch.cuda, "empty_cache", lambda: None)
    rp, rec = T.tune(None, 1000, 0, _cams(size), None, store=str(tmp_path / "t.json"))
    assert len(timed) == programs and len(rec["trials"]) == 24
    # of candidates that launch the same, the one with the default batch
    assert (rp.tile_w, rp.tile_h, rp.super_tile, rp.lds_batch) == (16, 16, 8, 64)
    assert json.load(open(tmp_path / "t.json"))["w"]["choice"]["lds_batch"] == 64
    again, rec2 = T.tune(None, 1000, 0, _cams(size), None, store=str(tmp_path / "t.json"))
    assert again == rp and rec2["reused"] and len(timed) == programs
