"""The density step's write around its workgroups' sizes and with one outcome
for all inputs: the new set against the oracle's, copies and moments bit for
bit, children within FP32 rounding, nothing past the set touched."""
import numpy as np
import pytest

from oracle import densify as OD
from paper_2603_08997_amd import scenes as S
from tests.gpu_util import rel_max_err, require_gpu, say, sg
from tests.test_gpu_densify import _gpu_densify, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 257, 2049, 6200, 262145])
@pytest.mark.parametrize("outcome", ["mixed", "keep", "clone", "split", "prune"])
def test_write(n, outcome):
    require_gpu()
    deg = 1
    P, m, v, g, count, normals = _inputs(n, deg, 90 + n)
    if outcome != "mixed":
        P[10, :n] = -50.0 if outcome == "prune" else 1.0
        count[:] = 3
        g[:] = 0.0 if outcome == "keep" else 1.0
        P[3:6, :n] = 2.0 if outcome == "split" else -20.0
    args = dict(grad_threshold=2e-4, percent_dense=0.01, scene_extent=2.0, min_opacity=0.005)
    op, om, ov = OD.densify(P, m, v, g, count, normals, OD.DensifyParams(**args))
    keep, clone, split = OD.decisions(P, g, count, OD.DensifyParams(**args))
    K, Cn = int(keep.sum()), int(clone.sum())
    say(f"densify write n={n} {outcome}: keep {K} clone {Cn} split {int(split.sum())}")
    n_out, (gp, gm, gv) = _gpu_densify(sg().DensifyParams(**args), P, m, v, g, count, normals, n, deg,
                                       S.padded_stride(2 * n))
    assert n_out == op.shape[1]
    assert np.array_equal(gp[:, :K + Cn], op[:, :K + Cn].astype(np.float32))
    assert np.array_equal(gm[:, :n_out], om.astype(np.float32))
    assert np.array_equal(gv[:, :n_out], ov.astype(np.float32))
    if n_out > K + Cn:
        kids = slice(K + Cn, n_out)
        assert rel_max_err(gp[0:3, kids], op[0:3, kids]) < 1e-5
        assert np.abs(gp[3:6, kids] - op[3:6, kids]).max() < 2e-6
        assert np.array_equal(gp[6:, kids], op[6:, kids].astype(np.float32))
    for x in (gp, gm, gv):
        assert np.isnan(x[:, n_out:]).all()
