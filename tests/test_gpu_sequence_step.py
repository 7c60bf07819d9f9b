"""The training step in one call: the view of the sequence picked by the
projection, the loss summed and the compositing backward prepared within the
loss backward. Against the view picked by its own call and the iteration stage
by stage: views, losses, gates and step counts equal, images bit for bit,
parameters up to the order of the compositing backward's atomic additions."""
import pytest
import torch

from paper_2603_08997_amd import scenes as S
from paper_2603_08997_amd import train as T
from tests.gpu_util import require_gpu, say, sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("start", [0, 2, (1 << 32) - 2])
@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("n,w,h", [(1, 64, 64), (700, 33, 18), (9000, 640, 416)])
def test_one_call_equals_the_stages(n, w, h, gated, start):
    require_gpu()
    m = sg()
    cams = [S.look_at_camera((3.0, 0.2 * k, 1.0), w, h) for k in range(3)]
    rp, cap = m.RasterParams(), 1 << 20
    targets = T.render_targets(S.tiny_scene(1, n), cams, rp, cap)
    seq = [2, 0, 1, 2, 2]
    # a gate that skips every view from its second visit on
    gate = m.GateParams(n_views=3, warmup=0, calibrate=False, budget=False, delta=10.0) if gated else None
    init = S.tiny_scene(3, n)
    one, stages = (T.Trainer(init, cams, targets, rp, gate, cap, gated=gated, sequence=seq)
                   for _ in range(2))
    one.seq_pos.fill_(start)
    slot = torch.zeros(1, dtype=torch.int32, device="cuda")
    counts = []
    for k in range(5):
        one.step()
        v = seq[(start + k) % 5]
        stages.view.fill_(v)
        stages.iteration(v, stages.view, slot)
        assert one.view.item() == v and one.seq_pos.item() == start + k + 1
        assert one.gate.item() == slot.item()
        counts.append(one.step_count.item())
        assert counts[-1] == stages.step_count.item()
        if k == 0:   # the same parameters so far
            assert torch.equal(one.rgb, stages.rgb) and torch.equal(one.loss, stages.loss)
        # at most one learning rate apart where a gradient's sign is that of its rounding
        assert (one.rgb - stages.rgb).abs().max().item() < 1e-2
    say(f"sequence step n={n} {w}x{h} gated={gated}: counts {counts}")
    assert counts[-1] == (3 if gated else 5)
    for a, b in ((one.m, stages.m), (one.v, stages.v)):
        scale = b.abs().amax(1, keepdim=True).clamp_min(1e-30)
        assert ((a - b).abs() / scale).max().item() < 1e-3
