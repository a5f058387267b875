"""The workspace budget changes how steps run, not what they compute: with a budget
below any full workspace every step takes a compact one, and each frame's end
pose and every session's map are bitwise those served in full workspaces."""
import pytest
import torch

from paper_2510_06644_amd import serving
from paper_2510_06644_amd.serving import Engine, GpuExecutor, ServeConfig, SessionSpec
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("async_mapping", [False, True])
def test_served_results_do_not_depend_on_the_budget(async_mapping):
    say(f"test_served_results_do_not_depend_on_the_budget async_mapping={async_mapping}")
    specs = [SessionSpec(320, 240, 20_000, "c0", 70 + k) for k in range(2)]
    trace = serving.poisson_trace(len(specs), 60.0, 0.2, 23)
    out, sizes = [], []
    for budget in (40e9, 1.0):
        ex = GpuExecutor(0, n_targets=2, record_poses=True)
        cfg = ServeConfig(track_iters=4, map_iters=5, keyframe_every=4, downsample=True,
                          async_mapping=async_mapping, ws_budget=budget)
        eng = Engine(specs, ex, cfg)
        rep = eng.run(trace)
        ex.verify()
        assert ex.overflows == 0 and rep["frames"] == len(trace)
        sizes.append(ex._workspace_bytes([20_000], [320], [240], ex._cap(specs[0])))
        out.append(ex)
    assert sizes[1] < sizes[0]
    a, b = out
    assert a.frame_poses.keys() == b.frame_poses.keys() and len(a.frame_poses) == len(trace)
    for k in a.frame_poses:
        assert torch.equal(a.frame_poses[k], b.frame_poses[k]), k
    for s in range(len(specs)):
        for x, y in zip(a.sessions[s]["params"], b.sessions[s]["params"]):
            assert torch.equal(x, y)
