"""What a workspace held before a forward is of no account: images and gradients are
bitwise the same in memory of zeros and of ones, with short lists, lists of more
than 2048 entries, tiles without a list, and a forward without a backward between."""
import numpy as np
import pytest
import torch

from paper_2510_06644_amd import rtgs, synth
from tests.gpu_util import dev_scene, eye_view, rcam, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,n", [(64, 48, 3000), (333, 97, 700), (1200, 680, 2000)])
@pytest.mark.parametrize("compact", [False, True])
def test_contents_do_not_matter(w, h, n, compact):
    say(f"test_workspace_contents {w}x{h} n={n} compact={compact}")
    cam = synth.make_camera(w, h)
    sc = synth.make_scene(synth.SceneSpec("s", w, h, n, 7, log_scale_mean=-2.5), cam)
    scene, view, rc = dev_scene(sc), torch.from_numpy(eye_view()).cuda(), rcam(cam)
    rng = np.random.default_rng(2)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    up = d(rng.normal(size=(3, h, w))), d(rng.normal(size=(h, w)))
    handle, cap = rtgs.Handle(0), 600_000
    size = rtgs.rtgs_workspace_size(n, w, h, cap, rtgs.RTGS_FWD_COMPACT_SUMS if compact else 0)
    got = []
    for fill in (0, 255):
        ws = torch.full((size,), fill, dtype=torch.uint8, device="cuda")
        e = lambda *s: torch.full(s, 7.0, device="cuda")
        for _ in range(2):
            out = [e(3, h, w), e(h, w), e(h, w), e(h, w),
                   torch.zeros(h, w, dtype=torch.int32, device="cuda")]
            rtgs.render_fwd(handle, *scene, view, rc, ws, cap, *out)
        g = [e(n, 3), e(n, 3), e(n, 4), e(n), e(n, 3), e(6)]
        rtgs.render_bwd(handle, *scene, view, rc, ws, cap, out[3], out[4], *up, None,
                        rtgs.RTGS_GRAD_POSE | rtgs.RTGS_GRAD_MAP, *g)
        code, pairs, _ = rtgs.rtgs_query(handle)
        assert code == rtgs.RTGS_OK and pairs > 0
        got.append(out + g)
    for k, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a, b), k
