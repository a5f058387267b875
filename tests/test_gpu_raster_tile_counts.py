"""The raster backward's builds by the number of tiles (up to 1024, and more): a
downsampled frame of more than 1024 coarse tiles against the same mask on the pixel
grid (up to the order of summation, GRAD_TOL), and batches on either side against
single-session calls, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2510_06644_amd import rtgs, synth
from tests.gpu_util import GRAD_TOL, eye_view, norm_err, rcam, say

pytestmark = pytest.mark.gpu
MAP = dict(g_means=3, g_log_scales=3, g_quats=4, g_opacity_logits=0, g_colors=3)


def _item(w, h, n, j, seed, map_grads):
    cam = synth.make_camera(w, h)
    rng = np.random.default_rng(seed)
    z = rng.uniform(1.5, 6.0, n)
    means = np.stack([(rng.uniform(0, w, n) - cam.cx) / cam.fx * z,
                      (rng.uniform(0, h, n) - cam.cy) / cam.fy * z, z], 1)
    px = np.exp(rng.uniform(np.log(0.4), np.log(25.0), (n, 3)))
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    e = lambda *s: torch.full(s, 7.0, device="cuda")
    it = dict(scene=(d(means), d(np.log(px * z[:, None] / cam.fx)), d(rng.normal(size=(n, 4))),
                     d(rng.uniform(-2, 2, n)), d(rng.uniform(0, 1, (n, 3)))),
              viewmat=d(eye_view()), cam=rcam(cam), sample_log2=j, color=e(3, h, w),
              depth=e(h, w), alpha=e(h, w), final_T=e(h, w),
              last_idx=torch.empty(h, w, dtype=torch.int32, device="cuda"),
              dL_dcolor=d(rng.normal(size=(3, h, w))), dL_ddepth=d(rng.normal(size=(h, w))),
              g_pose6=e(6), g_viewmat=e(12))
    if map_grads:
        it.update({k: e(n, c) if c else e(n) for k, c in MAP.items()})
    if j:
        it["pixel_mask"] = torch.empty(h, w, dtype=torch.uint8, device="cuda")
        rtgs.downsample_mask(d(rng.uniform(size=(h, w))), j, it["pixel_mask"])
    return it


def _run(handle, items, map_grads, cap=500_000):
    ws = torch.empty(rtgs.rtgs_workspace_size_batched(
        [len(i["scene"][0]) for i in items], [i["cam"].width for i in items],
        [i["cam"].height for i in items], cap), dtype=torch.uint8, device="cuda")
    rtgs.render_fwd_batched(handle, items, ws, cap)
    rtgs.render_bwd_batched(handle, items, ws, cap,
                            rtgs.RTGS_GRAD_POSE | (rtgs.RTGS_GRAD_MAP if map_grads else 0))
    assert rtgs.rtgs_query(handle)[0] == rtgs.RTGS_OK


@pytest.mark.parametrize("map_grads", [False, True])
def test_downsampled_frame_of_many_tiles(map_grads):
    say(f"test_downsampled_frame_of_many_tiles map={map_grads}")
    handle = rtgs.Handle(0)
    a, b = (_item(1200, 680, 6000, 1, 3, map_grads) for _ in range(2))
    b["sample_log2"] = 0
    for it in (a, b):
        _run(handle, [it], map_grads)
    for k in ("color", "depth", "alpha", "final_T"):
        assert torch.equal(a[k], b[k]), k
    for k in a:
        if k.startswith("g_"):
            e = norm_err(a[k].cpu().numpy(), b[k].cpu().numpy())
            say(f"  {k}: {e:.2e}")
            assert e < GRAD_TOL, k


@pytest.mark.parametrize("frames", [
    [(320, 240, 2000, 0), (320, 240, 1500, 0)], [(320, 240, 2000, 2), (97, 71, 300, 0)],
    [(640, 480, 3000, 0), (97, 71, 300, 0)], [(1200, 680, 3000, 1), (97, 71, 300, 3)]])
@pytest.mark.parametrize("map_grads", [False, True])
def test_batches_equal_single_sessions(frames, map_grads):
    say(f"test_batches_equal_single_sessions {frames} map={map_grads}")
    handle = rtgs.Handle(0)
    mk = lambda: [_item(*f, 20 + k, map_grads) for k, f in enumerate(frames)]
    batch, single = mk(), mk()
    _run(handle, batch, map_grads)
    for it in single:
        _run(handle, [it], map_grads)
    for a, b in zip(batch, single):
        for k in a:
            if k in ("color", "depth", "alpha", "final_T", "last_idx") or k.startswith("g_"):
                same = a[k] == b[k]
                if k == "last_idx":              # positions of the batch's lists
                    same = (a[k] >= 0) == (b[k] >= 0)
                assert bool(same.all()), k
