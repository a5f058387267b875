"""Batches whose tiles or binning chunks are scanned through global memory (more
than 12288 tiles, or more than 4096 chunks of 1024 Gaussians): tile ranges, ids,
images and gradients bit for bit those of single-session calls, or of the same
frame without the Gaussians that lie behind the camera."""
import numpy as np
import pytest
import torch

from paper_2510_06644_amd import rtgs, synth
from tests.gpu_util import eye_view, rcam, say

pytestmark = pytest.mark.gpu
GRADS = dict(g_means=3, g_log_scales=3, g_quats=4, g_opacity_logits=0, g_colors=3)


def _scene(w, h, n, seed, px_hi):
    cam = synth.make_camera(w, h)
    rng = np.random.default_rng(seed)
    z = rng.uniform(1.5, 6.0, n)
    means = np.stack([(rng.uniform(0, w, n) - cam.cx) / cam.fx * z,
                      (rng.uniform(0, h, n) - cam.cy) / cam.fy * z, z], 1)
    px = np.exp(rng.uniform(np.log(0.5), np.log(px_hi), (n, 3)))
    return cam, [np.ascontiguousarray(a, np.float32) for a in
                 (means, np.log(px * z[:, None] / cam.fx), rng.normal(size=(n, 4)),
                  rng.uniform(-2, 2, n), rng.uniform(0, 1, (n, 3)))]


def _item(cam, arrays, seed):
    w, h, n = cam.width, cam.height, len(arrays[0])
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    rng = np.random.default_rng(seed)
    e = lambda *s: torch.full(s, 7.0, device="cuda")
    it = dict(scene=tuple(d(a) for a in arrays), viewmat=d(eye_view()), cam=rcam(cam),
              color=e(3, h, w), depth=e(h, w), alpha=e(h, w), final_T=e(h, w),
              last_idx=torch.empty(h, w, dtype=torch.int32, device="cuda"),
              dL_dcolor=d(rng.normal(size=(3, h, w))), dL_ddepth=d(rng.normal(size=(h, w))),
              g_pose6=e(6), g_viewmat=e(12))
    it.update({k: e(n, c) if c else e(n) for k, c in GRADS.items()})
    return it


def _run(handle, items, cap):
    """Renders, differentiates; (ranges, ids) of the batch."""
    ns = [len(i["scene"][0]) for i in items]
    ws_, hs = [i["cam"].width for i in items], [i["cam"].height for i in items]
    ws = torch.empty(rtgs.rtgs_workspace_size_batched(ns, ws_, hs, cap), dtype=torch.uint8,
                     device="cuda")
    rtgs.render_fwd_batched(handle, items, ws, cap)
    tiles = sum(-(-w // 16) * -(-h // 16) for w, h in zip(ws_, hs))
    ranges = torch.empty(tiles, 2, dtype=torch.int32, device="cuda")
    ids = torch.empty(cap, dtype=torch.int32, device="cuda")
    rtgs.rtgs_debug_stage(ns, ws_, hs, cap, ws, ranges=ranges, ids=ids)
    rtgs.render_bwd_batched(handle, items, ws, cap)
    code, pairs, _ = rtgs.rtgs_query(handle)
    assert code == rtgs.RTGS_OK
    return ranges.cpu().numpy(), ids.cpu().numpy()[:pairs]


def test_many_tiles():
    say("test_many_tiles")
    handle = rtgs.Handle(0)
    frames = [_scene(1200, 680, 3000, 1, 40.0), _scene(1200, 680, 1500, 2, 5.0),
              _scene(1200, 680, 2047, 3, 120.0), _scene(1200, 680, 1, 4, 9.0),
              _scene(333, 97, 900, 5, 20.0)]
    mk = lambda: [_item(c, a, 10 + k) for k, (c, a) in enumerate(frames)]
    batch, single = mk(), mk()
    ranges, ids = _run(handle, batch, 1_500_000)
    assert len(ranges) > 12288
    t0 = p0 = g0 = 0
    for a, b in zip(batch, single):
        r1, i1 = _run(handle, [b], 1_500_000)
        assert len(i1) > 0
        assert np.array_equal(ranges[t0:t0 + len(r1)] - p0, r1)
        assert np.array_equal(ids[p0:p0 + len(i1)] - g0, i1)
        t0, p0, g0 = t0 + len(r1), p0 + len(i1), g0 + len(a["scene"][0])
        for k in ("color", "depth", "alpha", "final_T", "g_pose6", "g_viewmat", *GRADS):
            assert torch.equal(a[k], b[k]), k
    assert (t0, p0) == (len(ranges), len(ids))


def test_many_chunks():
    say("test_many_chunks")
    handle = rtgs.Handle(0)
    cam, few = _scene(160, 96, 90, 6, 6.0)
    n = 4097 * 1024 + 5
    at = np.sort(np.random.default_rng(7).choice(n, 90, replace=False))
    many = [np.zeros((n,) + a.shape[1:], np.float32) for a in few]
    many[0][:, 2] = -1.0                           # behind the camera
    many[2][:, 0] = 1.0
    for m, a in zip(many, few):
        m[at] = a
    a, b = _item(cam, many, 8), _item(cam, few, 8)
    ranges, ids = _run(handle, [a], 50_000)
    r1, i1 = _run(handle, [b], 50_000)
    assert np.array_equal(ranges, r1) and np.array_equal(ids, at[i1])
    for k in ("color", "depth", "alpha", "final_T"):
        assert torch.equal(a[k], b[k]), k
    rows = torch.from_numpy(at).cuda()
    for k in GRADS:
        assert torch.equal(a[k][rows], b[k]), k
        a[k][rows] = 0
        assert not bool(a[k].any()), k
