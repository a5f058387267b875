"""Backwards in compact workspaces (the pairs in passes): images and gradients
bitwise those of a full workspace, also when one forward is followed by backwards
of both forms."""
import numpy as np
import pytest
import torch

from paper_2510_06644_amd import rtgs, synth
from tests.gpu_util import eye_view, rcam, say

pytestmark = pytest.mark.gpu


def _item(w, h, n, j, seed):
    cam = synth.make_camera(w, h)
    rng = np.random.default_rng(seed)
    z = rng.uniform(1.5, 6.0, n)
    means = np.stack([(rng.uniform(0, w, n) - cam.cx) / cam.fx * z,
                      (rng.uniform(0, h, n) - cam.cy) / cam.fy * z, z], 1)
    px = np.exp(rng.uniform(np.log(0.4), np.log(60.0), (n, 3)))
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    it = dict(scene=(d(means), d(np.log(px * z[:, None] / cam.fx)), d(rng.normal(size=(n, 4))),
                     d(rng.uniform(-2, 2, n)), d(rng.uniform(0, 1, (n, 3)))),
              viewmat=d(eye_view()), cam=rcam(cam), sample_log2=j,
              dL_dcolor=d(rng.normal(size=(3, h, w))), dL_ddepth=d(rng.normal(size=(h, w))))
    if seed % 2:
        it["dL_dalpha"] = d(rng.normal(size=(h, w)))
    if j:
        it["pixel_mask"] = torch.empty(h, w, dtype=torch.uint8, device="cuda")
        rtgs.downsample_mask(d(rng.uniform(size=(h, w))), j, it["pixel_mask"])
    return it


def _outputs(it, map_grads):
    w, h, n = it["cam"].width, it["cam"].height, it["scene"][0].shape[0]
    e = lambda *s: torch.full(s, 7.0, device="cuda")
    out = dict(color=e(3, h, w), depth=e(h, w), alpha=e(h, w), final_T=e(h, w),
               last_idx=torch.empty(h, w, dtype=torch.int32, device="cuda"), g_pose6=e(6),
               g_viewmat=e(12))
    if map_grads:
        out.update(g_means=e(n, 3), g_log_scales=e(n, 3), g_quats=e(n, 4), g_opacity_logits=e(n),
                   g_colors=e(n, 3))
    return out


# one session, several with a downsampled one, few and many tiles; the capacities
# put the passes' ends into the pairs (also inside a merge window), after them, and
# at them
@pytest.mark.parametrize("frames", [[(97, 71, 900, 0)], [(640, 521, 900, 0)], [(640, 521, 900, 2)],
                                    [(97, 71, 900, 0), (320, 240, 700, 2), (131, 67, 1, 0)]])
@pytest.mark.parametrize("slack", [0, 1000, 1_000_000])
@pytest.mark.parametrize("map_grads", [False, True])
@pytest.mark.parametrize("balance", [False, True])
def test_backward_in_passes(frames, slack, map_grads, balance):
    say(f"test_backward_in_passes {frames} slack={slack} map={map_grads} balance={balance}")
    items = [_item(w, h, n, j, 5 + k) for k, (w, h, n, j) in enumerate(frames)]
    sizes = [f[2] for f in frames], [f[0] for f in frames], [f[1] for f in frames]
    handle = rtgs.Handle(0)
    fwd = rtgs.RTGS_FWD_SAVE_STATE | (rtgs.RTGS_FWD_BALANCE_LANES if balance else 0)
    bwd = (rtgs.RTGS_GRAD_POSE | (rtgs.RTGS_GRAD_MAP if map_grads else 0)
           | (rtgs.RTGS_GRAD_BALANCED_LANES if balance else 0))

    def run(buf, cap, ss):
        rtgs.render_bwd_batched(handle, ss, buf, cap, bwd)

    def forward(buf, cap):
        ss = [dict(it, **_outputs(it, map_grads)) for it in items]
        rtgs.render_fwd_batched(handle, ss, buf, cap, fwd)
        return ss

    big = torch.empty(rtgs.rtgs_workspace_size_batched(*sizes, 400_000), dtype=torch.uint8,
                      device="cuda")
    forward(big, 400_000)
    code, pairs, _ = rtgs.rtgs_query(handle)
    assert code == rtgs.RTGS_OK and pairs > 4000
    cap = pairs + slack
    size = lambda flag: rtgs.rtgs_workspace_size_batched(*sizes, cap, flag)
    bufs = [torch.empty(size(f), dtype=torch.uint8, device="cuda")
            for f in (0, rtgs.RTGS_FWD_COMPACT_SUMS)]
    assert bufs[1].numel() < bufs[0].numel()
    full, part = forward(bufs[0], cap), forward(bufs[1], cap)
    run(bufs[0], cap, full)
    run(bufs[1], cap, part)
    assert rtgs.rtgs_query(handle)[0] == rtgs.RTGS_OK
    for a, b in zip(full, part):
        for k in _outputs(a, map_grads):
            assert torch.equal(a[k], b[k]), k
    # again on the same forwards, the full workspace seen as a compact one first
    for buf in (bufs[0][:bufs[1].numel()], bufs[0], bufs[1]):
        again = [dict(it, **{k: v for k, v in _outputs(it, map_grads).items()
                             if k.startswith("g_")},
                      final_T=a["final_T"], last_idx=a["last_idx"]) for it, a in zip(items, full)]
        run(buf, cap, again)
        for a, b in zip(full, again):
            for k in b:
                if k.startswith("g_"):
                    assert torch.equal(a[k], b[k]), k


def test_renderer_over_its_share_takes_compact_workspaces():
    say("test_renderer_over_its_share")
    it = _item(320, 240, 700, 0, 3)
    grads = []
    for share in (1 << 40, 0):
        r = rtgs.Renderer(0, check="every")
        r._room.limit = share
        st = r.forward(it["scene"], it["viewmat"], it["cam"])
        flag = 0 if share else rtgs.RTGS_FWD_COMPACT_SUMS
        assert st.ws.numel() == rtgs.rtgs_workspace_size(700, 320, 240, st.cap, flag)
        st.stage()
        grads.append(r.backward(it["scene"], it["viewmat"], it["cam"], st, it["dL_dcolor"],
                                it["dL_ddepth"], it["dL_dalpha"]))
    for k, a in grads[0].items():
        assert torch.equal(a, grads[1][k]), k
