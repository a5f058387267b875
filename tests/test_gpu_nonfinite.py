"""A colour that is not finite on a Gaussian that no pixel blends: its footprint
(radius 0.38 px at the alpha floor, centred on a pixel corner) reaches a quadrant
but none of its pixel centres, so the gradients of the others are bitwise those
of the scene without it, and its own are zero."""
import numpy as np
import pytest
import torch

from paper_2510_06644_amd import rtgs, synth
from tests.gpu_util import eye_view, rcam, say

pytestmark = pytest.mark.gpu

MODES = {"plain": {}, "fragments": dict(save_fragments=True), "balanced": dict(balance=True)}


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("j", [0, 2, 4])
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("map_grads", [False, True])
def test_unblended_gaussian_with_nonfinite_colour(value, j, mode, map_grads):
    say(f"test_unblended_nonfinite value={value} j={j} {mode} map={map_grads}")
    cam = synth.Camera(32, 32, 32.0, 32.0, 16.0, 16.0)
    # (u, v, z, sigma in px, opacity): one in front, one behind, the unblended
    # one between them in depth and last in index
    rows = [(9.0, 7.5, 1.0, 4.0, 0.6), (7.0, 9.0, 2.0, 5.0, 0.7), (4.0, 4.0, 1.5, 1e-4, 0.005)]
    u, v, z, s, o = np.array(rows).T
    means = np.stack([(u - 16) / 32 * z, (v - 16) / 32 * z, z], 1)
    scales = np.log(s * z / 32)[:, None].repeat(3, 1) + np.array([0.0, 0.2, 0.4])
    quats = np.tile([1.0, 0.2, -0.1, 0.3], (3, 1))
    colors = np.array([[0.2, 0.5, 0.8], [0.7, 0.4, 0.1], [0.3, value, 0.6]])
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    scene = (d(means), d(scales), d(quats), d(np.log(o) - np.log1p(-o)), d(colors))
    view, rc = d(eye_view()), rcam(cam)
    rng = np.random.default_rng(3)
    up = [d(rng.normal(size=(3, 32, 32))), d(rng.normal(size=(32, 32))),
          d(rng.normal(size=(32, 32)))]
    r = rtgs.Renderer(0, check="every")
    kw = dict(sample_log2=j)
    pm = None
    if j:
        pm = torch.empty(32, 32, dtype=torch.uint8, device="cuda")
        rtgs.downsample_mask(d(rng.uniform(size=(32, 32))), j, pm)
        kw["pixel_mask"] = pm
    got = []
    for k in (2, 3):
        part = tuple(t[:k].contiguous() for t in scene)
        st = r.forward(part, view, rc, **MODES[mode], **kw)
        g = r.backward(part, view, rc, st, *up, pose=True, map_grads=map_grads, pixel_mask=pm)
        got.append((st, g))
    (a, ga), (b, gb) = got
    assert int(b.visible[2]) == 1
    assert torch.equal(a.final_T, b.final_T)
    for k in ga:
        if k in ("pose", "viewmat"):
            assert torch.equal(ga[k], gb[k]), k
        else:
            assert torch.equal(ga[k], gb[k][:2]), k
            assert not bool(gb[k][2].any()), k
