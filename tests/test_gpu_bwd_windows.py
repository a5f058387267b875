"""The backward's per-quadrant sums and their merge by windows of 512 pairs: gradients against
the float64 oracle where windows, binning chunks and groups of eight entries begin and end.

Small Gaussians of one tile each (so Gaussian i is pair i) put the ends of windows and chunks
(1024 Gaussians) at chosen Gaussians; one that covers every tile straddles a window's end.  The
frame is ragged, so edge quadrants are partly or wholly outside it."""
import numpy as np
import pytest
import torch

from paper_2510_06644_amd import rtgs, synth
from tests.gpu_util import dev_scene, eye_view, full_frame_parity, rcam

pytestmark = pytest.mark.gpu

CAM = synth.make_camera(90, 74)            # 6 x 5 tiles, the last ones ragged


def _scene(n, big, seed):
    """n Gaussians inside one tile each; those of `big` cover the frame."""
    rng = np.random.default_rng(seed)
    z = rng.uniform(1.0, 3.0, n)
    tile = np.arange(n) % 20               # 5 x 4 whole tiles
    u = (tile % 5) * 16 + 8 + rng.uniform(-2, 2, n)
    v = (tile // 5) * 16 + 8 + rng.uniform(-2, 2, n)
    # three different axes: an isotropic Gaussian has no gradient to its rotation
    ls = np.log(np.array([0.2, 0.5, 0.9]) / CAM.fx) + np.log(z)[:, None]
    eta = rng.uniform(-3.5, -1.0, n)
    for b in big:
        u[b], v[b] = 45.0, 37.0
        ls[b] = np.log(np.array([25.0, 30.0, 40.0]) / CAM.fx * z[b])
    means = np.stack([(u - CAM.cx) * z / CAM.fx, (v - CAM.cy) * z / CAM.fy, z], 1)
    q = rng.normal(size=(n, 4))
    return synth.Scene(*(np.ascontiguousarray(a, np.float32) for a in
                         (means, ls, q, eta, rng.random((n, 3)))))


@pytest.mark.parametrize("n,big", [(1, ()), (7, (3,)), (9, ()), (511, ()), (512, ()), (513, (0,)),
                                   (700, (500,)), (1024, (1023,)), (1025, (1024,)),
                                   (1100, (490, 498, 505))])
def test_window_ends(n, big):
    full_frame_parity(rtgs.Renderer(0), _scene(n, big, n), CAM, eye_view(), seed=n,
                      label=f"n={n}")


def test_backward_twice_and_reused_lists_start_from_clean_flags():
    """The merge leaves the flags clean: a second backward of the same forward, one of another
    gradient set, and a backward on reused lists after it give what fresh ones give, bit for
    bit."""
    sc, cam = _scene(900, (100, 600), 3), rcam(CAM)
    d, view = dev_scene(sc), torch.from_numpy(eye_view()).cuda()
    gc, gd, _ = (torch.from_numpy(a).cuda() for a in synth.upstream_grads(CAM.width, CAM.height, 5))
    R = rtgs.Renderer(0)

    def grads(st, **kw):
        return {k: v.clone() for k, v in R.backward(d, view, cam, st, gc, gd, **kw).items()}

    fresh = grads(R.forward(d, view, cam))
    fresh_pose = grads(R.forward(d, view, cam), map_grads=False)
    st = R.forward(d, view, cam)
    grads(st, map_grads=False)
    second = grads(st)
    third = grads(st, map_grads=False)
    mask = torch.zeros(900, dtype=torch.uint8, device="cuda")
    mask[::3] = 1
    again = R.forward(d, view, cam, gauss_mask=mask, reuse_lists_of=st)
    masked = {k: v.clone() for k, v in R.backward(d, view, cam, again, gc, gd,
                                                  gauss_mask=mask).items()}
    base = R.forward(d, view, cam)
    alone = R.forward(d, view, cam, gauss_mask=mask, reuse_lists_of=base)
    masked_alone = R.backward(d, view, cam, alone, gc, gd, gauss_mask=mask)
    for a, b in ((fresh, second), (fresh_pose, third), (masked_alone, masked)):
        for k in a:
            assert torch.equal(a[k], b[k]), k
    assert bool((masked["means"][::3] == 0).all()) and bool((masked["means"] != 0).any())
