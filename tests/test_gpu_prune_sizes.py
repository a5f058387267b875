"""The pruning selection, the pair change and the compaction at sizes around a
wave, a workgroup, the histogram grid (256 x 1024), the change grid (128 x
1024) and the grid of the final passes (2048 x 1024), with scores whose
threshold is settled by each of the three radix passes.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

from oracle import binning, selection
from paper_2510_06644_amd import rtgs
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def _scores(kind, n, rng):
    """||dL/dmu|| of a vector along x: its length, exact in float32."""
    bits = {"spread": lambda: rng.integers(0, 0x7f800000, n),
            "middle": lambda: 0x3f800000 | rng.integers(0, 4, n) << 12 | rng.integers(0, 8, n) << 7,
            "low": lambda: 0x3f800000 | rng.integers(0, 1024, n),
            "equal": lambda: np.full(n, 0x3f812345),
            "zeros": lambda: np.where(rng.random(n) < 0.9, 0, rng.integers(0, 0x7f800000, n)),
            "infinite": lambda: np.where(rng.random(n) < 0.5, 0x7f800000, 0)}[kind]()
    return bits.astype(np.uint32).view(np.float32)


@pytest.mark.parametrize("n,kind", [
    (1, "equal"), (63, "low"), (65, "spread"), (1023, "middle"), (1025, "low"), (2048, "equal"),
    (131_073, "spread"), (262_145, "low"), (262_145, "infinite"), (300_001, "zeros"),
    (2_097_153, "middle"), (2_100_000, "equal")])
def test_selection_at_grid_edges(n, kind):
    say(f"test_selection n={n} {kind}")
    rng = np.random.default_rng(n)
    gm = np.zeros((n, 3), np.float32)
    gm[:, 0] = _scores(kind, n, rng)
    vis = (rng.random(n) < 0.9).astype(np.uint8)
    mask = (rng.random(n) < 0.05).astype(np.uint8)
    d = lambda a: torch.from_numpy(a).cuda()
    out = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
    count = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    h = rtgs.Handle(0)
    gm_d, gc_d, vis_d = d(gm), torch.zeros(n, 6, device="cuda"), d(vis)
    for ratio in (0.0, 0.1, 0.37, 0.5):
        rtgs.prune_by_grad(h, gm_d, gc_d, vis_d, d(mask), 0.8, ratio, out, count)
        want, k = selection.prune_select(gm[:, 0], vis.astype(bool), mask.astype(bool),
                                         float(np.float32(ratio)))
        assert int(count) == k
        assert np.array_equal(out.cpu().numpy().astype(bool), want)


@pytest.mark.parametrize("n", [1, 64, 1023, 1025, 131_073, 400_001])
def test_pair_change_at_grid_edges(n):
    say(f"test_pair_change n={n}")
    rng = np.random.default_rng(n)

    def rects():
        lo = rng.integers(0, 60, (n, 2))
        return np.concatenate([lo, lo + rng.integers(-1, 12, (n, 2))], 1).astype(np.int32)

    a, b, skip = rects(), rects(), (rng.random(n) < 0.3).astype(np.uint8)
    out = torch.full((2,), -5, dtype=torch.int64, device="cuda")
    for sk in (None, skip):
        rtgs.tile_pair_change(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(),
                              None if sk is None else torch.from_numpy(sk).cuda(), out)
        assert tuple(out.tolist()) == tuple(
            binning.pair_change(a, b, None if sk is None else sk.astype(bool)))


@pytest.mark.parametrize("n", [1, 1024, 1025, 1_048_577, 1_200_000])
def test_compaction_at_scan_edges(n):
    say(f"test_compaction n={n}")
    g = torch.Generator(device="cuda").manual_seed(n)
    src = torch.arange(n, dtype=torch.int32, device="cuda")
    drop = (torch.rand(n, generator=g, device="cuda") < 0.3).to(torch.uint8)
    dst = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    kept = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    rtgs.compact_by_mask(drop, [(src, dst)], kept)
    want = src[drop == 0]
    assert int(kept) == want.numel()
    assert torch.equal(dst[:want.numel()], want)
