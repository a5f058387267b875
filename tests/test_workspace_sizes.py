"""Workspace sizes on the CPU: a compact workspace takes no more than one slot
of sums, key, id and mask byte per pair (61 bytes a pair: the bounds are the
recorded bytes of such a layout), a renderer's states over its share of the card
are compact, and a serving step admits the frames that 61 bytes a pair admit."""
import pytest

from paper_2510_06644_amd import rtgs, serving
from paper_2510_06644_amd.serving import GpuExecutor, ServeConfig, SessionSpec

COMPACT = rtgs.RTGS_FWD_COMPACT_SUMS
BOUNDS = [(128, 128, 2_000, 24_256, 1_929_984), (320, 240, 20_000, 241_200, 18_133_760),
          (640, 480, 100_000, 2_409_600, 163_594_496),
          (1200, 680, 300_000, 3_612_900, 271_550_208),
          (1200, 680, 500_000, 12_025_800, 813_767_424),
          (1200, 680, 1_500_000, 36_025_800, 2_422_865_408)]


@pytest.mark.parametrize("w,h,n,cap,bound", BOUNDS)
def test_compact_workspace_is_within_the_bound(w, h, n, cap, bound):
    full = rtgs.rtgs_workspace_size(n, w, h, cap)
    assert rtgs.rtgs_workspace_size(n, w, h, cap, COMPACT) <= bound < full
    assert rtgs.rtgs_workspace_size_batched([n, n], [w, w], [h, h], 2 * cap, COMPACT) <= 2 * bound


@pytest.mark.parametrize("cap", [0, 1, 511, 512, 682, 683, 2_000, (1 << 31) - 1])
def test_compact_is_never_larger(cap):
    full = rtgs.rtgs_workspace_size(1000, 64, 48, cap)
    assert rtgs.rtgs_workspace_size(1000, 64, 48, cap, COMPACT) <= full
    # saved fragments come with the full form
    frag = rtgs.RTGS_FWD_SAVE_FRAGMENTS
    assert (rtgs.rtgs_workspace_size(1000, 64, 48, cap, frag | COMPACT)
            == rtgs.rtgs_workspace_size(1000, 64, 48, cap, frag))


def test_states_over_the_share_are_compact_and_freed_ones_count_no_more():
    room = rtgs._Room(250)
    mk = lambda: room.workspace(lambda flag: 40 if flag & COMPACT else 100, "cpu")
    a, b, c = mk(), mk(), mk()
    assert [t.numel() for t in (a, b, c)] == [100, 100, 40]
    del a
    d, e = mk(), mk()
    assert [t.numel() for t in (d, e)] == [100, 40]
    del b, c, d, e
    assert [t.numel() for t in [mk() for _ in range(3)]] == [100, 100, 40]


def _executor(budget):
    ex = object.__new__(GpuExecutor)        # sizes only: no GPU needed
    ex.rtgs, ex.capacity_factor, ex.ws_budget = rtgs, 2.0, budget
    return ex


@pytest.mark.parametrize("spec,full", [(SessionSpec(1200, 680, 1_500_000), False),
                                       (serving.serving_mix()[-1], True)])
def test_a_step_of_sixteen_large_frames(spec, full):
    cfg = ServeConfig()
    ex = _executor(cfg.ws_budget)
    assert 16 * ex.step_bytes(spec, None) <= cfg.ws_budget
    args = [spec.n] * 16, [spec.width] * 16, [spec.height] * 16, 16 * ex._cap(spec)
    got = ex._workspace_bytes(*args)
    assert got <= cfg.ws_budget
    assert got == rtgs.rtgs_workspace_size_batched(*args, 0 if full else COMPACT)


def test_bytes_of_a_gaussian():
    # record 64, rectangle 16, count, first slot and key 12, merged gradient 40, list entry
    # 8, and two bytes for what a chunk of 1024 adds
    a, b = (rtgs.rtgs_workspace_size(n, 16, 16, 0) for n in (1 << 20, 1 << 21))
    assert (b - a) / (1 << 20) <= 64 + 16 + 12 + 40 + 8 + 2
