"""The differentiable render frees its workspace with its outputs (no reference
cycle): device memory does not grow from call to call with the garbage
collector off, whether the backward ran or not."""
import gc

import pytest
import torch

from paper_2510_06644_amd import autograd, rtgs
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("state", ["save", "recompute", "fragments"])
@pytest.mark.parametrize("backward", [False, True])
def test_workspace_is_freed_with_the_outputs(state, backward):
    say(f"test_workspace_is_freed {state} {backward}")
    g = torch.Generator(device="cuda").manual_seed(3)
    n = 500
    f = lambda *s: torch.rand(*s, generator=g, device="cuda")
    leaves = [t.requires_grad_(True) for t in (
        torch.cat([f(n, 2) * 2 - 1, f(n, 1) + 1.5], 1), f(n, 3) - 4, f(n, 4) + 0.1, f(n), f(n, 3))]
    vm = torch.eye(4, device="cuda")[:3].clone().requires_grad_(True)
    cam = rtgs.Cam(64, 48, 60.0, 60.0, 32.0, 24.0)
    r = rtgs.Renderer(0, check="every")

    def call():
        for t in leaves + [vm]:
            t.grad = None
        c, d, a, _ = autograd.render(*leaves, vm, cam, renderer=r, state=state)
        if backward:
            (c.sum() + d.sum() + a.sum()).backward()

    gc.collect()
    gc.disable()
    try:
        call()
        call()
        before = torch.cuda.memory_allocated()
        for _ in range(5):
            call()
        assert torch.cuda.memory_allocated() == before
    finally:
        gc.enable()
