"""Runs on multi-step expanded tiles (buffers at odd addresses) equal thread-level
steps for step counts on both sides of every change of their launch plan."""
import pytest

from gpu_common import gpu_fractal, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,r", [("triangle", 9), ("carpet", 6), ("vicsek", 6)])
def test_unaligned_runs_equal_thread_level_steps(name, r):
    torch = torch_or_skip()
    F = gpu_fractal(name, r)
    start = F.fill_bernoulli(11, 0.45)
    buf = torch.empty(2 * F.cells + 64, dtype=torch.uint8, device="cuda")
    a, b = buf[1:1 + F.cells], buf[F.cells + 2:2 * F.cells + 2]
    x, y = start.clone(), torch.empty_like(start)
    for steps in range(1, 12):
        F.compact_step(x, y, impl="cell")
        x, y = y, x
        a.copy_(start)
        assert torch.equal(F.compact_run(a, b, steps), x), steps
