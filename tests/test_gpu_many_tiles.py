"""Life on a fractal with more tiles than one launch of a workgroup per tile can
hold (2^26 tiles of 64 lanes are 2^32 lanes): s = 3 with 4 replicas at level 17,
17,179,869,184 cells in tiles of level 4.  Steps and runs equal the thread-level
kernel."""
import pytest

from gpu_common import torch_or_skip

pytestmark = pytest.mark.gpu


def test_more_tiles_than_a_launch_holds():
    torch = torch_or_skip()
    import paper_2201_00613_amd as sqz

    F = sqz.Fractal(3, [(0, 0), (1, 0), (1, 1), (2, 2)], 17)
    assert F.xtile_level == 4 and F.cells // 4 ** F.xtile_level == 1 << 26
    a = F.fill_bernoulli(5, 0.4)
    b, want = torch.empty_like(a), torch.empty_like(a)
    F.compact_step(a, want, impl="cell")
    F.compact_step(a, b)
    assert torch.equal(b, want)
    F.compact_step(want, b, impl="cell")
    res = F.compact_run(a, want, 2)
    assert res is a and torch.equal(a, b)
    del a, b, want, res
    torch.cuda.empty_cache()
