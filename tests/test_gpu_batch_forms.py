"""The launches over all tiled instances of a batch (persistent, and a workgroup
per tile) where more tiles than fit the chip at once share workgroups: numbers of
tiles that are no multiple of a workgroup's, fractals too small to tile, launches
of one and of several steps.  Every instance equals its own single-fractal run."""
import pytest

from gpu_common import torch_or_skip

pytestmark = pytest.mark.gpu

# 1, 3, 9 and 729 tiles of the triangles beside the other patterns: 2,600 in all
MANY = [("triangle", 14), ("triangle", 9), ("triangle_paper", 14), ("vicsek", 9), ("carpet", 6), ("triangle", 8),
        ("triangle", 4), ("vicsek", 2), ("triangle_paper", 10), ("vicsek", 3), ("triangle_paper", 14), ("triangle", 13)]


@pytest.mark.parametrize("form,steps_per_launch,wg", [("per_tile", 0, 0), ("per_tile", 3, 0), ("persistent", 0, 0),
                                                     ("persistent", 4, 1)])
def test_many_tiles_equal_single_runs(form, steps_per_launch, wg):
    torch = torch_or_skip()
    import fractals as FR
    import paper_2201_00613_amd as sqz

    fr = [sqz.Fractal(*FR.ALL[n], r) for n, r in MANY]
    B = sqz.Batch(fr)
    B.set_tiled_launch(form, steps_per_launch, wg)
    seeds = [90 + i for i in range(len(fr))]
    for steps in (1, 2, 7, 12):
        a = B.fill_bernoulli(seeds, 0.45)
        res = B.run(a, torch.full_like(a, 7), steps)
        for i, F in enumerate(fr):
            x = F.fill_bernoulli(seeds[i], 0.45)
            y = F.compact_run(x, torch.empty_like(x), steps)
            assert torch.equal(B.instance(res, i), y), (form, MANY[i], steps)
