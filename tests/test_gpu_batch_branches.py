"""A run of a batch whose launches are branches of one graph: replays, with
other work on the stream between them, equal steps launched one by one, for
every mix of pattern groups and instances without one (triangle, its mirror
image, Vicsek cross, carpet; patterns without a kernel of their own; fractals
of a few cells)."""
import pytest

from gpu_common import gpu_fractal, torch_or_skip

pytestmark = pytest.mark.gpu

MIXES = [["carpet3"], ["full2x2_6"], ["carpet5", "full2x2_6"], ["triangle9", "vicsek5", "carpet4"],
         ["triangle8", "triangle_paper10", "vicsek6", "carpet5", "full2x2_8", "triangle2", "carpet1", "triangle9"]]


@pytest.mark.parametrize("steps", [2, 13, 31])
@pytest.mark.parametrize("mix", range(len(MIXES)))
def test_replays_equal_single_steps(mix, steps):
    torch = torch_or_skip()
    import paper_2201_00613_amd as sqz

    fr = [sqz.Fractal(2, [(0, 0), (1, 0), (0, 1), (1, 1)], int(n[8:])) if n.startswith("full") else
          gpu_fractal(n.rstrip("0123456789"), int(n[len(n.rstrip("0123456789")):])) for n in MIXES[mix]]
    B = sqz.Batch(fr)
    a, b = B.empty_state(), B.empty_state()
    x, y = B.empty_state(), B.empty_state()
    for rep in range(4):
        a.bernoulli_(0.5, generator=torch.Generator("cuda").manual_seed(10 * mix + rep))
        x.copy_(a)
        res = B.run(a, b, steps)
        got = [B.instance(res, i).clone() for i in range(len(fr))]
        u, v = x, y
        for _ in range(steps):
            B.step(u, v)
            u, v = v, u
        for i in range(len(fr)):
            assert torch.equal(got[i], B.instance(u, i)), (rep, MIXES[mix][i])
        torch.cuda.synchronize()
