"""GPU parity of Life runs on the smallest fractals, which one workgroup takes
as a whole: a single cell, partial and full waves, 1000 and 1024 cells (the
largest) and the first fractal beyond, with and without aligned buffers,
against the CPU oracle (whole numbers, compared exactly)."""
import pytest

from gpu_common import mismatch, to_np, torch_or_skip

pytestmark = pytest.mark.gpu

TRIANGLE = (2, ((0, 0), (1, 0), (0, 1)))
VICSEK = (3, ((1, 0), (0, 1), (1, 1), (2, 1), (1, 2)))
CARPET = (3, tuple((x, y) for y in range(3) for x in range(3) if (x, y) != (1, 1)))
SQUARE = (2, ((0, 0), (1, 0), (0, 1), (1, 1)))
TEN = (4, ((0, 0), (1, 0), (3, 0), (0, 1), (2, 1), (3, 1), (1, 2), (2, 2), (0, 3), (3, 3)))


@pytest.mark.parametrize("pattern,r", [(TRIANGLE, 0), (TRIANGLE, 1), (TRIANGLE, 4), (TRIANGLE, 6), (TRIANGLE, 7),
                                       (VICSEK, 4), (VICSEK, 5), (CARPET, 2), (CARPET, 3), (SQUARE, 3), (SQUARE, 5),
                                       (TEN, 3)])
def test_runs_against_oracle(pattern, r):
    torch = torch_or_skip()
    import oracle
    import paper_2201_00613_amd as sqz

    F, O = sqz.Fractal(*pattern, r), oracle.Fractal(*pattern, r)
    state, at = O.fill_compact(3, 0.4), 0
    start = F.fill_bernoulli(3, 0.4)
    for steps in (0, 1, 2, 3, 10, 37):
        state, at = O.life_steps(state, steps - at), steps
        for pad in (0, 1):
            a = torch.full((F.cells + 2,), 5, dtype=torch.uint8, device="cuda")
            b = a.clone()
            x, y = a[pad:pad + F.cells], b[pad:pad + F.cells]
            x.copy_(start)
            mismatch(to_np(F.compact_run(x, y, steps)), state, f"{steps} steps, offset {pad}")
            for t in (a, b):
                assert bool((t[:pad] == 5).all()) and bool((t[pad + F.cells:] == 5).all())
