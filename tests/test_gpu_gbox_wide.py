"""GPU parity of Life runs on general replica patterns at the step counts where
the wider border of few tiles begins and ends (17 to 33 steps and their
multiples), and on both sides of the tile count up to which it is used, against
the CPU oracle (whole numbers, compared exactly)."""
import pytest

from gpu_common import mismatch, to_np, torch_or_skip

pytestmark = pytest.mark.gpu

WIDE = (4, ((0, 0), (1, 0), (3, 0), (0, 1), (2, 1), (3, 1), (1, 2), (2, 2), (0, 3), (3, 3)))
SQUARE = (2, ((0, 0), (1, 0), (0, 1), (1, 1)))
FIVE = (3, ((0, 0), (2, 0), (1, 1), (0, 2), (2, 2)))
SEVEN = (3, ((0, 0), (1, 0), (2, 0), (0, 1), (2, 1), (0, 2), (1, 2)))
SIX = (5, ((0, 0), (4, 0), (2, 1), (1, 3), (2, 2), (4, 4)))
CASES = [(WIDE, 4), (WIDE, 6), (SQUARE, 7), (SQUARE, 9), (SQUARE, 11), (SQUARE, 12), (FIVE, 8), (SEVEN, 6), (SIX, 5)]


@pytest.mark.parametrize("pattern,r", CASES)
def test_runs_against_oracle(pattern, r):
    torch = torch_or_skip()
    import oracle
    import paper_2201_00613_amd as sqz

    F, O = sqz.Fractal(*pattern, r), oracle.Fractal(*pattern, r)
    state, at = O.fill_compact(3, 0.5), 0
    start = F.fill_bernoulli(3, 0.5)
    for steps in (15, 18, 21, 25, 31, 32, 40, 63):
        state, at = O.life_steps(state, steps - at), steps
        mismatch(to_np(F.compact_run(start.clone(), torch.empty_like(start), steps)), state, f"{steps} steps")
