"""GPU parity of Life on general replica patterns through bit rows of an
expanded tile (Section "Moving from Thread-level to Block-level"): one step and
runs around the step counts at which a launch ends, on sparse and dense
patterns, side 2 to 16, single tiles and many, tile sizes that are not a
multiple of four cells, and start addresses without alignment, against the CPU
oracle (whole numbers, compared exactly)."""
import pytest

from gpu_common import mismatch, to_np, torch_or_skip

pytestmark = pytest.mark.gpu

WIDE = (4, ((0, 0), (1, 0), (3, 0), (0, 1), (2, 1), (3, 1), (1, 2), (2, 2), (0, 3), (3, 3)))
SQUARE = (2, ((0, 0), (1, 0), (0, 1), (1, 1)))
PAIR = (2, ((0, 0), (1, 1)))
FIVE = (3, ((0, 0), (2, 0), (1, 1), (0, 2), (2, 2)))        # five corners and centre: 5^M cells a tile
SEVEN = (3, ((0, 0), (1, 0), (2, 0), (0, 1), (2, 1), (0, 2), (1, 2)))
BIG = (16, tuple((i % 16, i // 16) for i in range(256) if i % 7 != 3)[:90])
CASES = [(WIDE, 1), (WIDE, 3), (WIDE, 4), (WIDE, 5), (SQUARE, 4), (SQUARE, 8), (PAIR, 9), (FIVE, 4), (FIVE, 6),
         (SEVEN, 5), (BIG, 1), (BIG, 2)]


@pytest.mark.parametrize("pattern,r", CASES)
def test_runs_against_oracle(pattern, r):
    torch = torch_or_skip()
    import oracle
    import paper_2201_00613_amd as sqz

    F, O = sqz.Fractal(*pattern, r), oracle.Fractal(*pattern, r)
    state, at = O.fill_compact(8, 0.5), 0
    start = F.fill_bernoulli(8, 0.5)
    got = F.compact_step(start, torch.empty_like(start))
    for steps in (1, 2, 3, 4, 5, 16, 17, 33):
        state, at = O.life_steps(state, steps - at), steps
        if steps == 1:
            mismatch(to_np(got), state, "one step")
        for pad in (0, 1):
            a = torch.full((F.cells + 2,), 5, dtype=torch.uint8, device="cuda")
            b = a.clone()
            x, y = a[pad:pad + F.cells], b[pad:pad + F.cells]
            x.copy_(start)
            mismatch(to_np(F.compact_run(x, y, steps)), state, f"{steps} steps, offset {pad}")
            for t in (a, b):
                assert bool((t[:pad] == 5).all()) and bool((t[pad + F.cells:] == 5).all())
