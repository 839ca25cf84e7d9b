"""GPU parity of the carpet's bit-row tiles (Section "Moving from Thread-level
to Block-level") at the step counts where a launch's border is used up (fifteen
steps; single tiles take a whole run in one launch), in runs and in batches, on
one tile of every size and on several, against the CPU oracle (whole numbers,
compared exactly)."""
import pytest

from gpu_common import gpu_fractal, mismatch, oracle_fractal, to_np, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [4, 5, 6, 7])
def test_runs_against_oracle(r):
    torch = torch_or_skip()
    F, O = gpu_fractal("carpet", r), oracle_fractal("carpet", r)
    state, at = O.fill_compact(6, 0.4), 0
    start = F.fill_bernoulli(6, 0.4)
    for steps in (2, 3, 4, 13, 15, 16, 31, 46):
        state, at = O.life_steps(state, steps - at), steps
        a, b = start.clone(), torch.full_like(start, 7)
        mismatch(to_np(F.compact_run(a, b, steps)), state, f"{steps} steps")


@pytest.mark.parametrize("levels", [(4, 5), (6, 4, 6), (3, 7)])
def test_batch_against_runs(levels):
    torch_or_skip()
    import paper_2201_00613_amd as sqz

    fr = [gpu_fractal("carpet", r) for r in levels]
    B = sqz.Batch(fr)
    for form in ("groups", "persistent", "per_tile"):
        B.set_tiled_launch(form)
        for steps in (15, 16, 50):
            a = B.fill_bernoulli(range(2, 2 + len(fr)), 0.5)
            starts = [B.instance(a, i).clone() for i in range(len(fr))]
            got = B.run(a, B.empty_state(), steps)
            for i, (F, s) in enumerate(zip(fr, starts)):
                want = F.compact_run(s.clone(), s.clone(), steps)
                mismatch(to_np(B.instance(got, i)), to_np(want), f"{form}, instance {i}, {steps} steps")
