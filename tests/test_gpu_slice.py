"""GPU parity of the Life runs on tiles bit-sliced across subtrees (Section
"Moving from Thread-level to Block-level"): both run forms around the step
counts at which ring subtrees are exchanged or a launch ends (31 steps for the
triangles, 27 for the Vicsek cross), launches whose last one updates in place,
and every tile configuration.  Small fractals against the CPU oracle, larger
ones against one-step launches; results are whole numbers, compared exactly."""
import pytest

from gpu_common import gpu_fractal, mismatch, oracle_fractal, to_np, torch_or_skip

pytestmark = pytest.mark.gpu

CASES = [("triangle", 5), ("triangle", 6), ("triangle", 8), ("triangle", 9), ("triangle", 11), ("triangle_paper", 9),
         ("vicsek", 3), ("vicsek", 6), ("vicsek", 7)]


def step_counts(name):
    k = 27 if name == "vicsek" else 31
    return [2, k - 1, k, k + 1, 2 * k, 2 * k + 1]


@pytest.mark.parametrize("form", ["launches", "resident"])
@pytest.mark.parametrize("name,r", CASES)
def test_runs_against_oracle(name, r, form):
    torch = torch_or_skip()
    F, O = gpu_fractal(name, r), oracle_fractal(name, r)
    want, at = O.fill_compact(31, 0.5), 0
    start = F.fill_bernoulli(31, 0.5)
    for steps in step_counts(name):
        want, at = O.life_steps(want, steps - at), steps
        a, b = start.clone(), torch.full_like(start, 7)  # the other buffer's contents must not matter
        mismatch(to_np(F.compact_run(a, b, steps, form=form)), want, f"{name} r={r} {form} {steps} steps")


@pytest.mark.parametrize("name,r", [("triangle", 13), ("triangle", 15), ("triangle", 16), ("triangle", 17),
                                    ("triangle_paper", 16), ("triangle_paper", 17), ("vicsek", 10), ("vicsek", 11)])
def test_runs_equal_single_steps(name, r):
    torch = torch_or_skip()
    F = gpu_fractal(name, r)
    start = F.fill_bernoulli(5, 0.5)
    x, y, at = start.clone(), torch.empty_like(start), 0
    for steps in step_counts(name)[1:5]:
        for _ in range(steps - at):
            F.compact_step(x, y)
            x, y = y, x
        at = steps
        for form in ["launches"] + (["resident"] if F.resident_run else []):
            a, b = start.clone(), torch.full_like(start, 7)
            assert torch.equal(F.compact_run(a, b, steps, form=form), x), (form, steps)


def test_runs_one_cell_into_a_buffer():
    """Subtiles start at odd addresses; the cells before and after the state stay as they were."""
    torch = torch_or_skip()
    F = gpu_fractal("triangle", 9)
    start = F.fill_bernoulli(3, 0.5)
    want = F.compact_run(start.clone(), torch.empty_like(start), 32, form="launches")
    for form in ("launches", "resident"):
        for steps in (32, 33):
            a = torch.full((F.cells + 64,), 9, dtype=torch.uint8, device="cuda")
            b = a.clone()
            x, y = a[32:32 + F.cells], b[32:32 + F.cells]
            x.copy_(start)
            res = F.compact_run(x, y, steps, form=form)
            if steps == 32:
                assert torch.equal(res, want), form
            for t in (a, b):
                assert bool((t[:32] == 9).all()) and bool((t[32 + F.cells:] == 9).all()), (form, steps)


@pytest.mark.parametrize("steps", [1, 27, 31, 32, 63])
def test_batch_equals_single_runs(steps):
    """A batch's own tiles (level 8, level 6): fractals whose single runs use larger ones included."""
    torch = torch_or_skip()
    import paper_2201_00613_amd as sqz

    fr = [gpu_fractal(n, r) for n, r in [("triangle", 5), ("triangle", 9), ("triangle", 14), ("triangle", 15),
                                         ("triangle_paper", 14), ("vicsek", 4), ("vicsek", 7), ("vicsek", 10)]]
    B = sqz.Batch(fr)
    a = B.fill_bernoulli([11 * i for i in range(len(fr))], 0.5)
    res = B.run(a, B.empty_state(), steps)
    for i, F in enumerate(fr):
        x = F.fill_bernoulli(11 * i, 0.5)
        assert torch.equal(B.instance(res, i), F.compact_run(x, torch.empty_like(x), steps)), (i, steps)


@pytest.mark.parametrize("steps", [1, 2, 3, 4, 31, 32, 33, 62, 63, 64])
def test_batch_plans_against_single_runs(steps):
    """A batch's launches, among them those of one step that set the parity, around the
    most steps of a launch (27 for the Vicsek cross, 31 for the triangles)."""
    torch = torch_or_skip()
    import paper_2201_00613_amd as sqz

    fr = [gpu_fractal(*n) for n in (("triangle", 9), ("triangle", 5), ("vicsek", 7), ("triangle_paper", 10), ("vicsek", 4),
                                    ("triangle", 12), ("carpet", 5))]
    B = sqz.Batch(fr)
    a, b = B.empty_state(), B.empty_state()
    starts = []
    for i, F in enumerate(fr):
        starts.append(F.fill_bernoulli(40 + i, 0.5))
        B.instance(a, i).copy_(starts[i])
    res = B.run(a, b, steps) if steps > 1 else B.step(a, b)
    for i, F in enumerate(fr):
        x, y = starts[i], torch.empty_like(starts[i])
        for _ in range(steps):
            F.compact_step(x, y, impl="cell")
            x, y = y, x
        assert torch.equal(B.instance(res, i), x), i


@pytest.mark.parametrize("name,r", [("triangle", 8), ("triangle", 9), ("triangle", 16), ("vicsek", 6), ("vicsek", 8), ("vicsek", 10)])
def test_resident_runs_without_and_with_exchanges(name, r):
    """The resident form where it takes the plain kernel (one launch, no exchange) and
    around its exchanges, run after run on the same state (their counts carry over)."""
    torch = torch_or_skip()
    F = gpu_fractal(name, r)
    x = F.fill_bernoulli(6, 0.5)
    y, a = torch.empty_like(x), x.clone()
    b = torch.empty_like(a)
    for steps in (3, 2, 27, 28, 31, 32, 1, 55, 63, 94, 4):
        res = F.compact_run(a, b, steps, form="resident")
        if res is not a:
            a, b = b, a
        for _ in range(steps):
            F.compact_step(x, y)
            x, y = y, x
        assert torch.equal(res, x), steps
