"""Resident runs long enough to exchange their ring subtrees (every 31 steps for the
triangles, 27 for the Vicsek cross; shorter odd runs need none): around every
exchange against the oracle, runs in a row whose exchange counts carry over, and
replays of a captured run with exchanges, between eager runs of other counts."""
import pytest

from gpu_common import gpu_fractal, mismatch, oracle_fractal, to_np, torch_or_skip

pytestmark = pytest.mark.gpu

K_OF = {"triangle": 31, "triangle_paper": 31, "vicsek": 27}


@pytest.mark.parametrize("name,r", [("triangle", 9), ("triangle", 12), ("triangle_paper", 10), ("vicsek", 7)])
def test_steps_around_exchanges(name, r):
    torch = torch_or_skip()
    F, O = gpu_fractal(name, r), oracle_fractal(name, r)
    assert F.resident_run
    K = K_OF[name]
    start, nb = O.fill_compact(31, 0.45), O.neighbour_table()
    state, t = start, 0
    for steps in (K - 1, K, K + 1, 2 * K - 1, 2 * K, 2 * K + 1, 3 * K + 2):
        state, t = O.life_steps(state, steps - t, nb), steps
        a = F.fill_bernoulli(31, 0.45)
        res = F.compact_run(a, torch.full_like(a, 7), steps, form="resident")
        mismatch(to_np(res), state, f"{name} r={r} {steps} steps")


@pytest.mark.parametrize("name,r", [("triangle", 12), ("triangle", 16), ("triangle_paper", 13), ("vicsek", 8), ("vicsek", 10)])
def test_exchange_counts_carry_over(name, r):
    torch = torch_or_skip()
    F = gpu_fractal(name, r)
    assert F.resident_run
    K = K_OF[name]
    a = F.fill_bernoulli(77, 0.5)
    x, y = a.clone(), torch.empty_like(a)
    u, v = a.clone(), torch.empty_like(a)
    for steps in (K + 1, 2 * K + 1, 3 * K + 1, 2, K, 2 * K, 5, K + 2, 4 * K + 3):  # 1, 2, 3, 0, 0, 1, 0, 1, 4 exchanges
        r1 = F.compact_run(x, y, steps, form="resident")
        x, y = (x, y) if r1 is x else (y, x)
        r2 = F.compact_run(u, v, steps, form="launches")
        u, v = (u, v) if r2 is u else (v, u)
        assert torch.equal(x, u), steps


@pytest.mark.parametrize("name,r", [("triangle", 12), ("vicsek", 8)])
def test_replays_between_eager_runs(name, r):
    torch = torch_or_skip()
    F = gpu_fractal(name, r)
    K = K_OF[name]
    steps = 2 * K + 2  # an even count: two exchanges, the result in place
    a = F.fill_bernoulli(17, 0.5)
    x, y = a.clone(), torch.empty_like(a)
    p, q = a.clone(), torch.empty_like(a)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        F.compact_run(p, q, steps, form="resident")
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        assert F.compact_run(x, y, steps, form="resident") is x
    torch.cuda.synchronize()
    assert torch.equal(x, a)
    u, v = a.clone(), torch.empty_like(a)
    for k, eager in enumerate((K + 1, 0, 3 * K + 1, 2 * K + 1, 1)):  # 1, 0, 3, 2, 0 exchanges between the replays
        g.replay()
        torch.cuda.synchronize()
        u = F.compact_run(u, v, steps, form="launches")
        assert torch.equal(x, u), k
        p.copy_(a)
        res = F.compact_run(p, q, eager, form="resident").clone()
        p.copy_(a)
        assert torch.equal(res, F.compact_run(p, q, eager, form="launches")), (k, eager)
    del g
