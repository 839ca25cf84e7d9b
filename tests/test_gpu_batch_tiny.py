"""Batches with fractals too small for a subtile to hold a block (level-3 and -4
triangles, the level-2 Vicsek cross): they run in their pattern's launches, in
every launch form, and their batches take the launch choices of any tiled batch."""
import pytest

from gpu_common import mismatch, oracle_fractal, to_np, torch_or_skip

pytestmark = pytest.mark.gpu

TINY = [("triangle", 3), ("triangle", 4), ("vicsek", 2), ("triangle_paper", 4), ("triangle_paper", 3)]
SPECS = {"one": [("triangle", 3)], "tiny": TINY * 3,
         "mixed": TINY + [("triangle", 5), ("triangle", 9), ("vicsek", 3), ("vicsek", 6), ("carpet", 5), ("triangle_paper", 8)]}


@pytest.mark.parametrize("name", sorted(SPECS))
def test_tiny_instances_against_oracle(name):
    torch = torch_or_skip()
    import fractals as FR
    import paper_2201_00613_amd as sqz

    spec = SPECS[name]
    B = sqz.Batch([sqz.Fractal(*FR.ALL[n], r) for n, r in spec])
    assert B.tiled_launch["form"] == "groups" and B.tiled_launch["steps_per_launch"] == 7
    assert B.steps_per_launch == 7  # the level-3 triangle's side less one
    seeds = [40 + i for i in range(len(spec))]
    ora = []
    for (n, r), s in zip(spec, seeds):
        O = oracle_fractal(n, r)
        ora.append((O, O.fill_compact(s, 0.5), O.neighbour_table()))
    for form, k, wg in (("groups", 0, 0), ("groups", 2, 0), ("persistent", 3, 2), ("per_tile", 7, 0)):
        B.set_tiled_launch(form, k, wg)
        for steps in (1, 2, 7, 10, 31):
            a, b = B.fill_bernoulli(seeds, 0.5), torch.full((B.total_bytes,), 7, dtype=torch.uint8, device="cuda")
            res = B.run(a, b, steps)
            for i, (O, start, nb) in enumerate(ora):
                mismatch(to_np(B.instance(res, i)), O.life_steps(start, steps, nb), f"{form} {spec[i]} {steps} steps")
