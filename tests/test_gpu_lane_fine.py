"""GPU parity of the diffusion runs on fractals that do not fill the chip, where
a lane holds a level-1 block (blocks of Section "Moving from Thread-level to
Block-level"): bit for bit equal to one-step launches of the expanded-tile
kernel at the levels where the kernel or its tile changes and at the step
counts where a launch ends (15 steps for triangles and carpets, 27 for the
Vicsek cross)."""
import pytest

from gpu_common import gpu_fractal, torch_or_skip

pytestmark = pytest.mark.gpu

CASES = [("triangle", 1), ("triangle", 6), ("triangle", 7), ("triangle", 10), ("triangle", 12), ("triangle", 13),
         ("triangle_paper", 1), ("triangle_paper", 7), ("triangle_paper", 12), ("triangle_paper", 13), ("vicsek", 1),
         ("vicsek", 4), ("vicsek", 7), ("vicsek", 10), ("carpet", 1), ("carpet", 3), ("carpet", 6), ("carpet", 7)]
LIMIT = {"triangle": 15, "triangle_paper": 15, "vicsek": 27, "carpet": 15}
TYPES = [("f32", "nearest"), ("bf16", "nearest"), ("bf16", "stochastic")]


@pytest.mark.parametrize("dtype,rounding", TYPES)
@pytest.mark.parametrize("name,r", CASES)
def test_runs_equal_one_step_launches(name, r, dtype, rounding):
    torch = torch_or_skip()
    F = gpu_fractal(name, r)
    u = F.fill_uniform(4)
    start = u if dtype == "f32" else F.bf16_encode(u, 0.5)
    x, y, at = start.clone(), torch.empty_like(start), 0
    k = LIMIT[name]
    for steps in (2, 3, k, k + 1, k + 4):
        for s in range(at, steps):
            F.diffuse_step(x, y, 0.1, dtype=dtype, step=100 + s, rounding=rounding, impl="xtile", seed=9)
            x, y = y, x
        at = steps
        got = F.diffuse_run(start.clone(), torch.empty_like(start), steps, 0.1, dtype=dtype, first_step=100,
                            rounding=rounding, seed=9)
        assert torch.equal(got.view(torch.uint8), x.view(torch.uint8)), steps
