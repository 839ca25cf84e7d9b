"""GPU parity of the diffusion runs with a block of cells per lane (several
steps per launch, blocks of Section "Moving from Thread-level to Block-level"):
bit for bit equal to one-step launches of the expanded-tile kernel, around the
step counts at which a launch ends (15 steps for the triangles, 27 for the
Vicsek cross, 18 for the carpet), in every tile configuration and storage
type; start addresses that are only element-aligned, and fields with
infinities and NaN."""
import pytest

from gpu_common import gpu_fractal, torch_or_skip

pytestmark = pytest.mark.gpu

CASES = [("triangle", 2), ("triangle", 8), ("triangle", 9), ("triangle", 11), ("triangle", 14), ("triangle_paper", 10),
         ("vicsek", 2), ("vicsek", 5), ("vicsek", 6), ("vicsek", 8), ("vicsek", 9), ("carpet", 2), ("carpet", 4),
         ("carpet", 5), ("carpet", 8)]
LIMIT = {"triangle": 15, "triangle_paper": 15, "vicsek": 27, "carpet": 18}
TYPES = [("f32", "nearest"), ("bf16", "nearest"), ("bf16", "stochastic")]


def start(torch, F, dtype, pad=0):
    u = F.fill_uniform(4)
    v = u if dtype == "f32" else F.bf16_encode(u, 0.5)
    whole = torch.zeros(F.cells + pad, dtype=v.dtype, device="cuda")
    whole[pad:] = v
    return whole[pad:]


@pytest.mark.parametrize("dtype,rounding", TYPES)
@pytest.mark.parametrize("name,r", CASES)
def test_runs_equal_one_step_launches(name, r, dtype, rounding):
    torch = torch_or_skip()
    F = gpu_fractal(name, r)
    k = LIMIT[name]
    x, at = start(torch, F, dtype).clone(), 0
    y = torch.empty_like(x)
    for steps in (1, 2, k, k + 1, 2 * k + 1):
        for s in range(at, steps):
            F.diffuse_step(x, y, 0.1, dtype=dtype, step=100 + s, rounding=rounding, impl="xtile", seed=9)
            x, y = y, x
        at = steps
        a = start(torch, F, dtype).clone()
        b = torch.empty_like(a)
        res = F.diffuse_run(a, b, steps, 0.1, dtype=dtype, first_step=100, rounding=rounding, seed=9)
        assert torch.equal(res.view(torch.uint8), x.view(torch.uint8)), steps


@pytest.mark.parametrize("dtype,rounding", TYPES)
@pytest.mark.parametrize("name,r", [("triangle", 9), ("vicsek", 7), ("carpet", 6)])
def test_element_aligned_buffers(name, r, dtype, rounding):
    torch = torch_or_skip()
    F = gpu_fractal(name, r)
    want = F.diffuse_run(start(torch, F, dtype).clone(), start(torch, F, dtype).clone(), 5, 0.1, dtype=dtype,
                         rounding=rounding, seed=3)
    a, b = start(torch, F, dtype, pad=1), start(torch, F, dtype, pad=3)
    res = F.diffuse_run(a, b, 5, 0.1, dtype=dtype, rounding=rounding, seed=3)
    assert torch.equal(res.contiguous().view(torch.uint8), want.view(torch.uint8))


@pytest.mark.parametrize("name,r", [("triangle", 9), ("vicsek", 6), ("carpet", 5)])
def test_infinities_and_nan(name, r):
    torch = torch_or_skip()
    F = gpu_fractal(name, r)
    u = F.fill_uniform(4)
    u[F.cells // 3], u[F.cells // 2], u[F.cells - 1] = float("inf"), float("nan"), -float("inf")
    x, y = u.clone(), torch.empty_like(u)
    for s in range(4):
        F.diffuse_step(x, y, 0.1, impl="xtile", step=s)
        x, y = y, x
    got = F.diffuse_run(u.clone(), torch.empty_like(u), 4, 0.1)
    assert torch.equal(torch.isnan(got), torch.isnan(x))
    assert torch.equal(torch.nan_to_num(got, 0.0), torch.nan_to_num(x, 0.0))


def test_cells_beyond_32_bits():
    """10.46e9 cells: the rounding hash of cells on both sides of index 2^32."""
    torch = torch_or_skip()
    F = gpu_fractal("triangle", 21)
    a = torch.empty(F.cells, dtype=torch.uint16, device="cuda")
    a.view(torch.bfloat16).uniform_(-0.5, 0.5, generator=torch.Generator("cuda").manual_seed(5))
    x, y, b = a.clone(), torch.empty_like(a), torch.empty_like(a)
    for s in range(3):
        F.diffuse_step(x, y, 0.1, dtype="bf16", step=7 + s, rounding="stochastic", impl="xtile", seed=9)
        x, y = y, x
    res = F.diffuse_run(a, b, 3, 0.1, dtype="bf16", first_step=7, rounding="stochastic", seed=9)
    for at in range(0, F.cells, 1 << 30):  # in pieces: comparison needs a copy
        assert torch.equal(res[at:at + (1 << 30)].view(torch.int16), x[at:at + (1 << 30)].view(torch.int16)), at
