"""The binary64 mass (its fixed summation order, bit for bit, in torch) and the
bfloat16 conversions at sizes around their vector widths and batches of loads,
at aligned and element-aligned addresses."""
import pytest

from gpu_common import gpu_fractal, torch_or_skip

pytestmark = pytest.mark.gpu

GRID = 1024 * 256  # sums of the fixed grid

# cells: 1, 3, 8, 81, 59049 (less than the grid), 262144 = the grid, 531441, 4.8e6 (a batch and a ragged
# rest), 1.7e7 (whole batches)
SIZES = [("triangle", 0), ("triangle", 1), ("carpet", 1), ("triangle", 4), ("triangle", 10), ("carpet", 6),
         ("triangle", 12), ("triangle", 14), ("carpet", 8)]


def tree(v):  # [.., 256] -> [..]
    while v.shape[-1] > 1:
        v = v[..., :v.shape[-1] // 2] + v[..., v.shape[-1] // 2:]
    return v[..., 0]


def mass_in_order(torch, u, offset):
    acc = torch.zeros(GRID, dtype=torch.float64, device="cuda")
    for at in range(0, u.numel(), GRID):
        row = u[at:at + GRID].double()
        acc[:row.numel()] += row
    part = tree(acc.view(1024, 256))
    lane = torch.zeros(256, dtype=torch.float64, device="cuda")
    for row in part.view(4, 256):
        lane = lane + row
    return float(tree(lane)) + u.numel() * offset


@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("name,r", SIZES)
def test_mass_and_conversions(name, r, pad):
    torch = torch_or_skip()
    F = gpu_fractal(name, r)
    g = torch.Generator("cuda").manual_seed(r)
    u = torch.empty(F.cells + pad, device="cuda").uniform_(-1.0, 1.0, generator=g)[pad:]
    assert float(F.mass_f64(u, offset=0.25)) == mass_in_order(torch, u, 0.25)
    want = (u - 0.25).to(torch.bfloat16)
    b = torch.zeros(F.cells + 2 * pad, dtype=torch.uint16, device="cuda")
    F.bf16_encode(u, 0.25, out=b[pad:pad + F.cells])
    h = b[pad:pad + F.cells]
    assert torch.equal(h.view(torch.int16), want.view(torch.int16))
    assert not pad or (int(b.view(torch.int16)[0]) == 0 and int(b.view(torch.int16)[-1]) == 0)
    assert float(F.mass_f64(h, dtype="bf16", offset=0.25)) == mass_in_order(torch, want, 0.25)
    out = torch.full((F.cells + 2 * pad,), 9.0, device="cuda")
    F.bf16_decode(h, 0.25, out=out[pad:pad + F.cells])
    assert torch.equal(out[pad:pad + F.cells], want.float() + 0.25)
    assert not pad or (float(out[0]) == 9.0 and float(out[-1]) == 9.0)
