"""The space maps against the oracle at counts around their pairs, passes and the
change to the form for many elements, at element-aligned addresses, with
indices and points outside the fractal; 32- and 64-bit indices."""
import numpy as np
import pytest

from gpu_common import gpu_fractal, mismatch, oracle_fractal, to_np, torch_or_skip

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 3, 511, 513, 2047, 2048, 2049, 100_001, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, 5_000_003]


@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("name,r", [("triangle", 0), ("triangle", 16), ("carpet", 5), ("triangle", 22)])
def test_counts(name, r, pad):
    torch = torch_or_skip()
    F, O = gpu_fractal(name, r), oracle_fractal(name, r)
    rng = np.random.default_rng(r)
    most = COUNTS[-1]
    c = rng.integers(0, F.cells, most, dtype=np.uint64)
    c[::1001] = F.cells + 5
    inside = c < F.cells
    xy = np.full((most, 2), -1, dtype=np.int32)
    xy[inside] = O.lam(c[inside])
    pts = rng.integers(-1, F.n + 1, (most, 2)).astype(np.int32)
    pts[::2] = xy[::2]
    nu = O.nu(pts.astype(np.int64))
    dc = torch.zeros(most + pad, dtype=torch.int64, device="cuda")
    dp = torch.zeros((most + pad, 2), dtype=torch.int32, device="cuda")
    dc[pad:] = torch.from_numpy(c.view(np.int64))
    dp[pad:] = torch.from_numpy(pts)
    for n in COUNTS:
        got = torch.full((n + 2 * pad, 2), 77, dtype=torch.int32, device="cuda")
        F.lambda_map(dc[pad:pad + n], out=got[pad:pad + n])
        mismatch(to_np(got[pad:pad + n]), xy[:n], f"lambda {n}")
        idx = torch.full((n + 2 * pad,), 77, dtype=torch.int64, device="cuda")
        F.nu_map(dp[pad:pad + n], out=idx[pad:pad + n])
        mismatch(to_np(idx[pad:pad + n]), nu[:n], f"nu {n}")
        if pad:
            assert (to_np(got[[0, -1]]) == 77).all() and (to_np(idx[[0, -1]]) == 77).all()
