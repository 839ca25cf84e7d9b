"""A batch whose runs keep changing length and buffers: each change replaces the
captured run while launches of the former may still be under way on one or two
streams, and the batch itself goes with work queued.  Results equal one-step
launches."""
import pytest

from gpu_common import gpu_fractal, torch_or_skip

pytestmark = pytest.mark.gpu


def test_replaced_runs_finish():
    torch = torch_or_skip()
    import paper_2201_00613_amd as sqz

    fr = [gpu_fractal("triangle", 12), gpu_fractal("carpet", 6), gpu_fractal("vicsek", 8)]
    B = sqz.Batch(fr)
    start = B.fill_bernoulli([1, 2, 3], 0.45)
    lengths = [2, 5, 3, 12, 4, 7, 31, 6, 2, 9, 33, 8, 5, 3, 16, 4, 10, 2, 21, 6, 3, 5]
    x, y = start.clone(), torch.empty_like(start)
    for _ in range(sum(lengths)):
        B.step(x, y)
        x, y = y, x
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    a, b = start.clone(), torch.empty_like(start)
    c, d = start.clone(), torch.empty_like(start)
    side.wait_stream(torch.cuda.current_stream())
    for n in lengths:  # no synchronisation: up to two runs in flight, one per stream
        res = B.run(a, b, n)
        a, b = (a, b) if res is a else (b, a)
        with torch.cuda.stream(side):
            res = B.run(c, d, n)
            c, d = (c, d) if res is c else (d, c)
    torch.cuda.current_stream().wait_stream(side)
    B.close()  # with work queued
    for i in range(len(fr)):
        off = B.offsets[i]
        n = fr[i].cells
        assert torch.equal(a[off:off + n], x[off:off + n]) and torch.equal(c[off:off + n], x[off:off + n]), i
