"""Inference on a handful of patterns (the popcount rows kernel and the line to
the tiled kernels) against plain integer products, bit for bit: widths around
its 64-word rounds and 8-row waves, rows of odd word counts, column tails,
class counts on either side of the classifier kernel's limit, bits set past
the inputs' end, more than eight layers, and the entry point without
allocation."""
import numpy as np
import pytest

from paper_2412_00119_amd import bmlp as B

from gpu_common import Pair, note, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("widths,c", [
    ((1, 64), 2), ((63, 7, 65), 9), ((64, 128, 70), 16), ((4096, 130, 64), 17), ((4097, 525, 4160), 100),
    ((130, 8200, 72), 300), ((100,) + (24,) * 10, 129),
])
def test_few_patterns(widths, c, n):
    torch = torch_cuda()
    rng = np.random.default_rng(sum(widths) + c + n)
    note(f"few patterns {widths} c={c} n={n}")
    p = Pair(widths, c, 7, 8, 0, 0.25, seed=c + n)
    x = np.where(rng.random((n, widths[0])) < 0.5, 1, -1).astype(np.int8)
    x[0] = 1
    xb, _ = p.to_dev(x)
    if widths[0] % 64:   # bits past the last input do not count
        xb[:, -1] |= -1 << (widths[0] % 64)
    out = p.gpu.forward(xb)
    again = torch.full_like(out, -7)
    B.bmlp_forward_noalloc(p.gpu.ctx, xb.data_ptr(), n, again.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    a = x.astype(np.int64)
    for l in range(1, len(widths)):
        a = np.where(a @ p.ora.W(l).astype(np.int64).T >= 0, 1, -1)
        want = a @ p.ora.P[l - 1].astype(np.int64).T
        np.testing.assert_array_equal(out[l - 1].cpu().numpy(), want)
        np.testing.assert_array_equal(again[l - 1].cpu().numpy(), want)
