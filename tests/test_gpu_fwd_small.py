"""The forward over small and large tile counts against the oracle, bit for
bit: K around the chunks and load rounds of the split-K kernel, row and
column tails, more column tiles than divide over the XCDs, and shapes on
either side of the line between the two kernels (rows of an odd number of
words among them, which the large-tile kernel loads four bytes at a time)."""
import numpy as np
import pytest

from paper_2412_00119_amd.synth import random_pm1

from gpu_common import Pair, note, pack_np, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k0,k1,gamma,n", [
    (1, 64, 64, 1), (63, 128, 64, 31), (255, 64, 64, 32), (256, 70, 10, 33), (257, 192, 64, 65),
    (1024, 64, 64, 40), (1025, 130, 13, 7), (2049, 64, 64, 33), (4097, 128, 64, 3), (5000, 81, 81, 34),
    (300, 1600, 64, 20),      # 25 column tiles: four a XCD, the last XCD has one
    (130, 4096, 64, 260),     # 576 tiles of few chunks
    (1100, 4096, 64, 260),    # 576 tiles: the large-tile kernel
    (130, 2112, 64, 1020),    # 1056 tiles, rows of 3 words
    (1090, 2040, 85, 640),    # 640 tiles, rows of 18 words, general groups
])
def test_forward_shapes(k0, k1, gamma, n):
    rng = np.random.default_rng(k0 + k1 + n)
    note(f"forward {k0}->{k1} gamma={gamma} n={n}")
    p = Pair((k0, k1), 5, 15, n, gamma, 0.25, seed=k0 + 1)
    x = random_pm1((n, k0), rng)
    x[0] = 1
    y = rng.integers(0, 5, n).astype(np.int32)
    p.step(x, y, 0, 0.5)


@pytest.mark.parametrize("c,n", [(130, 5), (300, 64)])
def test_many_class_products(c, n):
    """y_hat of several layers in one launch of the split-K kernel."""
    torch = torch_cuda()
    rng = np.random.default_rng(c)
    widths = (100, 128, 320, 70)
    note(f"products c={c} n={n}")
    p = Pair(widths, c, 7, n, 0, 0.25, seed=c)
    x = random_pm1((n, widths[0]), rng)
    xb, _ = p.to_dev(x)
    out = p.gpu.forward(xb)
    torch.cuda.synchronize()
    a = x.astype(np.int64)
    for l in range(1, 4):
        z = a @ p.ora.W(l).astype(np.int64).T
        a = np.where(z >= 0, 1, -1)
        np.testing.assert_array_equal(out[l - 1].cpu().numpy(), a @ p.ora.P[l - 1].astype(np.int64).T)


@pytest.mark.parametrize("k0,k1,gamma,n", [
    (1024, 4096, 64, 449),    # 256 tiles of 64 rows, one row in the last; K without a remainder
    (1200, 4096, 64, 500),    # rows of 19 words (four-byte loads)
    (1200, 4096, 64, 520),    # 288 tiles of 64 rows: tiles of 128
    (1130, 4030, 65, 449),    # a column tail, groups across tiles
    (2600, 2304, 0, 900),     # the group-size rule, row tail 4
    (513, 8128, 127, 225),    # K one past a step, 64 column tiles
])
def test_forward_half_tiles(k0, k1, gamma, n):
    """The 64-row tiles of the large-tile kernel, and the line to its 128-row tiles."""
    test_forward_shapes(k0, k1, gamma, n)


def test_many_class_products_half_tiles():
    """y_hat of three layers in one launch of 243 tiles of 64 rows."""
    test_many_class_products(300, 1700)


@pytest.mark.parametrize("widths,n", [
    ((130, 2111, 33), 1900),      # 255 tiles of 128 rows, the last column tile of 63 columns
    ((600, 4000, 4097), 1025),    # one row and one column past a tile
    ((64, 8129, 2080), 700),
])
def test_inference_column_tails(widths, n):
    """The large-tile kernel without a selection: signs of ragged widths, and
    zeros in a_l past the last column."""
    torch = torch_cuda()
    rng = np.random.default_rng(sum(widths))
    note(f"inference {widths} n={n}")
    p = Pair(widths, 7, 7, n, 1, 0.25, seed=n)
    x = random_pm1((n, widths[0]), rng)
    xb, _ = p.to_dev(x)
    for l in range(1, len(widths)):
        p.gpu.trace(l, n)["a"].fill_(-1)
    out = p.gpu.forward(xb)
    torch.cuda.synchronize()
    a = x.astype(np.float64)
    for l in range(1, len(widths)):
        a = np.where(a @ p.ora.W(l).astype(np.float64).T >= 0, 1.0, -1.0)
        rows = p.gpu.trace(l, n)["a"].cpu().numpy().view(np.uint64)
        np.testing.assert_array_equal(rows, pack_np(a.astype(np.int8), rows.shape[1]))
        want = (a @ p.ora.P[l - 1].astype(np.float64).T).astype(np.int64)
        np.testing.assert_array_equal(out[l - 1].cpu().numpy(), want)
