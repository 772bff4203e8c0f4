"""GPU parity of the input side with the oracle, bit for bit: per-feature
medians, median binarisation, and the fixed random ±1 expansion layer
(single and multiple input passes, ragged column and pattern tails), and a
few training steps on expanded inputs."""
import numpy as np
import pytest

import oracle.bmlp as ob
from paper_2412_00119_amd import bmlp as B

from gpu_common import Pair, note, pack_np, torch_cuda

pytestmark = pytest.mark.gpu


def _int8(rng, shape):
    return rng.integers(-128, 128, shape).astype(np.int8)


@pytest.mark.parametrize("n,k", [(1, 5), (2, 70), (999, 300), (1000, 129)])
def test_median_and_binarize(n, k):
    torch = torch_cuda()
    rng = np.random.default_rng(n + k)
    x = _int8(rng, (n, k))
    x[:, 3 % k] = 7                                  # a constant column
    xd = torch.from_numpy(x).cuda()
    note(f"median n={n} k={k}")
    med = B.feature_median(xd)
    bits = B.binarize(xd, med)
    torch.cuda.synchronize()
    m = ob.feature_median(x)
    np.testing.assert_array_equal(med.cpu().numpy(), m)
    np.testing.assert_array_equal(bits.cpu().numpy().view(np.uint64),
                                  pack_np(ob.median_binarize(x, m), bits.shape[1]))


@pytest.mark.parametrize("n,k", [(3, 7), (4, 8), (5, 9), (1023, 15), (8192, 16), (8193, 17), (17500, 23), (40, 1040),
                                 (130, 1025)])
def test_median_and_binarize_edges(n, k):
    """Feature tiles that overlap at the end of a row, rows shorter than a
    load, row counts around the passes of a work-group, rows that start at
    any byte, and columns of extreme or few values."""
    torch = torch_cuda()
    rng = np.random.default_rng(7 * n + k)
    x = _int8(rng, (n, k))
    x[:, 0] = np.where(rng.random(n) < 0.5, -128, 127)
    x[:, k - 1] = rng.integers(-1, 2, n)
    note(f"median edges n={n} k={k}")
    xd = torch.from_numpy(x).cuda()
    med = B.feature_median(xd)
    bits = B.binarize(xd, med)
    packed = torch.empty_like(bits)
    B.bmlp_pack(xd.data_ptr(), n, k, packed.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    m = ob.feature_median(x)
    np.testing.assert_array_equal(med.cpu().numpy(), m)
    np.testing.assert_array_equal(bits.cpu().numpy().view(np.uint64),
                                  pack_np(ob.median_binarize(x, m), bits.shape[1]))
    np.testing.assert_array_equal(packed.cpu().numpy().view(np.uint64), pack_np(x, bits.shape[1]))


@pytest.mark.parametrize("n,k", [(2048, 20), (2049, 16), (4097, 15), (6200, 31), (65000, 40), (5000, 4097), (9000, 129)])
def test_median_split(n, k):
    """Rows counted in one and in several parts (the last shorter than the
    others), feature tiles that overlap at the end of a row, and the same
    without scratch memory."""
    torch = torch_cuda()
    rng = np.random.default_rng(5 * n + k)
    x = _int8(rng, (n, k))
    x[:, 0] = np.where(np.arange(n) < (n + 1) // 2, 127, -128)
    x[:, k - 1] = rng.integers(-1, 2, n)
    note(f"median split n={n} k={k}")
    xd = torch.from_numpy(x).cuda()
    med = B.feature_median(xd)
    alone = torch.empty_like(med)
    B.bmlp_feature_median(xd.data_ptr(), n, k, alone.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    m = ob.feature_median(x)
    np.testing.assert_array_equal(med.cpu().numpy(), m)
    np.testing.assert_array_equal(alone.cpu().numpy(), m)


@pytest.mark.parametrize("n,k", [(1, 1), (255, 64), (256, 65), (257, 130), (129, 8193), (300, 8191), (128, 8256), (140, 9000),
                                 (2500, 8200)])
def test_median_wide(n, k):
    """64 features per work-group (few rows, or many features): row counts
    around its passes of 128, feature tails, and columns of extreme values."""
    test_median_split(n, k)


@pytest.mark.parametrize("n,k", [(100, 1000), (37, 33), (64, 47), (65, 49), (3, 63), (130, 16), (20, 1039),
                                 (1, 1), (300, 2), (1025, 13), (77, 15)])
def test_row_tails(n, k):
    """Rows that end at every place of a lane's 16 columns, and zeros past
    them in the last word."""
    test_median_and_binarize_edges(n, k)


@pytest.mark.parametrize("n,k", [(3, (1 << 25) + 9), (1, (1 << 28) + 70)])
def test_median_very_wide(n, k):
    """More features than work-groups of 8 or of 64 fit one launch."""
    torch = torch_cuda()
    g = torch.Generator(device="cuda").manual_seed(k)
    note(f"median n={n} k={k}")
    x = torch.randint(-128, 128, (n, k), generator=g, device="cuda", dtype=torch.int8)
    med = B.feature_median(x)
    want = x[0] if n == 1 else torch.maximum(torch.minimum(x[0], x[1]),
                                             torch.minimum(torch.maximum(x[0], x[1]), x[2]))
    assert bool((med == want).all())


@pytest.mark.parametrize("n,k_raw,k0", [(5, 1, 64), (300, 37, 100), (70, 300, 257), (257, 5000, 64),
                                        (64, 4096, 128)])
def test_expand(n, k_raw, k0):
    torch = torch_cuda()
    rng = np.random.default_rng(k_raw + k0)
    x = _int8(rng, (n, k_raw))
    seed = 0xFEEDFACE12345
    note(f"expand n={n} k_raw={k_raw} k0={k0}")
    bits = B.expand(torch.from_numpy(x).cuda(), k0, seed)
    torch.cuda.synchronize()
    want = ob.expand(x, ob.expansion_matrix(seed, k_raw, k0))
    np.testing.assert_array_equal(bits.cpu().numpy().view(np.uint64), pack_np(want, bits.shape[1]))


@pytest.mark.parametrize("n,k_raw,k0", [(1, 16, 64), (129, 128, 129), (127, 129, 65), (130, 1024, 200), (64, 1025, 128),
                                        (3, 2177, 96), (520, 33, 32767)])
def test_expand_edges(n, k_raw, k0):
    """Stages, chunks of drawn bits and tiles with remainders, rows that
    start at any byte, a work-group that walks two row tiles (the last
    size), and rows of equal extreme features."""
    torch = torch_cuda()
    rng = np.random.default_rng(n + 3 * k_raw + k0)
    x = _int8(rng, (n, k_raw))
    x[0] = -128
    x[n // 2] = 127
    seed = 0x8000000180000001
    note(f"expand edges n={n} k_raw={k_raw} k0={k0}")
    bits = B.expand(torch.from_numpy(x).cuda(), k0, seed)
    torch.cuda.synchronize()
    want = ob.expand(x, ob.expansion_matrix(seed, k_raw, k0))
    np.testing.assert_array_equal(bits.cpu().numpy().view(np.uint64), pack_np(want, bits.shape[1]))


@pytest.mark.parametrize("n", [3, 130])
@pytest.mark.parametrize("k_raw", [2, 15, 17, 30, 47, 79, 113, 140, 191, 1029])
def test_expand_row_tails(n, k_raw):
    """Rows that end at every place of a 16-byte load, and rows shorter than
    one."""
    test_expand_edges(n, k_raw, 70)


def test_expand_most_rows():
    """As many rows as the argument holds (rounding their number up to tiles
    must not pass 2^31)."""
    torch = torch_cuda()
    n, seed = 2**31 - 1, 99
    note(f"expand n={n}")
    x = torch.empty((n, 1), dtype=torch.int8, device="cuda")
    x.view(-1)[:] = 5
    x[:3, 0] = torch.tensor([-1, 0, 127], dtype=torch.int8)
    x[-3:, 0] = torch.tensor([0, -128, -3], dtype=torch.int8)
    bits = B.expand(x, 64, seed)
    few = torch.cat([x[:3], x[-3:], x[5:6]])
    want = ob.expand(few.cpu().numpy(), ob.expansion_matrix(seed, 1, 64))
    rows = pack_np(want, 1).view(np.int64)
    np.testing.assert_array_equal(torch.cat([bits[:3], bits[-3:]]).cpu().numpy(), rows[:6])
    for i in range(3, n - 3, 2**27):   # all the others are alike
        assert bool((bits[i:min(i + 2**27, n - 3)] == int(rows[6, 0])).all())


def test_training_on_expanded_inputs():
    torch = torch_cuda()
    p = Pair((256, 128), 5, 15, 64, 64, 0.25, seed=3)
    rng = np.random.default_rng(8)
    seed = 77
    R = ob.expansion_matrix(seed, 40, 256)
    for t in range(3):
        x = _int8(rng, (64, 40))
        y = rng.integers(0, 5, 64).astype(np.int32)
        a0 = ob.expand(x, R)
        xb = B.expand(torch.from_numpy(x).cuda(), 256, seed)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(xb.cpu().numpy().view(np.uint64), pack_np(a0, xb.shape[1]))
        note(f"expanded step {t}")
        p.step(a0, y, t, 0.5, tag=f"step {t}")
