"""The update with a group's rows spread over two to 64 work-groups, against
the oracle, bit for bit: groups of one row, of a width that the parts do not
divide, of several column chunks, and one group that is a whole layer."""
import numpy as np
import pytest

from paper_2412_00119_amd import bmlp as B
from paper_2412_00119_amd.synth import random_pm1

from gpu_common import Pair, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variants", [0, B.BMLP_VARIANT_SEQUENTIAL_CLIP])
@pytest.mark.parametrize("widths,gamma,bound,n", [
    ((70, 7), 1, 3, 20), ((70, 26), 13, 7, 90), ((2100, 64), 64, 15, 70), ((130, 1024), 1024, 31, 900),
    ((4100, 243), 81, 101, 50), ((100, 2048, 192), 64, 127, 33),
])
def test_split_rows(widths, gamma, bound, n, variants):
    rng = np.random.default_rng(sum(widths) + n)
    p = Pair(widths, 4, bound, n, gamma, 0.25, seed=11, variants=variants)
    for t in range(2):
        note(f"split {widths} gamma={gamma} variants={variants} step {t}")
        x = random_pm1((n, widths[0]), rng)
        y = rng.integers(0, 4, n).astype(np.int32)
        p.step(x, y, t, 0.5, tag=f"step {t}")


@pytest.mark.parametrize("widths,gamma,n", [
    ((8300, 64), 64, 90), ((6200, 78), 13, 70), ((33, 4200, 24), 3, 50), ((10300, 12), 1, 40), ((4200, 256), 256, 120),
])
def test_rows_of_several_chunks(widths, gamma, n):
    """Rows of two to six column chunks, which are taken in another order in
    each chunk, with few rows a work-group and many, when patterns that are
    alike choose the same few rows."""
    rng = np.random.default_rng(sum(widths) + n)
    p = Pair(widths, 3, 31, n, gamma, 0.25, seed=23)
    protos = random_pm1((3, widths[0]), rng)
    for t in range(3):
        note(f"chunks {widths} gamma={gamma} step {t}")
        y = rng.integers(0, 3, n).astype(np.int32)
        flip = rng.random((n, widths[0])) < 0.01
        x = np.where(flip, -protos[y], protos[y]).astype(np.int8)
        p.step(x, y, t, 0.5, tag=f"step {t}")
