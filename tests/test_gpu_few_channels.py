"""Backward-data passes into one to three channels on the banded-filter kernel: window sizes on either side of its
register classes (7, 12 and 32 values per lane), fewer and more channels than wavefronts, one and several
tiles with ragged edges, sources with and without pooling, every way the derivative is formed."""
import pytest

pytest.importorskip("torch")

from paper_1804_04512_amd.workloads import ConvSpec

import test_gpu_parity as T

pytestmark = pytest.mark.gpu

CASES = [
    ConvSpec(2, 1, 16, 16, 1, 3, 3, 1, "relu", 2), ConvSpec(3, 1, 19, 35, 4, 5, 5, 0, "sigmoid", 1),
    ConvSpec(2, 2, 33, 30, 5, 3, 3, 0, "identity", 1), ConvSpec(1, 3, 18, 20, 9, 5, 5, 2, "relu", 2),
    ConvSpec(2, 3, 22, 24, 17, 7, 7, 0, "sigmoid", 2), ConvSpec(1, 1, 28, 30, 12, 11, 11, 0, "identity", 2),
    ConvSpec(1, 2, 20, 17, 3, 12, 12, 5, "relu", 1), ConvSpec(1, 1, 41, 18, 6, 30, 3, 0, "relu", 2),
    ConvSpec(1, 3, 12, 9, 2, 2, 2, 0, "relu", 1), ConvSpec(1, 1, 17, 33, 40, 8, 17, 2, "sigmoid", 1),
]


@pytest.mark.parametrize("i", range(len(CASES)), ids=[f"C{c.C}_{c.H}x{c.W}_K{c.K}_{c.R}x{c.S}p{c.pad}_{c.act}_pool{c.pool}" for c in CASES])
def test_few_channels(i):
    T.check_trio(CASES[i], *T.rand_layer(CASES[i], 8000 + i))
