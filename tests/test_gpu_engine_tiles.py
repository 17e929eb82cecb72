"""The generic convolution instance where its tiles and batches end: maps of 8, 9, 16, 17 and 33 columns (8-, 16- and 32-wide tiles),
channel counts on either side of a chunk (balanced chunks: 17 are 9 + 8), more values per thread than one batch holds, filter
groups of 16, 32 and 48, a launch that splits its output channels, every source form of the backward-data pass."""
import pytest

pytest.importorskip("torch")

from paper_1804_04512_amd.workloads import ConvSpec

import test_gpu_parity as T

pytestmark = pytest.mark.gpu

CASES = [
    ConvSpec(2, 5, 10, 8, 7, 3, 3, 1, "relu", 2), ConvSpec(1, 17, 9, 9, 18, 4, 2, 0, "sigmoid", 1),
    ConvSpec(3, 16, 16, 16, 24, 3, 3, 1, "relu", 2), ConvSpec(2, 33, 12, 17, 33, 3, 5, 1, "relu", 1),
    ConvSpec(2, 12, 14, 16, 40, 3, 3, 1, "sigmoid", 2), ConvSpec(1, 4, 40, 33, 49, 9, 9, 4, "identity", 1),
    ConvSpec(1, 50, 20, 70, 5, 5, 5, 2, "sigmoid", 2), ConvSpec(2, 7, 8, 40, 50, 12, 12, 11, "relu", 1),
    ConvSpec(130, 6, 18, 34, 20, 3, 3, 0, "relu", 2), ConvSpec(1, 3, 7, 7, 64, 7, 7, 3, "identity", 1),
]


@pytest.mark.parametrize("i", range(len(CASES)), ids=[f"N{c.N}C{c.C}_{c.H}x{c.W}_K{c.K}_{c.R}x{c.S}p{c.pad}_{c.act}_pool{c.pool}" for c in CASES])
def test_engine_tiles(i):
    T.check_trio(CASES[i], *T.rand_layer(CASES[i], 9000 + i))
