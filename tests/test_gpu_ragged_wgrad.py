"""Filter gradient on rows that are not whole 16-byte groups: every remainder of the width by four, one
and several 32-column tiles, both staging depths (one round for a few channels of a small filter, several
beyond), pooled (the pooling bytes then start at any byte) and unpooled, each way the derivative is formed.
Compared with the CPU oracle like every layer; an element of the neighbouring row that slipped in would be
an error of the order of the result."""
import pytest

pytest.importorskip("torch")

from paper_1804_04512_amd.workloads import ConvSpec

import test_gpu_parity as T

pytestmark = pytest.mark.gpu

CASES = [ConvSpec(3, 2, 11, 31 + r, 5, 3, 3, 1, act, 1) for r, act in enumerate(["identity", "sigmoid", "relu", "identity"])]
CASES += [ConvSpec(2, 17, 13, 66 + r, 33, 3, 3, 0, act, 1) for r, act in enumerate(["relu", "identity", "sigmoid", "relu"])]
CASES += [ConvSpec(3, 1, 12, 2 * r + 2, 9, 3, 3, 1, act, 2) for r, act in enumerate(["relu", "sigmoid", "identity", "relu"])]
CASES += [ConvSpec(2, 9, 10, 2 * r + 62, 40, 5, 5, 2, act, 2) for r, act in enumerate(["identity", "relu", "sigmoid", "relu"])]
CASES += [ConvSpec(1, 3, 9, 9, 4, 9, 9, 0, "sigmoid", 1)]   # one output pixel


@pytest.mark.parametrize("i", range(len(CASES)), ids=[f"C{c.C}_{c.H}x{c.W}_K{c.K}_{c.R}x{c.S}_{c.act}_pool{c.pool}" for c in CASES])
def test_ragged_widths(i):
    T.check_trio(CASES[i], *T.rand_layer(CASES[i], 7000 + i))
