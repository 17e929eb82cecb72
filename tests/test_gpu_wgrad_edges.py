"""Filter gradients where a map ends inside the 8 x 32 tiles: one to eight groups of four columns, zero to two rows of a
wavefront, pooled and not, rows of whole 16-byte groups and not."""
import pytest

pytest.importorskip("torch")

from paper_1804_04512_amd.workloads import ConvSpec

import test_gpu_parity as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Wo", [1, 4, 6, 8, 10, 16, 18, 24, 26, 32, 34, 40, 60])
@pytest.mark.parametrize("Ho,pool", [(2, 2), (7, 1), (9, 1), (12, 2), (17, 1)])
def test_map_edges(Wo, Ho, pool):
    cs = ConvSpec(3, 2, Ho + 2, Wo + Wo % pool + 2, 17, 3, 3, 0, "sigmoid", pool)
    T.check_trio(cs, *T.rand_layer(cs, 4100 + Wo))
