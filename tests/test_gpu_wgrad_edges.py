"""Filter gradients where a map ends inside the 8 x 32 tiles: one to eight groups of four columns, zero to two rows of a
wavefront, pooled and not.  `test_map_edges` goes through the widths on one instance (rows that are no whole 16-byte groups,
one staging round); `test_instances` goes through the others on fewer widths: whole and ragged rows, one and several staging
rounds, each number of tap tiles, with and without the layer output, element-wise staging; `test_crbm_steps` through
those with two gradients and the visible sums in one launch.  test_host_rules.py checks that these lists reach them."""
import pytest

pytest.importorskip("torch")

from oracle import oracle as orc
from paper_1804_04512_amd import workloads as wl
from paper_1804_04512_amd.workloads import ConvSpec

import test_gpu_parity as T
import test_gpu_rbm_dense as R
from helpers import odesc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Wo", [1, 4, 6, 8, 10, 16, 18, 24, 26, 32, 34, 40, 60])
@pytest.mark.parametrize("Ho,pool", [(2, 2), (7, 1), (9, 1), (12, 2), (17, 1)])
def test_map_edges(Wo, Ho, pool):
    cs = ConvSpec(3, 2, Ho + 2, Wo + Wo % pool + 2, 17, 3, 3, 0, "sigmoid", pool)
    T.check_trio(cs, *T.rand_layer(cs, 4100 + Wo))


def _layers():
    """Padded so that a map is as wide as its image: whole 16-byte groups of one are whole groups of the other."""
    out = []
    for C, K, r in ((2, 17, 3), (3, 20, 5), (2, 40, 7), (16, 35, 3)):   # 2 (one round), 5, 7 and 9 tap tiles
        for i, (wo, ho, pool, act) in enumerate([(4, 7, 1, "sigmoid"), (8, 12, 2, "relu"), (20, 9, 1, "identity"), (24, 8, 1, "relu"), (40, 10, 2, "sigmoid"),
                                                 (6, 2, 1, "relu"), (10, 12, 2, "sigmoid"), (18, 17, 1, "identity"), (57, 9, 1, "sigmoid"), (34, 6, 2, "relu")]):
            out.append(ConvSpec(2 + i % 2, C, ho, wo, K, r, r, r // 2, act, pool))
    out += [ConvSpec(3, 16, ho + 8, wo, k, 9, 1, 0, act, pool)   # 16 lines of halo per channel: more than the staging registers hold
            for k, wo, ho, pool, act in ((17, 4, 7, 1, "relu"), (9, 18, 9, 1, "identity"), (40, 40, 10, 2, "relu"), (5, 24, 2, 2, "sigmoid"))]
    return out


LAYERS = _layers()
CRBM = [ConvSpec(3, 2, 12, 20, 17, 3, 3, 1), ConvSpec(2, 3, 11, 18, 35, 3, 3, 0),      # one staging round: whole rows, ragged ones
        ConvSpec(2, 1, 25, 28, 40, 9, 9, 0), ConvSpec(1, 16, 9, 8, 20, 5, 5, 2), ConvSpec(3, 16, 16, 16, 8, 3, 3, 1),   # several, whole rows
        ConvSpec(2, 3, 13, 26, 20, 5, 5, 0), ConvSpec(1, 16, 18, 19, 33, 3, 3, 0),     # several, ragged rows
        ConvSpec(2, 16, 18, 20, 9, 9, 1, 0)]                                           # element-wise


def _name(c):
    return f"C{c.C}_{c.H}x{c.W}_K{c.K}_{c.R}x{c.S}p{c.pad}_{c.act}_pool{c.pool}"


@pytest.mark.parametrize("i", range(len(LAYERS)), ids=lambda i: _name(LAYERS[i]))
def test_instances(i):
    T.check_trio(LAYERS[i], *T.rand_layer(LAYERS[i], 4200 + i))


@pytest.mark.parametrize("i", range(len(CRBM)), ids=lambda i: _name(CRBM[i]))
def test_crbm_steps(i):
    """The visible sums of few images fill a few of a channel's 32 slices, or (3 x 16 x 16) three."""
    w = wl.crbm_units(CRBM[i], "binary", 1)
    g = R.run_crbm_units_gpu(w, "binary", 1, w.lr)
    Wn, bn, cn = w.W.copy(), w.b.copy(), w.c.copy()
    o = orc.crbm_cd1_step_units(odesc(CRBM[i]), R.VIS["binary"], 1, w.v0, Wn, bn, cn, None, h0_sample_in=g["h0_sample"], lr=w.lr)
    R.check_step_outputs(g, o, (w.W, w.b, w.c), (Wn, bn, cn))
