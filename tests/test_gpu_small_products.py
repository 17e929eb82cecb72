"""Dense products on the small-product kernels at the sizes where their tiles end: the RBM step (states in
the product's epilogue, the two-phase weight gradient, the column sums and the reconstruction error of the
closing launch) around the 16 x 16, 32 x 32 and 64 x 32 tiles and the 16- and 32-wide k groups, rows that are no whole
16-byte groups, and steps on either side of every line to the persistent kernel (LINES; test_host_rules.py holds them to
their side): least extents up to 64, up to 256 and beyond, odd batches below and from 128 on, rows that are no whole
groups, for which the persistent kernel has its element-wise form."""
import pytest

pytest.importorskip("torch")

import test_gpu_rbm_dense as T
from paper_1804_04512_amd import workloads as wl
from test_host_rules import LINES

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (16, 32, 64), (17, 33, 65), (15, 31, 63), (33, 130, 66), (64, 64, 128), (100, 30, 5), (3, 784, 129),
         (131, 519, 257), (512, 24, 16), (512, 1024, 1024), (513, 1025, 1024)]


@pytest.mark.parametrize("batch,n_vis,n_hid", SIZES)
@pytest.mark.parametrize("visible", ["binary", "gaussian"])
def test_rbm_step_sizes(batch, n_vis, n_hid, visible):
    T.test_rbm_cd1_step((batch, n_vis, n_hid), visible)


@pytest.mark.parametrize("batch,n_vis,n_hid", [c for pair in LINES for c in pair])
def test_rbm_step_lines(batch, n_vis, n_hid):
    T.test_rbm_cd1_step((batch, n_vis, n_hid), "binary")


@pytest.mark.parametrize("batch,sizes", [(1, (5, 3, 2)), (17, (33, 65, 31, 7)), (64, (130, 66, 258, 17)), (100, (784, 499, 251, 10))])
def test_network_step_sizes(batch, sizes):
    T.check_dense_net(wl.paper_mnist_dense(batch, sizes))
