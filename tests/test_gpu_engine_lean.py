"""The lean convolution kernel (launches of two workgroups per compute unit and more, short gradients, planes past the other
kernel's offsets): each of its four instances, ragged tiles, chunks and filter groups, every source of the backward pass.
test_host_rules.py holds the same cases to the kernel they are meant for."""
import pytest

torch = pytest.importorskip("torch")

from paper_1804_04512_amd import binding as B
from paper_1804_04512_amd.workloads import ConvSpec

import test_gpu_parity as T
from test_host_rules import LEAN

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("i", range(len(LEAN)), ids=["x".join(map(str, c[:7])) + f"p{c[7]}_{c[8]}_pool{c[9]}" for _, c, _ in LEAN])
def test_lean_layers(i):
    cs = ConvSpec(*LEAN[i][1])
    T.check_trio(cs, *T.rand_layer(cs, 9500 + i))


def test_rows_past_the_32_bit_offsets():
    """Three rows of 30 million columns: the 18 rows a tile may touch are 2 GiB apart.  Against the nine shifted products
    in 64 bits; the sum of nine rounds to a few 2^-24 of the largest term."""
    cs = ConvSpec(1, 1, 3, 30_000_000, 4, 3, 3, 0, "identity", 1)
    g = torch.Generator("cuda").manual_seed(5)
    x = torch.randn(cs.x_shape, device="cuda", generator=g)
    w = torch.randn(cs.w_shape, device="cuda", generator=g)
    y = torch.full(cs.y_shape, float("nan"), device="cuda")
    B.dll_conv_valid_fwd(cs, x, w, None, y)
    for k in range(cs.K):
        ref = torch.zeros(cs.Wo, dtype=torch.float64, device="cuda")
        for r in range(3):
            for s in range(3):
                ref += x[0, 0, r, s:s + cs.Wo].double() * w[k, 0, r, s].double()
        assert float((y[0, k, 0].double() - ref).abs().max() / ref.abs().max()) <= 1e-6
