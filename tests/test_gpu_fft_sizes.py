"""The Fourier route of the full convolution over its padded sides (every power of two from 2 to 64, equal and
not), the edges of the product kernel's 4 x 4 tiles of image pairs and channels and, where there is work for them, 4 x 8
ones, odd batches, a single map, and a workspace that holds no product spectra (the route in two launches instead of
three, in tiles of one or, where there is work for them, 2 x 2)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as orc
from paper_1804_04512_amd import binding as B
from paper_1804_04512_amd.workloads import ConvSpec

from helpers import max_rel_err, odesc
from test_gpu_parity import dev, host

pytestmark = pytest.mark.gpu

# a sum of K products per frequency and two transforms of log2(4096) = 12 butterfly levels each way: relative to
# the largest output, a few times sqrt(12 + K) x 2^-24, at most 2e-6 here
TOL = 4e-6

SIDES = [ConvSpec(2, 2, h + r - 1, w + s - 1, 3, r, s, 0, "identity", 1)
         for h, r, w, s in [(1, 2, 1, 1), (2, 2, 3, 3), (5, 4, 4, 5), (8, 9, 20, 7), (18, 15, 1, 64), (64, 1, 2, 2), (50, 15, 25, 8), (33, 2, 9, 9)]]
TILES = [ConvSpec(n, c, 20, 37, k, 6, 9, 3, "identity", 1) for n, c, k in [(1, 1, 1), (7, 5, 2), (16, 8, 3), (17, 9, 4), (33, 17, 5)]]
# enough work for tiles of 4 x 8 (2048 wavefronts of them) and 2 x 2 (1024 image pairs x channels), short at both ends
TILES += [ConvSpec(63, 33, 48, 48, 5, 15, 15, 0, "identity", 1), ConvSpec(61, 35, 50, 40, 3, 9, 6, 2, "identity", 1)]


@pytest.mark.parametrize("cs", SIDES + TILES, ids=lambda c: f"N{c.N}C{c.C}K{c.K}_{c.Ho}x{c.Wo}_{c.R}x{c.S}p{c.pad}")
@pytest.mark.parametrize("room", ["all", "no product spectra"])
def test_fft_sizes(cs, room):
    r = np.random.default_rng(cs.N + 100 * cs.C + cs.Ho)
    dy, w = r.standard_normal(cs.y_shape).astype(np.float32), r.standard_normal(cs.w_shape).astype(np.float32)
    size = B.dll_conv_full_fft_workspace_bytes(cs)
    if room != "all":
        f = (1 << max(1, (cs.Ho + cs.R - 2).bit_length())) * (1 << max(1, (cs.Wo + cs.S - 2).bit_length()))
        size = sum(-(-8 * f * maps // 256) * 256 for maps in ((cs.N + 1) // 2 * cs.K, cs.K * cs.C))
    dx = torch.full(cs.x_shape, float("nan"), device="cuda")
    B.dll_conv_full_bwd_fft(cs, dev(dy), None, None, dev(w), dx, torch.empty(max(size, 256), dtype=torch.uint8, device="cuda"))
    assert max_rel_err(host(dx), orc.conv_full_bwd(odesc(cs), dy, None, None, w)) <= TOL
