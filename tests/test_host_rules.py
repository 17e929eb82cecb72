"""What the library settles on the host before it launches anything: workspace sizes, and which kernel takes a call
(launches are noted instead of run: no GPU needed)."""
import re
import struct

import pytest

from paper_1804_04512_amd import binding as B
from paper_1804_04512_amd.workloads import ConvSpec

from launch_record import record


@pytest.mark.parametrize("shape", [(256, 1, 64, 64, 8, 3, 3, 1), (64, 1, 28, 28, 40, 9, 9, 0), (16, 3, 32, 32, 16, 5, 5, 2),
                                   (128, 16, 24, 24, 32, 3, 3, 1), (2, 1, 9, 9, 4, 4, 4, 0)])
def test_crbm_workspace_ignores_pooling_and_activation(shape):
    """The CRBM step ignores the descriptor's activation and pooling mode: it needs the same bytes whatever they
    are (a size taken from the pooled layer's plan was up to 1 MB short of what the step writes)."""
    sizes = {B.dll_crbm_workspace_bytes(ConvSpec(*shape, act, pool)) for act in ("identity", "relu") for pool in (1, 2)}
    assert len(sizes) == 1 and sizes.pop() > 0


# pass, layer, the lean kernel's instance <16-filter groups, row pairs>
LEAN = [
    ("fwd", (130, 3, 40, 40, 8, 3, 3, 0, "relu", 2), (1, 2)), ("bwd", (130, 9, 33, 47, 18, 2, 3, 1, "sigmoid", 1), (1, 2)),
    ("fwd", (260, 2, 8, 40, 5, 3, 3, 1, "sigmoid", 1), (1, 1)), ("fwd", (171, 20, 10, 69, 7, 5, 4, 0, "identity", 1), (1, 1)),
    ("fwd", (260, 15, 8, 34, 18, 3, 2, 0, "relu", 1), (2, 1)), ("bwd", (260, 18, 7, 40, 17, 3, 3, 0, "relu", 1), (2, 1)),
    ("fwd", (258, 3, 8, 40, 33, 3, 3, 1, "relu", 2), (3, 1)), ("bwd", (130, 40, 14, 20, 3, 3, 3, 1, "relu", 2), (3, 1)),
    ("bwd", (3, 5, 20, 36, 4, 5, 5, 2, "sigmoid", 2), (1, 1)),
]


def test_lean_layers_reach_the_lean_kernel(tmp_path):
    got = record([[what, *c] for what, c, _ in LEAN], tmp_path)
    for (what, c, (nt, rp)), (status, launches) in zip(LEAN, got):
        assert status == 0 and f"conv_engine_lean_kernelILi{nt}ELi{rp}E" in launches[0][0], (what, c, launches)


def test_full_launches_that_stay_pipelined(tmp_path):
    """Large filters, of which LDS holds no more workgroups than the pipelined kernel's registers, and forward passes
    into 17 to 32 channels with chunks to pipeline."""
    calls = [["bwd", 64, 32, 43, 43, 64, 9, 9, 0, "sigmoid", 1], ["fwd", 260, 17, 8, 34, 18, 3, 2, 0, "relu", 1],
             ["fwd", 60, 32, 56, 56, 8, 7, 7, 0, "relu", 2], ["bwd", 186, 8, 48, 48, 40, 7, 7, 3, "relu", 2]]
    for call, (status, launches) in zip(calls, record(calls, tmp_path)):
        assert status == 0 and "conv_engine_kernel" in launches[0][0], (call, launches)


def test_layers_past_the_pipelined_kernel(tmp_path):
    """Rows of a tile or filters of a workgroup 2 GiB apart, and maps of few columns whose narrow tiles would be more
    than a launch can have: neither is refused."""
    calls = [["fwd", 1, 1, 3, 30_000_000, 4, 3, 3, 0, "identity", 1], ["fwd", 1, 3_000_000, 4, 20, 5, 2, 2, 0, "identity", 1],
             ["fwd", 9_000_000, 1, 12, 8, 1, 1, 1, 0, "identity", 1], ["bwd", 9_000_000, 1, 10, 9, 1, 1, 1, 0, "relu", 1]]
    for call, (status, launches) in zip(calls, record(calls, tmp_path)):
        assert status == 0 and "conv_engine_lean_kernel" in launches[0][0], (call, launches)


def test_products_with_an_operand_of_2_gib(tmp_path):
    """The header allows tensors of fewer than 2^31 elements; the small-product kernel's buffers end at 2 GiB.  Products
    beyond are the persistent kernel's, however few multiply-adds they have (they were refused)."""
    calls = [["infer", [], [[20000, 32768], [32768, 10]], 10, 1], ["train", [], [[20000, 32768], [32768, 10]], 10, 1],
             ["rbm", 1, 32768, 20000], ["rbm", 1, 20000, 32768], ["infer", [], [[2000, 1]], 1, 300000],
             ["train", [], [[2001, 1]], 1, 300000], ["rbm", 2, 16384, 32768], ["train", [], [[3, 5], [5, 40000000], [40000000, 3]], 3, 5],
             ["infer", [], [[16384, 32769], [32769, 3]], 3, 1], ["infer", [], [[16384, 32751], [32751, 3]], 3, 1]]
    got = record(calls, tmp_path)
    for call, (status, launches) in zip(calls, got):
        assert status == 0 and launches, call
    assert "gemm_small" not in got[-2][1][0][0] and "gemm_small" in got[-1][1][0][0]   # either side of the line


def test_forward_products_do_not_mind_an_odd_batch(tmp_path):
    """What a forward product takes is settled by its rows' lengths: the batch is no row (odd batches of large layers ran
    on the small-product kernel, up to a third slower).  Rows that are no multiples of four take it up to 2^30 multiply-adds."""
    calls = [["infer", [], [[1696, 1912], [1912, 8]], 8, b] for b in (254, 255, 256)]
    calls += [["infer", [], [[1696, 1911], [1911, 8]], 8, 256], ["rbm", 127, 3012, 2392], ["rbm", 903, 2148, 136], ["rbm", 500, 1600, 1001]]
    first = [launches[0][0] for _, launches in record(calls, tmp_path)]
    assert all("gemm_fast" in f for f in first[:3]) and "gemm_small" in first[3]
    assert "gemm_fast" in first[4] and "gemm_small" in first[5] and "gemm_small" in first[6]


def test_narrow_3x3_layers(tmp_path):
    """Maps of at most 16 columns that leave the chip half empty: two channels are the few-output kernel's, as on any
    layer that the 3x3 instance does not take (they had come to the generic one, two of whose 16 columns they fill);
    gradients of few channels stay with the 3x3 instance from two thirds of the other layers' number of tiles on."""
    calls = [["bwd", 100, 2, 16, 16, 16, 3, 3, 1, "relu", 2], ["fwd", 100, 20, 16, 16, 2, 3, 3, 1, "relu", 1],
             ["bwd", 128, 16, 16, 16, 8, 3, 3, 1, "relu", 1], ["bwd", 129, 16, 16, 16, 8, 3, 3, 1, "relu", 1],
             ["bwd", 192, 32, 16, 16, 8, 3, 3, 1, "relu", 1], ["bwd", 193, 32, 16, 16, 8, 3, 3, 1, "relu", 1]]
    names = [launches[0][0] for _, launches in record(calls, tmp_path)]
    want = ["conv_fewout_kernel", "conv_fewout_kernel", "conv_engine_kernel", "conv3x3c16_kernel", "conv_engine_kernel", "conv3x3c16_kernel"]
    assert all(w in n for w, n in zip(want, names)), names


def test_grids_past_what_a_launch_can_have(tmp_path):
    """A launch holds 2^24 - 1 workgroups of 256 threads along x.  Layers of more tiles, transforms or sums than that are
    not refused where a kernel or a sequence of fewer exists."""
    calls = [["bwd", 9_000_000, 1, 4, 20, 1, 3, 3, 1, "identity", 2],     # two 16 x 16 tiles an image, or one of 32 columns
             ["fft", 16_000_000, 4, 2, 2, 2, 2, 2, 0, "identity", 1],     # 32 million inverse transforms, or 8 million of 2 x 2
             ["fft", 2, 4096, 2, 2, 4095, 2, 2, 0, "identity", 1],        # as many transforms as fit
             ["fft", 2, 4095, 2, 2, 4096, 2, 2, 0, "identity", 1],        # one operand after the other
             ["crbm", 1, 600_000, 2, 2, 1, 1, 1, 0],                      # 19 million visible sums, on 512 planes
             ["rbm", 1, 400_000_000, 1]]                                  # 25 million column sums
    got = record(calls, tmp_path)
    for call, (status, launches) in zip(calls, got):
        assert status == 0 and launches, call
    forward = [[l for l in launches if "fft2_forward" in l[0]] for _, launches in got]
    assert [len(f) for f in forward[1:4]] == [1, 1, 2] and forward[2][0][1] == (1 << 24) - 1


def test_crbm_step_that_cannot_be_finished_is_not_begun(tmp_path):
    """A step of more channels than its closing launch holds is refused before its first launch: the visible sums, which
    run before the closing launch, would count places past 2^31 (and write there) from 33.5 million channels on."""
    calls = [["crbm", 1, c, 1, 1, 1, 1, 1, 0] for c in (8_000_000, 9_000_000, 34_000_000, 70_000_000, 2_000_000_000)]
    got = record(calls, tmp_path)
    assert got[0][0] == 0 and len(got[0][1]) == 5
    for call, (status, launches) in zip(calls[1:], got[1:]):
        assert status == 5 and not launches, (call, status, launches)


def test_crbm_step_launches(tmp_path):
    """Five launches; both phases' filter gradients in one, on two planes of workgroups, and a workgroup for each of the 32
    visible sums per channel on the planes behind them, however few tiles the images have (they were walked in turn by one
    plane of as many workgroups as a filter gradient has)."""
    calls = [["crbm", 64, 1, 28, 28, 40, 9, 9, 0], ["crbm", 8, 16, 16, 16, 8, 3, 3, 0], ["crbm", 1, 64, 16, 16, 8, 3, 3, 1],
             ["crbm", 1, 3, 16, 17, 33, 5, 5, 0], ["crbm", 2, 16, 20, 20, 9, 9, 1, 0], ["crbm", 1, 8_000_000, 1, 1, 1, 1, 1, 0]]
    for call, (status, launches) in zip(calls, record(calls, tmp_path)):
        assert status == 0 and len(launches) == 5, (call, launches)
        name, x, y, z, _ = launches[3]
        assert "wgrad_kernel" in name and name.split("EEEv")[0].endswith("Lb1") and "step_tail_kernelILb0E" in launches[4][0], (call, launches)
        assert 32 * call[2] <= x * y * (z - 2) < 32 * call[2] + x * y, (call, launches)


def test_outputs_over_inputs(tmp_path):
    """A one-layer network's probabilities over its input and an RBM step's reconstruction over the states it starts from:
    nothing writes there while a product still reads (both had come to be written by that product itself)."""
    calls = [["infer_in_place", [], [[12, 10]], 10, 50], ["infer", [], [[12, 10]], 10, 50], ["rbm_in_place", 40, 48, 48], ["rbm", 40, 48, 48]]
    names = [[l[0] for l in launches] for _, launches in record(calls, tmp_path)]
    assert [len(n) for n in names] == [2, 1, 5, 4]
    assert "softmax" in names[0][1] and "copy" in names[2][4]


def test_fourier_tile_sizes_have_a_test(tmp_path):
    """test_gpu_fft_sizes.py reaches every instance of the product kernels."""
    cases = [(n, c, h, w, k, r, s, p) for n, c, k, h, w, r, s, p in [(63, 33, 5, 48, 48, 15, 15, 0), (61, 35, 3, 50, 40, 9, 6, 2), (33, 17, 5, 20, 37, 6, 9, 3)]]
    calls = [[what, *c, "identity", 1] for c in cases for what in ("fft", "fft_less")]
    names = ["".join(l[0] for l in launches) for _, launches in record(calls, tmp_path)]
    want = ["product_kernelILi4ELi8E", "product_inverse_kernelILi2ELi2E"] * 2 + ["product_kernelILi4ELi4E", "product_inverse_kernelILi1ELi1E"]
    assert all(w in n for w, n in zip(want, names)), names


def _kernel_resources(path):
    """Name -> resources of every kernel in a built library, from the notes of the code objects in it."""
    msgpack = pytest.importorskip("msgpack")
    data, out = open(path, "rb").read(), {}
    for m in re.finditer(rb"\x7fELF\x02\x01\x01\x40", data):   # 64 bits, AMD GPU
        elf = data[m.start():]
        (table,), (size, count) = struct.unpack_from("<Q", elf, 0x28), struct.unpack_from("<HH", elf, 0x3A)
        for i in range(count):
            _, kind, _, _, at, _ = struct.unpack_from("<IIQQQQ", elf, table + i * size)
            if kind != 7:
                continue
            name, body, note = struct.unpack_from("<III", elf, at)
            if note == 32:
                start = at + 12 + (name + 3) // 4 * 4
                for k in msgpack.unpackb(elf[start:start + body], strict_map_key=False)["amdhsa.kernels"]:
                    out[k[".name"]] = k
    return out


def test_filter_gradient_registers_leave_the_planned_wavefronts():
    """plan_wgrad sizes its grid by the wavefronts a SIMD has room for beside the registers of the instances with layer
    output.  Checks in the product loop had taken one from <2, 9> unpooled (a layer there 27 % slower) and from five of
    the ragged instances."""
    plan = {1: [[4, 3, 3, 2], [3, 2, 2, 2], [2, 1, 1, 1]], 2: [[5, 4, 3, 3], [4, 3, 2, 2], [3, 2, 2, 2]]}   # [pool][filters / 16 - 1][tap tiles]
    one_round = {1: [5, 3, 2], 2: [7, 5, 4]}
    # <filters / 16, tap tiles, pool, staging> that have one less: ragged rows (3) but for one
    less = {(1, 2, 1, 3), (2, 2, 1, 1), (2, 2, 1, 3), (2, 9, 1, 3), (1, 2, 2, 3), (1, 5, 2, 3), (2, 2, 2, 3), (2, 5, 2, 3), (3, 9, 2, 3)}
    kernels = _kernel_resources(B.LIB_PATH)
    for pool in (1, 2):
        for m in (1, 2, 3):
            for j, ntt in enumerate((2, 5, 7, 9)):
                for fast in (1, 2, 3, 4) if ntt == 2 else (1, 3):
                    name = f"_ZN4dllk12_GLOBAL__N_112wgrad_kernelILi{m}ELi{ntt}ELi{pool}ELi{fast}ELb1ELb0EEEvNS0_11WgradParamsE"
                    waves = min(8, 512 // ((kernels[name][".vgpr_count"] + 7) // 8 * 8))
                    want = (plan if fast in (1, 3) else one_round)[pool][m - 1]
                    want = (want[j] if fast in (1, 3) else want) - ((m, ntt, pool, fast) in less)
                    assert waves >= want, (name, kernels[name][".vgpr_count"], waves, want)


def test_map_edge_lists_reach_the_instances(tmp_path):
    """test_gpu_wgrad_edges.py: every staging form and number of tap tiles, pooled and not, with and without the layer
    output; whole rows and ragged ones with two gradients in one launch."""
    import test_gpu_wgrad_edges as E
    fields = lambda c: [c.N, c.C, c.H, c.W, c.K, c.R, c.S, c.pad, c.act, c.pool]
    got = record([["wgrad", *fields(c)] for c in E.LAYERS] + [["crbm", *fields(c)[:8]] for c in E.CRBM], tmp_path)
    names = [next(l[0] for l in launches if "wgrad_kernel" in l[0]) for status, launches in got if status == 0]
    assert len(names) == len(got)
    seen = {tuple(map(int, re.search(r"wgrad_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)ELb(\d)ELb(\d)E", n).groups()))[1:] for n in names}
    want = {(2, pool, fast, y, 0) for fast in (2, 4) for pool, y in ((1, 0), (1, 1), (2, 1))}
    want |= {(ntt, pool, fast, y, 0) for ntt in (5, 7, 9) for fast in (1, 3) for pool, y in ((1, 0), (1, 1), (2, 1))}
    want |= {(9, 1, 0, 1, 0), (2, 1, 2, 0, 1), (2, 1, 4, 0, 1), (7, 1, 1, 0, 1), (9, 1, 1, 0, 1), (5, 1, 3, 0, 1), (9, 1, 3, 0, 1), (9, 1, 0, 1, 1)}
    assert want <= seen, sorted(want - seen)


# RBM steps (batch, visible, hidden units): the largest of their kind in the small-product kernels, and the next beyond
LINES = [((64, 1024, 4096), (64, 1024, 4100)), ((128, 1024, 1536), (128, 1024, 1540)), ((512, 1024, 1024), (516, 1024, 1024)),
         ((127, 1024, 4124), (127, 1024, 4132)), ((129, 2048, 4064), (129, 2048, 4068)), ((513, 1025, 2041), (513, 1025, 2045))]


def test_rbm_steps_on_either_side_of_the_lines(tmp_path):
    got = record([["rbm", *c] for pair in LINES for c in pair], tmp_path)
    small = ["step_tail_kernelILb1E" in launches[-1][0] and len(launches) == 4 for _, launches in got]
    assert small == [True, False] * len(LINES), small
    assert any("11gemm_kernel" in l[0] for l in got[-1][1])   # the element-wise form
