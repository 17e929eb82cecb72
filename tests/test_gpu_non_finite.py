"""An infinity or NaN in an input reaches the outputs that are sums over it and no others: the neighbouring columns of
the banded few-output kernel (zeros of whose bands meet it), the next row's first elements in the last 16-byte
group of a ragged row (filter gradient, dense products)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as orc
from paper_1804_04512_amd import binding as B
from paper_1804_04512_amd.workloads import ConvSpec, DenseSpec

from helpers import TOL_GRAD, max_rel_err, odesc
from test_gpu_parity import dev, host, rand_layer

pytestmark = pytest.mark.gpu


def same_where_finite(got, ref):
    fin = np.isfinite(ref)
    differ = int(np.count_nonzero(np.isfinite(got) != fin))
    assert differ == 0, f"{differ} outputs finite on one side only"
    assert max_rel_err(got[fin], ref[fin]) <= TOL_GRAD


# every way the few-output kernel comes by its source: pooled and not, with and without the layer output, one to three outputs
FEW = [ConvSpec(2, 1, 18, 40, 6, 3, 3, 1, "identity", 2), ConvSpec(2, 2, 33, 30, 5, 3, 3, 0, "identity", 1),
       ConvSpec(1, 3, 24, 36, 17, 7, 7, 0, "sigmoid", 2), ConvSpec(1, 1, 17, 33, 40, 8, 17, 2, "sigmoid", 1),
       ConvSpec(1, 3, 22, 26, 9, 5, 5, 2, "relu", 2)]


@pytest.mark.parametrize("i", range(len(FEW)), ids=lambda i: f"C{FEW[i].C}K{FEW[i].K}_{FEW[i].R}x{FEW[i].S}_{FEW[i].act}_pool{FEW[i].pool}")
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_few_channels_backward(i, value):
    cs = FEW[i]
    x, w, b, dy = rand_layer(cs, 9800 + i)
    y, idx = orc.conv_valid_fwd(odesc(cs), x, w, b)
    at = np.unravel_index(int(np.argmax(np.where(np.arange(y.shape[3]) > y.shape[3] // 2, y, -np.inf))), y.shape)   # an active unit
    dy[at] = value
    ref = orc.conv_full_bwd(odesc(cs), dy, y, idx, w)
    assert np.isfinite(ref).any() and not np.isfinite(ref).all()
    dx = torch.full(cs.x_shape, 1.0, device="cuda")
    B.dll_conv_full_bwd(cs, dev(dy), dev(y), dev(idx) if cs.pool == 2 else None, dev(w), dx)
    same_where_finite(host(dx), ref)


@pytest.mark.parametrize("W", [37, 38, 39])
@pytest.mark.parametrize("pool", [1, 2])
def test_ragged_filter_gradient(W, pool):
    """The first element of a row is the neighbour of the row before it."""
    cs = ConvSpec(2, 3, 14, W + (W & 1 if pool == 2 else 0), 6, 3, 3, 0, "identity", pool)
    x, w, b, dy = rand_layer(cs, 9900 + W)
    y, idx = orc.conv_valid_fwd(odesc(cs), x, w, b)
    x[1, 1, 6, 0] = np.inf
    dw_o, db_o = orc.conv_valid_wgrad(odesc(cs), x, dy, y, idx)
    dw, db = torch.full(cs.w_shape, 1.0, device="cuda"), torch.full((cs.K,), 1.0, device="cuda")
    B.dll_conv_valid_wgrad(cs, dev(x), dev(dy), dev(y), dev(idx) if pool == 2 else None, dw, db, B.workspace(B.dll_conv_workspace_bytes(cs)))
    got = host(dw)
    assert np.isfinite(got[:, [0, 2]]).all() and np.isfinite(got[:, 1, :, 1:]).all() and not np.isfinite(got[:, 1, :, 0]).all()
    keep = np.isfinite(got) & np.isfinite(dw_o)
    assert max_rel_err(got[keep], dw_o[keep]) <= TOL_GRAD and max_rel_err(host(db), db_o) <= TOL_GRAD


@pytest.mark.parametrize("n_in", [5, 33, 130, 785])
def test_dense_rows_of_any_length(n_in):
    """A sample's infinities stay in its own outputs, whatever lies in the last 16 bytes of the row before."""
    rng = np.random.default_rng(n_in)
    x = rng.standard_normal((19, n_in)).astype(np.float32)
    ps = [rng.standard_normal(s).astype(np.float32) for s in [(37, n_in), (37,), (11, 37), (11,)]]
    net = B.net_desc([], [DenseSpec(n_in, 37, "sigmoid"), DenseSpec(37, 11)], 11, batch=19)
    ws = B.workspace(B.dll_cnn_forward_workspace_bytes(net))

    def run(a):
        logits, prob = torch.empty(19, 11, device="cuda"), torch.empty(19, 11, device="cuda")
        B.dll_cnn_forward(net, [dev(p) for p in ps], dev(a), logits, prob, ws=ws)
        return host(logits), host(prob)
    clean = run(x)
    x[7] = np.nan
    for got, want in zip(run(x), clean):
        others = np.arange(19) != 7
        assert np.array_equal(got[others], want[others]) and not np.isfinite(got[7]).any()
