"""The calls whose speed is watched: what programs have this library do, through its public entry points.

A case is a dict of plain values.  `listed()` names a dozen of them, `draw(rng)` gives more of the same
ranges, `prepare` builds what a program holds before the call (device tensors, network handle, workspace),
`run` is one pass, `exact` is the same result in 64-bit torch, without this library.

Kinds of case:
  layer_trio    forward, backward-data and filter gradient of one unpooled layer, as an autograd layer calls them
  layer_fwd     forward pass of one ReLU + max-pooling layer
  layer_bwd     both backward passes of one layer from the outputs its forward pass left
  cnn_train     one training step of a convolutional network (plain descent)
  cnn_infer     one inference pass of a convolutional network
  dense_train   one momentum step of a fully-connected network
  rbm           one CD-1 step of a fully-connected RBM
  crbm          one CD-1 step of a convolutional RBM
  full_fft      backward-data pass of a layer with large filters through the Fourier transform
"""
import math

import torch
import torch.nn.functional as F

from paper_1804_04512_amd import binding as B
from paper_1804_04512_amd.workloads import ConvSpec, DenseSpec


# ---------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: a sigmoid layer on eight MNIST-sized images, three calls of a few microseconds
        dict(name="layer_trio_mnist_b8", kind="layer_trio", N=8, C=1, H=28, W=28, K=8, R=5, S=5, pad=0, act="sigmoid"),
        # a middle layer of the large-image network, forward alone
        dict(name="layer_fwd_128x128_16", kind="layer_fwd", N=128, C=16, H=128, W=128, K=16, R=3, S=3, pad=1),
        # the backward passes of an unpooled layer on odd maps with channel counts that fill no tile
        dict(name="layer_bwd_odd_45x51", kind="layer_bwd", N=33, C=24, H=45, W=51, K=40, R=3, S=3, pad=1, act="relu", pool=1),
        # the small MNIST network's training step: a dozen dependent launches
        dict(name="cnn_train_mnist_b100", kind="cnn_train", net="mnist", batch=100),
        # the colour-image network's training step
        dict(name="cnn_train_cifar_b100", kind="cnn_train", net="cifar", batch=100),
        # the large-image network's training step: the headline workload and the largest case
        dict(name="cnn_train_imagenet_b128", kind="cnn_train", net="imagenet", batch=128, image=256, hidden=2048, classes=1000),
        # one image through the MNIST network, as a server answers a single request
        dict(name="cnn_infer_mnist_b1", kind="cnn_infer", net="mnist", batch=1),
        # a batch of large images through the five-block network
        dict(name="cnn_infer_imagenet_b128", kind="cnn_infer", net="imagenet5", batch=128, image=256, hidden=2048, classes=1000),
        # the fully-connected MNIST network's momentum step
        dict(name="dense_train_mnist_b100", kind="dense_train", batch=100, h1=500, h2=250),
        # its first layer pre-trained as an RBM
        dict(name="rbm_784_500_b100", kind="rbm", batch=100, n_vis=784, n_hid=500, visible="binary"),
        # a convolutional RBM on MNIST-sized images
        dict(name="crbm_mnist_b64", kind="crbm", N=64, C=1, H=28, W=28, K=40, R=9, S=9, pad=0, visible="binary", hidden_pool=1),
        # large filters: the full convolution by the Fourier route
        dict(name="full_fft_12x12_b64", kind="full_fft", N=64, C=32, H=43, W=43, K=32, R=12, S=12, pad=0),
    ]


_MAX_FLOP = 8e9          # of a drawn single layer: well under the large training step in time
_MAX_ELEMENTS = 1 << 25  # of any tensor of a drawn single layer


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_layer(rng, kind):
    while True:
        R = rng.choice([3, 3, 3, 5, 5, 7, 9])
        pad = rng.choice([0, R // 2])
        C = rng.choice([1, 3, _log(rng, 1, 64)])
        K = _log(rng, 4, 64)
        H = _log(rng, 12, 160)
        W = rng.choice([H, _log(rng, 12, 160)])
        N = _log(rng, 1, 128)
        if H + 2 * pad < R or W + 2 * pad < R:
            continue
        pool = {"layer_trio": 1, "layer_fwd": 2}.get(kind) or rng.choice([1, 2])
        if pool == 2:   # pooled maps are even
            H, W = H - (H + 2 * pad - R + 1) % 2, W - (W + 2 * pad - R + 1) % 2
        case = dict(kind=kind, N=N, C=C, H=H, W=W, K=K, R=R, S=R, pad=pad)
        if kind == "layer_trio":
            case.update(act=rng.choice(["identity", "sigmoid"]))
        elif kind == "layer_bwd":
            case.update(act=rng.choice(["identity", "sigmoid", "relu", "relu"]), pool=pool)
        cs = _conv_spec(case)
        passes = {"layer_trio": 3, "layer_fwd": 1, "layer_bwd": 2}[kind]
        if 2 * passes * cs.macs_nominal() <= _MAX_FLOP and max(N * C * H * W, N * K * cs.Ho * cs.Wo) <= _MAX_ELEMENTS:
            return case


def draw(rng):
    kind = rng.choice(["layer_trio", "layer_fwd", "layer_bwd", "cnn_train", "cnn_infer", "dense_train", "rbm", "crbm", "full_fft"])
    if kind in ("layer_trio", "layer_fwd", "layer_bwd"):
        return _draw_layer(rng, kind)
    if kind in ("cnn_train", "cnn_infer"):
        net = rng.choice(["mnist", "cifar", "imagenet", "imagenet5"])
        if net in ("mnist", "cifar"):
            return dict(kind=kind, net=net, batch=_log(rng, 16 if kind == "cnn_train" else 1, 512))
        return dict(kind=kind, net=net, batch=_log(rng, 8 if kind == "cnn_train" else 1, 128), image=32 * rng.randint(2, 8),
                    hidden=_log(rng, 256, 2048), classes=_log(rng, 10, 1000))
    if kind == "dense_train":
        return dict(kind=kind, batch=_log(rng, 16, 512), h1=_log(rng, 100, 1000), h2=_log(rng, 50, 500))
    if kind == "rbm":
        return dict(kind=kind, batch=_log(rng, 16, 512), n_vis=_log(rng, 100, 1600), n_hid=_log(rng, 64, 2048),
                    visible=rng.choice(["binary", "gaussian"]))
    if kind == "crbm":
        while True:
            C, R = rng.choice([(1, 5), (1, 7), (1, 9), (1, 11), (3, 5), (3, 7), (16, 3)])
            pad = rng.choice([0, R // 2])
            side, K, N = _log(rng, 16, 48), _log(rng, 8, 64), _log(rng, 8, 128)
            hidden_pool = rng.choice([1, 2])
            if hidden_pool == 2:   # pooled hidden maps are even
                side -= (side + 2 * pad - R + 1) % 2
            case = dict(kind=kind, N=N, C=C, H=side, W=side, K=K, R=R, S=R, pad=pad, visible=rng.choice(["binary", "gaussian"]),
                        hidden_pool=hidden_pool)
            if 10 * _conv_spec(case).macs_nominal() <= _MAX_FLOP:
                return case
    while True:
        R = rng.randint(6, 16)
        out = rng.randint(8, 65 - R)   # the full convolution's side is out + R - 1 <= 64
        N, C, K = _log(rng, 1, 64), _log(rng, 3, 32), _log(rng, 3, 32)
        pad = rng.choice([0, 0, R // 2])
        H = out + R - 1 - 2 * pad
        if H >= 1:
            return dict(kind="full_fft", N=N, C=C, H=H, W=H, K=K, R=R, S=R, pad=pad)


# ---------------------------------------------------------------------------------------
# shapes
# ---------------------------------------------------------------------------------------
def _conv_spec(case):
    pool = 2 if case["kind"] == "layer_fwd" else case.get("pool", 1)
    act = "relu" if case["kind"] == "layer_fwd" else case.get("act", "identity")
    return ConvSpec(case["N"], case["C"], case["H"], case["W"], case["K"], case["R"], case["S"], case["pad"], act, pool)


def _net_spec(case):
    """(conv layers, dense layers, classes, learning rate) of the networks the library is benchmarked on."""
    n, net, train = case["batch"], case["net"], case["kind"] == "cnn_train"
    if net == "mnist":
        act = "relu" if train else "sigmoid"
        conv = [ConvSpec(n, 1, 28, 28, 8, 5, 5, 0, act, 2), ConvSpec(n, 8, 12, 12, 8, 5, 5, 0, act, 2)]
        return conv, [DenseSpec(128, 150, act), DenseSpec(150, 10)], 10, 0.1
    if net == "cifar":
        p, feat = (1, 1536) if train else (0, 864)   # trained with padded convolutions, served without
        conv = [ConvSpec(n, 3, 32, 32, 12, 5, 5, 2 * p, "relu", 2),
                ConvSpec(n, 12, 14 + 2 * p, 14 + 2 * p, 24, 3, 3, p, "relu", 2)]
        return conv, [DenseSpec(feat, 64, "relu"), DenseSpec(64, 10)], 10, 0.001
    chans = [3, 16, 16, 32, 32, 32][:5 if net == "imagenet" else 6]
    conv, side = [], case["image"]
    for c, k in zip(chans, chans[1:]):
        conv.append(ConvSpec(n, c, side, side, k, 3, 3, 1, "relu", 2))
        side //= 2
    return conv, [DenseSpec(32 * side * side, case["hidden"], "relu"), DenseSpec(case["hidden"], case["classes"])], case["classes"], 0.001


def _dense_spec(case):
    return [DenseSpec(784, case["h1"], "sigmoid"), DenseSpec(case["h1"], case["h2"], "sigmoid"), DenseSpec(case["h2"], 10)]


# ---------------------------------------------------------------------------------------
# inputs: made on the device from the seed alone
# ---------------------------------------------------------------------------------------
class _Draws:
    def __init__(self, seed):
        self.g = torch.Generator("cuda").manual_seed(1804 * 1000003 + int(seed))

    def normal(self, *shape, sigma=1.0):
        t = torch.randn(shape, generator=self.g, device="cuda")
        return t.mul_(sigma) if sigma != 1.0 else t

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.g, device="cuda")

    def on(self, p, *shape):
        return (self.uniform(*shape) < p).float()

    def whole(self, n, *shape, dtype=torch.int32):
        return torch.randint(0, n, shape, generator=self.g, device="cuda", dtype=dtype)


def _params(conv, dense, d):
    ps = []
    for c in conv:
        ps += [d.normal(*c.w_shape, sigma=math.sqrt(2.0 / (c.C * c.R * c.S))), d.normal(c.K, sigma=0.01)]
    for q in dense:
        ps += [d.normal(q.out, q.in_, sigma=math.sqrt(2.0 / q.in_)), d.normal(q.out, sigma=0.01)]
    return ps


def _inputs(case, seed):
    d, kind = _Draws(seed), case["kind"]
    if kind in ("layer_trio", "layer_fwd", "layer_bwd", "full_fft"):
        cs = _conv_spec(case)
        s = dict(cs=cs, w=d.normal(*cs.w_shape, sigma=math.sqrt(2.0 / (cs.C * cs.R * cs.S))))
        if kind != "full_fft":
            s.update(x=d.normal(*cs.x_shape), bias=d.normal(cs.K, sigma=0.1))
        if kind != "layer_fwd":
            s.update(dy=d.normal(*cs.y_shape))
        if kind == "layer_bwd":
            y = d.normal(*cs.y_shape)
            s["y"] = {"identity": y, "sigmoid": torch.sigmoid(y), "relu": torch.relu(y)}[cs.act]
            if cs.pool == 2:   # position of the maximum; a ReLU layer flags its inactive units
                s["idx"] = d.whole(4, *cs.y_shape, dtype=torch.uint8) + (4 * (s["y"] == 0).to(torch.uint8) if cs.act == "relu" else 0)
        return s
    if kind in ("cnn_train", "cnn_infer"):
        conv, dense, classes, lr = _net_spec(case)
        x = d.uniform(*conv[0].x_shape) if case["net"] == "mnist" else d.normal(*conv[0].x_shape)
        return dict(conv=conv, dense=dense, classes=classes, lr=lr, x=x, params=_params(conv, dense, d),
                    labels=d.whole(classes, case["batch"]))
    if kind == "dense_train":
        dense = _dense_spec(case)
        ps = _params([], dense, d)
        return dict(dense=dense, x=d.uniform(case["batch"], 784), labels=d.whole(10, case["batch"]), params=ps,
                    velocity=[d.normal(*p.shape, sigma=1e-3) for p in ps])
    if kind == "rbm":
        n, nv, nh = case["batch"], case["n_vis"], case["n_hid"]
        return dict(v0=d.on(0.2, n, nv) if case["visible"] == "binary" else d.normal(n, nv), W=d.normal(nh, nv, sigma=0.05),
                    b=d.normal(nh, sigma=0.1), c=d.normal(nv, sigma=0.1), u=d.uniform(n, nh))
    cs = _conv_spec(case)
    p = case["hidden_pool"]
    return dict(cs=cs, v0=d.on(0.2, *cs.x_shape) if case["visible"] == "binary" else d.normal(*cs.x_shape),
                W=d.normal(*cs.w_shape, sigma=0.05), b=d.normal(cs.K, sigma=0.1), c=d.normal(cs.C, sigma=0.1),
                u=d.uniform(cs.N, cs.K, cs.Ho // p, cs.Wo // p))


def _empty(*shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    s, kind = _inputs(case, seed), case["kind"]
    s["kind"] = kind
    if kind in ("layer_trio", "layer_fwd", "layer_bwd"):
        cs = s["cs"]
        s["ws"] = B.workspace(B.dll_conv_workspace_bytes(cs))
        if kind != "layer_bwd":
            s["y"] = _empty(*cs.y_shape)
        if kind == "layer_fwd":
            s["idx"] = _empty(*cs.y_shape, dtype=torch.uint8)
        else:
            s.update(dx=_empty(*cs.x_shape), dw=_empty(*cs.w_shape), db=_empty(cs.K))
    elif kind == "full_fft":
        cs = s["cs"]
        s.update(dx=_empty(*cs.x_shape), ws=B.workspace(B.dll_conv_full_fft_workspace_bytes(cs)))
    elif kind in ("cnn_train", "cnn_infer", "dense_train"):
        n = case["batch"]
        s["net"] = B.net_desc(s.get("conv", []), s["dense"], s.get("classes", 10), batch=n)
        s["logits"] = _empty(n, s.get("classes", 10))
        if kind == "cnn_infer":
            s.update(prob=_empty(n, s["classes"]), ws=B.workspace(B.dll_cnn_forward_workspace_bytes(s["net"])))
        else:
            s.update(loss=_empty(1), ws=B.workspace(B.dll_cnn_workspace_bytes(s["net"])))
    elif kind == "rbm":
        n, nv, nh = case["batch"], case["n_vis"], case["n_hid"]
        s.update(n=n, nv=nv, nh=nh, visible=B.VISIBLE[case["visible"]], dW=_empty(nh, nv), db=_empty(nh), dc=_empty(nv),
                 mse=_empty(1), ws=B.workspace(B.dll_rbm_workspace_bytes(n, nv, nh)))
    else:
        cs = s["cs"]
        s.update(visible=B.VISIBLE[case["visible"]], hidden_pool=case["hidden_pool"], dW=_empty(*cs.w_shape), db=_empty(cs.K),
                 dc=_empty(cs.C), h0p=_empty(*cs.y_shape), mse=_empty(1), ws=B.workspace(B.dll_crbm_workspace_bytes(cs)))
    return s


# ---------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------
_RBM_LR = 0.01
_MOMENTUM_LR, _MOMENTUM, _DECAY = 0.1, 0.9, 1e-4


def run(s):
    kind = s["kind"]
    if kind == "layer_trio":
        B.dll_conv_valid_fwd(s["cs"], s["x"], s["w"], s["bias"], s["y"])
        B.dll_conv_full_bwd(s["cs"], s["dy"], s["y"], None, s["w"], s["dx"])
        B.dll_conv_valid_wgrad(s["cs"], s["x"], s["dy"], s["y"], None, s["dw"], s["db"], s["ws"])
        return dict(y=s["y"], dx=s["dx"], dw=s["dw"], db=s["db"])
    if kind == "layer_fwd":
        B.dll_conv_valid_fwd(s["cs"], s["x"], s["w"], s["bias"], s["y"], s["idx"])
        return dict(y=s["y"], idx=s["idx"])
    if kind == "layer_bwd":
        B.dll_conv_full_bwd(s["cs"], s["dy"], s["y"], s.get("idx"), s["w"], s["dx"])
        B.dll_conv_valid_wgrad(s["cs"], s["x"], s["dy"], s["y"], s.get("idx"), s["dw"], s["db"], s["ws"])
        return dict(dx=s["dx"], dw=s["dw"], db=s["db"])
    if kind == "full_fft":
        B.dll_conv_full_bwd_fft(s["cs"], s["dy"], None, None, s["w"], s["dx"], s["ws"])
        return s["dx"]
    if kind == "cnn_train":
        B.dll_cnn_train_step(s["net"], s["params"], None, s["x"], s["labels"], s["lr"], s["loss"], s["logits"], ws=s["ws"])
        return dict(loss=s["loss"], logits=s["logits"], params=s["params"])
    if kind == "cnn_infer":
        B.dll_cnn_forward(s["net"], s["params"], s["x"], s["logits"], s["prob"], ws=s["ws"])
        return dict(logits=s["logits"], prob=s["prob"])
    if kind == "dense_train":
        B.dll_cnn_train_step_momentum(s["net"], s["params"], s["velocity"], None, s["x"], s["labels"], _MOMENTUM_LR, _MOMENTUM,
                                      _DECAY, s["loss"], s["logits"], ws=s["ws"])
        return dict(loss=s["loss"], logits=s["logits"], params=s["params"], velocity=s["velocity"])
    if kind == "rbm":
        B.dll_rbm_cd1_step(s["n"], s["nv"], s["nh"], s["visible"], s["v0"], s["W"], s["b"], s["c"], s["u"], None, _RBM_LR, s["dW"],
                           s["db"], s["dc"], recon_mse=s["mse"], ws=s["ws"])
        return dict(W=s["W"], b=s["b"], c=s["c"], dW=s["dW"], db=s["db"], dc=s["dc"], mse=s["mse"])
    B.dll_crbm_cd1_step_units(s["cs"], s["visible"], s["hidden_pool"], s["v0"], s["W"], s["b"], s["c"], s["u"], None, _RBM_LR,
                              s["dW"], s["db"], s["dc"], h0_prob=s["h0p"], recon_mse=s["mse"], ws=s["ws"])
    return dict(W=s["W"], b=s["b"], c=s["c"], dW=s["dW"], db=s["db"], dc=s["dc"], h0p=s["h0p"], mse=s["mse"])


# ---------------------------------------------------------------------------------------
# work: what a pass cannot do without
# ---------------------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind in ("layer_trio", "layer_fwd", "layer_bwd", "full_fft", "crbm"):
        cs = _conv_spec(case)
        x, w, y = (4 * math.prod(t) for t in (cs.x_shape, cs.w_shape, cs.y_shape))
        macs = cs.macs_exact()
        if kind == "layer_fwd":
            return dict(bytes=x + w + y + y // 4, flops=2 * macs)
        if kind == "layer_trio":
            return dict(bytes=2 * x + 2 * w + 2 * y, flops=6 * macs)
        if kind == "layer_bwd":
            return dict(bytes=2 * x + 2 * w + 2 * y + (y // 4 if cs.pool == 2 else 0), flops=4 * macs)
        if kind == "crbm":   # v0, u, W in; W, dW, hidden probabilities out
            return dict(bytes=x + 2 * y + 3 * w, flops=10 * macs)
        # a real transform per map and filter, a complex product per pair of spectra, an inverse per output map
        p = 1 << (cs.Ho + cs.R - 2).bit_length()
        f = p * p
        one = 2.5 * f * math.log2(f)
        return dict(bytes=x + w + y, flops=one * (cs.N * cs.K + cs.K * cs.C + cs.N * cs.C) + 4.0 * f * cs.N * cs.K * cs.C)
    if kind == "rbm":
        n, nv, nh = case["batch"], case["n_vis"], case["n_hid"]
        return dict(bytes=4 * (n * nv + n * nh + 3 * nv * nh), flops=10 * n * nv * nh)
    conv, dense = ([], _dense_spec(case)) if kind == "dense_train" else _net_spec(case)[:2]
    n = case["batch"]
    size_p = sum(math.prod(c.w_shape) + c.K for c in conv) + sum(q.in_ * q.out + q.out for q in dense)
    size_x = math.prod(conv[0].x_shape) if conv else n * dense[0].in_
    out = n * dense[-1].out
    train = kind != "cnn_infer"
    flops = 0
    for i, c in enumerate(conv):
        flops += 2 * c.macs_exact() * ((2 if i == 0 else 3) if train else 1)
    for i, q in enumerate(dense):
        flops += 2 * n * q.in_ * q.out * ((2 if i == 0 and not conv else 3) if train else 1)
    return dict(bytes=4 * (size_x + out * (1 if train else 2) + size_p * ({"cnn_train": 2, "dense_train": 4}.get(kind, 1))), flops=flops)


# ---------------------------------------------------------------------------------------
# tolerances
# ---------------------------------------------------------------------------------------
# About four times what single- and double-precision results differ by on these inputs.
def tolerance(case):
    kind = case["kind"]
    if kind in ("layer_trio", "layer_bwd", "full_fft"):
        return dict(rel=2e-6, max=2e-5)
    if kind == "layer_fwd":   # near-equal maxima of a window may go to either position
        return dict(rel=2e-6, max=2e-5, differ=1e-5)
    if kind == "cnn_infer":
        return dict(rel=8e-6, max=1e-4)
    if kind == "dense_train":
        return dict(rel=2e-6, max=2e-5)
    if kind == "cnn_train":   # a near-tie of a pooling window or a ReLU moves one unit's gradient
        return dict(rel=2e-5, max=2e-3)
    return dict(rel=1e-3, max=5e-2)   # a sample whose probability equals its uniform number to rounding may go either way


# ---------------------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------------------
def _valid64(x, w, b, pad):
    (n, c, h, wd), (k, _, r, s) = x.shape, w.shape
    xp = F.pad(x, (pad, pad, pad, pad))
    ho, wo = h + 2 * pad - r + 1, wd + 2 * pad - s + 1
    z = torch.zeros((n, k, ho * wo), dtype=x.dtype, device=x.device)
    if b is not None:
        z += b.view(1, k, 1)
    for i in range(r):
        for j in range(s):
            z += torch.matmul(w[:, :, i, j], xp[:, :, i:i + ho, j:j + wo].reshape(n, c, ho * wo))
    return z.view(n, k, ho, wo)


def _full64(dz, w, pad, h, wd):
    (n, k, ho, wo), (_, c, r, s) = dz.shape, w.shape
    dxp = torch.zeros((n, c, h + 2 * pad, wd + 2 * pad), dtype=dz.dtype, device=dz.device)
    flat = dz.reshape(n, k, ho * wo)
    for i in range(r):
        for j in range(s):
            dxp[:, :, i:i + ho, j:j + wo] += torch.matmul(w[:, :, i, j].t().contiguous(), flat).view(n, c, ho, wo)
    return dxp[:, :, pad:pad + h, pad:pad + wd].contiguous()


def _grad64(x, dz, r, s, pad):
    (n, c, _, _), (_, k, ho, wo) = x.shape, dz.shape
    xp = F.pad(x, (pad, pad, pad, pad))
    flat = dz.reshape(n, k, ho * wo)
    dw = torch.zeros((k, c, r, s), dtype=x.dtype, device=x.device)
    for i in range(r):
        for j in range(s):
            part = xp[:, :, i:i + ho, j:j + wo].reshape(n, c, ho * wo).transpose(1, 2).contiguous()
            dw[:, :, i, j] = torch.matmul(flat, part).sum(0)
    return dw


def _act64(z, act):
    return torch.sigmoid(z) if act == "sigmoid" else torch.relu(z) if act == "relu" else z


def _slope64(y, act):
    return y * (1 - y) if act == "sigmoid" else (y > 0).to(y.dtype) if act == "relu" else torch.ones_like(y)


def _blocks64(z):
    """[N,K,H,W] as [N,K,H/2,W/2,4], the four values of each 2x2 block in row-major order."""
    n, k, h, w = z.shape
    return z.view(n, k, h // 2, 2, w // 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(n, k, h // 2, w // 2, 4)


def _unblocks64(b):
    n, k, h, w, _ = b.shape
    return b.view(n, k, h, w, 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(n, k, 2 * h, 2 * w)


def _unpool64(g, pos):
    return _unblocks64(torch.zeros(g.shape + (4,), dtype=g.dtype, device=g.device).scatter_(-1, pos.unsqueeze(-1), g.unsqueeze(-1)))


_NEAR_TIE = 5e-7    # of a layer's values: which of two so close is the larger is a matter of single-precision rounding


def _layer64(cs, x, w, b):
    """(output, position of each pooled maximum or None, whether every maximum and ReLU is decided beyond rounding)."""
    z = _valid64(x, w, b, cs.pad)
    near = _NEAR_TIE * float(z.square().mean().sqrt())
    if cs.pool == 1:
        return _act64(z, cs.act), None, cs.act != "relu" or float(z.abs().min()) > near
    top, pos = _blocks64(z).topk(2, -1)
    live = top[..., 0] > -near if cs.act == "relu" else torch.ones_like(top[..., 0], dtype=torch.bool)
    clear = not bool((live & (top[..., 0] - top[..., 1] < near)).any())
    if cs.act == "relu":
        clear = clear and float(top[..., 0].abs().min()) > near
    return _act64(top[..., 0], cs.act), pos[..., 0], clear


def _back64(cs, dy, y, pos):
    dz = dy * _slope64(y, cs.act)
    return dz if cs.pool == 1 else _unpool64(dz, pos)


def _net64(conv, dense, params, x, labels=None):
    """(logits, gradients in the order of params or None, loss or None).  The gradients of a convolution layer are
    None where a pooling window or ReLU of that layer or a later one is decided by rounding alone."""
    acts, poss, clears, h = [x], [], [], x
    for l, cs in enumerate(conv):
        h, pos, clear = _layer64(cs, h, params[2 * l], params[2 * l + 1])
        acts.append(h)
        poss.append(pos)
        clears.append(clear)
    L = len(conv)
    h = h.reshape(h.shape[0], -1)
    ins = []
    for q, dd in enumerate(dense):
        ins.append(h)
        h = h @ params[2 * (L + q)].t() + params[2 * (L + q) + 1]
        if q < len(dense) - 1:
            h = _act64(h, dd.act)
    if labels is None:
        return h, None, None
    n = h.shape[0]
    logp = torch.log_softmax(h, 1)
    loss = -logp[torch.arange(n, device=h.device), labels.long()].mean()
    g = (logp.exp() - F.one_hot(labels.long(), h.shape[1]).to(h.dtype)) / n
    grads = [None] * len(params)
    for q in reversed(range(len(dense))):
        grads[2 * (L + q)], grads[2 * (L + q) + 1] = g.t() @ ins[q], g.sum(0)
        g = g @ params[2 * (L + q)]
        if q > 0:
            g = g * _slope64(ins[q], dense[q - 1].act)
    if L:
        g = g.view_as(acts[L])
    for l in reversed(range(L)):
        cs = conv[l]
        if not clears[l]:
            break
        dz = _back64(cs, g, acts[l + 1], poss[l])
        grads[2 * l], grads[2 * l + 1] = _grad64(acts[l], dz, cs.R, cs.S, cs.pad), dz.sum((0, 2, 3))
        if l:
            g = _full64(dz, params[2 * l], cs.pad, cs.H, cs.W)
    return h, grads, loss.view(1)


_UNDECIDED = 1e-7   # a uniform number this close to its threshold: which side the sample falls on is a matter of rounding


def _hidden64(z, p):
    """Probabilities of the hidden units and, with 2x2 blocks, the four of each block."""
    if p == 1:
        return torch.sigmoid(z), None
    b = _blocks64(z)
    m = b.max(-1, keepdim=True).values.clamp(min=0)
    e = torch.exp(b - m)
    q = e / (torch.exp(-m) + e.sum(-1, keepdim=True))
    return _unblocks64(q), q


def exact(case, seed):
    t, kind = _inputs(case, seed), case["kind"]
    d = {k: v.double() if isinstance(v, torch.Tensor) and v.dtype == torch.float32 else v for k, v in t.items()}
    if kind in ("layer_trio", "layer_fwd", "layer_bwd", "full_fft"):
        cs = d["cs"]
        if kind == "full_fft":
            return _full64(d["dy"], d["w"], cs.pad, cs.H, cs.W)
        if kind == "layer_fwd":
            return dict(y=_layer64(cs, d["x"], d["w"], d["bias"])[0], idx=None)
        y = d["y"] if kind == "layer_bwd" else _layer64(cs, d["x"], d["w"], d["bias"])[0]
        dz = _back64(cs, d["dy"], y, (d["idx"] & 3).long() if "idx" in d else None)
        out = dict(dx=_full64(dz, d["w"], cs.pad, cs.H, cs.W), dw=_grad64(d["x"], dz, cs.R, cs.S, cs.pad), db=dz.sum((0, 2, 3)))
        return out if kind == "layer_bwd" else dict(out, y=y)
    if kind in ("cnn_train", "cnn_infer", "dense_train"):
        ps = [p.double() for p in t["params"]]
        logits, grads, loss = _net64(d.get("conv", []), d["dense"], ps, d["x"], None if kind == "cnn_infer" else t["labels"])
        if kind == "cnn_infer":
            # the softmax multiplies the rounding of large logits: there the logits alone are held against 64 bits
            return dict(logits=logits, prob=torch.softmax(logits, 1) if float(logits.abs().max()) < 4 else None)
        if kind == "cnn_train":
            return dict(loss=loss, logits=logits, params=[None if g is None else p - d["lr"] * g for p, g in zip(ps, grads)])
        vs = [_MOMENTUM * v.double() - _MOMENTUM_LR * (g + (_DECAY * p if p.dim() > 1 else 0)) for p, v, g in zip(ps, t["velocity"], grads)]
        return dict(loss=loss, logits=logits, params=[p + v for p, v in zip(ps, vs)], velocity=vs)
    # the RBM steps
    conv, p = kind == "crbm", case.get("hidden_pool", 1)
    v0, W, b, c, u = d["v0"], d["W"], d["b"], d["c"], d["u"]
    n = v0.shape[0]
    if conv:
        cs = d["cs"]
        hidden = lambda v: _hidden64(_valid64(v, W, b, cs.pad), p)                             # noqa: E731
        visible = lambda h: _full64(h, W, cs.pad, cs.H, cs.W) + c.view(1, -1, 1, 1)            # noqa: E731
        stat = lambda v, h: _grad64(v, h, cs.R, cs.S, cs.pad)                                  # noqa: E731
        per = (0, 2, 3)
    else:
        hidden = lambda v: (torch.sigmoid(v @ W.t() + b), None)                                # noqa: E731
        visible = lambda h: h @ W + c                                                          # noqa: E731
        stat = lambda v, h: h.t() @ v                                                          # noqa: E731
        per = (0,)
    h0p, q = hidden(v0)
    if q is None:
        h0s, near = (u < h0p).double(), (u - h0p).abs().min()
    else:   # unit i of a block is on where the running sums of the block's probabilities enclose u
        s = q.cumsum(-1)
        below = torch.cat([torch.zeros_like(s[..., :1]), s[..., :3]], -1)
        uu = u.unsqueeze(-1)
        h0s, near = _unblocks64(((below <= uu) & (uu < s)).double()), (uu - s).abs().min()
    v1 = visible(h0s)
    if case["visible"] == "binary":
        v1 = torch.sigmoid(v1)
    h1p, _ = hidden(v1)
    dW, db, dc = (stat(v0, h0p) - stat(v1, h1p)) / n, (h0p - h1p).sum(per) / n, (v0 - v1).sum(per) / n
    out = dict(W=W + _RBM_LR * dW, b=b + _RBM_LR * db, c=c + _RBM_LR * dc, dW=dW, db=db, dc=dc, mse=(v0 - v1).square().mean().view(1))
    if float(near) < _UNDECIDED:
        out = {k: None for k in out}
    return dict(out, h0p=h0p) if conv else out
