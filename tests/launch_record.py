"""Which kernels a call would launch, found out without a GPU: `record` compiles the stand-in for the HIP runtime beside
this file, and makes the calls in a process of its own that holds that instead of the runtime.  Pointers are made up
(the library never follows one on the host), so the sizes may be any that the header allows."""
import ctypes as C
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
WORKSPACE = 1 << 62   # "as much as is asked for"


def record(calls, folder, root=None):
    """calls: [[entry point, descriptor, ...]], see `_make`.  Returns [(status, [(kernel, grid x, y, z, block x), ...]), ...]."""
    shim = os.path.join(str(folder), "launch_record.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wall", "-o", shim, os.path.join(HERE, "launch_record.c")], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), shim, root or os.path.dirname(HERE)], input=json.dumps(calls),
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr
    return [(st, [tuple(l) for l in ls]) for st, ls in json.loads(r.stdout.splitlines()[-1])]


class _Pointers:
    """Made-up device addresses, far apart, 4 KiB aligned."""
    def __init__(self):
        self.next = 1 << 40

    def __call__(self):
        self.next += 1 << 40
        return self.next


def _make(B, L, what, *args):
    """One call by name: 'fwd' / 'bwd' / 'wgrad' / 'fft' / 'fft_less' / 'crbm' (ConvSpec fields), 'rbm' (batch, n_vis, n_hid),
    'infer' / 'train' (conv layers, dense layers, classes, batch); 'rbm_in_place' writes v1 over h0_sample_in,
    'infer_in_place' the probabilities over x."""
    from paper_1804_04512_amd.workloads import ConvSpec, DenseSpec
    p, ws = _Pointers(), C.c_void_p(1 << 20)
    if what in ("fwd", "bwd", "wgrad", "fft", "fft_less", "crbm"):
        d = B.conv_desc(ConvSpec(*args))
        ref, idx = C.byref(d), p() if d.pool == 2 else None
        if what == "fwd":
            return L.dll_conv_valid_fwd(ref, p(), p(), p(), p(), idx, None, 0, None)
        if what == "bwd":
            return L.dll_conv_full_bwd(ref, p(), None if d.act == 0 else p(), idx, p(), p(), None, 0, None)
        if what == "wgrad":
            return L.dll_conv_valid_wgrad(ref, p(), p(), None if d.act == 0 else p(), idx, p(), p(), ws, WORKSPACE, None)
        if what in ("fft", "fft_less"):   # less: a workspace without the product spectra
            room = WORKSPACE if what == "fft" else L.dll_conv_full_fft_workspace_bytes(ref) - 256
            return L.dll_conv_full_bwd_fft(ref, p(), None if d.act == 0 else p(), idx, p(), p(), ws, room, None)
        return L.dll_crbm_cd1_step_units(ref, 0, 1, p(), p(), p(), p(), p(), None, 0.1, p(), p(), p(), *([None] * 6), ws, WORKSPACE, None)
    if what == "rbm_in_place":
        h = p()
        return L.dll_rbm_cd1_step(*args, 0, p(), p(), p(), p(), None, h, 0.1, p(), p(), p(), None, None, h, None, p(), ws, WORKSPACE, None)
    if what == "rbm":
        return L.dll_rbm_cd1_step(*args, 0, p(), p(), p(), p(), p(), None, 0.1, p(), p(), p(), *([None] * 4), p(), ws, WORKSPACE, None)
    conv, dense, classes, batch = args
    net = B.net_desc([ConvSpec(*c) for c in conv], [DenseSpec(*q) for q in dense], classes, batch)
    params = (C.c_void_p * (2 * (len(conv) + len(dense))))(*[p() for _ in range(2 * (len(conv) + len(dense)))])
    ref = C.byref(net.desc)
    if what == "infer_in_place":
        x = p()
        return L.dll_cnn_forward(ref, params, x, None, x, ws, WORKSPACE, None)
    if what == "infer":
        return L.dll_cnn_forward(ref, params, p(), None, p(), ws, WORKSPACE, None)
    return L.dll_cnn_train_step(ref, params, None, p(), p(), 0.1, p(), None, None, ws, WORKSPACE, None)


def _main():
    shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)   # before anything that brings the runtime along
    sys.path.insert(0, sys.argv[2])
    from paper_1804_04512_amd import binding as B
    L = B.lib()
    room = 1 << 18
    text = C.create_string_buffer(room)
    shim.take_launches.argtypes = [C.c_char_p, C.c_size_t]
    out = []
    for call in json.load(sys.stdin):
        status = _make(B, L, *call)
        shim.take_launches(text, room)
        lines = [l.rsplit(" ", 4) for l in text.value.decode().splitlines()]
        out.append([status, [[l[0], *map(int, l[1:])] for l in lines]])
    print(json.dumps(out))


if __name__ == "__main__":
    _main()
