"""bf16 pointwise layers (1x1 convs at stride 1 and 2, linear layers): the forms their
kernels take at the sizes where they can go wrong (channels and pixels past whole steps
and granules, inputs smaller than one load, windows that reach past x, split and unsplit
K loops, lists of any block height, several tiles per workgroup), against the fp64 oracle
with the gates of the other layers."""

from __future__ import annotations

import numpy as np
import pytest

from synthetic import COL, DENSE, ROW, ROWCOL, UNSTRUCTURED, ConvLayer, LinearLayer, draw_layer

from tests.helpers import DT, from_dev, gate_conv, gate_linear, oracle_mask, out_to_f64, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_11581_amd as B
    B.lib()
    return B


# n, cin, h, w, cout, stride, (bh, bw), regularity, rate, bias and ReLU, output type
CONVS = [
    (1, 1, 1, 3, 5, 1, (0, 0), DENSE, 1, True, "bf16"),            # x smaller than one load
    (1, 3, 1, 1, 17, 2, (0, 0), DENSE, 1, False, "f32"),
    (3, 33, 7, 7, 40, 1, (16, 16), ROW, 2, True, "bf16"),          # odd plane, a step of one channel
    (2, 70, 5, 9, 130, 1, (0, 0), UNSTRUCTURED, 4, False, "f32"),
    (2, 64, 13, 13, 48, 2, (16, 16), ROW, 2, True, "bf16"),        # stride 2, odd width
    (3, 40, 6, 5, 33, 2, (0, 0), DENSE, 1, True, "f32"),           # last granule past the row
    (5, 96, 15, 8, 64, 2, (16, 0), ROW, 2, True, "bf16"),          # stride 2, kept filters only
    (2, 300, 9, 11, 70, 1, (0, 0), ROW, 3, True, "bf16"),          # kept filters only
    (1, 1024, 6, 6, 96, 1, (32, 32), ROW, 2, True, "bf16"),        # split K loop
    (40, 96, 14, 14, 64, 1, (0, 0), DENSE, 1, False, "bf16"),      # several tiles per workgroup
    (2, 64, 10, 10, 96, 1, (32, 32), COL, 4, True, "bf16"),
    (3, 61, 7, 7, 50, 1, (16, 16), COL, 2, False, "f32"),          # ragged blocks and channels
    (2, 96, 12, 12, 100, 1, (48, 32), COL, 2, True, "bf16"),       # three m-tiles per list
    (2, 48, 11, 13, 40, 2, (8, 16), COL, 2, True, "bf16"),         # lists at stride 2
    (2, 256, 9, 9, 64, 1, (32, 64), COL, 8, False, "bf16"),        # an eighth kept: the other kernel
    (1, 512, 5, 5, 64, 1, (64, 32), COL, 4, True, "bf16"),         # lists, split K loop
    (2, 64, 8, 8, 64, 1, (16, 32), ROWCOL, 2, False, "bf16"),
]
# in, out, batch, (bh, bw), regularity, rate, bias and ReLU, output type
LINEARS = [
    (5, 3, 1, (0, 0), DENSE, 1, True, "f32"),
    (100, 65, 7, (16, 16), ROW, 2, False, "bf16"),
    (2048, 100, 9, (0, 0), DENSE, 1, True, "f32"),                 # split K loop
    (257, 300, 513, (32, 32), ROW, 2, True, "bf16"),
    (160, 128, 33, (32, 32), COL, 2, True, "bf16"),
    (512, 96, 130, (16, 64), COL, 4, False, "f32"),
    (640, 64, 20, (64, 64), COL, 10, False, "bf16"),               # a tenth kept: the other kernel
    (2112, 1040, 3, (16, 32), COL, 2, False, "bf16"),              # lists too long for one workgroup to pack
]


def _out(B, shape, out_dt):
    """An output that ends where its buffer does: a store past it would change the guard."""
    import torch
    buf = torch.full((int(np.prod(shape)) + 64,), 7.0, device="cuda",
                     dtype=torch.float32 if out_dt == "f32" else torch.bfloat16)
    return buf, buf[:-64].view(shape)


def _bias(d):
    import torch
    return None if d.get("bias") is None else torch.from_numpy(d["bias"].astype(np.float32)).cuda()


@pytest.mark.parametrize("i", range(len(CONVS)))
def test_pointwise_conv_matches_oracle(B, i):
    import torch
    from paper_2111_11581_amd.layers import PackedLayer
    n, cin, h, w, cout, s, (bh, bw), reg, rate, br, out_dt = CONVS[i]
    layer = ConvLayer(f"pointwise {i}", n, cin, h, w, cout, 1, 1, s, s, 0, 0, bh, bw, reg, rate, "bf16",
                      ("normal", 0, 1.0), ("normal", 0, (2.0 / cin) ** 0.5), relu=br)
    d = draw_layer(layer, 10, i, with_bias=br)
    conv = B.ConvShape(n, cin, h, w, 1, 1, s, s, 0, 0)
    L = PackedLayer(layer.scheme, B.BF16, to_dev(d["w"].reshape(cout, -1), "bf16"), conv=conv)
    m = L.mask.cpu().numpy().reshape(cout, -1)
    assert np.array_equal(m, oracle_mask(d["w"], "bf16", layer.scheme))
    x = to_dev(d["x"], "bf16")
    for _ in range(2):   # a second pass finds other values in LDS
        buf, y = _out(B, layer.y_shape, out_dt)
        L.conv2d(x, y, n, DT[out_dt], _bias(d), br)
        torch.cuda.synchronize()
        assert torch.all(buf[-64:] == 7.0)
        gate_conv(out_to_f64(from_dev(y, out_dt), out_dt), d["x"], d["w"], m, "bf16", out_dt, layer, bias=d.get("bias"),
                  relu=br)


@pytest.mark.parametrize("i", range(len(LINEARS)))
def test_pointwise_linear_matches_oracle(B, i):
    import torch
    from paper_2111_11581_amd.layers import PackedLayer
    cin, cout, n, (bh, bw), reg, rate, br, out_dt = LINEARS[i]
    layer = LinearLayer(f"linear {i}", n, cin, cout, bh, bw, reg, rate, "bf16", ("normal", 0, 1.0),
                        ("normal", 0, (2.0 / cin) ** 0.5), relu=br)
    d = draw_layer(layer, 10, 100 + i, with_bias=br)
    L = PackedLayer(layer.scheme, B.BF16, to_dev(d["w"], "bf16"))
    m = L.mask.cpu().numpy().reshape(cout, cin)
    assert np.array_equal(m, oracle_mask(d["w"], "bf16", layer.scheme))
    buf, y = _out(B, layer.y_shape, out_dt)
    L.linear(to_dev(d["x"], "bf16"), y, n, DT[out_dt], _bias(d), br)
    torch.cuda.synchronize()
    assert torch.all(buf[-64:] == 7.0)
    gate_linear(out_to_f64(from_dev(y, out_dt), out_dt), d["x"], d["w"], m, "bf16", out_dt, bias=d.get("bias"), relu=br)


@pytest.mark.parametrize("sizes", [(24, 18), (20, 24)])
def test_a_layer_runs_as_in_a_thread_of_its_own(B, sizes):
    """Planes that share packed tiles (nothing in them depends on the size), called in either
    order: every output has the bits of a thread that called nothing before."""
    import threading

    import torch
    from paper_2111_11581_amd.layers import PackedLayer
    cin, cout, n = 512, 128, 4
    w = to_dev(draw_layer(ConvLayer("w", n, cin, 8, 8, cout, 1, 1, 1, 1, 0, 0, 0, 0, DENSE, 1, "bf16", ("normal", 0, 1.0),
                                    ("normal", 0, 0.06)), 10, 200)["w"].reshape(cout, -1), "bf16")
    x = {s: torch.randn(n, cin, s, s, device="cuda").to(torch.bfloat16) for s in sizes}
    layers = {s: PackedLayer(B.Scheme(cout, cin, 0, 0, DENSE, 1, 1), B.BF16, w, conv=B.ConvShape(n, cin, s, s, 1, 1, 1, 1, 0, 0))
              for s in sizes}

    def outputs(order):
        out = {}

        def call():
            for s in order:
                y = torch.empty(n, cout, s, s, device="cuda")
                layers[s].conv2d(x[s], y, n, B.F32)
                torch.cuda.synchronize()
                out[s] = y
        t = threading.Thread(target=call)
        t.start()
        t.join()
        return out

    alone = {s: outputs([s])[s] for s in sizes}
    for order in (sizes, sizes[::-1], sizes + sizes):
        for s, y in outputs(order).items():
            assert torch.equal(y, alone[s]), (order, s)


# regularity, (bh, bw), counts: lists that the gathered kernel, which splits K loops, does not take
NO_WORKSPACE = [(COL, (32, 32), True), (COL, (48, 32), False), (ROWCOL, (48, 16), False)]


def _captured(i):
    """In a process of its own: the first forward of a layer is captured into a graph, which a
    call that allocates the workspace cannot be, and replayed."""
    import torch
    import paper_2111_11581_amd as B
    from paper_2111_11581_amd.layers import PackedLayer
    reg, (bh, bw), counted = NO_WORKSPACE[i]
    cin, cout, n = 512, 96, 20
    scheme = B.Scheme(cout, cin, bh, bw, reg, 2, 1)
    if counted:
        scheme.set_counts([[8 + (i + j) % 9 for j in range(cin // bw)] for i in range(cout // bh)])
    w = torch.randn(cout, cin, device="cuda").to(torch.bfloat16)
    layer = PackedLayer(scheme, B.BF16, w)
    x = torch.randn(cin, n, device="cuda").to(torch.bfloat16)
    y = torch.empty(cout, n, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        layer.linear(x, y, n, B.F32)
    wm, xd = w.double() * layer.mask.view(cout, cin), x.double()
    ref, bound = wm @ xd, 2 * (cin + 2) * 2.0 ** -24 * (wm.abs() @ xd.abs())   # fp32 sums in any order
    for _ in range(3):
        y.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.all((y - ref).abs() <= bound)


@pytest.mark.parametrize("i", range(len(NO_WORKSPACE)))
def test_lists_outside_the_gathered_kernel_need_no_workspace(B, i):
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", f"from tests.test_pointwise_gpu import _captured; _captured({i})"],
                       cwd=root, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stderr[-2000:]
