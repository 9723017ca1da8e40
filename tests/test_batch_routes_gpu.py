"""Layers whose tiles are packed for two kernels, at batches that either of them runs (which
does is fixed on the host by tests/native/both.cpp): both outputs match the fp64 oracle, tiles
of another plan give NaN on both routes, and calls on several streams and graphs replayed at
once do not disturb each other."""

from __future__ import annotations

import os
import subprocess
import sys

import numpy as np
import pytest

from synthetic import COL, DENSE, PUNCHED, ConvLayer, LinearLayer, draw_layer

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


# cin, h, w, cout, kernel, stride, regularity, (bh, bw), rate, batches
CONVS = [
    (512, 14, 14, 512, 3, 2, COL, (16, 32), 4, (1, 64)),
    (648, 16, 16, 214, 3, 2, COL, (64, 32), 2, (1, 64)),
    (512, 4, 4, 512, 3, 1, DENSE, (0, 0), 1, (4,)),
    (516, 7, 10, 163, 3, 2, PUNCHED, (64, 16), 2, (1, 70)),
    (454, 25, 25, 24, 1, 1, COL, (64, 64), 4, (1, 64)),
    (214, 63, 63, 41, 1, 1, COL, (32, 32), 2, (1, 64)),
]


@pytest.mark.parametrize("i", range(len(CONVS)))
def test_conv_matches_oracle_at_either_batch(B, i):
    import torch
    from paper_2111_11581_amd.layers import PackedLayer
    cin, h, w, cout, k, s, reg, (bh, bw), rate, batches = CONVS[i]
    p = k // 2
    L = None
    for n in batches:
        layer = ConvLayer(f"batch {i}", n, cin, h, w, cout, k, k, s, s, p, p, bh, bw, reg, rate, "bf16", ("normal", 0, 1.0),
                          ("normal", 0, (2.0 / (cin * k * k)) ** 0.5), relu=True)
        d = draw_layer(layer, 13, i, with_bias=True)
        if L is None:   # packed once for every batch
            L = PackedLayer(layer.scheme, B.BF16, to_dev(d["w"].reshape(cout, -1), "bf16"),
                            conv=B.ConvShape(1, cin, h, w, k, k, s, s, p, p))
            m = L.mask.cpu().numpy().reshape(cout, -1)
            assert np.array_equal(m, oracle_mask(d["w"], "bf16", layer.scheme))
        images = sorted({0, n // 2, n - 1})
        bias = torch.from_numpy(d["bias"].astype(np.float32)).cuda()
        buf = torch.full((int(np.prod(layer.y_shape)) + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
        y = buf[:-64].view(layer.y_shape)
        L.conv2d(to_dev(d["x"], "bf16"), y, n, DT["bf16"], bias, True)
        torch.cuda.synchronize()
        assert torch.all(buf[-64:] == 7.0)
        gate_conv(out_to_f64(from_dev(y[images], "bf16"), "bf16"), d["x"], d["w"], m, "bf16", "bf16", layer, bias=d["bias"],
                  relu=True, images=images)
        # tiles of another plan (their header does not match)
        other = L.tiles.clone()
        other[4] += 1
        L.tiles, mine = other, L.tiles
        L.conv2d(to_dev(d["x"], "bf16"), y, n, DT["bf16"], bias, False)
        L.tiles = mine
        assert torch.isnan(y.float()).all()


@pytest.mark.parametrize("n", [1, 554])
def test_linear_matches_oracle_at_either_batch(B, n):
    import torch
    from paper_2111_11581_amd.layers import PackedLayer
    layer = LinearLayer("batch fc", n, 3960, 424, 64, 32, COL, 4, "bf16", ("normal", 0, 1.0), ("normal", 0, 0.03))
    d = draw_layer(layer, 13, 50)
    L = PackedLayer(layer.scheme, B.BF16, to_dev(d["w"], "bf16"))
    m = L.mask.cpu().numpy().reshape(424, 3960)
    y = torch.empty(layer.y_shape, dtype=torch.float32, device="cuda")
    L.linear(to_dev(d["x"], "bf16"), y, n, DT["f32"])
    torch.cuda.synchronize()
    gate_linear(out_to_f64(from_dev(y, "f32"), "f32"), d["x"], d["w"], m, "bf16", "f32")


def _captured():
    """In a process of its own: the first forward of a small batch, captured and replayed."""
    import torch
    import paper_2111_11581_amd as B
    from paper_2111_11581_amd.layers import PackedLayer
    w = torch.randn(512, 512 * 9, device="cuda").to(torch.bfloat16)
    layer = PackedLayer(B.Scheme(512, 512 * 9, 0, 0, B.DENSE, 1, 1), B.BF16, w, conv=B.ConvShape(4, 512, 4, 4, 3, 3, 1, 1, 1, 1))
    x = torch.randn(4, 512, 4, 4, device="cuda").to(torch.bfloat16)
    y = torch.empty(4, 512, 4, 4, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        layer.conv2d(x, y, 4, B.F32)
    cols = torch.nn.functional.unfold(x.double(), 3, padding=1)
    ref = (w.double() @ cols).view(4, 512, 4, 4)
    bound = 2 * (4608 + 2) * 2.0 ** -24 * (w.double().abs() @ cols.abs()).view(4, 512, 4, 4)   # fp32 sums in any order
    for _ in range(3):
        y.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.all((y - ref).abs() <= bound)
    layer.conv2d(x, y, 4, B.F32)   # and with the workspace
    assert torch.all((y - ref).abs() <= bound)


def test_a_first_call_inside_a_capture_runs(B):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", "from tests.test_batch_routes_gpu import _captured; _captured()"],
                       cwd=root, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stderr[-2000:]


def test_streams_do_not_share_a_buffer(B):
    """Different inputs on ten streams, all at once, several times."""
    import torch
    from paper_2111_11581_amd.layers import PackedLayer
    w = torch.randn(512, 512 * 9, device="cuda").to(torch.bfloat16)
    layer = PackedLayer(B.Scheme(512, 512 * 9, 0, 0, B.DENSE, 1, 1), B.BF16, w, conv=B.ConvShape(4, 512, 4, 4, 3, 3, 1, 1, 1, 1))
    n_streams = 10
    xs = [torch.randn(4, 512, 4, 4, device="cuda").to(torch.bfloat16) for _ in range(n_streams)]
    cols = [torch.nn.functional.unfold(x.double(), 3, padding=1) for x in xs]
    refs = [(w.double() @ c).view(4, 512, 4, 4) for c in cols]
    bounds = [2 * (4608 + 2) * 2.0 ** -24 * (w.double().abs() @ c.abs()).view(4, 512, 4, 4) for c in cols]
    streams = [torch.cuda.Stream() for _ in range(n_streams)]
    ys = [[torch.full((4, 512, 4, 4), 7.0, device="cuda") for _ in range(5)] for _ in range(n_streams)]
    torch.cuda.synchronize()
    for r in range(5):
        for s, x, y in zip(streams, xs, ys):
            layer.conv2d(x, y[r], 4, B.F32, stream=s)
    torch.cuda.synchronize()
    for y, ref, bound in zip(ys, refs, bounds):
        for r in range(5):
            assert torch.all((y[r] - ref).abs() <= bound)


def test_graphs_of_one_stream_do_not_share_a_buffer(B):
    """Graphs captured one after the other on a stream that has run the layer, replayed on
    streams of their own while that stream runs it again: every output as in an eager call
    alone, bit for bit (so the captured calls take the same kernel)."""
    import torch
    from paper_2111_11581_amd.layers import PackedLayer
    w = torch.randn(512, 512 * 9, device="cuda").to(torch.bfloat16)
    layer = PackedLayer(B.Scheme(512, 512 * 9, 0, 0, B.DENSE, 1, 1), B.BF16, w, conv=B.ConvShape(4, 512, 4, 4, 3, 3, 1, 1, 1, 1))
    n_graphs = 4
    xs = [torch.randn(4, 512, 4, 4, device="cuda").to(torch.bfloat16) for _ in range(n_graphs + 1)]
    refs = [torch.empty(4, 512, 4, 4, device="cuda") for _ in xs]
    ys = [torch.empty(4, 512, 4, 4, device="cuda") for _ in xs]
    main = torch.cuda.Stream()
    torch.cuda.synchronize()
    for x, ref in zip(xs, refs):
        layer.conv2d(x, ref, 4, B.F32, stream=main)
        torch.cuda.synchronize()
    graphs = []
    for i in range(n_graphs):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=main):
            layer.conv2d(xs[i], ys[i], 4, B.F32, stream=main)
        graphs.append(g)
    streams = [torch.cuda.Stream() for _ in range(n_graphs)]
    for _ in range(3):
        for y in ys:
            y.fill_(7.0)
        torch.cuda.synchronize()
        for _ in range(10):
            for g, s in zip(graphs, streams):
                with torch.cuda.stream(s):
                    g.replay()
            layer.conv2d(xs[-1], ys[-1], 4, B.F32, stream=main)
        torch.cuda.synchronize()
        for y, ref in zip(ys, refs):
            assert torch.equal(y, ref)
