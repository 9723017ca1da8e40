"""3-wide bf16 convs: the forms their kernel takes at the sizes where it can go wrong
(group and row remainders, windows that reach past x, paddings wider than the image,
tiles over several images, lists whose steps span more channels than the registers hold,
block-rows of any height), against the fp64 oracle with the gates of the other convs."""

from __future__ import annotations

import numpy as np
import pytest

from synthetic import COL, DENSE, PUNCHED, ROW, ROWCOL, UNSTRUCTURED, ConvLayer, draw_layer

from tests.helpers import DT, from_dev, gate_conv, oracle_mask, out_to_f64, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_11581_amd as B
    B.lib()
    return B


# n, cin, h, w, cout, kh, (sh, sw), (ph, pw), (bh, bw), regularity, rate, bias and ReLU, output type
CASES = [
    (1, 1, 2, 3, 5, 3, (1, 1), (1, 1), (0, 0), DENSE, 1, True, "bf16"),          # x smaller than one load
    (1, 2, 5, 1, 16, 3, (1, 1), (1, 2), (0, 0), DENSE, 1, False, "f32"),         # padding wider than the image
    (2, 8, 9, 5, 24, 3, (1, 1), (1, 1), (8, 16), COL, 2, True, "f32"),           # partial groups, fp32 stores
    (3, 40, 7, 7, 33, 3, (1, 1), (1, 1), (16, 32), COL, 4, True, "bf16"),        # tiles over images, ragged rows
    (2, 24, 11, 9, 40, 3, (1, 1), (2, 2), (0, 0), UNSTRUCTURED, 4, False, "bf16"),
    (2, 16, 12, 8, 32, 3, (1, 1), (0, 3), (16, 16), ROW, 2, True, "bf16"),
    (1, 20, 6, 62, 48, 3, (1, 1), (1, 1), (48, 32), COL, 2, False, "bf16"),      # three m-tiles per list
    (2, 12, 9, 130, 64, 3, (1, 1), (1, 1), (64, 36), COL, 4, True, "bf16"),      # wide rows
    (5, 96, 13, 13, 64, 3, (2, 2), (1, 1), (16, 32), COL, 4, True, "bf16"),      # stride 2, odd width
    (2, 17, 10, 16, 24, 3, (2, 2), (1, 1), (8, 8), ROWCOL, 2, False, "f32"),
    (1, 3, 7, 21, 70, 3, (2, 2), (2, 2), (0, 0), DENSE, 1, True, "bf16"),
    (2, 32, 9, 12, 32, 1, (1, 1), (0, 1), (16, 24), COL, 4, False, "bf16"),      # 1 x 3
    (2, 10, 14, 10, 32, 5, (1, 2), (2, 1), (32, 30), COL, 3, True, "bf16"),      # 5 x 3, strides 1 and 2
    (2, 12, 13, 8, 16, 3, (3, 1), (1, 1), (16, 36), COL, 2, False, "bf16"),      # rows skipped
    (1, 256, 18, 18, 32, 3, (1, 1), (1, 1), (32, 0), COL, 16, False, "bf16"),    # steps over very many channels
    (1, 256, 30, 30, 16, 3, (2, 2), (1, 1), (16, 64), COL, 16, True, "bf16"),
    (3, 64, 10, 14, 96, 3, (1, 1), (1, 1), (32, 32), PUNCHED, 4, True, "bf16"),
    (2, 30, 9, 9, 80, 3, (1, 1), (1, 1), (0, 0), ROW, 4, True, "bf16"),          # kept filters only
    (70, 16, 6, 6, 24, 3, (1, 1), (1, 1), (8, 16), COL, 2, False, "bf16"),       # more images than planned for
    # columns before the image in many chunks: neither the first nor the last
    (2, 256, 14, 14, 48, 3, (1, 1), (2, 2), (0, 0), DENSE, 1, True, "bf16"),
    (2, 256, 9, 11, 40, 3, (1, 1), (1, 3), (16, 32), COL, 2, False, "bf16"),
    (1, 256, 15, 13, 32, 3, (2, 2), (2, 2), (0, 0), DENSE, 1, False, "f32"),
    (3, 192, 10, 16, 32, 3, (2, 2), (1, 3), (16, 16), COL, 2, True, "bf16"),
    (1, 256, 12, 12, 33, 3, (1, 1), (2, 2), (16, 32), PUNCHED, 2, True, "bf16"),
    (1, 300, 3, 2, 33, 1, (1, 1), (0, 5), (0, 0), DENSE, 1, False, "bf16"),      # units with no column in the image
    # units past the registers: smaller tiles of several pixel waves on the planned layout
    (8, 32, 46, 46, 18, 3, (1, 1), (1, 1), (16, 64), COL, 4, True, "bf16"),
    (8, 32, 46, 46, 31, 3, (1, 1), (1, 1), (16, 32), PUNCHED, 4, False, "f32"),
    (66, 32, 46, 46, 18, 3, (2, 2), (1, 1), (16, 64), PUNCHED, 4, True, "bf16"),
    # block-rows shorter than a tile, stored with zeros
    (2, 20, 33, 30, 62, 3, (1, 1), (1, 1), (6, 36), COL, 2, True, "bf16"),
    (2, 24, 25, 23, 60, 3, (1, 1), (1, 1), (4, 12), COL, 4, False, "f32"),
    (2, 24, 33, 30, 62, 3, (1, 1), (1, 1), (2, 4), PUNCHED, 4, True, "bf16"),
    (3, 32, 46, 46, 62, 3, (2, 2), (1, 1), (2, 12), COL, 4, False, "bf16"),
]


def _run(B, layer, x, w, out_dt, bias):
    import torch
    from paper_2111_11581_amd.layers import PackedLayer
    conv = B.ConvShape(layer.n, layer.cin, layer.h, layer.w, layer.kh, layer.kw, layer.sh, layer.sw, layer.ph, layer.pw)
    L = PackedLayer(layer.scheme, B.BF16, to_dev(w.reshape(layer.cout, -1), "bf16"), conv=conv)
    tdt = torch.float32 if out_dt == "f32" else torch.bfloat16
    # the output ends where its buffer does: a store past it would change the guard
    buf = torch.full((int(np.prod(layer.y_shape)) + 64,), 7.0, dtype=tdt, device="cuda")
    y = buf[:-64].view(layer.y_shape)
    bd = None if bias is None else torch.from_numpy(bias.astype(np.float32)).cuda()
    L.conv2d(to_dev(x, "bf16"), y, layer.n, DT[out_dt], bd, layer.relu)
    torch.cuda.synchronize()
    assert torch.all(buf[-64:] == 7.0)
    return L, y


def _layer(i):
    n, cin, h, w, cout, kh, (sh, sw), (ph, pw), (bh, bw), reg, rate, br, out = CASES[i]
    return ConvLayer(f"conv3 {i}", n, cin, h, w, cout, kh, 3, sh, sw, ph, pw, bh, bw, reg, rate, "bf16",
                     ("normal", 0, 1.0), ("normal", 0, (2.0 / (cin * kh * 3)) ** 0.5), relu=br), br, out


@pytest.mark.parametrize("i", range(len(CASES)))
def test_conv3_matches_oracle(B, i):
    layer, br, out_dt = _layer(i)
    d = draw_layer(layer, 9, i, with_bias=br)
    L, y = _run(B, layer, d["x"], d["w"], out_dt, d.get("bias"))
    m = L.mask.cpu().numpy().reshape(layer.cout, -1)
    assert np.array_equal(m, oracle_mask(d["w"], "bf16", layer.scheme))
    gate_conv(out_to_f64(from_dev(y, out_dt), out_dt), d["x"], d["w"], m, "bf16", out_dt, layer, bias=d.get("bias"),
              relu=layer.relu)


@pytest.mark.parametrize("i", [3, 8])
def test_conv3_keeps_images_apart(B, i):
    """An image of NaN and Inf changes no other image's output (tiles span images, and a
    row's pads are neighbours of other rows' values in memory)."""
    layer, br, out_dt = _layer(i)
    d = draw_layer(layer, 9, i, with_bias=br)
    _, y = _run(B, layer, d["x"], d["w"], out_dt, d.get("bias"))
    x2 = d["x"].copy()
    x2[1, ::2], x2[1, 1::2] = 0x7fc0, 0x7f80
    _, y2 = _run(B, layer, x2, d["w"], out_dt, d.get("bias"))
    a, b = from_dev(y, out_dt), from_dev(y2, out_dt)
    for k in range(layer.n):
        assert k == 1 or np.array_equal(a[k], b[k]), k
