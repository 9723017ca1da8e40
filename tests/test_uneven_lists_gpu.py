"""Whole-width column blocks, whose kept columns may lie anywhere, packed from weights of
uneven scale: the layers are accepted whatever the mask and match the fp64 oracle."""

from __future__ import annotations

import numpy as np
import pytest

from synthetic import COL, ROWCOL, ConvLayer, LinearLayer, bf16_bits_to_f32, draw_layer
from synthetic.gen import f32_to_bf16_bits

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


# in, out, batch or (images, height and width, kernel, stride), block rows, regularity, rate
CASES = [
    (2048, 512, 40, 32, COL, 2),
    (2048, 512, 40, 32, COL, 4),
    (1024, 64, (2, 14, 1, 1), 16, COL, 2),
    (512, 64, (2, 14, 3, 2), 16, COL, 4),       # 7x7 planes
    (512, 48, (3, 4, 3, 1), 16, COL, 2),        # 4x4 planes
    (64, 64, (2, 14, 3, 1), 16, COL, 4),        # a window of the whole input
    (256, 64, (1, 14, 3, 1), 16, COL, 8),       # stored with zeros
    (128, 48, (1, 28, 3, 2), 16, ROWCOL, 4),
    (64, 40, (2, 9, 1, 1), 16, ROWCOL, 2),
]


def _scales(cin, kind):
    """Per input channel: half of them 0.7 of the others, or only both ends kept."""
    s = np.ones(cin)
    if kind == "halves":
        s[cin // 2:] = 0.7
    else:
        s[cin // 8:-(cin // 8)] = 1e-3
    return s


@pytest.mark.parametrize("kind", ["halves", "ends"])
@pytest.mark.parametrize("i", range(len(CASES)))
def test_uneven_channel_scales(B, i, kind):
    import torch
    from paper_2111_11581_amd.layers import PackedLayer
    cin, cout, geo, bh, reg, rate = CASES[i]
    if isinstance(geo, int):
        layer = LinearLayer(f"uneven {i}", geo, cin, cout, bh, 0, reg, rate, "bf16", ("normal", 0, 1.0),
                            ("normal", 0, 0.05))
    else:
        n, hw, k, s = geo
        layer = ConvLayer(f"uneven {i}", n, cin, hw, hw, cout, k, k, s, s, k // 2, k // 2, bh, 0, reg, rate, "bf16",
                          ("normal", 0, 1.0), ("normal", 0, 0.05))
    d = draw_layer(layer, 12, i)
    w = bf16_bits_to_f32(d["w"]).reshape(cout, cin, -1) * _scales(cin, kind).astype(np.float32)[None, :, None]
    w = f32_to_bf16_bits(w).reshape(d["w"].shape)
    conv = None if isinstance(geo, int) else B.ConvShape(n, cin, hw, hw, k, k, s, s, k // 2, k // 2)
    L = PackedLayer(layer.scheme, B.BF16, to_dev(w.reshape(cout, -1), "bf16"), conv=conv)
    m = L.mask.cpu().numpy().reshape(cout, -1)
    assert np.array_equal(m, oracle_mask(w, "bf16", layer.scheme))
    y = torch.empty(layer.y_shape, dtype=torch.float32, device="cuda")
    x = to_dev(d["x"], "bf16")
    if conv is None:
        L.linear(x, y, geo, DT["f32"])
    else:
        L.conv2d(x, y, n, DT["f32"])
    torch.cuda.synchronize()
    out = out_to_f64(from_dev(y, "f32"), "f32")
    if conv is None:
        gate_linear(out, d["x"], w, m, "bf16", "f32")
    else:
        gate_conv(out, d["x"], w, m, "bf16", "f32", layer)
