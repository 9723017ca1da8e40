"""Column lists whose scan takes several rounds, ends inside a thread's 8 columns or inside
a wave, and block-rows of one row, of ragged height and taller than a launch's row
workgroups: mask, lists, offsets and values are exactly the oracle's, and unpack gives the
masked matrix back."""

from __future__ import annotations

import numpy as np
import pytest

from oracle import prune as OP
from synthetic import COL, PUNCHED, ROWCOL, draw, seed_for

from tests.helpers import DT, from_dev, oracle_mask, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_11581_amd as B
    B.lib()
    return B


# R, C, bh, bw, regularity, rate, khw, dtype
CASES = [
    (5, 7, 1, 3, COL, 2, 1, "bf16"),             # shorter than one thread's columns
    (33, 511, 16, 32, COL, 4, 1, "bf16"),        # last wave and thread in part, ragged block-row
    (40, 2048, 16, 32, COL, 4, 1, "f32"),        # exactly one round
    (24, 2049, 8, 32, COL, 2, 1, "bf16"),        # one column into the second
    (17, 4611, 16, 0, COL, 3, 1, "f32"),         # three rounds, whole-width block
    (1100, 40, 1100, 8, COL, 2, 1, "bf16"),      # more rows than a launch's workgroups
    (37, 2052, 8, 16, ROWCOL, 2, 1, "bf16"),     # a column kept by any row of the block
    (36, 2061, 8, 5, PUNCHED, 3, 9, "f32"),      # kernel locations
]


@pytest.mark.parametrize("i", range(len(CASES)), ids=[f"{c[0]}x{c[1]}-{c[4]}-{c[7]}" for c in CASES])
def test_column_lists_are_exact(B, i):
    from paper_2111_11581_amd.layers import PackedLayer
    R, C, bh, bw, reg, rate, khw, dtype = CASES[i]
    w = draw(seed_for(9, 90 + i, 1), (R, C), ("normal", 0, 1), dtype)
    scheme = B.Scheme(R, C, bh, bw, reg, rate, khw)
    layer = PackedLayer(scheme, DT[dtype], to_dev(w, dtype))
    m = oracle_mask(w, dtype, scheme)
    assert np.array_equal(layer.mask.cpu().numpy().reshape(R, C), m)
    back = from_dev(layer.unpack(), dtype).reshape(R, C)
    assert np.array_equal(back.view(np.uint8), np.where(m == 1, w, np.zeros_like(w)).view(np.uint8))
    pk = OP.pack(w, m, bh, bw, reg, rate)
    assert np.array_equal(layer.rowptr[:layer.n_rowptr].cpu().numpy(), pk["rowptr"])
    assert np.array_equal(layer.indices[:layer.n_indices].cpu().numpy(), pk["indices"])
    vals = from_dev(layer.values[:layer.n_values], dtype)
    assert np.array_equal(vals.view(np.uint8), np.ascontiguousarray(pk["values"]).view(np.uint8))
